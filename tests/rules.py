"""The rules that pick a kernel for the transposing conversions, stated again for tests that aim at one kernel: where a line moves, the
tests that no longer reach theirs fail.  test_col_small_rule.py compares them with the library's sources."""

KINDS = ("mxfp4", "align", "requant")


def small_tiles(kind, M, K, E=0, units=256):
    """Tiles of 128 x 128 take these rows (of E experts; 0: one matrix)."""
    pick = KINDS.index(kind)
    if E == 0:
        return 4 * (-(-M // 128) * (K // 128)) <= (11, 11, 12)[pick] * units
    if E > 256:
        return False
    padded = M % 128 == 0
    line = ((336, 336 if M <= 24 * E else 96, 336) if M <= 32 * E else (56, 24, 32) if M <= 64 * E else
            ((15, 12, 15) if padded else (24, 12, 15)) if M < 256 * E else (10, 10, 8) if padded else (14, 12, 12))[pick]
    return (2 * (M // 128) + E) * (K // 128) <= line * units


def own_rows(kind, M, K, E, units=256):
    """Not by small tiles, and the FP8-column kernels that write their own rows take these rows of E experts."""
    padded = M % 16 == 0 and (kind == "requant" or M % 128 != 0)
    return (not small_tiles(kind, M, K, E, units) and E <= 128 and padded and
            10 * (M // 128 + E) * -(-K // 256) <= 43 * units)


def times_as_wide(kind, M, K, E=0, units=256, own=False):
    """How often rows of K columns are repeated beside each other until small tiles leave them (to the FP8-column kernels that write
    their own rows, where `own`, else to those that do not)."""
    return next(n for n in range(1, 4000) if not small_tiles(kind, M, n * K, E, units) and
                (kind == "mxfp4" or E == 0 or own_rows(kind, M, n * K, E, units) == own))


def aligned_pieces(M, K, E, units=256):
    """Row -> column by tiles of 256 x 256 whose pieces are put together on 16-byte boundaries."""
    return E > 256 and 2 * (-(-M // 256) + E) * -(-K // 256) <= 3 * units
