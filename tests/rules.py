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


def aligned_pieces(M, K, E, units=256):
    """Row -> column by tiles of 256 x 256 whose pieces are put together on 16-byte boundaries."""
    return E > 256 and 2 * (-(-M // 256) + E) * -(-K // 256) <= 3 * units
