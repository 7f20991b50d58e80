"""GPU parity of the ragged FP8-column conversions where tiles write whole 64-byte segments of the output: splits around the
edges of pieces (16 rows), segments (64), scale groups (128) and tiles (256), outputs and inputs that begin off a segment, half
tiles along k, special scale bytes in the look-back rows, and both sides of the rule that leaves small padded launches to the
kernels that write their own rows.  Tiles of 128 x 128 take the narrow ones among these, so every case is repeated with its columns
beside each other until they do not."""
import numpy as np
import pytest
import torch

import paper_2603_02731_amd as mx
from oracle import ref
from paper_2603_02731_amd import synth
from tests.rules import own_rows, times_as_wide
from tests.test_gpu_parity import DEV, UNITS, assert_same, host

pytestmark = pytest.mark.gpu

SPLITS = {
    "pieces": [1, 15, 16, 17, 0, 31, 2, 241, 255, 257, 271, 272, 273],
    "segments": [63, 64, 65, 191, 192, 193, 319, 320, 321, 64, 448],
    "groups": [127, 128, 129, 383, 384, 385, 256, 511, 512, 513, 0, 769],
    "one": [1023],
    "long last tiles": [449, 455, 500, 511, 330, 505, 480, 496],  # nearly a whole tile behind a whole one
    "short last tiles": [268, 258, 780, 300, 524, 319, 1026],
    "by 16": [16, 272, 48, 528, 304, 1040, 32, 336],      # a total that is a multiple of 16: the small launch keeps its kernels
    "by 16 at length": [16 * n for n in (1, 3, 17, 33, 65, 20, 50, 31)] * 9,  # the same, above that line at K = 2176
    "by 64": [64, 320, 576, 192, 128, 832],               # k-rows of whole segments, of half lines
}


def run(rows, K, requant, q, sf, q_off=0, x_off=0, times=1):
    """The grouped call on the columns of q and sf, `times` beside each other, as an input q_off and an output x_off bytes past a
    256-byte boundary, guards around both outputs."""
    off = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    groups = [-(-r // 128) for r in rows]
    n, ns = times * K * int(off[-1]), times * K * sum(groups)
    src = torch.empty(times * q.size + 256, dtype=torch.uint8, device=DEV)[q_off:q_off + times * q.size].view(len(q), -1)
    src.copy_(torch.from_numpy(q).to(DEV).repeat(1, times))
    x = torch.full((n + 4096,), 0xA5, dtype=torch.uint8, device=DEV)
    s = torch.full((ns + 64,), -7.0, device=DEV)
    mx.mxfp4_row_to_fp8_col_grouped(src, torch.from_numpy(sf).to(DEV).repeat(1, times), torch.from_numpy(off).to(DEV),
                                    x_col=x[x_off:x_off + n], x_col_scale=s[:ns], requant=requant, offsets_host=off.tolist())
    want, want_s = ref.row_to_fp8_col_grouped(q, sf, off, requant=requant)
    got = host(x)
    assert (got[:x_off] == 0xA5).all() and (got[x_off + n:] == 0xA5).all(), "bytes around the output written"
    assert bool((s[ns:] == -7.0).all()), "scales behind the output written"

    def repeated(want, lengths):  # every expert's k-rows, `times`
        ends = np.cumsum([0] + [K * t for t in lengths])
        return np.concatenate([np.tile(want.reshape(-1)[a:b], times) for a, b in zip(ends, ends[1:])])

    assert_same(host(s)[:ns], repeated(want_s, groups), f"group scales K={times * K} requant={requant}")
    assert_same(got[x_off:x_off + n], repeated(want, rows), f"E4M3 bytes K={times * K} requant={requant}")


def above(rows, K, requant, own=False):
    """How often the columns go beside each other so that no small tiles take the rows: see tests/rules.py."""
    return times_as_wide("requant" if requant else "align", sum(rows), K, len(rows), UNITS, own)


@pytest.mark.parametrize("requant", [False, True])
@pytest.mark.parametrize("name", SPLITS)
def test_splits_around_the_edges(name, requant):
    rows = SPLITS[name]
    K = 2176 if name == "by 16 at length" else 384
    q, sf = synth.random_mxfp4(sum(rows), K, seed=len(rows), scale_spread=6)
    for times in {1, above(rows, K, requant)} | ({above(rows, K, requant, own=True)} if name == "by 16" else set()):
        run(rows, K, requant, q.numpy(), sf.numpy(), times=times)


@pytest.mark.parametrize("q_off,x_off", [(0, 16), (4, 0), (12, 48), (0, 64)])
def test_alignment_of_input_and_output(q_off, x_off):
    rows = [300, 128, 64, 513, 7]
    q, sf = synth.random_mxfp4(sum(rows), 256, seed=q_off + x_off, scale_spread=6)
    for requant in (False, True):
        for times in (1, above(rows, 256, requant)):
            run(rows, 256, requant, q.numpy(), sf.numpy(), q_off, x_off, times)


@pytest.mark.parametrize("requant", [False, True])
@pytest.mark.parametrize("center,spread,nan", [(250, 6, 0.0), (3, 4, 0.0), (127, 20, 0.02), (127, 127, 0.002)])
def test_special_scales_in_the_look_back_rows(center, spread, nan, requant):
    """Bytes beyond FP32, NaN, and maxima so small that the encoder's operand would be negative, in some groups only."""
    rows = [777, 130, 515]
    q, sf = synth.random_mxfp4(sum(rows), 384, seed=center, scale_center=127, scale_spread=3)
    q2, sf2 = synth.random_mxfp4(sum(rows), 384, seed=spread, scale_center=center, scale_spread=spread, nan_scale_frac=nan)
    q, sf = q.numpy(), sf.numpy()
    for lo, hi in ((150, 260), (420, 470), (640, 645), (1000, 1300)):  # far halves, near halves, tiles
        q[lo:hi], sf[lo:hi] = q2.numpy()[lo:hi], sf2.numpy()[lo:hi]
    q[300:384] = 0  # a look-back half without a non-zero element
    for times in (1, above(rows, 384, requant)):
        run(rows, 384, requant, q, sf, times=times)


@pytest.mark.parametrize("experts", [64, 65, 256, 257, 1024])
def test_expert_lookup_at_its_sizes(experts):
    rng = np.random.default_rng(experts)
    rows = [int(r) for r in rng.integers(0, 90, experts)]
    rows[experts // 2], rows[-1] = 600, 1
    q, sf = synth.random_mxfp4(sum(rows), 128, seed=experts, scale_spread=4)
    for times in {1, above(rows, 128, False)}:
        run(rows, 128, False, q.numpy(), sf.numpy(), times=times)


@pytest.mark.parametrize("requant", [False, True])
@pytest.mark.parametrize("experts,empty,last", [(65, (), 16), (65, (64,), 0), (100, (62, 63, 64), 528), (100, (0, 99), 0),
                                                (128, (63,), 272), (128, tuple(range(1, 64)), 784), (128, tuple(range(64, 127)), 16)])
def test_small_padded_launches_of_65_to_128_experts(experts, empty, last, requant):
    """The kernels that write their own rows look for one of up to 128 experts in two steps of 64: a total that is a multiple of
    16 and not of 128 and few tiles, experts without rows around the middle, experts of several tiles on both sides of it.  Of about
    256 rows on the average and more: small tiles take fewer."""
    rng = np.random.default_rng(experts + last)
    rows = [16 * int(n) for n in rng.integers(1, 44 * experts // (experts - len(empty)), experts)]
    rows[5], rows[63], rows[64], rows[-1] = 544, 288, 272, last
    if experts > 70:
        rows[70] = 1040
    for e in empty:
        rows[e] = 0
    if sum(rows) % 128 == 0:
        rows[10] += 16
    some = next(e for e, r in enumerate(rows) if r)
    while not any(own_rows("requant" if requant else "align", sum(rows), 128 * n, experts, UNITS) for n in range(1, 40)):
        rows[some] += 128  # between the two lines no whole number of columns fits every total
    assert sum(rows) % 16 == 0 and sum(rows) % 128 != 0 and rows[some] < 8192
    q, sf = synth.random_mxfp4(sum(rows), 128, seed=experts, scale_spread=6)
    run(rows, 128, requant, q.numpy(), sf.numpy(), times=above(rows, 128, requant, own=True))


@pytest.mark.parametrize("experts", [64, 65, 256, 257, 1024])
def test_expert_lookup_at_its_sizes_requantized(experts):
    rng = np.random.default_rng(experts + 1)
    rows = [int(r) for r in rng.integers(0, 70, experts)]
    rows[experts // 2], rows[-1] = 600, 1
    q, sf = synth.random_mxfp4(sum(rows), 128, seed=experts, scale_spread=4)
    for times in {1, above(rows, 128, True)}:
        run(rows, 128, True, q.numpy(), sf.numpy(), times=times)
