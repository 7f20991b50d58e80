"""GPU parity of the routed quantizers on both sides of every rule that picks a kernel: a gathered or scattered row is
the oracle's flat row, and bytes that no row owns keep their contents."""
import ctypes

import numpy as np
import pytest
import torch

import paper_2603_02731_amd as mx
from oracle import parallel as par
from paper_2603_02731_amd import binding, synth
from tests.test_gpu_parity import DEV, assert_same, dev, host

pytestmark = pytest.mark.gpu
GUARD = 256


def source(M, K, seed):
    """Activations with a NaN block and a zero row, and the oracle's packed rows plus one zero row at the end."""
    rng = np.random.default_rng(seed)
    x8, s = synth.student_t_fp8(M, K, seed=seed)
    x8, s = x8.numpy(), s.numpy()
    x8[rng.integers(0, M), rng.integers(0, K)] = 0x7F
    x8[rng.integers(0, M)] = 0
    q, sf = par.quant(x8, s)
    zero = np.zeros((1, q.shape[1]), np.uint8), np.zeros((1, sf.shape[1]), np.uint8)
    return rng, x8, s, np.concatenate([q, zero[0]]), np.concatenate([sf, zero[1]])


def outputs(rows, K, layout):
    """(buffer, q, sf, ld_q, ld_sf, views): records on 16-byte boundaries with a gap, or two planes with rows on
    8- and 4-byte boundaries or without gaps (dense: both on 16 bytes where K % 512 == 0); guard bytes around all of it."""
    nq, ns = K // 2, K // 32
    if layout == "records":
        ld_q = ld_sf = (nq + ns + 15) // 16 * 16 + 16
        at_q, at_sf, size = GUARD, GUARD + nq, GUARD + rows * ld_q
    else:
        step = {"planes": 16, "planes8": 8, "planes64": 64, "dense": 0}[layout]
        ld_q, ld_sf = nq + step, ns + step // 2
        at_q, at_sf = GUARD, (GUARD + rows * ld_q + 15) // 16 * 16
        size = at_sf + rows * ld_sf
    buf = torch.full((size + GUARD,), 0xA5, dtype=torch.uint8, device=DEV)
    return buf, buf[at_q:], buf[at_sf:], ld_q, ld_sf, (at_q, at_sf)


def check(buf, at, ld_q, ld_sf, K, rows, wq, wsf):
    """wq / wsf: oracle rows; rows: which output rows they are.  Everything else in buf is still 0xA5."""
    want = np.full(buf.numel(), 0xA5, np.uint8)
    for start, ld, w in ((at[0], ld_q, wq), (at[1], ld_sf, wsf)):
        place = start + rows.astype(np.int64)[:, None] * ld + np.arange(w.shape[1])[None, :]
        want[place] = w
    assert_same(host(buf), want, "routed rows")


@pytest.mark.parametrize("layout", ["records", "planes", "planes8"])
@pytest.mark.parametrize("K,M,fan", [(1920, 37, 3), (2048, 37, 3), (2048, 1023, 2), (2048, 1024, 2), (2176, 1025, 3),
                                     (2176, 9, 1), (5120, 21, 8), (6016, 6, 9), (6016, 1030, 1), (6144, 1024, 1),
                                     (6144, 13, 1), (6144, 13, 2), (6272, 5, 9), (7680, 1024, 1), (7808, 512, 1),
                                     (8192, 512, 1), (8192, 511, 1), (16896, 342, 1), (98304, 2, 2), (98304, 79, 1)])
def test_scatter_kernels(K, M, fan, layout):
    """Small launches and fan-outs of one, by a lane per chunk whatever the row length (98304 elements: of many tiles), and a wave or a
    workgroup per row; fan-outs of 1, 2 and past the eight indices read ahead; scale bytes as 16-byte pieces and as dwords."""
    rng, x8, s, wq, wsf = source(M, K, K + fan)
    M_out = M * fan + 5
    dst = rng.permutation(M_out)[: M * fan].reshape(M, fan).astype(np.int32)
    nowhere = rng.random(dst.shape) < 0.05
    dst[nowhere] = rng.choice(np.array([-1, M_out, 2 ** 31 - 1], np.int32), size=int(nowhere.sum()))
    buf, q, sf, ld_q, ld_sf, at = outputs(M_out, K, layout)
    mx.mxfp4_quant_from_fp8_scatter(dev(x8), dev(s), dev(dst), M_out, q=q, sf=sf, ld_q=ld_q, ld_sf=ld_sf)
    src, _ = np.nonzero(~nowhere)
    check(buf, at, ld_q, ld_sf, K, dst[~nowhere], wq[src], wsf[src])


@pytest.mark.parametrize("layout", ["records", "planes", "dense"])
@pytest.mark.parametrize("K,M,fan", [(1024, 301, 4), (1024, 301, 5), (640, 77, 17),  # destinations held by fours and eights, and past them
                                     (2048, 3072, 2), (2048, 3073, 2), (2176, 2891, 9), (2176, 2892, 9),  # lanes, a wave per row
                                     (6016, 1045, 3), (6016, 1046, 3), (6144, 256, 2), (6144, 257, 2), (6272, 251, 9), (7168, 221, 9),  # a workgroup
                                     (7808, 201, 4), (7808, 202, 4), (98304, 16, 2), (98304, 17, 2)])  # and rows of several segments
def test_scatter_sides_of_the_small_launches(K, M, fan, layout):
    """Both sides of the sizes up to which a lane takes a chunk of long rows, and the kernels above them, which take records and dense
    planes (scale rows on 16 bytes); other planes are the lanes'."""
    test_scatter_kernels(K, M, fan, layout)


@pytest.mark.parametrize("K,M,fan", [(5632, 11916, 4), (5632, 11915, 4), (5632, 15887, 3), (4608, 7282, 8), (4480, 7490, 8)])
def test_scatter_of_many_copies(K, M, fan):
    """Both sides of the size, the row length and the fan-out from which a workgroup takes a row of less than 6144 elements."""
    rng, x8, s, wq, wsf = source(M, K, K + M)
    M_out = M * fan + 3
    dst = rng.permutation(M_out)[: M * fan].reshape(M, fan).astype(np.int32)
    buf, q, sf, ld_q, ld_sf, at = outputs(M_out, K, "records")
    mx.mxfp4_quant_from_fp8_scatter(dev(x8), dev(s), dev(dst), M_out, q=q, sf=sf, ld_q=ld_q, ld_sf=ld_sf)
    want = torch.full_like(buf, 0xA5)
    rows = dev(dst.reshape(-1).astype(np.int64))
    for start, ld, w in ((at[0], ld_q, wq), (at[1], ld_sf, wsf)):
        want.as_strided((M_out, w.shape[1]), (ld, 1), start)[rows] = dev(w[:M]).repeat_interleave(fan, dim=0)
    assert torch.equal(buf, want)


@pytest.mark.parametrize("K,M", [(6144, 2047), (6144, 2048), (6272, 2049), (6144, 2303), (6144, 2304), (6144, 2561)])
def test_scatter_rows_in_runs(K, M):
    """Rows dealt to the XCDs in runs: below and from the number of rows on, with and without rows left over after the last
    round of runs; every row is written once, to all of its destinations."""
    rng, x8, s, wq, wsf = source(M, K, K + M)
    M_out = M * 2 + 3
    dst = rng.permutation(M_out)[: M * 2].reshape(M, 2).astype(np.int32)
    buf, q, sf, ld_q, ld_sf, at = outputs(M_out, K, "records")
    mx.mxfp4_quant_from_fp8_scatter(dev(x8), dev(s), dev(dst), M_out, q=q, sf=sf, ld_q=ld_q, ld_sf=ld_sf)
    src = np.repeat(np.arange(M), 2)
    check(buf, at, ld_q, ld_sf, K, dst.reshape(-1), wq[src], wsf[src])


# ---- gather by owners

GROUPS = 1 << (torch.cuda.get_device_properties(0).multi_processor_count.bit_length() - 1) if torch.cuda.is_available() else 256


def saved(M, K, n):
    """What the launch expects to save, in 10^-15 s."""
    return (139 * n - 158 * M) * K - 124000 * M


def least(M, K):
    """The smallest number of output rows from which M source rows are gathered by owners."""
    enough = (25 if K <= 7680 else 40) * 10 ** 9
    n = ((enough + 124000 * M) // K + 158 * M) // 139
    while saved(M, K, n) < enough:
        n += 1
    assert saved(M, K, n - 1) < enough and n <= 4096 * GROUPS
    return max(n, 2 * M)


def unsampled(n):
    """bool [n]: the places of the index at which no sample is taken (runs of 256, chosen by a hash of their number)."""
    samples = 1 if n >= 256 * GROUPS else 2 if n >= 128 * GROUPS else 4
    eighths = min(8, max(1, 2048 * GROUPS // n))
    run = np.arange(n) // 256
    step, u, wave = run // 64, run // 16 % 4, run % 16
    hashed = (step * 64 + wave) * 0x9E3779B1 % 2 ** 32
    return ((u - (hashed >> 30)) % 4 >= samples) | ((hashed >> 27 & 7) >= eighths)


def index_of(kind, M, n, rng):
    """int32 [n] gather indices into M source rows."""
    idx = (np.arange(n) % M).astype(np.int32)
    rng.shuffle(idx)
    at = np.arange(n)
    if kind == "padded":        # every fifth slot unused, some far outside
        idx[::5] = -1
        idx[7::50] = M
        idx[9::50] = 2 ** 31 - 1
    elif kind == "crowd":       # a quarter of the slots name one row: its owner's rows are dealt out
        idx[rng.random(n) < 0.25] = 5
    elif kind == "sixteenth":   # a crowd in every slot but each sixteenth
        idx[at % 16 != 0] = np.where(rng.random(n) < 0.5, 3, idx)[at % 16 != 0]
    elif kind == "hidden":      # a crowd only where no sample is taken: the list of its owner overflows
        idx[unsampled(n)] = 3
    elif kind == "two hidden":  # the same with rows dealt to that owner as well
        idx[unsampled(n)] = np.where(rng.random(n) < 0.9, 3, -1)[unsampled(n)]
    elif kind == "last slot":   # the last of every eight slots names row 0
        idx[at % 8 == 7] = 0
    elif kind == "one":         # all slots name the last row
        idx[:] = M - 1
    elif kind == "none":
        idx[:] = -(2 ** 31)
    elif kind == "sorted":
        idx.sort()
    elif kind == "quarter":     # only the first quarter of the source is in use
        idx[:] = rng.integers(0, M // 4, n)
    elif kind == "eighth row":  # rows at a stride of a power of two
        idx[:] = rng.integers(0, M // 8, n) * 8
    elif kind == "few":         # fewer rows than workgroups
        idx[:] = rng.integers(0, 100, n)
    elif kind == "power":
        idx[:] = (rng.random(n) ** 6 * M).astype(np.int32)
    return idx


def gathered(rng, x8, s, wq, wsf, idx, K, layout):
    """Gathers into guarded outputs through an index that starts at an odd multiple of 4 bytes; every byte of the
    buffer is compared."""
    n, M = len(idx), x8.shape[0]
    buf, q, sf, ld_q, ld_sf, at = outputs(n, K, layout)
    padded = torch.zeros(n + 1, dtype=torch.int32, device=DEV)
    padded[1:] = dev(idx)
    mx.mxfp4_quant_from_fp8(dev(x8), dev(s), padded[1:], q=q, sf=sf, ld_q=ld_q, ld_sf=ld_sf)
    src = dev(np.where((idx >= 0) & (idx < M), idx, M).astype(np.int64))
    want = torch.full_like(buf, 0xA5)
    for start, ld, w in ((at[0], ld_q, dev(wq)), (at[1], ld_sf, dev(wsf))):
        want.as_strided((n, w.shape[1]), (ld, 1), start).copy_(w[src])
    if not torch.equal(buf, want):
        bad = torch.nonzero(buf != want).view(-1)
        raise AssertionError(f"{bad.numel()} of {buf.numel()} bytes differ, the first at {int(bad[0])} (rows start at {at}, "
                             f"{ld_q} and {ld_sf} bytes apart)")


@pytest.mark.parametrize("layout", ["records", "planes8"])
@pytest.mark.parametrize("K,M,n,kind", [
    (2048, 1024, 19175, "mixed"), (2048, 1023, 21846, "mixed"), (1920, 1024, 32768, "mixed"), (7168, 4200, 8401, "sorted"),
    (7168, 4200, 8399, "sorted"), (2176, 1300, 30001, "padded"), (2048, 1029, 40003, "crowd"), (2048, 1024, 30010, "sixteenth"),
    (7808, 1030, 5003, "padded"), (8192, 1024, 5003, "mixed"), (2048, 2047, 24577, "one")])
def test_gather(K, M, n, kind, layout):
    """Short rows and small maps: one lane per chunk."""
    rng, x8, s, wq, wsf = source(M, K, K + n)
    gathered(rng, x8, s, wq, wsf, index_of(kind, M, n, rng), K, layout)


@pytest.mark.parametrize("layout", ["records", "planes8"])
@pytest.mark.parametrize("K,rows,over,kind", [
    (4096, 4, 0, "mixed"), (4096, 4, -1, "mixed"), (3968, 4, 1000, "mixed"),     # the rule's line, and rows too short for it
    (4096, 4, 0, "hidden"), (4096, 5, 1, "two hidden"), (4224, 5, 2, "hidden"),  # longer lists than there is room for
    (7168, 9, 3, "crowd"), (4224, 4, 0, "sixteenth"), (4096, 6, 1, "last slot"), (4096, 4, 5, "one"), (4096, 4, 2, "none"),
    (6272, 5, 0, "padded"), (7680, 4, 3, "sorted"), (7808, 4, 1, "power"), (8192, 4, 2, "quarter"), (4096, 16, 0, "eighth row"),
    (16896, 4, 3, "few"), (7168, 4, 40001, "mixed")])
def test_gather_by_owners(K, rows, over, kind, layout):
    """Both sides of the rule (`over` output rows above it; a few more source rows than `rows` per workgroup), ends of the
    index that are no whole quad, unused slots, crowds that the sample sees and ones that it does not, sources of which a part
    is used, rows of one and several segments, scale bytes as 16-byte pieces and as dwords."""
    M = rows * GROUPS + (rows > 4) * 7
    n = least(M, K) + over
    rng, x8, s, wq, wsf = source(M, K, K + n)
    gathered(rng, x8, s, wq, wsf, index_of(kind, M, n, rng), K, layout)


@pytest.mark.parametrize("layout", ["records", "planes", "planes64"])
@pytest.mark.parametrize("K,kind", [(6144, "power"), (6272, "power"), (6656, "mixed"), (7168, "power"), (7552, "crowd"), (7680, "power"),
                                    (7808, "mixed")])
def test_gather_by_owners_in_whole_lines(K, kind, layout):
    """Widths on both sides of the ones whose rows leave by whole lines, rows on and off 64-byte segments, workgroups that have
    more than their share of the output rows (a power law) and ones that have not."""
    M = 9 * GROUPS + 7
    rng, x8, s, wq, wsf = source(M, K, K)
    gathered(rng, x8, s, wq, wsf, index_of(kind, M, least(M, K) + 3, rng), K, layout)


@pytest.mark.parametrize("layout", ["records", "planes"])
@pytest.mark.parametrize("K,M,n,kind", [
    (1536, 9000, 150187, "mixed"), (1536, 9000, 150186, "mixed"),                              # the rule's line, 4 copies and more
    (2048, 40000, 131072, "mixed"), (2048, 40000, 131071, "mixed"),                            # the same, fewer copies
    (2048, 40001, 160003, "mixed"), (2048, 5001, 120047, "mixed"), (2048, 5001, 120048, "mixed"), (2048, 65536, 131071, "sorted"),
    (2048, 16391, 131085, "padded"), (2048, 16391, 131085, "crowd"), (2048, 16391, 131085, "none"), (2048, 16391, 131085, "one"),
    (2176, 9001, 120001, "few"), (2176, 9001, 120001, "power"), (2176, 9001, 120001, "eighth row"), (2176, 9001, 120001, "sorted"),
    (6144, 8001, 65537, "padded"), (6272, 8001, 40004, "crowd"), (6272, 8001, 40005, "padded"), (7168, 4099, 65536, "padded"),
    (7168, 4099, 40000, "one"), (7680, 4099, 33003, "power"), (7808, 8192, 33000, "crowd"), (12288, 6001, 22000, "padded"),
    (16896, 2047, 16000, "few"), (98304, 601, 2500, "padded"), (98304, 601, 3100, "crowd")])
def test_gather_by_lists(K, M, n, kind, layout):
    """Both sides of the rule, up to and from 65536 and 262144 entries on, windows that end early, rows by waves (of one and
    several segments) and by workgroups, unused entries, rows with more entries in a window than a list takes, scale bytes as
    16-byte pieces and as dwords."""
    rng, x8, s, wq, wsf = source(M, K, K + n)
    gathered(rng, x8, s, wq, wsf, index_of(kind, M, n, rng), K, layout)


@pytest.mark.parametrize("K,M,n,kind", [(7168, 4099, 65537, "padded"), (7168, 6401, 33003, "crowd"), (8192, 6001, 33001, "mixed"),
                                        (6656, 7001, 36003, "few"), (8192, 9001, 33001, "power"), (7168, 16385, 37450, "one"),
                                        (6272, 7001, 37003, "padded")])
def test_gather_by_lists_into_dense_planes(K, M, n, kind):
    """What a call without outputs gets: rows of five copies and more by workgroups, of fewer by waves, nibbles and scale bytes of a row
    in two places, as 16-byte pieces where K % 512 == 0."""
    rng, x8, s, wq, wsf = source(M, K, K + n)
    assert mx.lib().mxfp4_quant_from_fp8_gather_workspace(M, K, n, 64, K // 2) > 0
    gathered(rng, x8, s, wq, wsf, index_of(kind, M, n, rng), K, "dense")


@pytest.mark.parametrize("K,M,n,kind", [(1536, 33000, 524288, "padded"), (1536, 33000, 524289, "crowd"), (1536, 150000, 1048576, "mixed"),
                                        (1536, 150000, 1048577, "mixed"), (2048, 524000, 1048003, "padded")])
def test_gather_by_lists_of_a_long_index(K, M, n, kind):
    """More entries than lanes hold, more source rows than there are counters, and an index too long for it.  All rows are zero but
    the scale bytes' worth of them: the scale of source row i says which it is."""
    rng = np.random.default_rng(n)
    idx = index_of(kind, M, n, rng)
    x = torch.full((M, K), 0x38, dtype=torch.uint8, device=DEV)  # 1.0
    # blocks of the values 2^(i's digits): the scale byte of tile t is digit t of i in base 128, plus 60
    row = torch.arange(M, device=DEV)
    s = torch.ones(M, K // 128, device=DEV)
    for t in range(3):
        s[:, t] = torch.exp2(((row >> (7 * t)) % 128 - 60).float())
    q, sf = mx.mxfp4_quant_from_fp8(x, s, dev(idx))
    used = torch.from_numpy((idx >= 0) & (idx < M)).to(DEV)
    digits = torch.stack([sf[:, 4 * t].long() - 65 for t in range(3)], 1)  # 1.0 = 4.0 * 2^-2: byte 127 - 2 for a scale of 2^0
    got = digits[:, 0] + (digits[:, 1] << 7) + (digits[:, 2] << 14)
    assert torch.equal(got[used], dev(idx).long()[used])
    assert bool((q[used] == 0x66).all()) and not bool(q[~used].any()) and not bool(sf[~used].any())


def test_gather_in_stale_memory():
    """The memory to work in holds what an earlier call with another index left in it, or any bytes at all; too little of it, or
    none, is the plain call."""
    K, M, n = 2048, 16391, 131085
    rng, x8, s, wq, wsf = source(M, K, 7)
    x, xs = dev(x8), dev(s)
    L = mx.lib()
    q, sf = torch.empty(n, K // 2, dtype=torch.uint8, device=DEV), torch.empty(n, K // 32, dtype=torch.uint8, device=DEV)
    size = L.mxfp4_quant_from_fp8_gather_workspace(M, K, n, q.data_ptr(), K // 2)
    assert size > 0
    work = torch.zeros(size + 64, dtype=torch.uint8, device=DEV)
    wq, wsf = dev(wq), dev(wsf)
    maps = [index_of(k, M, n, rng) for k in ("mixed", "padded", "crowd", "mixed", "one", "mixed")]
    for i, idx in enumerate(maps * 2):
        if i == len(maps):
            work.random_(0, 4)  # small numbers are output rows of the first window
        given = [size, size, size - 1, size, 0, size][i % 6]
        d = dev(idx)
        q.fill_(1)
        sf.fill_(1)
        work[size:] = 0xA5
        assert L.mxfp4_quant_from_fp8_gather(x.data_ptr(), xs.data_ptr(), M, K, d.data_ptr(), n, q.data_ptr(), K // 2, sf.data_ptr(),
                                             K // 32, work.data_ptr() if given else None, given,
                                             torch.cuda.current_stream().cuda_stream) == 0
        src = dev(np.where((idx >= 0) & (idx < M), idx, M).astype(np.int64))
        assert torch.equal(q, wq[src]) and torch.equal(sf, wsf[src]), f"call {i}"
        assert bool((work[size:] == 0xA5).all())


def test_gather_by_lists_under_capture():
    """Replays of a captured gather, with the inputs changed and eager calls between the replays."""
    K, M, n = 2048, 16391, 131085
    rng, x8, s, _, _ = source(M, K, 1)
    x, xs = dev(x8), dev(s)
    idx = dev(index_of("padded", M, n, rng))
    q, sf = mx.mxfp4_quant_from_fp8(x, xs, idx)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        mx.mxfp4_quant_from_fp8(x, xs, idx, q=q, sf=sf)
    for i in range(4):
        y8, ys = synth.student_t_fp8(M, K, seed=20 + i)
        x.copy_(y8)
        xs.copy_(ys)
        idx.copy_(idx.roll(i * 977))
        want = mx.mxfp4_quant_from_fp8(x, xs, idx, stream=torch.cuda.current_stream())  # no memory to work in: by owners
        q.zero_()
        sf.fill_(7)
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(q, want[0]) and torch.equal(sf, want[1]), f"replay {i}"


def hip_runtime():
    """The HIP runtime that PyTorch has loaded."""
    with open("/proc/self/maps") as f:
        return ctypes.CDLL(next(line.split()[-1] for line in f if "libamdhip64" in line))


@pytest.mark.parametrize("by", ["torch", "hip"])
def test_memory_of_a_captured_gather(by, monkeypatch):
    """A graph of PyTorch's has a pool that its memory to work in stays in.  A graph that the program captures by HIP's own calls has
    none: it takes the kernels without, and what the allocator gives to other tensors afterwards is theirs."""
    K, M, n = 2048, 16391, 131085
    rng, x8, s, _, _ = source(M, K, 2)
    x, xs = dev(x8), dev(s)
    idx = dev(index_of("padded", M, n, rng))
    stream, routes = torch.cuda.Stream(), []

    class Recording:
        def __getattr__(self, name):
            routes.append(name)
            return getattr(library, name)

    library, recording = mx.lib(), Recording()
    q, sf = (torch.empty(n, w, dtype=torch.uint8, device=DEV) for w in (K // 2, K // 32))
    size = library.mxfp4_quant_from_fp8_gather_workspace(M, K, n, q.data_ptr(), K // 2)
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        mx.mxfp4_quant_from_fp8(x, xs, idx, q=q, sf=sf)  # its memory is with the allocator now
        stream.synchronize()
        monkeypatch.setattr(binding, "lib", lambda: recording)
        if by == "torch":
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=stream):
                mx.mxfp4_quant_from_fp8(x, xs, idx, q=q, sf=sf)
            replay = graph.replay
        else:
            hip, raw, handle = hip_runtime(), ctypes.c_void_p(), ctypes.c_void_p(stream.cuda_stream)
            assert hip.hipStreamBeginCapture(handle, 1) == 0  # 1: other threads may do as they like
            try:
                mx.mxfp4_quant_from_fp8(x, xs, idx, q=q, sf=sf)
            finally:
                ended = hip.hipStreamEndCapture(handle, ctypes.byref(raw))
            assert ended == 0
            executable = ctypes.c_void_p()
            assert hip.hipGraphInstantiate(ctypes.byref(executable), raw, None, None, ctypes.c_size_t(0)) == 0

            def replay():
                assert hip.hipGraphLaunch(executable, handle) == 0
        monkeypatch.undo()
        assert ("mxfp4_quant_from_fp8_gather" in routes) == (by == "torch") and ("mxfp4_quant_from_fp8" in routes) == (by == "hip")
        others = [torch.full((size,), 0x5A, dtype=torch.uint8, device=DEV) for _ in range(4)]
        for i in range(3):
            idx.copy_(idx.roll(i * 977))
            want = mx.mxfp4_quant_from_fp8(x, xs, idx)
            q.fill_(1)
            sf.fill_(7)
            replay()
            stream.synchronize()
            assert torch.equal(q, want[0]) and torch.equal(sf, want[1]), f"replay {i}"
            assert all(bool((t == 0x5A).all()) for t in others), f"replay {i}: another tensor was written to"
        if by == "hip":
            assert hip.hipGraphExecDestroy(executable) == 0 and hip.hipGraphDestroy(raw) == 0


def test_gather_where_there_is_no_memory_to_work_in():
    """An allocator at its limit, which frees what it holds before it gives up, is asked once, and the call is done without."""
    K, M, n = 2048, 16391, 131085
    rng, x8, s, _, _ = source(M, K, 3)
    x, xs, idx = dev(x8), dev(s), dev(index_of("padded", M, n, rng))
    want = mx.mxfp4_quant_from_fp8(x, xs, idx)
    q, sf = (torch.zeros(n, w, dtype=torch.uint8, device=DEV) for w in (K // 2, K // 32))
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    size = mx.lib().mxfp4_quant_from_fp8_gather_workspace(M, K, n, q.data_ptr(), K // 2)
    full = []
    torch.cuda.set_per_process_memory_fraction(torch.cuda.memory_reserved() / torch.cuda.get_device_properties(0).total_memory)
    try:
        with pytest.raises(torch.OutOfMemoryError):
            while len(full) < 10000:
                full.append(torch.empty(size, dtype=torch.uint8, device=DEV))
        before = torch.cuda.memory_stats()["num_ooms"]
        got = mx.mxfp4_quant_from_fp8(x, xs, idx, q=q, sf=sf)
        asked = torch.cuda.memory_stats()["num_ooms"] - before
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
    assert got[0] is q and torch.equal(q, want[0]) and torch.equal(sf, want[1])
    assert asked == 1


def test_gather_sides_of_the_row_counts():
    """Fewer rows than four per workgroup, and fewer than two output rows per source row, on the lane-wise side."""
    for M, n in ((4 * GROUPS - 1, least(4 * GROUPS, 7168) + 100), (32 * GROUPS, 64 * GROUPS - 1), (32 * GROUPS, 64 * GROUPS)):
        rng, x8, s, wq, wsf = source(M, 7168, n)
        gathered(rng, x8, s, wq, wsf, index_of("padded", M, n, rng), 7168, "records")


def test_gather_takes_no_map_to_one_workgroup():
    """Maps that name one row in the slots of a fixed sample, or use a part of the source: one workgroup doing their work
    alone takes 5 to 20 times as long as the workgroups together."""
    M, K, n = 32 * GROUPS, 7168, 256 * GROUPS
    x = torch.randint(0, 120, (M, K), dtype=torch.uint8, device=DEV)
    s = torch.ones(M, K // 128, device=DEV)
    q, sf = torch.empty(n, K // 2, dtype=torch.uint8, device=DEV), torch.empty(n, K // 32, dtype=torch.uint8, device=DEV)

    def us(idx):
        idx = dev(idx)
        times = []
        for _ in range(5):
            e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            mx.mxfp4_quant_from_fp8(x, s, idx, q=q, sf=sf)
            e[0].record()
            for _ in range(5):
                mx.mxfp4_quant_from_fp8(x, s, idx, q=q, sf=sf)
            e[1].record()
            torch.cuda.synchronize()
            times.append(e[0].elapsed_time(e[1]) * 200)
        return min(times)

    rng = np.random.default_rng(1)
    even = us(index_of("mixed", M, n, rng))
    every = np.arange(n)
    maps = {k: index_of(k, M, n, rng) for k in ("crowd", "sixteenth", "last slot", "one", "none", "quarter", "eighth row", "few")}
    for slots in (16, 32, 64):
        maps[f"last of {slots}"] = np.where(every % slots == slots - 1, 0, index_of("mixed", M, n, rng)).astype(np.int32)
        maps[f"first of {slots}"] = np.where(every % slots != 0, 0, index_of("mixed", M, n, rng)).astype(np.int32)
    slow = {k: round(t) for k, t in ((k, us(v)) for k, v in maps.items()) if t > 2.5 * even}
    assert not slow, f"{slow} us against {even:.0f} for an even map"


def test_gather_by_owners_under_capture():
    """Replays of a captured gather, with the inputs changed and eager work between the replays."""
    K, M = 4096, 4 * GROUPS
    n = least(M, K)
    rng, x8, s, _, _ = source(M, K, 1)
    x, xs = dev(x8), dev(s)
    idx = dev(index_of("padded", M, n, rng))
    q, sf = mx.mxfp4_quant_from_fp8(x, xs, idx)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        mx.mxfp4_quant_from_fp8(x, xs, idx, q=q, sf=sf)
    for i in range(4):
        y8, ys = synth.student_t_fp8(M, K, seed=10 + i)
        x.copy_(y8)
        xs.copy_(ys)
        idx.copy_(idx.roll(i * 977))
        want = mx.mxfp4_quant_from_fp8(x, xs, idx)
        q.zero_()
        sf.fill_(7)
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(q, want[0]) and torch.equal(sf, want[1]), f"replay {i}"
