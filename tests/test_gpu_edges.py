"""GPU parity at the sizes where a kernel or a dispatch rule changes over: the ends of a range on either side, through the
C ABI, against the CPU oracle or against calls that the oracle pins elsewhere.  Everything here is bit-exact."""
import numpy as np
import pytest
import torch

from oracle import gq_oracle as O

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2305_18627_amd as gq
    DEV = torch.device("cuda:0")
else:                                                  # collected but never run without a GPU
    gq = None
    DEV = None


def host(t):
    return t.detach().cpu().numpy()


# Exponential sums are formed in binary32 up to K 2^(s-1) = 2^24 where the kernel knows K (4, 8, 16, 32), else in integers.
@pytest.mark.parametrize("K,s", [(4, 22), (4, 23), (4, 24), (8, 21), (8, 22), (8, 23), (32, 20), (32, 21), (5, 21), (64, 25)])
def test_fused_exponential_sums_at_the_float_limit(K, s):
    d = 1031
    g = torch.Generator().manual_seed(K * 100 + s)
    xs = [torch.randn(d, generator=g) for _ in range(K)]
    for w, x in enumerate(xs):
        x.clamp_(-1.0, 1.0)
        x[:200] = 1.0                                  # every worker at the top level: the sum is K 2^(s-1)
        x[200:400] = -1.0
        x[400:600] = 1.0 if w else -2.0 ** -(s - 1)    # one unit below (K - 1) 2^(s-1): odd sums at the limit
    nf = np.float32(1.0)
    p = gq.make_params(gq.GQ_EXP, s, gq.GQ_PACK_I8, gq.GQ_AGG_I32, seed=99)
    agg = torch.zeros(d, dtype=torch.int32, device=DEV)
    lv = [torch.zeros(d, dtype=torch.uint8, device=DEV) for _ in range(K)]
    gq.fused_quantize_aggregate([x.to(DEV) for x in xs], torch.ones(1, device=DEV), p, 0, agg)
    want = O.quantize_aggregate([x.numpy() for x in xs], nf, O.EXP, s, 99, 0)
    assert np.array_equal(host(agg).astype(np.int64), want)
    assert int(want[0]) == K << (s - 1) and int(want[200]) == -(K << (s - 1))
    agg.zero_()
    gq.fused_quantize_aggregate([x.to(DEV) for x in xs], torch.ones(1, device=DEV), p, 0, agg, None, lv)
    assert np.array_equal(host(agg).astype(np.int64), want)
    assert np.array_equal(host(lv[-1]).view(np.int8), O.quantize(xs[-1].numpy(), nf, O.EXP, s, 99, K - 1, 0))


def lists_of(lv, d, p, cap=None, starts=True):
    """gq_compact's list of the int8 codes lv: (indices, values, count, table of tile starts), guard entries behind the list."""
    cap = d if cap is None else cap
    idx = torch.full((cap + 8,), -1, dtype=torch.int32, device=DEV)
    val = torch.full((cap + 8,), 0x5A, dtype=torch.int8, device=DEV)
    cnt = torch.full((1,), -1, dtype=torch.int64, device=DEV)
    tab = torch.full((gq.tile_starts_len(d),), -1, dtype=torch.int32, device=DEV)
    gq.compact(lv, d, p, idx[:cap], val[:cap], cnt, tile_starts_out=tab if starts else None)
    return idx, val, cnt, tab


def check_lists(q, got, cap=None):
    """A sender's output against the construction: numpy's nonzero and its running counts at the tiles."""
    idx, val, cnt, tab = (host(t) for t in got)
    at = np.flatnonzero(q)
    assert int(cnt[0]) == at.size
    n = at.size if cap is None else min(at.size, cap)
    assert np.array_equal(idx[:n].view(np.uint32), at[:n].astype(np.uint32)) and np.array_equal(val[:n], q[at[:n]])
    assert (idx[n:] == -1).all() and (val[n:] == 0x5A).all()
    edges = np.minimum(np.arange(tab.size, dtype=np.int64) * 4096, q.size)
    assert np.array_equal(tab.view(np.uint32), np.searchsorted(at, edges).astype(np.uint32))


# A sender's workgroup takes a span of 16384 codes (32768 from 2^25 codes on); up to 4096 entries of a span are staged whole,
# more go row by row; spans are grouped by 128 (64).
@pytest.mark.parametrize("d", [16_383, 16_384, 16_385, 32_769, 128 * 16_384, 128 * 16_384 + 1, 129 * 16_384 + 5, 70_001])
@pytest.mark.parametrize("fill", ["none", "one", "4096", "4097", "last", "all"])
def test_compact_at_span_and_staging_edges(d, fill):
    q = np.zeros(d, np.int8)
    if fill == "one":
        q[d // 2] = -128
    elif fill in ("4096", "4097"):                     # so many non-zeros in every span
        per = np.zeros(16_384, np.int8)
        per[np.random.default_rng(d).permutation(16_384)[:int(fill)]] = 5
        q = np.resize(per, d)
    elif fill == "last":
        q[-1] = 127
    elif fill == "all":
        q = (np.arange(d) % 127 + 1).astype(np.int8)
    p = gq.make_params(gq.GQ_LINEAR, 127, gq.GQ_PACK_I8, gq.GQ_AGG_I32, seed=1)
    lv = torch.from_numpy(q).view(torch.uint8).to(DEV)
    check_lists(q, lists_of(lv, d, p))
    if fill in ("4097", "all"):                        # a list that ends inside a span, and one of no entries at all
        check_lists(q, lists_of(lv, d, p, cap=16_384 + 77), cap=16_384 + 77)
        check_lists(q, lists_of(lv, d, p, cap=0), cap=0)


@pytest.mark.parametrize("d", [(1 << 25) - 1, (1 << 25), (1 << 25) + 32_769])
@pytest.mark.parametrize("density", [0.001, 0.3])
def test_compact_either_side_of_the_long_spans(d, density):
    g = torch.Generator(device=DEV).manual_seed(d)
    lv = torch.randint(1, 256, (d,), generator=g, device=DEV, dtype=torch.int16).to(torch.uint8)
    lv[torch.rand(d, generator=g, device=DEV) >= density] = 0
    p = gq.make_params(gq.GQ_LINEAR, 127, gq.GQ_PACK_I8, gq.GQ_AGG_I32, seed=1)
    check_lists(host(lv).view(np.int8), lists_of(lv, d, p))


# The list straight from the gradient: one level (s = 1, where the test for a non-zero code has its own case at the norm),
# densities either side of the staging limit, long spans from 2^27 coordinates on.
@pytest.mark.parametrize("scheme,s", [("linear", 1), ("exp", 1), ("linear", 127), ("exp", 16)])
@pytest.mark.parametrize("scale", [1e-6, 0.02, 0.25, 1.0])
@pytest.mark.parametrize("rng_bits", [32, 16])
@pytest.mark.parametrize("d", [16_385, 70_003])
def test_quantize_compact_at_span_and_density_edges(scheme, s, scale, rng_bits, d):
    g = torch.Generator(device=DEV).manual_seed(d + s)
    x = torch.randn(d, generator=g, device=DEV).clamp_(-1.0, 1.0).mul_(scale)
    x[::1001] = 1.0
    x[7::1001] = -float(np.nextafter(np.float32(1.0), np.float32(0.0)))
    x[5::4001] = float("nan")
    x[6::4001] = float("-inf")
    norm = torch.ones(1, device=DEV)
    p = gq.make_params(0 if scheme == "linear" else 1, s, gq.GQ_PACK_I8, gq.GQ_AGG_I32, seed=3, rng_bits=rng_bits)
    check_quantize_compact_equals_two_calls(x, norm, p)
    want = O.quantize(host(x), np.float32(1.0), 0 if scheme == "linear" else 1, s, 3, 9, 16, rng_bits)
    lv = torch.zeros(d, dtype=torch.uint8, device=DEV)
    gq.quantize(x, norm, p, 9, 16, lv)
    assert np.array_equal(host(lv).view(np.int8), want)


def check_quantize_compact_equals_two_calls(x, norm, p):
    d = x.numel()
    lv = torch.empty(d, dtype=torch.uint8, device=DEV)
    gq.quantize(x, norm, p, 9, 16, lv)
    want = lists_of(lv, d, p)
    idx, val = torch.full_like(want[0], -1), torch.full_like(want[1], 0x5A)
    cnt, tab = torch.full_like(want[2], -1), torch.full_like(want[3], -1)
    gq.quantize_compact(x, norm, p, 9, 16, idx[:d], val[:d], cnt, tile_starts_out=tab)
    for a, b in zip((idx, val, cnt, tab), want):
        assert torch.equal(a, b)


@pytest.mark.parametrize("scale", [0.002, 0.3])
@pytest.mark.parametrize("d", [(1 << 27) - 4, (1 << 27) + 32_771])
def test_quantize_compact_either_side_of_the_long_spans(d, scale):
    x = torch.randn(d, generator=torch.Generator(device=DEV).manual_seed(5), device=DEV).mul_(scale).clamp_(-1.0, 1.0)
    p = gq.make_params(gq.GQ_LINEAR, 7, gq.GQ_PACK_I8, gq.GQ_AGG_I32, seed=3)
    check_quantize_compact_equals_two_calls(x, torch.ones(1, device=DEV), p)


# From 20 groups of 64 words on, the counts of the four groups before a span's own are read span by span.  At these sizes
# gq_compact has spans of 32768 codes, 64 to a group, and gq_quantize_compact spans of 16384, 128 to a group.  Whole spans one
# short of the line and a last span of a single code on it: the first two for gq_compact (1279 and 1280 spans), the next two for
# gq_quantize_compact (2559 and 2560); beyond it a ragged group for both.  The first groups have fewer than four before them.
@pytest.mark.parametrize("scale", [0.002, 0.3])
@pytest.mark.parametrize("d", [1279 * 32_768, 1279 * 32_768 + 1, 2559 * 16_384, 2559 * 16_384 + 1, 1300 * 32_768 + 77])
def test_senders_either_side_of_the_window_of_groups(d, scale):
    x = torch.randn(d, generator=torch.Generator(device=DEV).manual_seed(6), device=DEV).mul_(scale).clamp_(-1.0, 1.0)
    norm = torch.ones(1, device=DEV)
    p = gq.make_params(gq.GQ_LINEAR, 7, gq.GQ_PACK_I8, gq.GQ_AGG_I32, seed=3)
    check_quantize_compact_equals_two_calls(x, norm, p)
    lv = torch.empty(d, dtype=torch.uint8, device=DEV)
    gq.quantize(x, norm, p, 9, 16, lv)
    check_lists(host(lv).view(np.int8), lists_of(lv, d, p))


# The receiver takes a segment of no more than two entries per lane both at once, a longer one four in a row per lane; lists may begin at
# any element of a buffer (indices 4-byte aligned, values anywhere) and end at the last entry of their capacity.
@pytest.mark.parametrize("K", [1, 2, 5, 8, 16, 33, 64])
@pytest.mark.parametrize("n", [1, 3, 7, 8, 9, 15, 16, 17, 18, 19, 31, 33, 63, 64, 65, 127, 129, 511, 513, 514, 515, 1023, 1024, 1025, 1026, 2050, 8192])
@pytest.mark.parametrize("tables", [True, False])
def test_sparse_aggregate_segment_lengths_and_offsets(K, n, tables):
    d = 2 * 8192 + 5
    rng = np.random.default_rng(n * 100 + K)
    p = gq.make_params(gq.GQ_LINEAR, 127, gq.GQ_PACK_I8, gq.GQ_AGG_I32, seed=1)
    want = np.zeros(d, np.int64)
    idx, val, cnt, tab = [], [], [], []
    for w in range(K):
        m = max(1, n - w % 4)                          # per worker and span, ragged between workers
        at = np.concatenate([np.sort(rng.choice(8192, m, replace=False)), 8192 + np.sort(rng.choice(8192, m, replace=False)), [d - 1]])
        q = rng.integers(1, 128, at.size) * rng.choice([-1, 1], at.size)
        want[at] += q
        off = w % 3                                    # the list ends with its buffer and begins `off` elements in
        bi = torch.zeros(off + at.size, dtype=torch.int32, device=DEV)
        bv = torch.zeros(off + at.size, dtype=torch.int8, device=DEV)
        bi[off:] = torch.from_numpy(at.astype(np.int32)).to(DEV)
        bv[off:] = torch.from_numpy(q.astype(np.int8)).to(DEV)
        idx.append(bi[off:]); val.append(bv[off:])
        cnt.append(torch.tensor([at.size], dtype=torch.int64, device=DEV))
        tab.append(torch.from_numpy(np.searchsorted(at, np.minimum(np.arange(gq.tile_starts_len(d)) * 4096, d)).astype(np.int32)).to(DEV))
    agg = torch.full((d,), 77, dtype=torch.int32, device=DEV)
    gq.sparse_aggregate(idx, val, cnt, d, p, agg, tile_starts=tab if tables else None)
    assert np.array_equal(host(agg).astype(np.int64), want)


# The tree reductions take workgroups of 1024 coordinates without guards and batches of up to eight workers without checks.
@pytest.mark.parametrize("d", [1023, 1024, 1025, 2047, 2048, 3 * 1024 + 3])
@pytest.mark.parametrize("K", [1, 2, 3, 7, 8, 9, 16, 17, 40, 64])
@pytest.mark.parametrize("kind,s", [("exp", 8), ("exp", 16), ("exp", 17), ("avg8", 127), ("avg4", 7)])
def test_tree_reductions_at_workgroup_edges(kind, s, K, d):
    rng = np.random.default_rng(K * 7 + d)
    qs = [rng.integers(-s, s + 1, d).astype(np.int8) for _ in range(K)]
    pack = gq.GQ_PACK_I4 if kind == "avg4" else gq.GQ_PACK_I8
    p = gq.make_params(gq.GQ_EXP if kind == "exp" else gq.GQ_LINEAR, s, pack, gq.GQ_AGG_I32, seed=21)
    lvs = [torch.from_numpy(O.pack(q, pack)[0]).to(DEV) for q in qs]
    red = torch.full((gq.levels_nbytes(d, pack) + 8,), 0xAB, dtype=torch.uint8, device=DEV)
    if kind == "exp":
        gq.exp_reduce(lvs, d, p, 64, None, red)
        want = O.exp_tree_reduce(qs, s, 21, 64)
    else:
        gq.avg_reduce(lvs, d, p, 64, None, red)
        want = O.avg_tree_reduce(qs, 21, 64)
    want = O.pack(np.asarray(want).astype(np.int8), pack)[0]
    assert np.array_equal(host(red)[:want.size], want) and (host(red)[want.size:] == 0xAB).all()


# Packed two's complement nibbles are summed without a table below 16 workers (byte sums on the linear grid, a byte look-up on the
# exponential one) and through a table from there; every nibble value, also -8, in whole workgroups of 1024 and in the ragged rest.
@pytest.mark.parametrize("K", [1, 2, 4, 7, 8, 15, 16, 17, 24, 31, 32, 33, 63, 64])
@pytest.mark.parametrize("scheme,lo", [("linear", -8), ("exp", -8)])
@pytest.mark.parametrize("agg", [0, 1])
def test_int_aggregate_every_nibble_value(K, scheme, lo, agg):
    d = 2 * 1024 + 7
    rng = np.random.default_rng(K)
    qs = [rng.integers(lo, 8, d).astype(np.int64) for _ in range(K)]
    for w, q in enumerate(qs):
        q[:16] = np.arange(-8, 8)                      # all workers alike: the extreme sums
        q[16:32] = -8
        q[1024:1040] = 7
    values = [np.sign(q) * ((1 << np.abs(q)) >> 1) if scheme == "exp" else q for q in qs]
    want = np.sum(values, axis=0)
    lvs = []
    for q in qs:
        n = np.concatenate([q & 15, [0]]).astype(np.uint8)
        lvs.append(torch.from_numpy(n[0::2] | (n[1::2] << 4)).to(DEV))
    p = gq.make_params(0 if scheme == "linear" else 1, 7, gq.GQ_PACK_I4, agg, seed=0)
    out = torch.full((d + 8,), 77, dtype=torch.int16 if agg else torch.int32, device=DEV)
    gq.int_aggregate(lvs, None, d, p, out)
    assert np.array_equal(host(out)[:d].astype(np.int64), want) and (host(out)[d:] == 77).all()


# Long launches bound the workgroups per compute unit by extra LDS (packed sums from 10e6 coordinates on, the average from 25e6, the
# fused call from 40e6, the quantiser from 50e6): the same outputs as the same work in short pieces, which are not bounded, in
# every format and worker count that has a bound of its own.
PIECE = 6_000_000


@pytest.mark.parametrize("K", [1, 4, 8, 16])
@pytest.mark.parametrize("pack,scheme", [(1, "linear"), (1, "exp"), (3, "linear")])
@pytest.mark.parametrize("agg", [0, 1])
def test_packed_sum_long_launch_equals_pieces(K, pack, scheme, agg):
    d = 10_000_001
    g = torch.Generator(device=DEV).manual_seed(8)
    lvs = [torch.randint(0, 256, ((d + 1) // 2 + 16,), generator=g, device=DEV, dtype=torch.int16).to(torch.uint8) for _ in range(K)]
    sps = [torch.randint(-2**31, 2**31 - 1, ((d + 31) // 32,), generator=g, device=DEV, dtype=torch.int64).to(torch.int32) for _ in range(K)] if pack == 3 else None
    p = gq.make_params(0 if scheme == "linear" else 1, 7, pack, agg, seed=3)
    a = torch.full((d,), 77, dtype=torch.int16 if agg else torch.int32, device=DEV)
    gq.int_aggregate(lvs, sps, d, p, a)
    for lo in range(0, d, PIECE):
        n = min(PIECE, d - lo)
        a1 = torch.empty(n, dtype=a.dtype, device=DEV)
        gq.int_aggregate([v[lo // 2:] for v in lvs], [v[lo // 32:] for v in sps] if sps else None, n, p, a1)
        assert torch.equal(a[lo:lo + n], a1)


@pytest.mark.parametrize("K", [4, 8])
@pytest.mark.parametrize("scheme,s,agg,mean", [("linear", 127, 0, True), ("linear", 7, 1, False), ("exp", 7, 1, True), ("exp", 16, 0, False)])
def test_fused_long_launch_equals_pieces(K, scheme, s, agg, mean):
    d = 40_000_003
    g = torch.Generator(device=DEV).manual_seed(8)
    xs = [torch.randn(d, generator=g, device=DEV).clamp_(-1.0, 1.0) for _ in range(K)]
    norm = torch.ones(1, device=DEV)
    p = gq.make_params(0 if scheme == "linear" else 1, s, gq.GQ_PACK_I8, agg, seed=3)
    typ = torch.int16 if agg else torch.int32
    a, m = torch.full((d,), 77, dtype=typ, device=DEV), torch.full((d,), 7.0, device=DEV) if mean else None
    gq.fused_quantize_aggregate(xs, norm, p, 0, a, m)
    for lo in range(0, d, PIECE):
        n = min(PIECE, d - lo)
        a1, m1 = torch.empty(n, dtype=typ, device=DEV), torch.empty(n, device=DEV) if mean else None
        gq.fused_quantize_aggregate([x[lo:lo + n] for x in xs], norm, p, lo, a1, m1)
        assert torch.equal(a[lo:lo + n], a1) and (not mean or torch.equal(m[lo:lo + n], m1))


# Up to 2^22 coordinates (with the codes stored up to 2^23 loads) the fused call and the quantiser have kernels of their own: either
# side of the lines the same outputs as in pieces that lie on the short side, in every worker count with a kernel of its own and
# where sums pass 2^24 (exponential, s = 22 to 24), and with the windows forced on, which keeps the other kernel.
@pytest.mark.parametrize("K", [1, 3, 4, 8, 16, 32, 61])
@pytest.mark.parametrize("scheme,s", [("linear", 127), ("exp", 16), ("exp", 24)])
@pytest.mark.parametrize("rng_bits", [32, 16])
@pytest.mark.parametrize("d", [(1 << 22) - 1, 1 << 22, (1 << 22) + 5])
def test_fused_either_side_of_the_short_launches(K, scheme, s, rng_bits, d):
    g = torch.Generator(device=DEV).manual_seed(9)
    pool = torch.randn(d + 64 * 4, generator=g, device=DEV).clamp_(-1.0, 1.0)
    xs = [pool[4 * w:4 * w + d] for w in range(K)]           # 16-byte aligned, every worker another vector
    norm = torch.ones(1, device=DEV)
    sch = 0 if scheme == "linear" else 1
    p = gq.make_params(sch, s, gq.GQ_PACK_I8, gq.GQ_AGG_I32, seed=3, rng_bits=rng_bits)
    on = gq.make_params(sch, s, gq.GQ_PACK_I8, gq.GQ_AGG_I32, seed=3, rng_bits=rng_bits, flags=gq.GQ_FLAG_WRITE_WINDOWS_ON)
    a, b, m = (torch.full((d,), 77, dtype=t, device=DEV) for t in (torch.int32, torch.int32, torch.float32))
    gq.fused_quantize_aggregate(xs, norm, p, 8, a, m)
    gq.fused_quantize_aggregate(xs, norm, on, 8, b)
    assert torch.equal(a, b)
    for lo in range(0, d, 1_000_008):
        n = min(1_000_008, d - lo)
        a1, m1 = torch.empty(n, dtype=torch.int32, device=DEV), torch.empty(n, device=DEV)
        gq.fused_quantize_aggregate([x[lo:lo + n] for x in xs], norm, p, 8 + lo, a1, m1)
        assert torch.equal(a[lo:lo + n], a1) and torch.equal(m[lo:lo + n], m1)


@pytest.mark.parametrize("K,d", [(2, (1 << 22) + 1), (2, 1 << 22), (8, 1 << 20), (8, (1 << 20) + 1), (3, 100_003)])
@pytest.mark.parametrize("pack", [0, 1, 2, 3])
@pytest.mark.parametrize("scheme", ["linear", "exp"])
@pytest.mark.parametrize("rng_bits", [32, 16])
def test_codes_either_side_of_the_short_launches(K, d, pack, scheme, rng_bits):
    g = torch.Generator(device=DEV).manual_seed(10)
    xs = [torch.randn(d, generator=g, device=DEV).clamp_(-1.0, 1.0) for _ in range(K)]
    norm = torch.ones(1, device=DEV)
    p = gq.make_params(0 if scheme == "linear" else 1, 7, pack, gq.GQ_AGG_I32, seed=3, rng_bits=rng_bits)
    planes = pack >= 2

    def buffers(n):
        return (torch.full((gq.levels_nbytes(n, pack) + 8,), 0xAB, dtype=torch.uint8, device=DEV),
                torch.full(((n + 31) // 32 + 1,), -1, dtype=torch.int32, device=DEV) if planes else None)

    codes = [buffers(d) for _ in xs]
    a = torch.full((d,), 77, dtype=torch.int32, device=DEV)
    gq.fused_quantize_aggregate(xs, norm, p, 8, a, None, [c[0] for c in codes], [c[1] for c in codes] if planes else None)
    a2 = torch.empty_like(a)
    gq.fused_quantize_aggregate(xs, norm, p, 8, a2)
    assert torch.equal(a, a2)
    for w, x in enumerate(xs):
        lv, sp = buffers(d)
        gq.quantize(x, norm, p, w, 8, lv, sp)
        assert torch.equal(lv, codes[w][0]) and (not planes or torch.equal(sp, codes[w][1]))
        for lo in range(0, d, 1_000_000):                    # a multiple of 32: planes and nibbles begin with their words
            n = min(1_000_000, d - lo)
            lv1, sp1 = buffers(n)
            gq.quantize(x[lo:lo + n], norm, p, w, 8 + lo, lv1, sp1)
            nb, at = gq.levels_nbytes(n, pack), lo if pack in (0, 2) else lo // 2
            assert torch.equal(lv[at:at + nb], lv1[:nb]) and (lv1[nb:] == 0xAB).all()
            if planes:
                assert torch.equal(sp[lo // 32:lo // 32 + (n + 31) // 32], sp1[:-1]) and int(sp1[-1]) == -1


@pytest.mark.parametrize("pack", [0, 1, 2, 3])
@pytest.mark.parametrize("scheme,s", [("linear", 7), ("exp", 7)])
@pytest.mark.parametrize("rng_bits", [32, 16])
def test_quantize_long_launch_equals_pieces(pack, scheme, s, rng_bits):
    d = 50_000_003
    x = torch.randn(d, generator=torch.Generator(device=DEV).manual_seed(8), device=DEV).clamp_(-1.0, 1.0)
    norm = torch.ones(1, device=DEV)
    p = gq.make_params(0 if scheme == "linear" else 1, s, pack, gq.GQ_AGG_I32, seed=3, rng_bits=rng_bits)
    planes = pack >= 2
    lv = torch.full((gq.levels_nbytes(d, pack),), 0xAB, dtype=torch.uint8, device=DEV)
    sp = torch.full(((d + 31) // 32,), -1, dtype=torch.int32, device=DEV) if planes else None
    gq.quantize(x, norm, p, 2, 0, lv, sp)
    for lo in range(0, d, PIECE):
        n = min(PIECE, d - lo)
        lv1 = torch.empty(gq.levels_nbytes(n, pack), dtype=torch.uint8, device=DEV)
        sp1 = torch.empty((n + 31) // 32, dtype=torch.int32, device=DEV) if planes else None
        gq.quantize(x[lo:lo + n], norm, p, 2, lo, lv1, sp1)
        at = lo if pack in (0, 2) else lo // 2
        assert torch.equal(lv[at:at + lv1.numel()], lv1)
        if planes:
            assert torch.equal(sp[lo // 32:lo // 32 + sp1.numel()], sp1)


@pytest.mark.parametrize("K", [8, 16, 32])
@pytest.mark.parametrize("pack", [0, 1])
def test_average_long_launch_equals_pieces(K, pack):
    d = 25_000_003
    g = torch.Generator(device=DEV).manual_seed(8)
    per = 1 if pack == 0 else 2
    codes = [torch.randint(-7, 8, (d // per + 16,), generator=g, device=DEV, dtype=torch.int16).to(torch.uint8) for _ in range(K)]
    p = gq.make_params(gq.GQ_LINEAR, 7, pack, gq.GQ_AGG_I32, seed=3)
    norm = torch.ones(1, device=DEV)
    red, mean = torch.full((gq.levels_nbytes(d, pack),), 0xAB, dtype=torch.uint8, device=DEV), torch.full((d,), 7.0, device=DEV)
    gq.avg_reduce(codes, d, p, 0, norm, red, mean)
    for lo in range(0, d, PIECE):
        n = min(PIECE, d - lo)
        red1, mean1 = torch.empty(gq.levels_nbytes(n, pack), dtype=torch.uint8, device=DEV), torch.empty(n, device=DEV)
        gq.avg_reduce([c[lo // per:] for c in codes], n, p, lo, norm, red1, mean1)
        assert torch.equal(red[lo // per:lo // per + red1.numel()], red1) and torch.equal(mean[lo:lo + n], mean1)


# gq_compact's waits end also where a span that it waits for never comes: in this build every third span, and every third group's
# sum, is published by nobody but the waves that wait for it.  The lists are the library's, bit for bit; grids with group sums
# alone and with a window of groups before the own one, short and long spans, ragged ends.
@pytest.fixture(scope="module")
def mute():
    import ctypes

    from paper_2305_18627_amd import build
    lib = ctypes.CDLL(build.MUTE_LIB)
    real, f = gq.lib().gq_compact, lib.gq_compact
    f.restype, f.argtypes = real.restype, real.argtypes
    return lib


@pytest.mark.parametrize("d", [3 * 16_384 + 5, 40 * 16_384, 130 * 16_384 + 77, 700 * 16_384 + 1, 1300 * 32_768 + 77, 4100 * 32_768 + 4099])
@pytest.mark.parametrize("density", [0.0, 0.001, 0.1, 0.6])
def test_senders_whose_spans_are_mute(mute, d, density):
    import ctypes
    g = torch.Generator(device=DEV).manual_seed(d)
    lv = torch.randint(1, 256, (d,), generator=g, device=DEV, dtype=torch.int16).to(torch.uint8)
    lv[torch.rand(d, generator=g, device=DEV) >= density] = 0
    p = gq.make_params(gq.GQ_LINEAR, 127, gq.GQ_PACK_I8, gq.GQ_AGG_I32, seed=3)
    want = lists_of(lv, d, p)
    ws = torch.full((gq.compact_workspace_bytes(d),), 0xFF, dtype=torch.uint8, device=DEV)
    got = [torch.full_like(want[0], -1), torch.full_like(want[1], 0x5A), torch.full_like(want[2], -1), torch.full_like(want[3], -1)]
    st = mute.gq_compact(lv.data_ptr(), d, ctypes.byref(p), got[0].data_ptr(), got[1].data_ptr(), d, got[2].data_ptr(), got[3].data_ptr(),
                         ws.data_ptr(), ws.numel(), torch.cuda.current_stream().cuda_stream)
    assert st == gq.GQ_OK
    torch.cuda.synchronize()
    for a, b in zip(got, want):
        assert torch.equal(a, b)


# Senders on two streams, each with its own workspace and lists, may share the chip: two of gq_compact, or one of it beside one of
# gq_quantize_compact.
@pytest.mark.parametrize("d", [25_600_003, 50_000_001])
def test_senders_on_two_streams(d):
    norm = torch.ones(1, device=DEV)
    p = gq.make_params(gq.GQ_LINEAR, 7, gq.GQ_PACK_I8, gq.GQ_AGG_I32, seed=3)
    side = [torch.cuda.Stream(), torch.cuda.Stream()]
    work = []
    for k in range(2):
        x = torch.randn(d, generator=torch.Generator(device=DEV).manual_seed(k), device=DEV).mul_(0.02).clamp_(-1.0, 1.0)
        lv = torch.empty(d, dtype=torch.uint8, device=DEV)
        gq.quantize(x, norm, p, 9, 16, lv)
        want = lists_of(lv, d, p)
        got = [torch.full_like(want[0], -1), torch.full_like(want[1], 0x5A), torch.full_like(want[2], -1), torch.full_like(want[3], -1)]
        work.append((x, lv, want, got, torch.empty(gq.compact_workspace_bytes(d), dtype=torch.uint8, device=DEV)))
    torch.cuda.synchronize()
    for turn in range(20):
        for k, ((x, lv, want, got, ws), s) in enumerate(zip(work, side)):
            if turn % 2 or k:
                gq.compact(lv, d, p, got[0][:d], got[1][:d], got[2], ws, stream=s, tile_starts_out=got[3])
            else:
                gq.quantize_compact(x, norm, p, 9, 16, got[0][:d], got[1][:d], got[2], ws, stream=s, tile_starts_out=got[3])
    torch.cuda.synchronize()
    for x, lv, want, got, ws in work:
        for a, b in zip(got, want):
            assert torch.equal(a, b)
