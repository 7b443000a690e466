"""The calls that a user of this library makes, as cases that can be timed and compared.

A case is one pass of a training program over resident gradients (or stored codes, or lists) through the public entry
points, with every buffer allocated beforehand as such a program keeps it.  Kinds:

  step     gq_global_norm -> gq_fused_quantize_aggregate -> gq_dequantize: one synchronisation step of Algorithm 1
  buckets  gq_bucketed_quantize_aggregate: the communication hook's schedule, every bucket under its own norm
  wire     gq_quantize for every worker -> gq_int_aggregate -> gq_dequantize: the encoder and the decoder of a deployment
  receive  gq_int_aggregate -> gq_dequantize on codes that arrived from the workers
  alg2     gq_exp_reduce: Algorithm 2 on the workers' codes
  average  gq_avg_reduce: low-bit linear codes averaged inside every reduce step
  sparse   gq_global_norm ((2,2) norm) -> gq_quantize_compact for every worker -> gq_sparse_aggregate -> gq_dequantize
  lists    gq_compact for every worker -> gq_sparse_aggregate on stored codes

Outputs are whole buffers; integer results depend on nothing but the inputs, so they are compared bit for bit.
"""
import math

import torch

import paper_2305_18627_amd as gq

QUANT_SEED = 0xC0FFEE
NORMS = {"linf": gq.GQ_NORM_LINF, "l2": gq.GQ_NORM_L2, "l2max": gq.GQ_NORM_L2_MAX}
SCHEMES = {"linear": gq.GQ_LINEAR, "exp": gq.GQ_EXP}
PACKS = {"i8": gq.GQ_PACK_I8, "i4": gq.GQ_PACK_I4, "u8s": gq.GQ_PACK_U8_SIGNPLANE, "u4s": gq.GQ_PACK_U4_SIGNPLANE}
AGGS = {"i32": gq.GQ_AGG_I32, "i16": gq.GQ_AGG_I16}
CHUNK = 1 << 24
M32 = 0xFFFFFFFF


def _case(name, kind, d, K, dist, norm, scheme, s, pack, agg, rng_bits=32, codes=False, fused_mean=False, bucket=0):
    return {"name": name, "kind": kind, "d": d, "K": K, "dist": dist, "norm": norm, "scheme": scheme, "s": s, "pack": pack,
            "agg": agg, "rng_bits": rng_bits, "codes": codes, "fused_mean": fused_mean, "bucket": bucket}


def listed():
    return [
        # a small odd gradient (one layer): latency and launches
        _case("step_100k_k4", "step", 100_003, 4, "outliers", "linf", "linear", 127, "i8", "i32"),
        # a small model's whole gradient, L2 norm
        _case("step_1m_k4_l2", "step", 1_048_576, 4, "normal", "l2", "linear", 127, "i8", "i32"),
        # one 25 MB gradient bucket as a data-parallel hook gets it, short draws, mean written by the fused call, odd length
        _case("bucket_6.5m_k8_exp", "step", 6_553_601, 8, "student", "linf", "exp", 7, "i4", "i16", rng_bits=16, fused_mean=True),
        # an image model's gradient, exponential grid, the codes kept beside the sum
        _case("step_25.6m_k8_exp_codes", "step", 25_600_000, 8, "layers", "l2", "exp", 16, "i8", "i32", codes=True),
        # the benchmark's step: 110e6 coordinates, 16 workers, max norm, 127 levels
        _case("step_110m_k16", "step", 110_000_000, 16, "outliers", "linf", "linear", 127, "i8", "i32"),
        # a long gradient cut into buckets of 2^26, each under its own norm, last bucket short
        _case("buckets_1.5b_k8", "buckets", 1_500_000_000, 8, "mixture", "l2", "linear", 15, "u4s", "i32", fused_mean=True, bucket=1 << 26),
        # encode, sum and decode one bucket of 2^26 in 4 bits with sign planes
        _case("wire_67m_k8_u4s", "wire", 1 << 26, 8, "mixture", "l2", "linear", 15, "u4s", "i32"),
        # decode packed 4-bit codes of 32 workers into 16-bit sums
        _case("receive_350m_k32_i4", "receive", 350_000_000, 32, "student", "linf", "exp", 7, "i4", "i16"),
        # Algorithm 2 over 32 workers
        _case("alg2_50m_k32", "alg2", 50_000_003, 32, "student", "linf", "exp", 7, "i8", "i32"),
        # in-step averaging of int8 codes
        _case("average_25.6m_k8", "average", 25_600_001, 8, "normal", "linf", "linear", 127, "i8", "i32"),
        # the sparse branch from gradients to the mean, under the norm that makes the codes sparse
        _case("sparse_110m_k16_l2", "sparse", 110_000_000, 16, "outliers", "l2", "linear", 127, "i8", "i32"),
        # the sparse branch on stored codes of a max norm: one code in six is not zero
        _case("lists_25.6m_k8", "lists", 25_600_003, 8, "outliers", "linf", "linear", 127, "i8", "i32"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "buckets", "wire", "receive", "alg2", "average", "sparse", "lists"])
    K = min(64, _log_int(rng, 1, 64))
    d = _log_int(rng, 20_000, min(600_000_000, 3_000_000_000 // K))
    d += rng.randrange(8)
    dist = rng.choice(["normal", "outliers", "student", "mixture", "layers"])
    norm = rng.choice(["linf", "linf", "l2", "l2max"])
    scheme = rng.choice(["linear", "exp"])
    pack = rng.choice(["i8", "i4", "u8s", "u4s"])
    if kind == "alg2":
        scheme, pack = "exp", "i8"
    elif kind == "average":
        scheme, pack = "linear", rng.choice(["i8", "i4"])
    elif kind == "sparse":
        norm, pack = "l2", "i8"
    elif kind == "lists":
        pack = "i8"
    if scheme == "linear":
        s = {"i8": 127, "i4": 7, "u8s": 255, "u4s": 15}[pack]
    else:
        s = {"i8": rng.choice([7, 8, 16]), "i4": 7, "u8s": 16, "u4s": 15}[pack]
    unit = s if scheme == "linear" else 1 << (s - 1)
    agg = "i16" if K * unit <= 32767 and kind not in ("sparse", "lists") and rng.random() < 0.5 else "i32"
    bucket = 8 * _log_int(rng, max(8, d // 400), max(8, d // 8)) if kind == "buckets" else 0
    return {k: v for k, v in _case("", kind, d, K, dist, norm, scheme, s, pack, agg, rng_bits=rng.choice([32, 32, 16]),
                                   codes=kind == "step" and rng.random() < 0.3, fused_mean=rng.random() < 0.5,
                                   bucket=bucket).items() if k != "name"}


# ---- inputs -------------------------------------------------------------------------------------------------------

def _gradient(out, dist, seed, worker):
    """Overwrite the fp32 vector `out` with worker `worker`'s gradient."""
    g = torch.Generator(device=out.device)
    g.manual_seed(seed * 1_000_003 + worker)
    d = out.numel()
    if dist == "layers":                                  # blocks of their own scale, shared by the workers
        gs = torch.Generator()
        gs.manual_seed(seed * 1_000_003 + 999_983)
        std = torch.pow(10.0, -5.0 + 3.0 * torch.rand(160, generator=gs)).to(out.device)
    for lo in range(0, d, CHUNK):
        v = out[lo:lo + CHUNK]
        n = v.numel()
        if dist == "normal":
            v.normal_(0.0, 1e-3, generator=g)
        elif dist == "outliers":
            v.normal_(0.0, 1e-3, generator=g)
            v.mul_(torch.where(torch.rand(n, generator=g, device=v.device) < 0.01, 100.0, 1.0))
        elif dist == "mixture":
            v.normal_(0.0, 1.0, generator=g)
            v.mul_(torch.where(torch.rand(n, generator=g, device=v.device) < 0.1, 1e-2, 1e-4))
        elif dist == "student":
            z = torch.empty(3, n, device=v.device).normal_(0.0, 1.0, generator=g)
            v.normal_(0.0, 1e-4, generator=g)
            v.div_(z.square_().mean(0).sqrt_())
        else:
            v.normal_(0.0, 1.0, generator=g)
            v.mul_(std[torch.arange(lo, lo + n, device=v.device).mul_(160).div_(d, rounding_mode="floor")])
    return out


def _gradients(case, seed):
    return [_gradient(torch.empty(case["d"], device="cuda"), case["dist"], seed, w) for w in range(case["K"])]


def _unit(case):
    return case["s"] if case["scheme"] == "linear" else 1 << (case["s"] - 1)


def _signed_codes(case, seed, worker):
    """int8 codes of one worker (int16 where they pass 127), rounded at random onto the case's grid under the worker's own max norm."""
    x = _gradient(torch.empty(case["d"], device="cuda"), case["dist"], seed, worker)
    g = torch.Generator(device="cuda")
    g.manual_seed(seed * 1_000_003 + 500_000 + worker)
    scale = _unit(case) / x.abs().max()
    q = torch.empty(case["d"], dtype=torch.int16 if case["s"] > 127 else torch.int8, device="cuda")
    for lo in range(0, case["d"], CHUNK):
        v = x[lo:lo + CHUNK]
        t = v.abs() * scale
        u = torch.rand(v.numel(), generator=g, device="cuda")
        if case["scheme"] == "linear":
            k = torch.floor(t + u).clamp_(max=case["s"])
        else:
            m, e = torch.frexp(t)                          # t = m 2^e, m in [1/2, 1)
            k = torch.where(t < 1.0, (u < t).float(), e.float() + (u < 2.0 * m - 1.0).float()).clamp_(max=case["s"])
        q[lo:lo + CHUNK] = (k * v.sign()).to(q.dtype)
    return q


def _packed(case, q, levels, plane):
    """Write the signed codes q into a level buffer (and a sign plane) in the case's format."""
    d, pack = case["d"], case["pack"]
    for lo in range(0, d, CHUNK):
        v = q[lo:lo + CHUNK].to(torch.int16)
        n = v.numel()
        if plane is not None:
            neg = torch.nn.functional.pad((v < 0).to(torch.int64), (0, -n % 32)).view(-1, 32)
            words = (neg << torch.arange(32, device="cuda")).sum(1)
            plane[lo // 32:lo // 32 + words.numel()] = torch.where(words >= 1 << 31, words - (1 << 32), words).to(torch.int32)
            v = v.abs()
        if pack in ("i8", "u8s"):
            levels[lo:lo + n] = (v & 255).to(torch.uint8)
        else:
            b = torch.nn.functional.pad(v & 15, (0, n & 1)).view(-1, 2)
            levels[lo // 2:lo // 2 + b.shape[0]] = (b[:, 0] | (b[:, 1] << 4)).to(torch.uint8)


def _rows(K, nbytes, dtype=torch.uint8, align=256):
    """K zeroed buffers as the rows of one tensor, each aligned."""
    per = align // torch.empty(0, dtype=dtype).element_size()
    return torch.zeros(K, -(-nbytes // per) * per, dtype=dtype, device="cuda")


def prepare(case, seed):
    d, K, kind = case["d"], case["K"], case["kind"]
    p = gq.make_params(SCHEMES[case["scheme"]], case["s"], PACKS[case["pack"]], AGGS[case["agg"]], seed=QUANT_SEED, rng_bits=case["rng_bits"])
    st = {"kind": kind, "K": K, "d": d, "params": p, "norm_kind": NORMS[case["norm"]], "fused_mean": case["fused_mean"],
          "bucket": case["bucket"]}
    agg_type = torch.int16 if case["agg"] == "i16" else torch.int32
    plane = case["pack"] in ("u8s", "u4s")
    st["norm"] = torch.full((1,), 0.05, device="cuda")
    st["flags"] = torch.zeros(1, dtype=torch.int32, device="cuda")
    if kind not in ("alg2", "average"):
        st["agg"] = torch.zeros(d, dtype=agg_type, device="cuda")
    if kind != "lists":
        st["mean"] = torch.zeros(d, device="cuda")
    if kind in ("step", "buckets", "wire", "sparse"):
        st["x"] = _gradients(case, seed)
    if kind in ("step", "wire", "sparse"):
        st["workspace"] = torch.empty(gq.norm_workspace_bytes(K, d), dtype=torch.uint8, device="cuda")
    if kind == "buckets":
        nb = -(-d // case["bucket"])
        st["norms"] = torch.zeros(nb, device="cuda")
        st["bucket_flags"] = torch.zeros(nb, dtype=torch.int32, device="cuda")
        st["workspace"] = torch.empty(gq.bucketed_workspace_bytes(K, d, case["bucket"]), dtype=torch.uint8, device="cuda")
    st["levels"] = st["planes"] = None
    if kind in ("wire", "receive", "alg2", "average", "lists") or case["codes"]:
        st["levels_all"] = _rows(K, gq.levels_nbytes(d, p.pack))
        st["levels"] = list(st["levels_all"])
        if plane:
            st["planes_all"] = _rows(K, gq.signplane_nwords(d), torch.int32)
            st["planes"] = list(st["planes_all"])
    if kind in ("receive", "alg2", "average", "lists"):
        for w in range(K):
            _packed(case, _signed_codes(case, seed, w), st["levels"][w], st["planes"][w] if plane else None)
    if kind in ("alg2", "average"):
        st["reduced"] = torch.zeros(gq.levels_nbytes(d, p.pack), dtype=torch.uint8, device="cuda")
    if kind in ("sparse", "lists"):
        # the lists: under the (2,2) norm as long as Theorem 1's bound asks for (a worker's share of it, with room), else a
        # third of the coordinates for these gradients' codes, or all of them
        bound = gq.sparse_nnz_bound(p, K, d) if kind == "sparse" else d / 3 if case["dist"] == "outliers" and case["scheme"] == "linear" else d
        room = d if kind == "lists" else int(bound / K * 2) + 1024
        if kind == "lists" and bound < d:
            room = int(bound) + 1024
        st["indices_all"] = _rows(K, min(room, d), torch.int32)
        st["values_all"] = _rows(K, st["indices_all"].shape[1], torch.int8, align=1)
        st["counts_all"] = torch.zeros(K, dtype=torch.int64, device="cuda")
        st["starts_all"] = torch.zeros(K, gq.tile_starts_len(d), dtype=torch.int32, device="cuda")
        st["indices"], st["values"] = list(st["indices_all"]), list(st["values_all"])
        st["counts"], st["starts"] = [c for c in st["counts_all"].view(K, 1)], list(st["starts_all"])
        st["scan"] = torch.empty(gq.compact_workspace_bytes(d), dtype=torch.uint8, device="cuda")
    return st


# ---- one pass -------------------------------------------------------------------------------------------------------

def run(st):
    kind, K, d, p = st["kind"], st["K"], st["d"], st["params"]
    if kind == "step":
        gq.global_norm(st["x"], st["norm_kind"], st["norm"], st["flags"], st["workspace"])
        if st["fused_mean"]:
            gq.fused_quantize_aggregate(st["x"], st["norm"], p, 0, st["agg"], st["mean"], st["levels"], st["planes"])
        else:
            gq.fused_quantize_aggregate(st["x"], st["norm"], p, 0, st["agg"], None, st["levels"], st["planes"])
            gq.dequantize(st["agg"], d, st["norm"], p, K, st["mean"])
        out = {"norm": st["norm"], "flags": st["flags"], "sum": st["agg"], "mean": st["mean"]}
        if st["levels"] is not None:
            out["codes"] = st["levels_all"]
            if st["planes"] is not None:
                out["signs"] = st["planes_all"]
        return out
    if kind == "buckets":
        gq.bucketed_quantize_aggregate(st["x"], st["bucket"], st["norm_kind"], p, st["norms"], st["bucket_flags"], st["agg"],
                                       st["mean"] if st["fused_mean"] else None, st["workspace"])
        out = {"norms": st["norms"], "flags": st["bucket_flags"], "sum": st["agg"]}
        if st["fused_mean"]:
            out["mean"] = st["mean"]
        return out
    if kind == "wire":
        gq.global_norm(st["x"], st["norm_kind"], st["norm"], st["flags"], st["workspace"])
        for w in range(K):
            gq.quantize(st["x"][w], st["norm"], p, w, 0, st["levels"][w], st["planes"][w] if st["planes"] else None)
        gq.int_aggregate(st["levels"], st["planes"], d, p, st["agg"])
        gq.dequantize(st["agg"], d, st["norm"], p, K, st["mean"])
        out = {"norm": st["norm"], "codes": st["levels_all"], "sum": st["agg"], "mean": st["mean"]}
        if st["planes"] is not None:
            out["signs"] = st["planes_all"]
        return out
    if kind == "receive":
        gq.int_aggregate(st["levels"], st["planes"], d, p, st["agg"])
        gq.dequantize(st["agg"], d, st["norm"], p, K, st["mean"])
        return {"sum": st["agg"], "mean": st["mean"]}
    if kind == "alg2":
        gq.exp_reduce(st["levels"], d, p, 0, st["norm"], st["reduced"], st["mean"])
        return {"reduced": st["reduced"], "mean": st["mean"]}
    if kind == "average":
        gq.avg_reduce(st["levels"], d, p, 0, st["norm"], st["reduced"], st["mean"])
        return {"reduced": st["reduced"], "mean": st["mean"]}
    if kind == "sparse":
        gq.global_norm(st["x"], st["norm_kind"], st["norm"], st["flags"], st["workspace"])
        for w in range(K):
            gq.quantize_compact(st["x"][w], st["norm"], p, w, 0, st["indices"][w], st["values"][w], st["counts"][w], st["scan"],
                                tile_starts_out=st["starts"][w])
    else:
        for w in range(K):
            gq.compact(st["levels"][w], d, p, st["indices"][w], st["values"][w], st["counts"][w], st["scan"], tile_starts_out=st["starts"][w])
    gq.sparse_aggregate(st["indices"], st["values"], st["counts"], d, p, st["agg"], tile_starts=st["starts"])
    out = {"indices": st["indices_all"], "values": st["values_all"], "counts": st["counts_all"], "starts": st["starts_all"], "sum": st["agg"]}
    if kind == "sparse":
        gq.dequantize(st["agg"], d, st["norm"], p, K, st["mean"])
        out["norm"], out["mean"] = st["norm"], st["mean"]
    return out


def work(case):
    """Bytes of one pass: every input read once, every output written once.  (The norm has to be known before the first
    code, so a pass over gradients that no cache holds cannot do with less than twice their bytes.)"""
    d, K, kind = case["d"], case["K"], case["kind"]
    agg = d * (2 if case["agg"] == "i16" else 4)
    codes = d * {"i8": 1.0, "i4": 0.5, "u8s": 1.125, "u4s": 0.625}[case["pack"]]
    if kind in ("step", "buckets"):
        mean = 4 * d if kind == "step" or case["fused_mean"] else 0
        return {"bytes": 4 * K * d + agg + mean + (K * codes if case["codes"] else 0), "flops": 0}
    if kind == "wire":
        return {"bytes": 4 * K * d + K * codes + agg + 4 * d, "flops": 0}
    if kind == "receive":
        return {"bytes": K * codes + agg + 4 * d, "flops": 0}
    if kind in ("alg2", "average"):
        return {"bytes": K * codes + codes + 4 * d, "flops": 0}
    if kind == "sparse":
        nnz = min(K * d, _unit(case) ** 2 + _unit(case) * math.sqrt(K * d)) * 0.3      # measured: about a third of the bound
        return {"bytes": 4 * K * d + 5 * nnz + agg + 4 * d, "flops": 0}
    return {"bytes": K * d + 5 * K * d / 6 + agg, "flops": 0}


def tolerance(case):
    """Everything is exact: the max norm is a maximum, the L2 norms are binary64 sums rounded once to binary32 (their order shows
    below 2^-45, and the rounding hides it), and codes, sums, lists and means are fixed by the norm and the counter-based random
    stream down to the last bit."""
    return "exact"


# ---- the same in 64 bits ----------------------------------------------------------------------------------------------

def _philox(c0, c1, c2, c3):
    """Philox4x32-10 (Salmon et al., SC'11) on int64 tensors that hold 32-bit words; the key is QUANT_SEED."""
    k0, k1 = QUANT_SEED & M32, QUANT_SEED >> 32
    for _ in range(10):
        p0, p1 = c0 * 0xD2511F53, c2 * 0xCD9E8D57          # products modulo 2^64: all their bits
        c0, c1, c2, c3 = ((p1 >> 32) & M32) ^ c1 ^ k0, p1 & M32, ((p0 >> 32) & M32) ^ c3 ^ k1, p0 & M32
        k0, k1 = (k0 + 0x9E3779B9) & M32, (k1 + 0xBB67AE85) & M32
    return torch.stack((c0, c1, c2, c3), 1)


def _words(lo, n, per, c2, c3):
    """The Philox words of coordinates lo .. lo+n-1 (lo a multiple of 8), `per` coordinates to a call: [calls, 4]."""
    call = torch.arange(lo // per, (lo + n + per - 1) // per, device="cuda")
    return _philox(call & M32, call >> 32, torch.full_like(call, c2), torch.full_like(call, c3))


def _values(case, x, lo, norm, worker):
    """Integer values (int64) of the codes of x = coordinates lo .. of one worker under the binary32 `norm`, by the documented rule."""
    n = x.numel()
    if case["rng_bits"] == 16:
        w = _words(lo, n, 8, worker, 0)
        r = torch.stack(((w << 16) & M32, w & 0xFFFF0000), 2).reshape(-1)[:n]
    else:
        r = _words(lo, n, 4, worker, 0).reshape(-1)[:n]
    ax, top = x.abs(), float(_unit(case))
    scale = torch.tensor(top, device="cuda") / norm
    if case["scheme"] == "linear":
        u = r.float().double() * (2.0 ** -32 - 2.0 ** -56)
        t = (ax.double() * scale.double() - u.float().double()).float()
        k = torch.ceil(t).clamp_(max=top)
    else:
        z = (ax * scale).clamp_(max=top)
        R = r >> 9
        bits = (z.view(torch.int32).to(torch.int64) + R) & 0x7F800000
        k = torch.where(z < 1.0, (torch.round(z.double() * 2.0 ** 23) + R >= 2 ** 23).float(), bits.to(torch.int32).view(torch.float32))
    k = torch.where(ax >= norm, torch.full_like(k, top), k)
    return (k.double() * x.sign().double()).to(torch.int64)


def _norm64(case, parts):
    if case["norm"] == "linf":
        return max(float(x.abs().max()) for x in parts)
    squares = [sum(float(x[i:i + CHUNK].double().square().sum()) for i in range(0, x.numel(), CHUNK)) for x in parts]
    return math.sqrt(sum(squares) if case["norm"] == "l2" else max(squares))


def _code_value(case, q):
    """The integer a signed code adds to the sum."""
    q = q.to(torch.int64)
    return q if case["scheme"] == "linear" else q.sign() * torch.where(q == 0, q, 1 << (q.abs() - 1).clamp_(min=0))


def _tree_alg2(case, codes, lo):
    """Algorithm 2 on int64 codes [K, n] of coordinates lo ..: the root's value, in units of 2^-e, as float64."""
    K, n = codes.shape
    s, pad = case["s"], 1
    while pad < K:
        pad *= 2
    width = 8 if s <= 8 else 16 if s <= 16 else 32
    per, levels = 32 // width, pad.bit_length() - 1
    # sign * 2^-e, e = s - k + 1 + log2(n'), scaled by 2^(s + 1 + log2 n'): sign * 2^k
    node = [None] * pad + [c.sign().double() * torch.exp2(c.abs().clamp(max=s).double()) for c in codes]
    node += [torch.zeros(n, dtype=torch.float64, device="cuda")] * (pad - K)
    groups = {}
    for h in range(pad - 1, 0, -1):
        if h // per not in groups:
            groups[h // per] = _words(lo, n, 4, h // per, 1).reshape(-1)[:n]
        r = (groups[h // per] >> (width * (h % per) + width - s)) & ((1 << s) - 1)
        k = torch.where(r == 0, s + 1, s - torch.floor(torch.log2(r.clamp(min=1).double())).to(torch.int64))
        a, b = node[2 * h], node[2 * h + 1]
        first = a.abs() >= b.abs()
        big, small = torch.where(first, a, b), torch.where(first, b, a)
        gap = torch.log2((big / small).abs())               # +inf or NaN next to a zero operand, which leaves the other alone
        same = big.sign() == small.sign()
        up, down = same & (k > gap), ~same & (small != 0) & (k > gap - 1)
        out = torch.where(up, big * 2.0, torch.where(down, big / 2.0, big))
        node[h] = torch.where(~same & (small != 0) & (gap == 0), torch.zeros_like(out), out)
        node[2 * h] = node[2 * h + 1] = None
    return node[1] * 2.0 ** -(s + 1 + levels), pad


def _tree_average(case, codes, lo):
    K, n = codes.shape
    pad = 1
    while pad < K:
        pad *= 2
    node = [None] * pad + list(codes) + [torch.zeros(n, dtype=torch.int64, device="cuda")] * (pad - K)
    coins = [_words(lo, n, 4, i, 2).reshape(-1)[:n] for i in range((pad + 31) // 32)]
    for h in range(pad - 1, 0, -1):
        node[h] = (node[2 * h] + node[2 * h + 1] + ((coins[h // 32] >> (h % 32)) & 1)) >> 1
    return node[1].double(), pad


def exact(case, seed):
    d, K, kind, unit = case["d"], case["K"], case["kind"], _unit(case)
    mean = torch.empty(d, dtype=torch.float64, device="cuda")
    if kind == "lists":                                      # whole numbers only
        return None
    if kind in ("receive", "alg2", "average"):
        norm = float(torch.tensor(0.05))                     # as the state holds it: binary32
        q = torch.stack([_signed_codes(case, seed, w) for w in range(K)])
        for lo in range(0, d, CHUNK // 4):
            c = q[:, lo:lo + CHUNK // 4]
            part = mean[lo:lo + CHUNK // 4]
            if kind == "receive":
                part.copy_(sum(_code_value(case, row) for row in c).double() * (norm / (K * unit)))
            elif kind == "alg2":
                root, pad = _tree_alg2(case, c.to(torch.int64), lo)
                part.copy_(root * (2.0 * pad * norm / K))
            else:
                root, pad = _tree_average(case, c.to(torch.int64), lo)
                part.copy_(root * (norm * pad / (K * case["s"])))
        return {"reduced": None, "sum": None, "mean": mean}
    xs = _gradients(case, seed)
    step = case["bucket"] if kind == "buckets" else d
    norms = []
    for b in range(0, d, step):
        parts = [x[b:b + step] for x in xs]
        norms.append(_norm64(case, parts))
        n32 = torch.tensor(norms[-1], device="cuda", dtype=torch.float32)
        for lo in range(b, min(b + step, d), CHUNK):
            hi = min(lo + CHUNK, b + step, d)
            total = sum(_values(case, x[lo:hi], lo, n32, w) for w, x in enumerate(xs))
            mean[lo:hi] = total.double() * (norms[-1] / (K * unit))
    norms = torch.tensor(norms, dtype=torch.float64)
    if kind == "buckets":
        return {"norms": norms, "mean": mean if case["fused_mean"] else None}
    return {"norm": norms, "mean": mean}
