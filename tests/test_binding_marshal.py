"""The binding's native argument marshalling: what it refuses (no GPU needed) and that every form of an argument that it
accepts reaches the library alike."""
import os
import subprocess
import sys

import pytest
import torch

import paper_2305_18627_amd as gq

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_refuses_what_is_not_a_fitting_cuda_tensor():
    p = gq.make_params(gq.GQ_LINEAR, 127)
    x, n = torch.zeros(8), torch.zeros(1)
    for call in (lambda: gq.global_norm([x], 0, n), lambda: gq.global_norm_static((x,), 0, n), lambda: gq.quantize(x, n, p, 0, 0, x),
                 lambda: gq.int_aggregate([x], None, 8, p, x), lambda: gq.dequantize(x, 8, n, p, 1, x),
                 lambda: gq.fused_quantize_aggregate([x], n, p, 0, x), lambda: gq.exp_reduce([x], 8, p, 0, n, x),
                 lambda: gq.avg_reduce([x], 8, p, 0, n, x), lambda: gq.compact(x, 8, p, x, x, n),
                 lambda: gq.quantize_compact(x, n, p, 0, 0, x, x, n), lambda: gq.sparse_aggregate([x], [x], [n], 8, p, x),
                 lambda: gq.bucketed_quantize_aggregate([x], 8, 0, p, n, None, x)):
        with pytest.raises(ValueError):
            call()
    for bad in (None, 3, "x", [x], [None]):
        with pytest.raises((TypeError, ValueError, AttributeError)):
            gq.quantize(bad, n, p, 0, 0, x)
        with pytest.raises((TypeError, ValueError, AttributeError)):
            gq.global_norm_static([bad], 0, n)
    with pytest.raises(TypeError):
        gq.dequantize(x, 8, n, b"not params", 1, x)
    # an iterator has no length, and its tensors may be nobody else's
    for call in (lambda it: gq.global_norm_static(it, 0, n), lambda it: gq.global_norm(it, 0, n, workspace=x), lambda it: gq.int_aggregate(it, None, 8, p, x),
                 lambda it: gq.int_aggregate([], it, 8, gq.make_params(gq.GQ_LINEAR, 7, gq.GQ_PACK_U4_SIGNPLANE), x),
                 lambda it: gq.fused_quantize_aggregate(it, n, p, 0, x), lambda it: gq.exp_reduce(it, 8, p, 0, n, x),
                 lambda it: gq.avg_reduce(it, 8, p, 0, n, x), lambda it: gq.sparse_aggregate(it, [], [], 8, p, x)):
        with pytest.raises(TypeError):
            call(t for t in ())
        with pytest.raises((TypeError, ValueError)):
            call(t for t in (x,))


def test_loads_where_torch_has_no_gpu_functions():
    code = ("import torch\n"
            "for name in ('_cuda_getDevice', '_cuda_getCurrentRawStream'):\n"
            "    if hasattr(torch._C, name): delattr(torch._C, name)\n"
            "import paper_2305_18627_amd as gq\n"
            "assert gq.version() > 0 and gq.compact_workspace_bytes(1000) > 0\n"
            "print('loaded')\n")
    r = subprocess.run([sys.executable, "-c", code], cwd=ROOT, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.strip().endswith("loaded"), r.stdout


def test_the_marshalling_says_what_it_was_built_for():
    from paper_2305_18627_amd import binding, build
    assert binding._m.built_for == build.built_for() and torch.__version__ in binding._m.built_for
    assert not build.is_stale()
    real = build.built_for
    try:                                               # another torch: the library has to be built again
        build.built_for = lambda: "torch 0.0, python 0.0"
        assert build.is_stale()
    finally:
        build.built_for = real


@pytest.mark.gpu
def test_sequences_streams_and_optional_arguments_reach_the_library_alike():
    dev = torch.device("cuda:0")
    K, d = 3, 5008                                     # rows of one tensor are 16-byte aligned
    both = torch.randn(K, d, device=dev)
    rows = [both[i] for i in range(K)]

    class Sequence:                                    # has a length and items, and nobody else holds these tensors
        def __len__(self):
            return K

        def __getitem__(self, i):
            if i >= K:
                raise IndexError(i)
            return both[i].clone()

    ref = None
    side = torch.cuda.Stream()
    p = gq.make_params(gq.GQ_LINEAR, 127, seed=4)
    for xs in (rows, tuple(rows), both, Sequence()):
        for stream in (None, torch.cuda.current_stream(), torch.cuda.current_stream().cuda_stream, side, side.cuda_stream):
            side.wait_stream(torch.cuda.current_stream())
            norm, flags = torch.zeros(1, device=dev), torch.zeros(1, dtype=torch.int32, device=dev)
            agg, mean = torch.zeros(d, dtype=torch.int32, device=dev), torch.zeros(d, device=dev)
            torch.cuda.synchronize()
            ws = gq.global_norm(xs, gq.GQ_NORM_LINF, norm, flags, stream=stream)
            assert ws.numel() >= gq.norm_workspace_bytes(K, d)
            gq.fused_quantize_aggregate(xs, norm, p, 0, agg, mean, stream=stream)
            torch.cuda.synchronize()
            got = (norm, flags, agg, mean)
            ref = ref or got
            assert all(torch.equal(a, b) for a, b in zip(got, ref))
    assert float(ref[0]) == float(both.abs().max())
    with torch.cuda.stream(side):                      # None is the stream that is current where the call is made
        norm2 = torch.zeros(1, device=dev)
        gq.global_norm_static(rows, gq.GQ_NORM_LINF, norm2)
        done = torch.cuda.Event()
        done.record(side)
    done.synchronize()
    assert torch.equal(norm2, ref[0])
    with pytest.raises(ValueError):
        gq.fused_quantize_aggregate(rows, norm, p, 0, agg, None, [torch.zeros(d, dtype=torch.uint8, device=dev)] * 2)
    with pytest.raises(gq.GQError):
        gq.global_norm([both[0]] * 65, gq.GQ_NORM_LINF, norm)
    with pytest.raises(ValueError):
        gq.global_norm(both.t()[:K], gq.GQ_NORM_LINF, norm)


@pytest.mark.gpu
@pytest.mark.parametrize("pack", [gq.GQ_PACK_I8, gq.GQ_PACK_I4, gq.GQ_PACK_U8_SIGNPLANE, gq.GQ_PACK_U4_SIGNPLANE])
def test_sign_planes_are_asked_for_where_the_format_has_them(pack):
    dev = torch.device("cuda:0")
    K, d = 2, 4099
    xs = [torch.randn(d, device=dev) for _ in range(K)]
    norm = torch.zeros(1, device=dev)
    gq.global_norm(xs, gq.GQ_NORM_LINF, norm)
    p = gq.make_params(gq.GQ_LINEAR, 7, pack, seed=4)
    planes = pack >= gq.GQ_PACK_U8_SIGNPLANE
    lvs = [torch.zeros(gq.levels_nbytes(d, pack), dtype=torch.uint8, device=dev) for _ in xs]
    sps = [torch.zeros(gq.signplane_nwords(d), dtype=torch.int32, device=dev) for _ in xs]
    want, got = torch.zeros(d, dtype=torch.int32, device=dev), torch.zeros(d, dtype=torch.int32, device=dev)
    gq.fused_quantize_aggregate(xs, norm, p, 0, want, None, lvs, sps)
    gq.int_aggregate(lvs, sps, d, p, got)
    assert torch.equal(got, want) and int(want.abs().sum()) > 0
    # one too few, none at all, too short ones: refused where they are used, ignored where not
    for some in ([], sps[:1], [sps[0], sps[1][:1]]):
        if planes:
            with pytest.raises(ValueError):
                gq.int_aggregate(lvs, some, d, p, got)
            with pytest.raises(ValueError):
                gq.fused_quantize_aggregate(xs, norm, p, 0, got, None, lvs, some)
        else:
            got.zero_()
            gq.int_aggregate(lvs, some, d, p, got)
            assert torch.equal(got, want)
            got.zero_()
            gq.fused_quantize_aggregate(xs, norm, p, 0, got, None, lvs, some)
            assert torch.equal(got, want)
        got.zero_()
        gq.fused_quantize_aggregate(xs, norm, p, 0, got, None, None, some)     # no codes stored
        assert torch.equal(got, want)
    if planes:
        with pytest.raises(gq.GQError):
            gq.int_aggregate(lvs, None, d, p, got)
    else:
        gq.int_aggregate(lvs, None, d, p, got)
