"""Thin ctypes binding of the C ABI in include/gqsgd.h.

Argument marshalling only: every step of the path runs in the HIP kernels of libgqsgd.so, and the
arguments are checked and converted in _marshal.so (csrc/marshal.cpp), which calls the library.
PyTorch is used for device memory (tensor.data_ptr()) and for the current HIP stream, nothing
else.  There is no CPU fallback: if the library has not been built, importing this module raises.
"""
import ctypes as C
import os

import torch

HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(HERE, "libgqsgd.so")
MARSHAL_PATH = os.path.join(HERE, "_marshal.so")

GQ_MAX_WORKERS = 64
GQ_OK, GQ_ERR_INVALID_ARG, GQ_ERR_UNSUPPORTED, GQ_ERR_OVERFLOW, GQ_ERR_WORKSPACE, GQ_ERR_DEVICE = range(6)
GQ_NORM_LINF, GQ_NORM_L2, GQ_NORM_L2_MAX = 0, 1, 2
GQ_LINEAR, GQ_EXP = 0, 1
GQ_PACK_I8, GQ_PACK_I4, GQ_PACK_U8_SIGNPLANE, GQ_PACK_U4_SIGNPLANE = 0, 1, 2, 3
GQ_AGG_I32, GQ_AGG_I16 = 0, 1
GQ_FLAG_WRITE_WINDOWS_OFF, GQ_FLAG_WRITE_WINDOWS_ON = 1, 2

# every symbol include/gqsgd.h declares
EXPORTS = ("gq_version", "gq_status_string", "gq_check_width", "gq_sparse_nnz_bound", "gq_norm_workspace_bytes", "gq_global_norm",
           "gq_global_norm_static", "gq_bucketed_workspace_bytes", "gq_bucketed_quantize_aggregate",
           "gq_quantize", "gq_int_aggregate", "gq_dequantize", "gq_fused_quantize_aggregate", "gq_exp_reduce", "gq_avg_reduce", "gq_compact_workspace_bytes", "gq_tile_starts_len", "gq_compact",
           "gq_quantize_compact",
           "gq_sparse_aggregate")


class gq_params(C.Structure):
    _fields_ = [("scheme", C.c_int32), ("s", C.c_int32), ("pack", C.c_int32), ("agg", C.c_int32),
                ("rng_bits", C.c_int32), ("flags", C.c_int32), ("seed", C.c_uint64)]


class GQError(RuntimeError):
    def __init__(self, status, where):
        self.status = int(status)
        name = _lib.gq_status_string(int(status)).decode() if _lib is not None else str(status)
        super().__init__("%s failed: %s" % (where, name))


def _load():
    for path in (LIB_PATH, MARSHAL_PATH):
        if not os.path.exists(path):
            raise ImportError("%s is missing: build it first (python -c 'import __graft_entry__ as g; g.build()' "
                              "or python paper_2305_18627_amd/build.py); there is no fallback path" % path)
    lib = C.CDLL(LIB_PATH)
    vp, i64, u32, i32, sz = C.c_void_p, C.c_int64, C.c_uint32, C.c_int, C.c_size_t
    pp = C.POINTER(gq_params)
    sigs = {
        "gq_version": (C.c_int, []),
        "gq_status_string": (C.c_char_p, [i32]),
        "gq_check_width": (i32, [pp, i32]),
        "gq_sparse_nnz_bound": (C.c_double, [pp, i32, i64]),
        "gq_norm_workspace_bytes": (sz, [i32, i64]),
        "gq_global_norm": (i32, [C.POINTER(vp), i32, i64, i32, vp, vp, vp, sz, vp]),
        "gq_global_norm_static": (i32, [C.POINTER(vp), i32, i64, i32, vp, vp, vp]),
        "gq_quantize": (i32, [vp, i64, vp, pp, u32, i64, vp, vp, vp]),
        "gq_int_aggregate": (i32, [C.POINTER(vp), C.POINTER(vp), i32, i64, pp, vp, vp]),
        "gq_dequantize": (i32, [vp, i64, vp, pp, i32, vp, vp]),
        "gq_bucketed_workspace_bytes": (sz, [i32, i64, i64]),
        "gq_bucketed_quantize_aggregate": (i32, [C.POINTER(vp), i32, i64, i64, i32, pp, vp, vp, vp, vp, vp, sz, vp, vp]),
        "gq_exp_reduce": (i32, [C.POINTER(vp), i32, i64, pp, i64, vp, vp, vp, vp]),
        "gq_avg_reduce": (i32, [C.POINTER(vp), i32, i64, pp, i64, vp, vp, vp, vp]),
        "gq_compact_workspace_bytes": (sz, [i64]),
        "gq_tile_starts_len": (i64, [i64]),
        "gq_compact": (i32, [vp, i64, pp, vp, vp, i64, vp, vp, vp, sz, vp]),
        "gq_quantize_compact": (i32, [vp, i64, vp, pp, u32, i64, vp, vp, i64, vp, vp, vp, sz, vp]),
        "gq_sparse_aggregate": (i32, [C.POINTER(vp), C.POINTER(vp), C.POINTER(vp), C.POINTER(i64), C.POINTER(vp), i32, i64, pp, vp, vp]),
        "gq_fused_quantize_aggregate": (i32, [C.POINTER(vp), i32, i64, vp, pp, i64, vp, vp, C.POINTER(vp),
                                               C.POINTER(vp), vp]),
    }
    for name, (res, args) in sigs.items():
        f = getattr(lib, name)
        f.restype = res
        f.argtypes = args
    return lib


_lib = None
_lib = _load()


try:
    from . import _marshal as _m  # noqa: E402
except ImportError as e:
    raise ImportError("%s does not load with torch %s: build it again" % (MARSHAL_PATH, torch.__version__)) from e
if not _m.built_for.startswith("torch %s, " % torch.__version__):
    raise ImportError("%s was built for %s, this is torch %s: build it again" % (MARSHAL_PATH, _m.built_for, torch.__version__))


def _current_raw_stream(device):
    return torch.cuda.current_stream(device).cuda_stream


# torch's own functions behind these two skip the Python objects; a torch without a GPU part has neither
_m.bind({name: C.cast(getattr(_lib, name), C.c_void_p).value for name in EXPORTS},
        getattr(torch._C, "_cuda_getDevice", torch.cuda.current_device),
        getattr(torch._C, "_cuda_getCurrentRawStream", _current_raw_stream))


def lib():
    """The loaded ctypes library (for tests that call the C ABI directly)."""
    return _lib


def _stream(stream):
    """A stream's address; None stands for the current stream (looked up where the call is made)."""
    if stream is None:
        return None
    return stream.cuda_stream if hasattr(stream, "cuda_stream") else int(stream)


def _check(st, where):
    if st != GQ_OK:
        raise GQError(st, where)


def _workspace(nbytes, like):
    return torch.empty(nbytes, dtype=torch.uint8, device=like.device)


def make_params(scheme, s, pack=GQ_PACK_I8, agg=GQ_AGG_I32, seed=0, rng_bits=32, flags=0):
    return gq_params(int(scheme), int(s), int(pack), int(agg), int(rng_bits), int(flags), int(seed))


def levels_nbytes(d, pack):
    return d if pack in (GQ_PACK_I8, GQ_PACK_U8_SIGNPLANE) else (d + 1) // 2


def signplane_nwords(d):
    return (d + 31) // 32


def status_string(st):
    return _lib.gq_status_string(int(st)).decode()


def version():
    return int(_lib.gq_version())


def check_width(params, K):
    """gq_check_width: the status code (GQ_OK / GQ_ERR_OVERFLOW / ...), not an exception."""
    return int(_lib.gq_check_width(C.byref(params), int(K)))


def sparse_nnz_bound(params, K, d):
    """gq_sparse_nnz_bound: the bound on the expected number of non-zero codes under the (2,2) norm; -1 for bad parameters."""
    return float(_lib.gq_sparse_nnz_bound(C.byref(params), int(K), int(d)))


def norm_workspace_bytes(K, d):
    return int(_lib.gq_norm_workspace_bytes(int(K), int(d)))


def global_norm(xs, kind, norm_out, status_flags=None, workspace=None, stream=None):
    """gq_global_norm over the K tensors xs (fp32, equal length).  Returns the workspace used."""
    if workspace is None:
        workspace = _workspace(max(norm_workspace_bytes(len(xs), xs[0].numel() if len(xs) else 0), 8), norm_out)
    _check(_m.global_norm(xs, int(kind), norm_out, status_flags, workspace, _stream(stream)), "gq_global_norm")
    return workspace


def global_norm_static(xs, kind, norm_out, status_flags=None, stream=None):
    """gq_global_norm_static: the norm with the library's own static scratch; nothing is allocated."""
    _check(_m.global_norm_static(xs, int(kind), norm_out, status_flags, _stream(stream)), "gq_global_norm_static")


def quantize(x, norm, params, worker, index_base, levels_out, signplane_out=None, stream=None):
    _check(_m.quantize(x, norm, params, int(worker), int(index_base), levels_out, signplane_out, _stream(stream)), "gq_quantize")


def int_aggregate(levels, signplanes, d, params, agg_out, stream=None):
    _check(_m.int_aggregate(levels, signplanes, int(d), params, agg_out, _stream(stream)), "gq_int_aggregate")


def dequantize(agg, d, norm, params, K, out, stream=None):
    _check(_m.dequantize(agg, int(d), norm, params, int(K), out, _stream(stream)), "gq_dequantize")


def fused_quantize_aggregate(xs, norm, params, index_base=0, agg_out=None, dequant_out=None,
                             levels_out=None, signplanes_out=None, stream=None):
    _check(_m.fused_quantize_aggregate(xs, norm, params, int(index_base), agg_out, dequant_out, levels_out, signplanes_out,
                                       _stream(stream)), "gq_fused_quantize_aggregate")


def bucketed_workspace_bytes(K, d, bucket):
    return int(_lib.gq_bucketed_workspace_bytes(int(K), int(d), int(bucket)))


def bucketed_quantize_aggregate(xs, bucket, kind, params, norms_out, status_flags=None, agg_out=None, dequant_out=None,
                                workspace=None, stream=None, side_stream=None):
    """gq_bucketed_quantize_aggregate: per bucket its own norm and fused quantize+aggregate; with side_stream the
    norm of the next bucket runs beside the fused call of the current one.  Returns the workspace used."""
    if workspace is None:
        workspace = _workspace(max(bucketed_workspace_bytes(len(xs), xs[0].numel() if len(xs) else 0, bucket), 8), norms_out)
    _check(_m.bucketed_quantize_aggregate(xs, int(bucket), int(kind), params, norms_out, status_flags, agg_out, dequant_out, workspace,
                                          _stream(stream), _stream(side_stream) or 0), "gq_bucketed_quantize_aggregate")
    return workspace


def exp_reduce(levels, d, params, index_base=0, norm=None, reduced_out=None, dequant_out=None, stream=None):
    _check(_m.exp_reduce(levels, int(d), params, int(index_base), norm, reduced_out, dequant_out, _stream(stream)), "gq_exp_reduce")


def avg_reduce(levels, d, params, index_base=0, norm=None, reduced_out=None, dequant_out=None, stream=None):
    _check(_m.avg_reduce(levels, int(d), params, int(index_base), norm, reduced_out, dequant_out, _stream(stream)), "gq_avg_reduce")


def compact_workspace_bytes(d):
    return int(_lib.gq_compact_workspace_bytes(int(d)))


def tile_starts_len(d):
    return int(_lib.gq_tile_starts_len(int(d)))


def compact(levels, d, params, indices_out, values_out, count_out, workspace=None, stream=None, tile_starts_out=None):
    """gq_compact: the non-zero int8 codes of one worker as (index, code) pairs, and optionally the table of where
    every tile of 4096 coordinates begins in the list.  Returns the workspace used."""
    if workspace is None:
        workspace = _workspace(compact_workspace_bytes(d), count_out)
    _check(_m.compact(levels, int(d), params, indices_out, values_out, count_out, workspace, tile_starts_out, _stream(stream)),
           "gq_compact")
    return workspace


def quantize_compact(x, norm, params, worker, index_base, indices_out, values_out, count_out, workspace=None, stream=None,
                     tile_starts_out=None):
    """gq_quantize_compact: the list gq_quantize + gq_compact would write, straight from the gradient.  Returns the
    workspace used."""
    if workspace is None:
        workspace = _workspace(compact_workspace_bytes(x.numel()), count_out)
    _check(_m.quantize_compact(x, norm, params, int(worker), int(index_base), indices_out, values_out, count_out, workspace,
                               tile_starts_out, _stream(stream)), "gq_quantize_compact")
    return workspace


def sparse_aggregate(indices, values, counts, d, params, agg_out, stream=None, tile_starts=None):
    _check(_m.sparse_aggregate(indices, values, counts, int(d), params, agg_out, tile_starts, _stream(stream)), "gq_sparse_aggregate")
