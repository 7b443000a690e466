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
