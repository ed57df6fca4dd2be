"""Every variant of the streamed product kernel that its plan can pick -- row fragments x column
blocks, bf16 and fp32, linear (LayerNorm and plain) and gated -- at ragged sizes: row blocks and
column groups that end inside, K that ends inside a chunk and, where such a call stays small, runs
past the ring's depth.  A CPU test checks that each size reaches its variant.

Bounds: the 2-norm bound of test_skinny, and the largest error of a row over the row's largest
value or the rms of all outputs, whichever is larger.  Variants of few columns need thousands of
rows, and among 8194 rows of 16 gated columns some have no value above a tenth of the rms; an
error's size follows the rms of the row's K products, not the row's largest output.  Linear: W'
rounds by 2^-9 / sqrt(3) rms, 1.1e-3 of that rms, and 5 sigma over 10^5 values are 6e-3, within the
2e-2 of the other tests.  Gated, silu(g) u: the errors g du and u dg are products of two normal
variables, whose tail falls as e^-t only and reaches t = 12 in 2 x 10^5 values; two of them,
in quadrature 1.4 x 12 x 1.1e-3 = 1.9e-2 of sigma_g sigma_u, over the outputs' rms of 0.66 of that:
3e-2.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2502_17728_amd import inputs as I
from tests import launch_rules as R
from tests.parity import TOL, cuda

# (row fragments, column blocks): (M, K, N)
LINEAR = {
    (2, 1): (17, 1800, 8), (2, 2): (17, 1312, 4136), (2, 3): (33, 1032, 4136), (2, 4): (33, 920, 6280),
    (2, 6): (33, 656, 8336), (2, 7): (33, 648, 12336), (3, 1): (8218, 1112, 8), (3, 2): (8235, 1040, 24),
    (3, 3): (8334, 904, 40), (3, 4): (33, 776, 14352), (3, 6): (33, 592, 16744), (3, 7): (65, 520, 12344),
    (4, 1): (12452, 1032, 8), (4, 2): (12637, 904, 24), (4, 3): (4141, 808, 120), (4, 4): (49, 648, 14368),
    (4, 6): (98, 520, 8232), (4, 7): (99, 520, 12344), (6, 1): (16403, 136, 8), (6, 2): (16390, 48, 24),
    (6, 3): (4119, 592, 200), (6, 4): (65, 520, 14728), (6, 6): (65, 464, 16392), (6, 7): (193, 456, 8216),
    (8, 1): (24578, 56, 8), (8, 2): (24617, 56, 24), (8, 3): (25029, 56, 40), (8, 4): (100, 456, 14440),
    (8, 6): (98, 392, 16528), (8, 7): (98, 392, 24648),
}
GATED = {
    (2, 2): (17, 1288, 8), (2, 4): (17, 912, 4104), (2, 6): (33, 648, 4192), (2, 8): (17, 528, 12464),
    (2, 14): (17, 392, 16888), (3, 2): (8194, 1032, 16), (3, 4): (33, 792, 6184), (3, 6): (33, 584, 8368),
    (3, 8): (33, 520, 14704), (3, 14): (33, 336, 16472), (4, 2): (12358, 904, 8), (4, 4): (4113, 664, 72),
    (4, 6): (49, 520, 8368), (4, 8): (145, 456, 4200), (4, 14): (49, 328, 16448), (6, 2): (16399, 48, 8),
    (6, 4): (65, 544, 6152), (6, 6): (65, 456, 8840), (6, 8): (65, 400, 12320), (8, 2): (24579, 56, 8),
    (8, 4): (8238, 456, 72), (8, 6): (97, 392, 8216), (8, 8): (97, 328, 12632),
}
F32_LINEAR = {
    (1, 1): (1, 1288, 8), (1, 2): (1, 904, 4112), (1, 3): (1, 648, 8216), (1, 4): (1, 520, 12456),
    (2, 1): (145, 912, 808), (2, 2): (86, 672, 2696), (2, 3): (17, 528, 8232), (2, 4): (33, 456, 6216),
    (2, 6): (1, 328, 16448), (4, 1): (681, 528, 360), (4, 2): (291, 456, 1608), (4, 3): (2783, 392, 200),
    (4, 4): (34, 336, 12440), (4, 6): (34, 264, 16528), (8, 1): (626, 296, 808), (8, 2): (323, 272, 2696),
    (8, 3): (8895, 264, 104), (8, 4): (67, 232, 12520), (8, 6): (65, 200, 16952),
}
F32_GATED = {
    (1, 2): (1, 904, 16), (1, 4): (1, 520, 4104), (2, 2): (4113, 648, 8), (2, 4): (17, 456, 4200),
    (2, 6): (1, 328, 8224), (4, 2): (8264, 456, 16), (4, 4): (33, 328, 6184), (4, 6): (65, 272, 4200),
    (8, 2): (16489, 264, 8), (8, 4): (65, 232, 6448), (8, 6): (66, 200, 8376),
}


@pytest.mark.parametrize("sizes,dtype,gated", [(LINEAR, R.BF16, False), (GATED, R.BF16, True),
                                               (F32_LINEAR, R.F32, False), (F32_GATED, R.F32, True)])
def test_sizes_reach_their_variants(sizes, dtype, gated):
    for plan, (M, K, N) in sizes.items():
        assert R.product(M, K, N, dtype, gated) == "streamed", (plan, M, K, N)
        assert R.streamed_plan(M, K, N, dtype, gated) == plan, (plan, M, K, N)


def _out(M, N, dtype):
    buf = torch.full((M + 2, N), 7.0, dtype=dtype, device="cuda")
    return buf, buf[1:M + 1]


def _compare(buf, ref, tol2, row_tol=TOL[torch.bfloat16]):
    torch.cuda.synchronize()
    out = buf.cpu()
    assert (out[0] == 7).all() and (out[-1] == 7).all()
    got = oracle.to_f64(out[1:-1])
    assert np.isfinite(got).all()
    scale = np.maximum(np.abs(ref).max(axis=1), np.sqrt((ref ** 2).mean()))
    if buf.dtype == torch.float32:
        row_tol = tol2 = TOL[torch.float32]
    assert (np.abs(got - ref).max(axis=1) / scale).max() <= row_tol
    assert np.linalg.norm(got - ref) <= tol2 * np.linalg.norm(ref)


def _silu(g):
    return g / (1.0 + np.exp(-g))


LINEAR_CASES = [(d, p, s) for d, t in (("bf16", LINEAR), ("f32", F32_LINEAR)) for p, s in t.items()]
GATED_CASES = [(d, p, s) for d, t in (("bf16", GATED), ("f32", F32_GATED)) for p, s in t.items()]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,plan,size", LINEAR_CASES)
def test_linear(dtype, plan, size):
    from paper_2502_17728_amd import ops
    M, K, N = size
    c = I.make_ln_case(M, K, N, dtype, seed=M + K)
    x, W = cuda(c["x"]), cuda(c["W"])
    buf, out = _out(M, N, x.dtype)
    ops.ln_linear_deferred(x, ops.ln_linear_prepare(W, cuda(c["gamma"]), cuda(c["beta"])), c["eps"], out=out)
    _compare(buf, oracle.norm_linear_matmul(c["x"], c["gamma"], c["beta"], c["W"], None, c["eps"]), 4e-3)
    if R.product(M, K, N, R.BF16 if dtype == "bf16" else R.F32, plain=True) == "streamed":
        bias = torch.linspace(-1, 1, N).to(x.dtype)
        buf, out = _out(M, N, x.dtype)
        ops.gemm(x, ops.ln_linear_prepare(W, torch.ones(K, dtype=x.dtype, device="cuda")), cuda(bias),
                 out=out.unsqueeze(0))
        _compare(buf, oracle.to_f64(c["x"]) @ oracle.to_f64(c["W"]) + oracle.to_f64(bias), 4e-3)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,plan,size", GATED_CASES)
def test_gated(dtype, plan, size):
    from paper_2502_17728_amd import ops
    M, K, N = size
    c = I.make_swiglu_case(M, K, N, dtype, seed=M + K)
    x = cuda(c["x"])
    buf, out = _out(M, N, x.dtype)
    ops.rms_swiglu_deferred(x, ops.swiglu_prepare(cuda(c["Wg"]), cuda(c["Wu"]), cuda(c["gamma"])), c["eps"], out=out)
    g, u = (oracle.norm_linear_matmul(c["x"], c["gamma"], None, c[w], None, c["eps"], rms=True) for w in ("Wg", "Wu"))
    _compare(buf, _silu(g) * u, 6e-3, 3e-2)
