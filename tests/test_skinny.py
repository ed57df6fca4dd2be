"""The streamed kernel (bf16 from 17 rows, fp32 of any) at small sizes where it can go wrong: row
counts around its row blocks, more than one row block, K that ends inside a 32- or 64-k chunk or
within the first stage, ragged column blocks; LayerNorm, RMSNorm, gated and plain.  Small outputs
take its smaller variants (every variant: test_skinny_plans).  Rows of guard values around the
output must survive.

Bounds: the row-normwise bound of the parity tests, and on the 2-norm of the whole error
4e-3 (gated 6e-3): W' and the output round to bf16 once each, 2^-9 / sqrt(3) rms at most
apiece (1.6e-3 together), the gated product has two such factors and K-long fp32 sums add
far less.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2502_17728_amd import inputs as I
from tests.parity import TOL, cuda, rowwise_rel_err

pytestmark = pytest.mark.gpu

SHAPES = [(17, 8, 8), (32, 40, 24), (33, 72, 136), (48, 64, 4104), (49, 1000, 264), (64, 200, 1000), (65, 96, 72),
          (96, 328, 520), (97, 136, 2056), (128, 2056, 40), (129, 1000, 1032), (200, 72, 4096), (257, 520, 776),
          (300, 768, 3072), (815, 104, 328)]


def _guarded(M, N):
    buf = torch.full((M + 2, N), 7.0, dtype=torch.bfloat16, device="cuda")
    return buf, buf[1:M + 1]


def _check(buf, ref, tol2):
    torch.cuda.synchronize()
    out = buf.cpu()
    assert (out[0] == 7).all() and (out[-1] == 7).all()
    got = out[1:-1]
    assert rowwise_rel_err(got, ref) <= TOL[torch.bfloat16]
    assert np.linalg.norm(oracle.to_f64(got) - ref) <= tol2 * np.linalg.norm(ref)


@pytest.mark.parametrize("M,K,N", SHAPES)
def test_linear(M, K, N):
    from paper_2502_17728_amd import ops
    for norm in ("layernorm", "rms"):
        c = I.make_ln_case(M, K, N, "bf16", seed=M + K, norm=norm)
        w = ops.ln_linear_prepare(cuda(c["W"]), cuda(c["gamma"]), cuda(c["beta"]))
        buf, out = _guarded(M, N)
        if norm == "rms":
            ops.rms_linear_deferred(cuda(c["x"]), w, c["eps"], out=out)
            ref = oracle.rms_linear(c["x"], c["gamma"], c["W"], None, c["eps"])
        else:
            ops.ln_linear_deferred(cuda(c["x"]), w, c["eps"], out=out)
            ref = oracle.ln_linear(c["x"], c["gamma"], c["beta"], c["W"], None, c["eps"])
        _check(buf, ref, 4e-3)


@pytest.mark.parametrize("M,K,N", [(17, 40, 24), (40, 72, 264), (64, 1000, 3592), (80, 328, 2056), (128, 136, 1032),
                                   (200, 64, 136)])
def test_gated(M, K, N):
    from paper_2502_17728_amd import ops
    c = I.make_swiglu_case(M, K, N, "bf16", seed=M + K)
    w = ops.swiglu_prepare(cuda(c["Wg"]), cuda(c["Wu"]), cuda(c["gamma"]))
    buf, out = _guarded(M, N)
    ops.rms_swiglu_deferred(cuda(c["x"]), w, c["eps"], out=out)
    _check(buf, oracle.rms_swiglu(c["x"], c["gamma"], c["Wg"], c["Wu"], c["eps"]), 6e-3)


@pytest.mark.parametrize("M,K,N", [(17, 40, 24), (50, 1000, 264), (128, 72, 1032), (300, 136, 520)])
def test_plain(M, K, N):
    # gemm on packed weights (gamma = 1), with a bias
    from paper_2502_17728_amd import ops
    c = I.make_ln_case(M, K, N, "bf16", seed=M)
    one = torch.ones(K, dtype=torch.bfloat16)
    w = ops.ln_linear_prepare(cuda(c["W"]), cuda(one))
    bias = torch.linspace(-1, 1, N).to(torch.bfloat16)
    buf, out = _guarded(M, N)
    ops.gemm(cuda(c["x"]), w, cuda(bias), out=out.unsqueeze(0))
    ref = oracle.to_f64(c["x"]) @ oracle.to_f64(c["W"]) + oracle.to_f64(bias)
    _check(buf, ref, 4e-3)


@pytest.mark.parametrize("M,K,N", [(1, 8, 8), (3, 40, 24), (16, 1000, 264), (17, 24, 136), (33, 72, 4104),
                                   (64, 328, 520), (65, 136, 72), (128, 768, 1032), (129, 200, 40), (300, 104, 776),
                                   (1000, 16, 328)])
def test_fp32(M, K, N):
    # every fp32 product on packed weights: LayerNorm, RMSNorm with its exported statistics, gated, plain
    from paper_2502_17728_amd import ops
    tol = TOL[torch.float32]
    c = I.make_ln_case(M, K, N, "f32", seed=M + K)
    x, W = cuda(c["x"]), cuda(c["W"])
    w = ops.ln_linear_prepare(W, cuda(c["gamma"]), cuda(c["beta"]))
    out = ops.ln_linear_deferred(x, w, c["eps"])
    assert rowwise_rel_err(out.cpu(), oracle.ln_linear(c["x"], c["gamma"], c["beta"], c["W"], None, c["eps"])) <= tol
    w = ops.ln_linear_prepare(W, cuda(c["gamma"]))
    out, y, stats = ops.linear_deferred_post(x, w, cuda(c["gamma"]), eps=c["eps"], rms=True)
    assert rowwise_rel_err(out.cpu(), oracle.rms_linear(c["x"], c["gamma"], c["W"], None, c["eps"])) <= tol
    assert rowwise_rel_err(y.cpu(), oracle.rmsnorm(c["x"], c["gamma"], c["eps"])) <= tol
    out = ops.gemm(x, ops.ln_linear_prepare(W, torch.ones(K, device="cuda")))
    assert rowwise_rel_err(out.cpu(), oracle.to_f64(c["x"]) @ oracle.to_f64(c["W"])) <= tol
    g = I.make_swiglu_case(M, K, N, "f32", seed=M)
    w = ops.swiglu_prepare(cuda(g["Wg"]), cuda(g["Wu"]), cuda(g["gamma"]))
    out = ops.rms_swiglu_deferred(cuda(g["x"]), w, g["eps"])
    assert rowwise_rel_err(out.cpu(), oracle.rms_swiglu(g["x"], g["gamma"], g["Wg"], g["Wu"], g["eps"])) <= tol


@pytest.mark.parametrize("M,K,dtype", [(3, 8, "f32"), (40, 24, "f32"), (300, 72, "f32"), (20, 8, "bf16"), (40, 40, "bf16"),
                                       (100, 328, "bf16"), (300, 200, "bf16")])
def test_infinite_weight_in_the_last_chunk(M, K, dtype):
    # an infinite weight of the last k row, where the last stage of chunks reaches past K: +-inf as the
    # plain product gives, in its column only
    from paper_2502_17728_amd import ops
    c = I.make_ln_case(M, K, 136, dtype, seed=M)
    W = c["W"].clone()
    W[K - 1, 5] = float("inf")
    out = ops.gemm(cuda(c["x"]), ops.ln_linear_prepare(cuda(W), torch.ones(K, dtype=W.dtype, device="cuda"))).cpu()
    x_last = c["x"][:, K - 1].float()
    assert (x_last != 0).all()
    assert torch.equal(out[:, 5].float(), torch.sign(x_last) * float("inf"))
    keep = [n for n in range(136) if n != 5]
    assert rowwise_rel_err(out[:, keep], (oracle.to_f64(c["x"]) @ oracle.to_f64(c["W"]))[:, keep]) <= TOL[W.dtype]
