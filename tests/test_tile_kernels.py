"""The MFMA tile kernels of the bf16 products past 128 rows -- pipelined 128 x 128, 256 x 256 and
256 x 192 tiles and the two-stage 128 x 128 loop (K not a multiple of 64) -- at ragged sizes that the
launch rule sends to each (checked on the CPU), LayerNorm, RMSNorm, gated and plain: values, row
moments exchanged between workgroups and reduced locally, exported and pre-computed statistics,
non-finite and degenerate rows, graph replays.  Bounds as in the parity tests.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2502_17728_amd import inputs as I
from tests import launch_rules as R
from tests.parity import TOL, cuda, rowwise_rel_err

LINEAR = {"tiles128": (194, 192, 7240), "tiles256": (1281, 192, 8072), "tiles256x192": (386, 192, 8216),
          "two_stage": (396, 200, 7200)}
GATED = {"tiles128": (129, 192, 4136), "tiles256": (515, 192, 8200), "tiles256x192": (257, 192, 5448),
         "two_stage": (262, 200, 5744)}
PLAIN = {"tiles128": (129, 192, 264), "tiles256": (1288, 192, 8112), "tiles256x192": (385, 192, 8232),
         "two_stage": (389, 200, 7336)}
TOL2 = TOL[torch.bfloat16]


def test_sizes_reach_their_kernels():
    for sizes, kw in ((LINEAR, {}), (GATED, {"gated": True}), (PLAIN, {"plain": True})):
        for kernel, size in sizes.items():
            assert R.product(*size, **kw) == kernel, (kernel, size)


def _linear(kernel, norm, seed):
    c = I.make_ln_case(*LINEAR[kernel], "bf16", seed=seed, outliers=2, norm=norm)
    beta = None if norm == "rms" else c["beta"]
    return c, beta


def _reference(c, beta, norm):
    return oracle.norm_linear_matmul(c["x"], c["gamma"], beta, c["W"], None, c["eps"], rms=norm == "rms")


def _call(ops, c, beta, norm, x=None):
    w = ops.ln_linear_prepare(cuda(c["W"]), cuda(c["gamma"]), cuda(beta))
    f = ops.rms_linear_deferred if norm == "rms" else ops.ln_linear_deferred
    return f(cuda(c["x"]) if x is None else x, w, c["eps"])


@pytest.mark.gpu
@pytest.mark.parametrize("norm", ["layernorm", "rms"])
@pytest.mark.parametrize("kernel", LINEAR)
def test_linear(kernel, norm, monkeypatch):
    from paper_2502_17728_amd import ops
    c, beta = _linear(kernel, norm, 3)
    ref = _reference(c, beta, norm)
    assert rowwise_rel_err(_call(ops, c, beta, norm).cpu(), ref) <= TOL2
    monkeypatch.setenv("DN_MOMENT_WAIT_TICKS", "0")  # every workgroup reduces its rows' moments itself
    assert rowwise_rel_err(_call(ops, c, beta, norm).cpu(), ref) <= TOL2


@pytest.mark.gpu
@pytest.mark.parametrize("kernel", LINEAR)
def test_statistics(kernel):
    # exported by the product's kernel, and taken from a pre-pass
    from paper_2502_17728_amd import ops
    c, beta = _linear(kernel, "layernorm", 4)
    M = LINEAR[kernel][0]
    g, b = cuda(c["gamma"]), cuda(beta)
    w = ops.ln_linear_prepare(cuda(c["W"]), g, b)
    ref = _reference(c, beta, "layernorm")
    out, y, st = ops.linear_deferred_post(cuda(c["x"]), w, g, b, c["eps"])
    assert rowwise_rel_err(out.cpu(), ref) <= TOL2
    sd, xd = st.cpu().double().reshape(M, 2).numpy(), oracle.to_f64(c["x"])
    np.testing.assert_allclose(sd[:, 0], xd.mean(1), rtol=1e-4, atol=1e-5)
    np.testing.assert_allclose(sd[:, 1], 1 / np.sqrt(xd.var(1) + c["eps"]), rtol=1e-4)
    assert rowwise_rel_err(ops.ln_linear_serial(cuda(c["x"]), w, c["eps"]).cpu(), ref) <= TOL2


@pytest.mark.gpu
@pytest.mark.parametrize("norm", ["layernorm", "rms"])
@pytest.mark.parametrize("kernel", LINEAR)
def test_nonfinite_and_degenerate_rows(kernel, norm):
    from paper_2502_17728_amd import ops
    c, beta = _linear(kernel, norm, 5)
    M, K, _ = LINEAR[kernel]
    x = c["x"].clone()
    x[1, K // 3], x[2, K - 1], x[M - 1, 0] = float("nan"), float("inf"), float("-inf")
    c["x"] = x
    out = _call(ops, c, beta, norm).cpu()
    assert torch.isnan(out[[1, 2, M - 1]].float()).all()
    assert rowwise_rel_err(out, _reference(c, beta, norm)) <= TOL2
    c, beta = _linear(kernel, norm, 6)  # eps = 0: a row without variance (RMSNorm: of zeros) is NaN
    x = c["x"].clone()
    x[0], x[M - 1] = (0, 0) if norm == "rms" else (0.75, -1.5)
    c["x"], c["eps"] = x, 0.0
    out = _call(ops, c, beta, norm).cpu()
    assert torch.isnan(out[[0, M - 1]].float()).all()
    assert rowwise_rel_err(out, _reference(c, beta, norm)) <= TOL2


@pytest.mark.gpu
@pytest.mark.parametrize("kernel", LINEAR)
def test_linear_graph_replays(kernel):
    from paper_2502_17728_amd import ops
    cases = [I.make_ln_case(*LINEAR[kernel], "bf16", seed=20 + i, outliers=2, mean_offset=0.5 * i) for i in range(3)]
    a = cases[0]
    w = ops.ln_linear_prepare(cuda(a["W"]), cuda(a["gamma"]), cuda(a["beta"]))
    x = cuda(a["x"])
    out = ops.ln_linear_deferred(x, w, a["eps"])
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        ops.ln_linear_deferred(x, w, a["eps"], out=out)
    for c in cases + cases[:1]:
        x.copy_(cuda(c["x"]))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        eager = ops.ln_linear_deferred(x, w, a["eps"])
        torch.cuda.synchronize()
        ref = oracle.norm_linear_matmul(c["x"], a["gamma"], a["beta"], a["W"], None, a["eps"])
        assert rowwise_rel_err(out.cpu(), ref) <= TOL2
        assert rowwise_rel_err(eager.cpu(), ref) <= TOL2


@pytest.mark.gpu
@pytest.mark.parametrize("kernel", GATED)
def test_gated(kernel, monkeypatch):
    from paper_2502_17728_amd import ops
    cases = [I.make_swiglu_case(*GATED[kernel], "bf16", seed=7 + i, outliers=2) for i in range(2)]
    a = cases[0]
    w = ops.swiglu_prepare(cuda(a["Wg"]), cuda(a["Wu"]), cuda(a["gamma"]))
    Wg, Wu = oracle.to_f64(a["Wg"]), oracle.to_f64(a["Wu"])
    refs = [oracle.rms_swiglu_matmul(c["x"], a["gamma"], Wg, Wu, a["eps"]) for c in cases]
    x = cuda(a["x"])
    out = ops.rms_swiglu_deferred(x, w, a["eps"])
    assert rowwise_rel_err(out.cpu(), refs[0]) <= TOL2
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        ops.rms_swiglu_deferred(x, w, a["eps"], out=out)
    for i in (0, 1, 0):
        x.copy_(cuda(cases[i]["x"]))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert rowwise_rel_err(out.cpu(), refs[i]) <= TOL2
    monkeypatch.setenv("DN_MOMENT_WAIT_TICKS", "0")
    assert rowwise_rel_err(ops.rms_swiglu_deferred(x, w, a["eps"]).cpu(), refs[0]) <= TOL2


@pytest.mark.gpu
@pytest.mark.parametrize("kernel", PLAIN)
def test_plain(kernel):
    from paper_2502_17728_amd import ops
    M, K, N = PLAIN[kernel]
    c = I.make_ln_case(M, K, N, "bf16", seed=9)
    bias = torch.linspace(-1, 1, N).to(torch.bfloat16)
    w = ops.ln_linear_prepare(cuda(c["W"]), torch.ones(K, dtype=torch.bfloat16, device="cuda"))
    out = ops.gemm(cuda(c["x"]), w, cuda(bias)).cpu()
    ref = oracle.to_f64(c["x"]) @ oracle.to_f64(c["W"]) + oracle.to_f64(bias)
    assert rowwise_rel_err(out, ref) <= TOL2
