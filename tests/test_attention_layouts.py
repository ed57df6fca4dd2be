"""attention_deferred on each of its prefill layouts (256, 128, 64 and 32 query rows per
workgroup, keys split 1, 2, 4 and 4 ways): ragged queries and keys around the tile edges,
causal and not, grouped queries, head counts that do and do not divide among 8 XCDs.

Bounds: the row-normwise bound of the other parity tests, and 4e-3 on the 2-norm of the
whole error -- the bf16 numerators and the bf16 output each round by 2^-9 / sqrt(3) rms at
most (1.6e-3 together), and a lost or doubled key tile moves it by far more.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2502_17728_amd import inputs as I
from tests.parity import TOL, cuda, rowwise_rel_err

pytestmark = pytest.mark.gpu

# (query heads, group, Lq, Lk, d, causal), by the layout the launcher's estimate picks
LAYOUTS = {
    256: [(96, 1, 513, 513, 128, True), (64, 4, 1025, 700, 128, False), (130, 1, 600, 600, 64, True),
          (120, 8, 1025, 129, 64, False), (260, 4, 250, 8, 128, False), (300, 1, 200, 200, 64, True),
          (100, 4, 700, 700, 128, True), (140, 1, 257, 384, 128, False),
          # the halves of a workgroup in step up to 3072 keys, one phase apart past that
          (128, 4, 511, 3072, 128, False), (128, 4, 511, 3073, 128, False), (160, 1, 511, 3200, 64, False),
          (128, 8, 500, 4999, 64, False)],
    128: [(48, 4, 520, 520, 128, True), (80, 1, 257, 640, 128, False), (64, 2, 520, 520, 64, True)],
    64: [(40, 1, 385, 300, 128, False), (96, 4, 385, 385, 64, True), (40, 1, 520, 1300, 64, False)],
    32: [(24, 8, 449, 449, 128, True), (16, 1, 193, 1500, 128, False), (3, 1, 40, 161, 128, False),
         (8, 4, 97, 97, 128, True), (5, 1, 33, 700, 64, False), (1, 1, 1, 1, 64, True), (2, 1, 17, 8, 128, False)],
}


@pytest.mark.parametrize("bq,shape", [(bq, s) for bq, shapes in LAYOUTS.items() for s in shapes])
def test_prefill_layouts(bq, shape):
    from paper_2502_17728_amd import ops
    H, g, Lq, Lk, d, causal = shape
    q = I.make_qkv_case(H, Lq, d, causal, seed=Lq + bq)["Q"]
    kv = I.make_qkv_case(H // g, Lk, d, causal, seed=Lk + 7)
    scale = 1.0 / d ** 0.5
    out = ops.attention_deferred(cuda(q), cuda(kv["K"]), cuda(kv["V"]), causal=causal, scale=scale).cpu()
    heads = sorted({0, H // 2, H - 1})  # first, a middle and the last head, every row
    rows = np.arange(len(heads) * Lq)
    ref = oracle.attention(q[heads].reshape(-1, d), kv["K"], kv["V"], scale,
                           head=np.array(heads)[rows // Lq] // g, qpos=rows % Lq if causal else None)
    got = out[heads].reshape(-1, d)
    assert rowwise_rel_err(got, ref) <= TOL[torch.bfloat16]
    assert np.linalg.norm(oracle.to_f64(got) - ref) <= 4e-3 * np.linalg.norm(ref)
    assert torch.isfinite(out.float()).all()
