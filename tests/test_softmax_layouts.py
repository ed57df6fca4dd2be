"""softmax_pv_deferred on each of its layouts (256, 128 and 64 queries per workgroup, and 32 with
the keys split), causal and not, ragged queries and keys.  Bounds as for the attention layouts."""
import numpy as np
import pytest
import torch

import oracle
from paper_2502_17728_amd import inputs as I
from tests.parity import TOL, cuda, rowwise_rel_err

pytestmark = pytest.mark.gpu


# (heads, L, d, causal): n256 = heads ceil(L / 256), n128 = heads ceil(L / 128) pick the layout
@pytest.mark.parametrize("BH,L,d,causal", [
    (520, 248, 64, True), (260, 264, 128, True), (171, 136, 128, False), (130, 264, 64, False),   # 256
    (170, 200, 128, True), (85, 488, 64, True), (100, 232, 64, False), (170, 120, 128, False),    # 128
    (3, 8, 64, True), (9, 200, 128, True), (50, 776, 64, True), (4, 1160, 128, False), (2, 64, 64, False),  # 64
    (5, 72, 128, False), (12, 512, 64, False), (20, 904, 128, False)])                            # split
def test_layouts(BH, L, d, causal):
    from paper_2502_17728_amd import ops
    c = I.make_sm_case(BH, L, d, causal, seed=BH + L)
    out = ops.softmax_pv_deferred(cuda(c["S"]), cuda(c["V"]), causal=causal).cpu()
    hs = sorted({0, BH // 2, BH - 1})
    rows = np.arange(len(hs) * L)
    ref = oracle.softmax_pv(c["S"][hs].reshape(-1, L), c["V"], head=np.array(hs)[rows // L],
                            qpos=rows % L if causal else None)
    got = out[hs].reshape(-1, d)
    assert rowwise_rel_err(got, ref) <= TOL[torch.bfloat16]
    assert np.linalg.norm(oracle.to_f64(got) - ref) <= 4e-3 * np.linalg.norm(ref)
    assert torch.isfinite(out.float()).all()
