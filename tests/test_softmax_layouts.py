"""softmax_pv_deferred on each of its layouts (256, 128, 64 and 32 queries per workgroup, and
32 with the keys split), causal and not, ragged queries and keys.  Bounds as for the attention layouts."""
import numpy as np
import pytest
import torch

import oracle
from paper_2502_17728_amd import inputs as I
from tests.parity import TOL, cuda, rowwise_rel_err

pytestmark = pytest.mark.gpu


# (heads, L, d, causal) by the layout the launcher picks
LAYOUTS = {
    "256": [(520, 248, 64, True), (260, 264, 128, True), (171, 136, 128, False), (130, 264, 64, False)],
    "128": [(170, 200, 128, True), (85, 488, 64, True), (50, 776, 64, True), (100, 232, 64, False),
            (170, 120, 128, False)],
    "64": [(9, 200, 128, True), (4, 1160, 128, True), (16, 1160, 128, False)],
    "32": [(3, 8, 64, True), (40, 200, 64, True), (2, 776, 64, True), (2, 64, 64, False), (5, 40, 128, False)],
    "split": [(5, 72, 128, False), (12, 512, 64, False), (20, 904, 128, False), (4, 1160, 128, False)],
}
# (heads, Lq, Lk, d): few queries against many keys, and the other way about
RAGGED = {
    "256": [(300, 1, 136, 64), (40, 1000, 72, 128)],
    "128": [(200, 33, 520, 128), (21, 1024, 8, 64)],
    "64": [(100, 100, 2056, 64), (40, 300, 1032, 128)],
    "32": [(3, 300, 64, 64), (7, 1, 8, 128), (2, 33, 56, 64)],
    "split": [(8, 32, 8192, 128), (1, 17, 4104, 64), (3, 1, 1032, 128), (5, 33, 2048, 64), (60, 100, 1096, 128),
              (80, 100, 2048, 64), (200, 30, 200, 128)],
}


@pytest.mark.parametrize("BH,Lq,Lk,d", [c for cs in RAGGED.values() for c in cs])
def test_ragged(BH, Lq, Lk, d):
    from paper_2502_17728_amd import ops
    g = torch.Generator().manual_seed(BH + Lk)
    S = (torch.randn(BH, Lq, Lk, generator=g) * 2).to(torch.bfloat16)
    V = torch.randn(BH, Lk, d, generator=g).to(torch.bfloat16)
    out = ops.softmax_pv_deferred(cuda(S), cuda(V)).cpu()
    hs = sorted({0, BH // 2, BH - 1})
    ref = oracle.softmax_pv(S[hs].reshape(-1, Lk), V, head=np.repeat(np.array(hs), Lq))
    got = out[hs].reshape(-1, d)
    assert rowwise_rel_err(got, ref) <= TOL[torch.bfloat16]
    assert np.linalg.norm(oracle.to_f64(got) - ref) <= 4e-3 * np.linalg.norm(ref)
    assert torch.isfinite(out.float()).all()


@pytest.mark.parametrize("BH,L,d,causal", [c for cs in LAYOUTS.values() for c in cs])
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
