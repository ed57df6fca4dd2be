"""Decode attention over every way the keys can be dealt: whole heads per workgroup, heads cut
between two workgroups, heads cut into many, runs that end one head and begin the next, cache
lengths around the 128-key unit and the 32-key steps, one key, and the smaller workspace that
cuts every head alike; with a workspace and (bitwise the same) without.  2-norm bound as for
prefill: 4e-3 (numerators and output round to bf16, 1.6e-3 rms together)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2502_17728_amd import inputs as I
from tests.parity import TOL, cuda, rowwise_rel_err

pytestmark = pytest.mark.gpu

CASES = [(1, 1, 1, 128), (2, 3, 31, 64), (3, 16, 33, 128), (5, 4, 127, 64), (5, 4, 128, 128), (7, 1, 129, 128),
         (1, 16, 20000, 64), (3, 2, 9001, 128), (100, 1, 700, 128), (255, 2, 260, 128), (256, 1, 300, 128),
         (257, 4, 257, 128), (300, 1, 1000, 64), (513, 1, 129, 64), (600, 3, 400, 64), (1100, 1, 200, 128)]


def _check(case, out, BH, Lq, d):
    torch.cuda.synchronize()
    hs = sorted({0, 1 % BH, BH // 3, BH // 2, BH - 2 if BH > 1 else 0, BH - 1})
    ref = oracle.attention(case["Q"][hs].reshape(-1, d), case["K"], case["V"], case["scale"],
                           head=np.repeat(np.array(hs), Lq))
    got = out.cpu()[hs].reshape(-1, d)
    assert rowwise_rel_err(got, ref) <= TOL[torch.bfloat16]
    assert np.linalg.norm(oracle.to_f64(got) - ref) <= 4e-3 * np.linalg.norm(ref)
    assert torch.isfinite(out.float()).all()


@pytest.mark.parametrize("BH,Lq,Lk,d", CASES)
def test_deal(BH, Lq, Lk, d):
    from paper_2502_17728_amd import ops
    case = I.make_decode_case(BH, Lq, Lk, d, seed=BH + Lk)
    q, k, v = cuda(case["Q"]), cuda(case["K"]), cuda(case["V"])
    n = ops.attention_decode_workspace_bytes(BH, Lq, Lk, d)
    ws = torch.full((n + 64,), 0xff, dtype=torch.uint8, device="cuda")  # NaN partials if any were read unwritten
    out = ops.attention_decode_deferred(q, k, v, scale=case["scale"], workspace=ws[:n])
    _check(case, out, BH, Lq, d)
    assert (ws[n:] == 0xff).all()
    assert torch.equal(out, ops.attention_decode_deferred_noalloc(q, k, v, scale=case["scale"]))
    # the least workspace: every head in the same number of ranges
    w, units = (512 if d == 64 else 256), -(-Lk // 128)
    want = max(1, min(units, -(-w // BH)))
    least = BH * -(-units // -(-units // want)) * Lq * (d + 4) * 4
    ws.fill_(0xff)
    out = ops.attention_decode_deferred(q, k, v, scale=case["scale"], workspace=ws[:least])
    _check(case, out, BH, Lq, d)
    assert (ws[least:] == 0xff).all()


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("hidden", [range(0, 8192), range(0, 8200), range(4096, 11000)])
def test_runs_of_minus_infinite_scores(d, hidden):
    # whole partials (of 128 keys: one head gives more than 64) whose scores are all -inf weigh
    # nothing, wherever they lie; a row with no other score is NaN
    from paper_2502_17728_amd import ops
    case = I.make_decode_case(1, 2, 11000, d, seed=d)
    q, k, v = case["Q"].clone(), case["K"].clone(), case["V"]
    q[:, :, 0] = 1.0
    hid = torch.zeros(11000, dtype=torch.bool)
    hid[list(hidden)] = True
    k[:, hid, 0] = float("-inf")
    ref = oracle.attention(q.reshape(-1, d), k[:, ~hid], v[:, ~hid], case["scale"], head=np.zeros(2, int))
    for f in (ops.attention_decode_deferred, ops.attention_decode_deferred_noalloc):
        got = f(cuda(q), cuda(k), cuda(v), scale=case["scale"]).cpu().reshape(-1, d)
        assert rowwise_rel_err(got, ref) <= TOL[torch.bfloat16]
    k[:, :, 0] = float("-inf")
    assert torch.isnan(ops.attention_decode_deferred(cuda(q), cuda(k), cuda(v), scale=case["scale"])).all()
