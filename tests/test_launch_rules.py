"""The parity tests' sizes against the launch rules (CPU): each reaches the kernel and layout its
test names, so that a change of a rule cannot leave a kernel untested."""
import pytest

from tests import launch_rules as R
from tests import test_attention_layouts, test_softmax_layouts


def test_attention_layout_sizes():
    for bq, shapes in test_attention_layouts.LAYOUTS.items():
        for H, _, Lq, Lk, d, causal in shapes:
            assert R.prefill(H, Lq, Lk, d, causal) == bq, (H, Lq, Lk, d, causal)
    phased = [(s, R.phased(s[3])) for s in test_attention_layouts.LAYOUTS[256]]
    for d in (64, 128):  # both schedules of the 256-query layout
        assert {p for s, p in phased if s[4] == d} == {True, False}


def test_softmax_layout_sizes():
    for name, shapes in test_softmax_layouts.LAYOUTS.items():
        for BH, L, d, causal in shapes:
            assert R.softmax(BH, L, L, d, causal) == name, (BH, L, d, causal)
    for name, shapes in test_softmax_layouts.RAGGED.items():
        for BH, Lq, Lk, d in shapes:
            assert R.softmax(BH, Lq, Lk, d, False) == name, (BH, Lq, Lk, d)


def test_few_row_rule():
    # calls that the streamed kernel takes and calls that it had slowed, by the measurements beside the rule
    for M, K, N, plain, name in [(512, 768, 2304, True, "streamed"), (4096, 768, 768, True, "tiles128"),
                                 (1500, 768, 2304, True, "tiles128"), (1500, 768, 2304, False, "streamed"),
                                 (4096, 768, 768, False, "tiles128"), (3300, 768, 768, False, "streamed"),
                                 (3000, 1024, 1024, False, "streamed"), (5500, 752, 1176, False, "two_stage"),
                                 (3100, 752, 1176, False, "streamed"), (17, 752, 1176, True, "streamed")]:
        assert R.product(M, K, N, plain=plain) == name, (M, K, N, plain)
    assert R.product(3100, 752, 1176, gated=True) == "two_stage"
