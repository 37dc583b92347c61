"""The split of short 16-bit backward launches (CPU only), each shape with what it was measured to take with the split of the
longer launches and with the one that is estimated shortest: two key groups where they gained, the first one where the other lost."""
import pytest

from plan_lib import _cu, backward_launch, backward_split


@pytest.mark.parametrize("docs,hq,hkv,d,step,steps,groups", [
    ([1054], 8, 1, 128, 4, 1, 2),           # 63 and 35 us
    ([1763], 8, 2, 128, 0, 1, 2),           # 79 and 49
    ([318, 457], 12, 2, 64, 6, 1, 2),       # 33 and 19
    ([1694], 8, 2, 64, 8, 1, 2),            # 55 and 34
    ([151], 24, 8, 64, 5, 3, 1),            # 19 and 25
    ([668], 8, 1, 64, 2, 6, 1),             # 50 and 66
    ([436], 12, 2, 64, 7, 5, 1),            # 45 and 57
    ([96, 102], 32, 8, 64, 3, 8, 1),        # 53 and 62
    ([403, 227], 32, 8, 128, 3, 7, 1),      # 147 and 159
    ([168], 24, 8, 128, 0, 5, 1),           # 28 and 30
    ([666], 8, 1, 128, 4, 4, 1),            # 45 and 61
])
def test_another_split_only_where_it_gains(docs, hq, hkv, d, step, steps, groups):
    *split, dq_groups = backward_launch(docs, hq, hkv, d, step, steps)
    assert dq_groups == groups
    assert groups == 2 or tuple(split) == backward_split(_cu(docs), hq, hkv, d, step, steps)
