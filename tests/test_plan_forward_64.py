"""The head_dim 64 forward's split (CPU only), each shape with what eight waves, four waves and two key groups were measured to take: one
document or several, first and late steps, few long workgroups, several rounds of the device and many short ones."""
import pytest

from plan_lib import forward_split


@pytest.mark.parametrize("docs,hq,hkv,step,steps,split", [
    ([1118], 12, 2, 0, 5, "four_waves"),              # 33, 25 and 33 us
    ([3318], 32, 8, 9, 1, "four_waves"),              # 98, 73 and 97
    ([247, 436], 64, 4, 9, 1, "four_waves"),          # 23, 18 and 22
    ([1499, 1468], 16, 16, 0, 5, "four_waves"),       # 105, 85 and 114
    ([8843], 12, 2, 4, 1, "four_waves"),              # 214, 166 and 197
    ([1414], 24, 8, 8, 1, "two_key_groups"),          # 46, 37 and 26
    ([444, 320], 24, 8, 9, 1, "two_key_groups"),      # 33, 23 and 17
    ([2493, 1235, 212], 12, 2, 3, 1, "two_key_groups"),   # 64, 58 and 41
    ([7640], 8, 2, 0, 1, "two_key_groups"),           # 151, 104 and 83
    ([3613, 2031], 12, 2, 5, 1, "two_key_groups"),    # 90, 83 and 59: a document that starts inside a wave's rows
    ([65536], 16, 4, 0, 7, "eight_waves"),            # more than sixteen of the largest workgroups to a unit
    ([497, 69], 24, 8, 10, 1, "two_key_groups"),      # short packed batches: 34, 23 and 17
    ([183, 183, 66], 16, 16, 10, 4, "two_key_groups"),    # 34, 22 and 16
    ([86, 145, 88], 32, 8, 3, 4, "four_waves"),       # 14, 11 and 17
    ([91, 146, 79], 64, 4, 10, 6, "eight_waves"),     # 27, 29 and 47
])
def test_the_split_that_was_measured_shortest(docs, hq, hkv, step, steps, split):
    assert forward_split(docs, hq, hkv, 64, "bf16", step, steps)[0] == split
