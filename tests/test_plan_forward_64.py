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
    ([65536], 16, 4, 0, 7, "eight_waves"),            # more than sixteen of the largest workgroups to a unit
    ([320, 319], 16, 16, 0, 1, "four_waves"),         # a packed batch of fewer than 640 tokens: by the number of workgroups
    ([320, 319], 14, 2, 0, 7, "eight_waves"),
])
def test_the_split_that_was_measured_shortest(docs, hq, hkv, step, steps, split):
    assert forward_split(docs, hq, hkv, 64, "bf16", step, steps)[0] == split
