"""The fp32 passes' choice between operands straight from memory and tiles in LDS (CPU only)."""
import pytest

from plan_lib import f32_direct


@pytest.mark.parametrize("d", [64, 128])
def test_offsets_hold_in_32_bits(d):
    """The forward tells rows up to four apart and 32 columns, the backward 32 rows and all columns by 32-bit byte offsets; strides are
    multiples of 8 elements."""
    ways = {st: f32_direct([40], 2, 1, d, 0, 1, q_st=st, kv_st=st) for st in ((1 << 25) - 8, 1 << 25, (1 << 28) - 8, 1 << 28)}
    assert list(ways.values()) == [(True, True), (True, False), (True, False), (False, False)]
    for st, (forward, backward) in ways.items():
        assert not forward or 4 * st * 4 + 31 * 4 < 1 << 32
        assert not backward or 31 * st * 4 + d * 4 <= 1 << 32
    assert f32_direct([40], 2, 1, d, 0, 1, q_st=1 << 28) == (True, False)   # (the forward reads rows of Q at 64-bit addresses)


@pytest.mark.parametrize("docs,hq,hkv,d,step,steps,forward", [
    ([476], 8, 1, 64, 2, 1, True),
    ([444], 8, 2, 128, 6, 1, True),         # tiles 113 us, memory 37
    ([8963], 64, 4, 64, 1, 1, False),       # 5995 and 6393
    ([4824], 64, 4, 64, 3, 1, False),       # 1822 and 1962
    ([3811], 32, 8, 64, 6, 5, False),       # 3059 and 3263
    ([5450], 32, 8, 64, 4, 3, False),       # 3514 and 3726
])
def test_forward_s_way_that_was_measured_shorter(docs, hq, hkv, d, step, steps, forward):
    assert f32_direct(docs, hq, hkv, d, step, steps)[0] == forward


@pytest.mark.parametrize("docs,hq,hkv,d,step,steps,backward", [
    ([476], 8, 1, 64, 2, 1, True),          # tiles 70 us, memory 28
    ([444], 8, 2, 128, 6, 1, True),         # 129 and 63
    ([14883], 16, 16, 64, 0, 1, True),      # 15056 and 14700
    ([16334], 8, 1, 64, 3, 3, True),        # 32152 and 26355
    ([2000], 32, 8, 128, 0, 2, False),      # 2391 and 2610
    ([876], 32, 32, 64, 2, 1, False),       # 162 and 182
    ([153] * 104, 16, 16, 64, 1, 1, False),     # 817 and 879
    ([1093], 32, 32, 128, 5, 1, False),     # 569 and 613
])
def test_backward_s_way_that_was_measured_shorter(docs, hq, hkv, d, step, steps, backward):
    assert f32_direct(docs, hq, hkv, d, step, steps)[1] == backward
