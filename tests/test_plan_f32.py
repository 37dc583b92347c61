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
