"""GPU parity of per-document step counts where one launch serves many runs of documents: more runs than a launch takes, runs
that share a 128-token tile's length, empty ones between them, more than 64 documents in one run beside others, both types,
and steps on both sides of the later blocks that one pass holds."""
import pytest

import test_gpu_docsteps as docsteps
from paper_2603_18567_amd.workloads import custom_workload

pytestmark = pytest.mark.gpu

CASES = [
    (custom_workload("slices_40", "bf16", [7, 40, 1, 33] * 10, 8, 2, 128, 4, 41), [1, 4, 2, 3] * 10),
    (custom_workload("slices_17_head64", "bf16", [20, 0, 130, 5] * 9, 6, 3, 64, 10, 42), [10, 3, 9, 0] * 9),
    (custom_workload("slices_16_many_heads", "bf16", [3, 30] * 8, 16, 1, 128, 9, 43), [9, 2] * 8),
    (custom_workload("slices_100_documents", "bf16", [200] + [2, 0, 3] * 30 + [64, 1], 4, 4, 128, 3, 44), [3] + [1] * 90 + [2, 3]),
    (custom_workload("slices_f32", "f32", [50, 1, 64, 17] * 5, 4, 2, 64, 3, 45), [2, 3, 1, 0] * 5),
    (custom_workload("slices_f32_head128", "f32", [33, 70, 5], 3, 3, 128, 4, 46), [4, 1, 2]),
]


@pytest.mark.parametrize("wl,steps", CASES, ids=[c[0].name for c in CASES])
def test_many_slices_match_oracle(wl, steps):
    docsteps.test_docsteps_match_oracle_and_leave_the_rest_alone(wl, steps)
