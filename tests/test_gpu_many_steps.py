"""GPU parity of the backward with more steps than one pass of the preprocess kernel holds later blocks for (7):
one block more, two full passes, and the first block of a third; all steps in one call, in the training order
with the fp32 carry, and in calls of several steps."""
import pytest
import torch

from paper_2603_18567_amd.workloads import custom_workload
from ttt_testlib import Case, compare_full

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k,d,calls", [(8, 128, 1), (9, 128, 1), (9, 64, 9), (15, 128, 15), (16, 64, 1), (16, 128, 3)])
def test_many_steps_match_oracle(k, d, calls):
    print(f"k={k} d={d} backward calls={calls}", flush=True)
    wl = custom_workload(f"steps_{k}_{d}", "bf16", [70, 1, 33], 4, 2, d, k, seed=60 + k)
    case = Case(wl, "cuda:0")
    case.run.forward()
    if calls == 1:
        case.run.backward(case.d_o)
    else:
        cuts = [round(k * i / calls) for i in range(calls + 1)]
        for i in reversed(range(calls)):
            case.run.backward(case.d_o, cuts[i], cuts[i + 1], accumulate=True)
    torch.cuda.synchronize()
    for key, (err, bound) in compare_full(case).items():
        assert err <= bound, f"{key}: {err:.3e} > {bound:.3e}"


def test_many_steps_times_heads_match_oracle():
    """32 steps of 41 query heads per kv head: the bf16 kernels set no limit on (step, head) pairs (1312 here; a
    preprocess that kept D in LDS would have room for 1280)."""
    wl = custom_workload("steps_32_heads_41", "bf16", [21, 5], 41, 1, 64, 32, seed=93)
    print("k=32 d=64 heads=41/1", flush=True)
    case = Case(wl, "cuda:0")
    case.run.forward()
    case.run.backward(case.d_o)
    torch.cuda.synchronize()
    for key, (err, bound) in compare_full(case).items():
        assert err <= bound, f"{key}: {err:.3e} > {bound:.3e}"
