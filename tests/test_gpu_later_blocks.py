"""GPU parity of the later blocks' dK, dV where they are made beside the streaming passes and where the preprocess launch makes
them: tokens and heads that do not fill a workgroup of either launch, one block, as many as one pass holds and one more, a
call that sees no later block, and one fp32 carry that calls of both ways continue."""
import pytest
import torch

from paper_2603_18567_amd.workloads import custom_workload
from plan_lib import later_blocks_apart
from ttt_testlib import Case, compare_full

pytestmark = pytest.mark.gpu

# documents, hq, hkv, head_dim, k, steps of the backward's calls (descending), made by the preprocess launch?
CASES = [
    ([1], 3, 3, 128, 2, [2], [False]),
    ([31], 6, 3, 64, 1, [1], [False]),
    ([33, 30], 6, 2, 64, 8, [8], [False]),
    ([20, 45], 5, 1, 128, 9, [1] * 9, [False] * 9),
    ([64, 1, 31], 32, 2, 128, 3, [2, 1], [False, False]),
    ([250, 51], 32, 8, 128, 9, [9], [True]),
    ([520, 3], 32, 8, 64, 10, [10], [True]),
    ([300, 221], 32, 8, 128, 9, [5, 1, 2, 1], [True, False, False, False]),
]


@pytest.mark.parametrize("docs,hq,hkv,d,k,calls,apart", CASES, ids=[f"{sum(c[0])}_{c[1]}_{c[2]}_{c[3]}_{c[4]}_{len(c[5])}" for c in CASES])
def test_later_blocks_match_oracle(docs, hq, hkv, d, k, calls, apart):
    print(f"documents={docs} heads={hq}/{hkv} head_dim={d} k={k} calls={calls}", flush=True)
    case = Case(custom_workload(f"later_{sum(docs)}_{d}", "bf16", docs, hq, hkv, d, k, seed=k + hq), "cuda:0")
    case.run.forward()
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    ways, end = [], k
    for n in calls:
        ways.append(later_blocks_apart(sum(docs), hq, hkv, d, end - n, n, n_cu))
        case.run.backward(case.d_o, end - n, end, accumulate=len(calls) > 1)
        end -= n
    assert end == 0 and ways == apart
    torch.cuda.synchronize()
    for key, (err, bound) in compare_full(case).items():
        assert err <= bound, f"{key}: {err:.3e} > {bound:.3e}"
