"""GPU parity of the forward where a row's diagonal keys come through more LDS slots than lie behind the key tiles: the slots and
the freed tile stages in turn, back to the slots, with 4, 2 and 1 query heads per workgroup, ragged last rows and as few key
tiles as one.  Forward only: the backward does not share this code."""
import pytest
import torch

import oracle as O
from paper_2603_18567_amd.workloads import custom_workload
from plan_lib import forward_split
from ttt_testlib import Case, check, to_np32

pytestmark = pytest.mark.gpu

CASES = [
    # documents, hq, hkv, head_dim, k, steps per call, split, heads per workgroup
    ([31], 4, 1, 128, 12, 1, "two_key_groups", 4),
    ([70, 1, 62], 12, 2, 128, 8, 1, "two_key_groups", 2),
    ([300, 70, 1, 29, 49], 64, 16, 128, 12, 12, "eight_waves", 4),
    ([300, 70, 1, 29, 49], 48, 8, 128, 12, 12, "eight_waves", 2),
    ([33, 64, 2], 8, 2, 64, 10, 1, "four_waves", 4),
    ([33, 64, 2], 48, 24, 64, 10, 10, "four_waves", 2),
    ([63, 200, 1, 41], 128, 32, 64, 12, 12, "eight_waves", 4),
    ([63, 200, 1, 41], 192, 96, 64, 15, 15, "eight_waves", 2),
    ([3, 1030, 40], 4, 1, 64, 9, 1, "two_key_groups", 4),
    ([1060], 3, 3, 64, 5, 1, "two_key_groups", 1),
]


@pytest.mark.parametrize("docs,hq,hkv,d,k,steps,split,heads", CASES, ids=[f"{sum(c[0])}_{c[1]}_{c[2]}_{c[3]}_{c[4]}" for c in CASES])
def test_many_diagonal_keys_match_oracle(docs, hq, hkv, d, k, steps, split, heads):
    print(f"documents={docs} heads={hq}/{hkv} head_dim={d} k={k}", flush=True)
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    assert forward_split(docs, hq, hkv, d, "bf16", k - steps, steps, n_cu) == (split, heads)
    wl = custom_workload(f"slots_{sum(docs)}_{hq}", "bf16", docs, hq, hkv, d, k, seed=hq + k)
    case = Case(wl, "cuda:0")
    for t in case.run.o + case.run.lse:
        t.fill_(float("nan"))
    for j in range(0, k, steps):
        case.run.forward(j, j + steps)
    torch.cuda.synchronize()
    Q, K, V, _ = case.oracle_inputs()
    o, lse = O.oracle_full(Q, K, V, wl.cu_seqlens, wl.scale, None, 0, k)[:2]
    for j in range(k):
        check(f"O[{j}]", to_np32(case.run.o[j]), o[j], wl.dtype, rows=True)
        check(f"LSE[{j}]", to_np32(case.run.lse[j]), lse[j], wl.dtype, lse=True)
