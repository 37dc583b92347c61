"""GPU parity of the forward where a workgroup's waves are split into two key groups (launches of few, long
workgroups): rows whose keys all lie in one group's tiles, an odd number of tiles, ragged last rows, document
starts inside a tile pair, 4, 2 and 1 query heads per workgroup, and no, one, two and more diagonal keys."""
import pytest
import torch

from paper_2603_18567_amd.workloads import custom_workload
from ttt_testlib import Case, compare_full

pytestmark = pytest.mark.gpu

CASES = [
    ("one_tile", [50], 8, 2, 2),
    ("two_tiles_ragged", [127], 8, 2, 3),
    ("odd_tiles", [321], 4, 1, 4),
    ("documents_inside_tile_pairs", [70, 1, 130, 64, 33], 8, 2, 4),
    ("two_heads_per_workgroup", [200, 95], 12, 2, 5),
    ("one_head_per_workgroup", [260, 3], 3, 3, 4),
]


# head_dim 64: two key groups while there are few, long workgroups; four waves while there are few; eight otherwise
CASES_64 = [
    ("two_key_groups", [1100], 4, 1, 2, 1),
    ("two_key_groups_documents", [3, 1030, 40], 2, 2, 3, 1),
    ("four_waves", [70, 1, 130, 64, 33], 8, 2, 4, 1),
    ("four_waves_one_head", [200, 95], 3, 3, 3, 1),
    ("eight_waves", [63, 200, 1, 336], 32, 8, 4, 4),
]


def run(name, docs, hq, hkv, d, k, steps_per_call):
    print(f"case {name} documents={docs} heads={hq}/{hkv} head_dim={d} k={k}", flush=True)
    wl = custom_workload(f"groups_{name}", "bf16", docs, hq, hkv, d, k, seed=len(docs) + 5)
    case = Case(wl, "cuda:0")
    for j in range(0, k, steps_per_call):
        case.run.forward(j, j + steps_per_call)
    case.run.backward(case.d_o)
    torch.cuda.synchronize()
    for key, (err, bound) in compare_full(case).items():
        assert err <= bound, f"{key}: {err:.3e} > {bound:.3e}"


@pytest.mark.parametrize("name,docs,hq,hkv,k", CASES, ids=[c[0] for c in CASES])
def test_two_key_groups_match_oracle(name, docs, hq, hkv, k):
    run(name, docs, hq, hkv, 128, k, 1)


@pytest.mark.parametrize("name,docs,hq,hkv,k,steps", CASES_64, ids=[c[0] for c in CASES_64])
def test_head_dim_64_splits_match_oracle(name, docs, hq, hkv, k, steps):
    run(name, docs, hq, hkv, 64, k, steps)


@pytest.mark.parametrize("docs,hq,hkv,d,k,steps", [([128], 4, 4, 64, 3, 3), ([300], 8, 2, 64, 1, 1), ([65, 1, 70], 8, 2, 64, 2, 1),
                                                   ([200, 3], 8, 1, 128, 2, 1), ([250], 3, 1, 64, 1, 1)])
def test_fp32_short_launches_match_oracle(docs, hq, hkv, d, k, steps):
    """fp32: two key groups in the forward (head_dim 64), query rows of a key tile split over workgroups in the
    backward, also into more parts than a tile has query tiles."""
    print(f"fp32 documents={docs} heads={hq}/{hkv} head_dim={d} k={k}", flush=True)
    case = Case(custom_workload(f"f32_{len(docs)}_{d}_{k}", "f32", docs, hq, hkv, d, k, seed=d + len(docs)), "cuda:0")
    for j in range(0, k, steps):
        case.run.forward(j, j + steps)
    for j in reversed(range(0, k, steps)):
        case.run.backward(case.d_o, j, j + steps, accumulate=steps < k)
    torch.cuda.synchronize()
    for key, (err, bound) in compare_full(case).items():
        assert err <= bound, f"{key}: {err:.3e} > {bound:.3e}"
