"""GPU parity of the forward's work splits.  Two key groups per workgroup (launches of few, long workgroups): rows
whose keys all lie in one group's tiles, an odd number of tiles, ragged last rows, document starts inside a tile
pair, 4, 2 and 1 query heads per workgroup, and no, one, two and more diagonal keys.  One key group (launches of
many workgroups): the same heads per workgroup, rows of several documents in a wave, and more documents than the
kernel looks up by itself.  Every test asserts the split that the launch rules choose for its calls."""
import pytest
import torch

import oracle as O
from paper_2603_18567_amd.workloads import custom_workload
from plan_lib import f32_direct, forward_split
from ttt_testlib import Case, check, compare_full, to_np32

pytestmark = pytest.mark.gpu

CASES = [
    ("one_tile", [50], 8, 2, 2),   # (without a diagonal key, at step 0, one key group is enough)
    ("two_tiles_ragged", [127], 8, 2, 3),
    ("odd_tiles", [321], 4, 1, 4),
    ("documents_inside_tile_pairs", [70, 1, 130, 64, 33], 8, 2, 4),
    ("two_heads_per_workgroup", [200, 95], 12, 2, 5),
    ("one_head_per_workgroup", [260, 3], 3, 3, 4),
]


# head_dim 64: two key groups for few, long workgroups; four waves for more or shorter ones; eight for many.  (The splits' estimates
# choose; with one or two heads to a workgroup eight waves are left for more than sixteen workgroups per compute unit.)
CASES_64 = [
    ("two_key_groups", [1100], 4, 1, 2, 1),
    ("two_key_groups_documents", [3, 1030, 40], 2, 2, 3, 1),
    ("four_waves", [70, 1, 130, 64, 33], 8, 2, 4, 1),
    ("four_waves_one_head", [200, 95], 96, 32, 3, 1),
    ("eight_waves", [63, 200, 1, 41], 128, 32, 11, 11),
    ("four_waves_two_heads", [33, 1, 130, 64], 128, 64, 4, 1),       # 64 rows: diagonal rows through LDS
    ("eight_waves_one_head", [63, 200, 1, 41], 128, 128, 17, 17),
    ("eight_waves_two_heads", [63, 200, 1, 41], 192, 96, 15, 15),
    ("eight_waves_70_documents", [9, 1, 0, 17, 5] * 14, 144, 48, 15, 15),
]


def compute_units():
    return torch.cuda.get_device_properties(0).multi_processor_count


def splits_of_calls(docs, hq, hkv, d, dtype, k, steps_per_call):
    return [forward_split(docs, hq, hkv, d, dtype, j, steps_per_call, compute_units()) for j in range(0, k, steps_per_call)]


def run(name, docs, hq, hkv, d, k, steps_per_call, split):
    print(f"case {name} documents={docs} heads={hq}/{hkv} head_dim={d} k={k}", flush=True)
    assert all(s == split for s, _ in splits_of_calls(docs, hq, hkv, d, "bf16", k, steps_per_call)[int(name == "one_tile"):])
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
    run(name, docs, hq, hkv, 128, k, 1, "two_key_groups")


@pytest.mark.parametrize("name,docs,hq,hkv,k,steps", CASES_64, ids=[c[0] for c in CASES_64])
def test_head_dim_64_splits_match_oracle(name, docs, hq, hkv, k, steps):
    run(name, docs, hq, hkv, 64, k, steps, next(s for s in ("two_key_groups", "four_waves", "eight_waves") if name.startswith(s)))


# head_dim 128, one key group: launches of more than six rounds of the device
ONE_GROUP = [
    # name, documents, hq, hkv, k, query heads per workgroup
    ("one_head", [300, 70, 1, 0, 29, 150, 47], 64, 64, 9, 1),
    ("one_head_of_three", [301, 70, 1, 29, 150, 149], 48, 16, 11, 1),
    ("two_heads", [300, 70, 1, 29, 150, 101], 32, 16, 17, 2),
    ("two_heads_of_six", [75, 300, 70, 1, 29, 176], 48, 8, 11, 2),
    ("one_head_100_documents", [5, 0, 11, 1, 13] * 20, 64, 64, 9, 1),
    ("two_heads_70_documents", [20, 7, 0, 1, 19, 13, 4] * 10, 32, 16, 17, 2),
    ("four_heads_80_documents", [30, 7, 17, 1] * 20, 32, 8, 11, 4),
]


@pytest.mark.parametrize("name,docs,hq,hkv,k,heads", ONE_GROUP, ids=[c[0] for c in ONE_GROUP])
def test_one_key_group_matches_oracle(name, docs, hq, hkv, k, heads):
    """Forward only: many heads and steps make the workgroups, and the backward does not depend on the split."""
    print(f"case {name} documents={docs} heads={hq}/{hkv} k={k}", flush=True)
    assert splits_of_calls(docs, hq, hkv, 128, "bf16", k, k) == [("eight_waves", heads)]
    wl = custom_workload(f"one_group_{name}", "bf16", docs, hq, hkv, 128, k, seed=len(docs) + 31)
    case = Case(wl, "cuda:0")
    for t in case.run.o + case.run.lse:
        t.fill_(float("nan"))
    case.run.forward()
    torch.cuda.synchronize()
    Q, K, V, _ = case.oracle_inputs()
    o, lse = O.oracle_full(Q, K, V, wl.cu_seqlens, wl.scale, None, 0, k)[:2]
    for j in range(k):
        check(f"O[{j}]", to_np32(case.run.o[j]), o[j], wl.dtype, rows=True)
        check(f"LSE[{j}]", to_np32(case.run.lse[j]), lse[j], wl.dtype, lse=True)


def run_fp32(docs, hq, hkv, d, k, steps):
    print(f"fp32 documents={docs} heads={hq}/{hkv} head_dim={d} k={k}", flush=True)
    case = Case(custom_workload(f"f32_{len(docs)}_{d}_{k}", "f32", docs, hq, hkv, d, k, seed=d + len(docs)), "cuda:0")
    for j in range(0, k, steps):
        case.run.forward(j, j + steps)
    for j in reversed(range(0, k, steps)):
        case.run.backward(case.d_o, j, j + steps, accumulate=steps < k)
    torch.cuda.synchronize()
    for key, (err, bound) in compare_full(case).items():
        assert err <= bound, f"{key}: {err:.3e} > {bound:.3e}"


@pytest.mark.parametrize("docs,hq,hkv,d,k,steps", [([128], 4, 4, 64, 3, 3), ([300], 8, 2, 64, 1, 1), ([65, 1, 70], 8, 2, 64, 2, 1),
                                                   ([200, 3], 8, 1, 128, 2, 1), ([250], 3, 1, 64, 1, 1)])
def test_fp32_short_launches_match_oracle(docs, hq, hkv, d, k, steps):
    """fp32 with work for few compute units: operands straight from memory in both passes."""
    assert all(f32_direct(docs, hq, hkv, d, j, steps, compute_units()) == (True, True) for j in range(0, k, steps))
    run_fp32(docs, hq, hkv, d, k, steps)


@pytest.mark.parametrize("docs,hq,hkv,k,steps,heads", [([98], 64, 4, 6, 2, 2), ([119, 7, 15], 64, 4, 3, 1, 2), ([46, 152, 101, 21], 24, 8, 6, 2, 1),
                                                       ([83, 175, 164, 13, 85, 30], 12, 12, 6, 2, 1)])
def test_fp32_two_key_groups_match_oracle(docs, hq, hkv, k, steps, heads):
    """fp32, head_dim 64: tiles in LDS in the forward, with two key groups."""
    for j in range(0, k, steps):
        assert not f32_direct(docs, hq, hkv, 64, j, steps, compute_units())[0]
    assert all(x == ("two_key_groups", heads) for x in splits_of_calls(docs, hq, hkv, 64, "f32", k, steps))
    run_fp32(docs, hq, hkv, 64, k, steps)


@pytest.mark.parametrize("docs,hq,hkv,d,k,backward", [([150, 1, 82], 32, 32, 64, 8, True), ([200, 60, 70], 64, 16, 64, 3, True), ([150, 1, 82, 290], 32, 8, 128, 5, True),
                                                      ([530, 1, 82], 32, 8, 128, 3, False)])
def test_fp32_full_launches_match_oracle(docs, hq, hkv, d, k, backward):
    """fp32 with work for every compute unit: tiles in LDS in the forward, with one key group; in the backward with long documents alone."""
    assert f32_direct(docs, hq, hkv, d, 0, k, compute_units()) == (False, backward)
    assert [s for s, _ in splits_of_calls(docs, hq, hkv, d, "f32", k, k)] == ["four_waves"]
    run_fp32(docs, hq, hkv, d, k, k)
