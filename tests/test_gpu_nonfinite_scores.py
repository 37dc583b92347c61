"""GPU: scores that are not finite.  A NaN reaches exactly the rows that see its key.
Every case asserts the way that the launch rules choose."""
import pytest
import torch

from paper_2603_18567_amd.workloads import custom_workload
from plan_lib import f32_direct, forward_split
from ttt_testlib import Case

pytestmark = pytest.mark.gpu

CASES = [
    # dtype, documents, hq, hkv, head_dim, k, steps per call, way
    ("f32", [40], 2, 1, 64, 4, 4, "direct"),
    ("f32", [40], 2, 1, 128, 4, 4, "direct"),
    ("f32", [40] * 40, 64, 4, 64, 2, 2, "four_waves"),
    ("f32", [530], 32, 8, 128, 3, 3, "four_waves"),
    ("bf16", [300], 8, 2, 128, 4, 1, "two_key_groups"),
    ("bf16", [300, 70, 1, 29, 49], 64, 16, 128, 12, 12, "eight_waves"),
    ("bf16", [500], 32, 8, 64, 4, 1, "two_key_groups"),
    ("bf16", [70, 1, 130, 64, 33], 8, 2, 64, 4, 1, "four_waves"),
    ("bf16", [63, 200, 1, 41], 128, 32, 64, 11, 11, "eight_waves"),
]


def way_of(dtype, docs, hq, hkv, d, step, steps):
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    if dtype == "f32" and f32_direct(docs, hq, hkv, d, step, steps, n_cu)[0]:
        return "direct"
    return forward_split(docs, hq, hkv, d, dtype, step, steps, n_cu)[0]


def prepare(dtype, docs, hq, hkv, d, k, steps, way, from_step=0):
    print(f"{dtype} documents={docs} heads={hq}/{hkv} head_dim={d} k={k} steps={steps}", flush=True)
    assert all(way_of(dtype, docs, hq, hkv, d, j, steps) == way for j in range(from_step, k, steps))
    return Case(custom_workload(f"nonfinite_{dtype}_{d}_{way}", dtype, docs, hq, hkv, d, k, seed=d + len(docs)), "cuda:0")


def forward(run, steps):
    for t in run.o + run.lse:
        t.fill_(77.0)
    for j in range(0, run.K, steps):
        run.forward(j, j + steps)
    torch.cuda.synchronize()
    return [t.clone() for t in run.o], [t.clone() for t in run.lse]


@pytest.mark.parametrize("dtype,docs,hq,hkv,d,k,steps,way", CASES, ids=[f"{c[0]}_{c[4]}_{c[7]}" for c in CASES])
def test_a_nan_in_a_later_block_reaches_its_row(dtype, docs, hq, hkv, d, k, steps, way):
    """A diagonal key with a NaN, in each later block in turn: O and LSE of its token are NaN from that step on, in the heads of
    its group, and nothing else is, also where it is the first key of the row that its wave sees."""
    case = prepare(dtype, docs, hq, hkv, d, k, steps, way, from_step=1 if way == "two_key_groups" else 0)   # (step 0 has no diagonal key)
    G, row, g = hq // hkv, 5, hkv - 1
    for block in range(1, min(k, 4)):
        was = case.run.k[block][row, g, 3].clone()
        case.run.k[block][row, g, 3] = float("nan")
        o, lse = forward(case.run, steps)
        case.run.k[block][row, g, 3] = was
        for j in range(k):
            hit = torch.zeros(hq, sum(docs), dtype=torch.bool, device="cuda:0")
            hit[g * G:(g + 1) * G, row] = j >= block
            assert torch.equal(lse[j].isnan(), hit), f"LSE[{j}], NaN in block {block}"
            assert torch.equal(o[j].isnan(), hit.T[..., None].expand_as(o[j])), f"O[{j}], NaN in block {block}"


@pytest.mark.parametrize("dtype,docs,hq,hkv,d,k,steps,way", CASES, ids=[f"{c[0]}_{c[4]}_{c[7]}" for c in CASES])
def test_a_later_block_s_score_of_minus_infinity_has_no_weight(dtype, docs, hq, hkv, d, k, steps, way):
    """The same O and LSE as with a score too low to count, also where it is the first key of the row that its wave sees."""
    case = prepare(dtype, docs, hq, hkv, d, k, steps, way, from_step=1 if way == "two_key_groups" else 0)
    for t in case.q:
        t[..., 0].abs_().add_(0.1)
    outputs = []
    for low in (-1e30, float("-inf")):
        for t in case.k[1:]:
            t[::3, :, 0] = low
        outputs.append(sum(forward(case.run, steps), []))
    for finite, infinite in zip(*outputs):
        assert bool(finite.isfinite().all())
        assert torch.equal(finite, infinite)


@pytest.mark.parametrize("dtype,docs,hq,hkv,d,k,steps,way", CASES, ids=[f"{c[0]}_{c[4]}_{c[7]}" for c in CASES])
def test_a_row_whose_scores_are_all_minus_infinity(dtype, docs, hq, hkv, d, k, steps, way):
    """The sum of its weights is 0: LSE is -inf and O is 0 / 0, in every split.  The rows that see other keys as well are finite."""
    case = prepare(dtype, docs, hq, hkv, d, k, steps, way, from_step=1 if way == "two_key_groups" else 0)
    for t in case.q:
        t[..., 0].abs_().add_(0.1)
    for t in case.k:
        t[0, :, 0] = float("-inf")
    o, lse = forward(case.run, steps)
    for j in range(k):
        assert bool((lse[j][:, 0] == float("-inf")).all()) and bool(lse[j][:, 1:].isfinite().all()), f"LSE[{j}]"
        assert bool(o[j][0].isnan().all()) and bool(o[j][1:].isfinite().all()), f"O[{j}]"
