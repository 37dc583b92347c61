"""GPU parity of the fp32 passes with operands straight from memory (rows, keys and documents that end inside a block of 32, more key
blocks and diagonal keys than waves, more than 64 documents, strided views) and of the tiles in LDS that large launches, the backward of
rows 2^25 elements apart and the forward of rows 2^28 apart take.  Every case asserts the way that the launch rules choose for its passes."""
import pytest
import torch

from paper_2603_18567_amd import TttAttnRunner
from paper_2603_18567_amd.workloads import custom_workload
from plan_lib import f32_direct
from ttt_testlib import Case, compare_full

pytestmark = pytest.mark.gpu

CASES = [
    # documents, hq, hkv, head_dim, k, steps per call, (forward, backward) straight from memory
    ([1], 2, 1, 64, 3, 1, (True, True)),
    ([32], 3, 1, 128, 2, 2, (True, True)),
    ([31, 1, 33], 4, 2, 64, 3, 3, (True, True)),
    ([300, 0, 65], 4, 2, 128, 2, 1, (True, True)),        # ten key blocks: some waves have two
    ([70], 4, 4, 128, 12, 12, (True, True)),              # eleven diagonal keys
    ([33, 40], 8, 1, 64, 11, 1, (True, True)),
    ([20, 30] * 35, 4, 1, 128, 2, 1, (True, True)),       # bounds per token
    ([700], 4, 1, 64, 2, 2, (True, True)),
    ([40] * 40, 64, 4, 64, 2, 2, (False, True)),
    ([513, 1, 6], 16, 16, 128, 6, 6, (True, False)),
    ([300, 64, 1, 500], 32, 32, 64, 2, 1, [(True, True), (True, False)]),   # one (step, head) pair: the later step's backward
    ([530], 32, 8, 128, 3, 3, (False, False)),
]


def passes(run, d_o, k, steps):
    for j in range(0, k, steps):
        run.forward(j, j + steps)
    for j in reversed(range(0, k, steps)):
        run.backward(d_o, j, j + steps, accumulate=steps < k)
    torch.cuda.synchronize()


@pytest.mark.parametrize("docs,hq,hkv,d,k,steps,direct", CASES, ids=[f"{sum(c[0])}_{len(c[0])}_{c[1]}_{c[2]}_{c[3]}_{c[4]}" for c in CASES])
def test_f32_matches_oracle(docs, hq, hkv, d, k, steps, direct):
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    print(f"documents={docs} heads={hq}/{hkv} head_dim={d} k={k} steps={steps}", flush=True)
    ways = [f32_direct(docs, hq, hkv, d, j, steps, n_cu) for j in range(0, k, steps)]
    assert ways == (direct if isinstance(direct, list) else [direct] * len(ways))
    case = Case(custom_workload(f"f32_direct_{sum(docs)}_{d}", "f32", docs, hq, hkv, d, k, seed=sum(docs) + k), "cuda:0")
    for t in case.run.o + case.run.lse:
        t.fill_(float("nan"))
    passes(case.run, case.d_o, k, steps)
    for key, (err, bound) in compare_full(case).items():
        assert err <= bound, f"{key}: {err:.3e} > {bound:.3e}"


@pytest.mark.parametrize("docs,hq,hkv,d,k,row,head,direct", [
    ([45, 50], 4, 2, 64, 3, 4 * 72 + 40, 72, (True, True)), ([66], 2, 2, 128, 2, 2 * 136, 136, (True, True)),
    ([40] * 40, 64, 4, 64, 2, 64 * 72, 72, (False, True)), ([530], 32, 8, 128, 3, 32 * 136, 136, (False, False)),
    ([31, 6], 2, 1, 64, 1, 1 << 25, 64, (True, False)), ([34], 2, 1, 128, 1, 1 << 25, 128, (True, False))],
    ids=["strided_64", "strided_128", "strided_tiles_64", "strided_tiles_128", "far_rows_64", "far_rows_128"])
def test_f32_strided_views_match_oracle(docs, hq, hkv, d, k, row, head, direct):
    """Rows `row` elements apart, heads `head`: what lies between keeps a sentinel."""
    print(f"documents={docs} heads={hq}/{hkv} head_dim={d} k={k} strides={row},{head}", flush=True)
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    assert f32_direct(docs, hq, hkv, d, 0, k, n_cu, row, row) == direct
    case = Case(custom_workload(f"f32_strided_{sum(docs)}_{d}", "f32", docs, hq, hkv, d, k, seed=k + d), "cuda:0")
    sentinel, bufs = 77.0, []

    def wide(t, copy=True):
        buf = torch.full(((t.shape[0] - 1) * row + t.shape[1] * head,), sentinel, device=t.device)
        view = buf.as_strided(t.shape, (row, head, 1))
        if copy:
            view.copy_(t)
        bufs.append((buf, view))
        return view

    run = TttAttnRunner([wide(t) for t in case.q], [wide(t) for t in case.k], [wide(t) for t in case.v], case.wl.cu_seqlens, case.wl.scale, "cuda:0")
    d_o = [wide(t) for t in case.d_o]
    run.o, run.dq = [wide(t, False) for t in case.q], [wide(t, False) for t in case.q]
    run.dk, run.dv = [wide(t, False) for t in case.k], [wide(t, False) for t in case.v]
    passes(run, d_o, k, k)
    case.run = run
    for key, (err, bound) in compare_full(case).items():
        assert err <= bound, f"{key}: {err:.3e} > {bound:.3e}"
    for buf, view in bufs:
        view.fill_(sentinel)
        assert bool((buf == sentinel).all())


@pytest.mark.parametrize("row,direct", [((1 << 28) - 8, True), (1 << 28, False)])
def test_f32_forward_with_rows_a_gibibyte_apart(row, direct):
    """K and V rows as far apart as the forward's 32-bit offsets can tell, and farther: the same O and LSE as with rows that
    follow each other."""
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    assert f32_direct([6], 2, 1, 64, 0, 1, n_cu, kv_st=row) == (direct, False)
    print(f"kv row stride={row}", flush=True)
    case = Case(custom_workload("f32_gibibyte", "f32", [6], 2, 1, 64, 1, seed=9), "cuda:0")
    case.run.forward()

    def far(t):
        buf = torch.full((5 * row + 64,), 77.0, device=t.device)
        view = buf.as_strided(t.shape, (row, 64, 1))
        view.copy_(t)
        return view

    run = TttAttnRunner(case.q, [far(t) for t in case.k], [far(t) for t in case.v], case.wl.cu_seqlens, case.wl.scale, "cuda:0")
    run.forward()
    torch.cuda.synchronize()
    for got, ref in zip(run.o + run.lse, case.run.o + case.run.lse):
        torch.testing.assert_close(got, ref, rtol=1e-5, atol=1e-5)   # (sums of six terms, in another order with tiles)


@pytest.mark.parametrize("d", [64, 128])
def test_f32_diagonal_scores_of_minus_infinity(d):
    """A diagonal key of score -inf has no weight, also where it is the first key that its wave sees: the same as a score too low to count."""
    print(f"head_dim={d}", flush=True)
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    assert f32_direct([40], 2, 1, d, 0, 3, n_cu)[0]
    case = Case(custom_workload(f"f32_minus_inf_{d}", "f32", [40], 2, 1, d, 3, seed=d), "cuda:0")
    for t in case.q:
        t[..., 0].abs_().add_(0.1)
    outputs = []
    for low in (-1e30, float("-inf")):
        for t in case.k[1:]:
            t[::3, :, 0] = low
        for t in case.run.o + case.run.lse:
            t.fill_(float("nan"))
        case.run.forward(0, 3)
        torch.cuda.synchronize()
        outputs.append([t.clone() for t in case.run.o + case.run.lse])
    for finite, infinite in zip(*outputs):
        assert bool(finite.isfinite().all())
        assert torch.equal(finite, infinite)
