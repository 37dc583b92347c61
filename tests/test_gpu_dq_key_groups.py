"""GPU parity of the 16-bit dQ tiles with two key groups (short launches): one row, rows and keys that end inside a block, a tile and
a group's half of a key tile, document starts inside a half, no, one, two and more diagonal keys, one step a call and all at once.
Every case asserts the key groups that the launch rules choose."""
import pytest
import torch

from paper_2603_18567_amd import TttAttnRunner
from paper_2603_18567_amd.workloads import custom_workload
from plan_lib import backward_launch
from ttt_testlib import Case, compare_full

pytestmark = pytest.mark.gpu

CASES = [
    # documents, hq, hkv, head_dim, k, steps per backward call
    ([1], 8, 1, 128, 6, 1),
    ([33], 8, 1, 128, 5, 1),
    ([129], 12, 2, 128, 4, 1),
    ([130, 33, 64], 8, 2, 128, 5, 1),
    ([63, 1, 65, 127, 200], 8, 1, 128, 5, 1),
    ([493], 12, 2, 128, 3, 1),
    ([257], 8, 2, 128, 4, 1),
    ([70, 260, 300], 4, 1, 128, 2, 2),
    ([900, 129], 3, 1, 128, 2, 2),
    ([31, 290], 16, 16, 64, 4, 1),
    ([449], 6, 6, 64, 3, 1),
    ([600, 41], 8, 1, 64, 2, 2),
]


@pytest.mark.parametrize("docs,hq,hkv,d,k,steps", CASES, ids=[f"{sum(c[0])}_{len(c[0])}_{c[1]}_{c[2]}_{c[3]}" for c in CASES])
def test_two_key_groups_match_oracle(docs, hq, hkv, d, k, steps):
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    print(f"documents={docs} heads={hq}/{hkv} head_dim={d} k={k} steps={steps}", flush=True)
    assert any(backward_launch(docs, hq, hkv, d, j, steps, n_cu)[2] == 2 for j in range(0, k, steps))
    case = Case(custom_workload(f"dq_groups_{sum(docs)}_{d}", "bf16", docs, hq, hkv, d, k, seed=sum(docs) + k), "cuda:0")
    case.run.forward()
    for j in reversed(range(0, k, steps)):
        case.run.backward(case.d_o, j, j + steps, accumulate=steps < k)
    torch.cuda.synchronize()
    for key, (err, bound) in compare_full(case).items():
        assert err <= bound, f"{key}: {err:.3e} > {bound:.3e}"


@pytest.mark.parametrize("docs,hq,hkv,d,row,head", [([257, 40], 8, 2, 128, 8 * 136 + 24, 136), ([449], 6, 6, 64, 6 * 72, 72)], ids=["head128", "head64"])
def test_two_key_groups_of_strided_views_on_a_side_stream_and_from_a_graph(docs, hq, hkv, d, row, head):
    """Rows `row` and heads `head` elements apart (the Q and dO rows of a dQ tile come by 32-bit offsets from row to row), first eagerly on a
    stream of their own, then recorded there and replayed: what lies between the rows keeps a sentinel, every replay is checked."""
    print(f"documents={docs} heads={hq}/{hkv} head_dim={d} strides={row},{head}", flush=True)
    k, sentinel, bufs = 3, 77.0, []
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    assert any(backward_launch(docs, hq, hkv, d, j, 1, n_cu)[2] == 2 for j in range(k))
    case = Case(custom_workload(f"dq_groups_strided_{d}", "bf16", docs, hq, hkv, d, k, seed=d), "cuda:0")

    def wide(t, copy=True):
        buf = torch.full(((t.shape[0] - 1) * row + t.shape[1] * head,), sentinel, device=t.device, dtype=t.dtype)
        view = buf.as_strided(t.shape, (row, head, 1))
        if copy:
            view.copy_(t)
        bufs.append((buf, view))
        return view

    run = TttAttnRunner([wide(t) for t in case.q], [wide(t) for t in case.k], [wide(t) for t in case.v], case.wl.cu_seqlens, case.wl.scale, "cuda:0")
    d_o = [wide(t) for t in case.d_o]
    run.o, run.dq = [wide(t, False) for t in case.q], [wide(t, False) for t in case.q]
    run.dk, run.dv = [wide(t, False) for t in case.k], [wide(t, False) for t in case.v]
    case.run = run

    def passes():
        for j in range(k):
            run.forward(j, j + 1)
        for j in reversed(range(k)):
            run.backward(d_o, j, j + 1, accumulate=True)

    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):   # the binding takes torch's current stream
        passes()
    torch.cuda.synchronize()
    compare_full(case)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        passes()
    for _ in range(3):
        for t in run.o + run.lse + run.dq + run.dk + run.dv:
            t.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        compare_full(case)
    for buf, view in bufs:
        view.fill_(sentinel)
        assert bool((buf == sentinel).all())
