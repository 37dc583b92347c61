"""GPU parity where the number of documents changes how their bounds are found: up to 64 the forward looks
them up in cu_seqlens itself (one per lane), beyond that they come from a kernel before it.  Documents of
one token, several inside one 32-row block, and boundaries on tile edges; both element types."""
import pytest
import torch

from paper_2603_18567_amd.workloads import custom_workload
from ttt_testlib import Case, compare_full

pytestmark = pytest.mark.gpu

DOCS = {
    "63_of_mixed_lengths": [1, 2, 5, 40] * 15 + [31, 33, 64],
    "64_with_edges_on_tiles": [64] * 3 + [1] * 32 + [7] * 28 + [100],
    "65": [3] * 64 + [90],
    "200_of_one_token": [1] * 200,
}


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("name", list(DOCS))
def test_many_documents_match_oracle(name, dtype):
    print(f"documents {name} dtype={dtype}", flush=True)
    wl = custom_workload(f"docs_{name}_{dtype}", dtype, DOCS[name], 8, 2, 64 if dtype == "f32" else 128, 3, seed=31)
    case = Case(wl, "cuda:0")
    case.run.forward()
    case.run.backward(case.d_o)
    torch.cuda.synchronize()
    for key, (err, bound) in compare_full(case).items():
        assert err <= bound, f"{key}: {err:.3e} > {bound:.3e}"
