"""GPU parity of the in-place log-softmax-loss backward (Alg. 3) against the fp64 oracle, element by
element, through the C ABI: rows held in registers by 256, 512 and 1024 threads, rows held in registers and LDS, rows that
are partly read twice, rows that start at any element, strided rows, masked rows (g = 0), and tensors above and
below the size from which the caches are passed by."""
import os
import sys

import numpy as np
import pytest
import torch

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
from oracle.loss_oracle import logsoftmax_loss_bwd   # noqa: E402

# fp32: the result is O(|g|); exp2 and the V-term sums carry a few fp32 ulps each.
# bf16: one rounding of the output (2^-9 relative) plus the rounding of nothing else (inputs are
# given rounded); elements where p*g and pi*s cancel are bounded relative to the row maximum.
TOL = {torch.float32: 2e-5, torch.bfloat16: 2e-2}


def make(n, v, dtype, seed, stride_pad=0):
    gen = torch.Generator().manual_seed(seed)
    z = (torch.randn(n, v + stride_pad, generator=gen) * 3).to(dtype)
    p = torch.rand(n, v + stride_pad, generator=gen) ** 6
    p = (p / p[:, :v].sum(1, keepdim=True)).to(dtype)
    g = torch.randn(n, generator=gen)
    if n > 2:
        g[1] = 0.0                     # a masked position
    return z, p, g


CASES = [   # name, rows, vocabulary, dtype, stride padding; the position in this list + 500 is the seed
    ("f32_small", 7, 1000, torch.float32, 0),
    ("f32_draft_vocab", 5, 32000, torch.float32, 0),
    ("bf16_draft_vocab", 5, 32000, torch.bfloat16, 0),
    ("f32_ragged_unaligned", 4, 4099, torch.float32, 0),        # vocab not a multiple of the vector width
    ("bf16_ragged", 4, 50257, torch.bfloat16, 0),
    ("f32_strided_rows", 6, 2048, torch.float32, 64),
    ("f32_odd_stride_elementwise", 3, 777, torch.float32, 3),   # rows start at any element: columns before the first vector
    ("f32_streamed_long_row", 3, 70001, torch.float32, 0),      # registers and LDS
    ("bf16_streamed_long_row", 2, 151936, torch.bfloat16, 0),   # the last slabs are read twice
    ("f32_vocab_1", 3, 1, torch.float32, 0),
    ("bf16_256_threads_last_size", 5, 16384, torch.bfloat16, 0),
    ("bf16_unaligned_rows", 5, 16385, torch.bfloat16, 0),       # contiguous odd vocabulary: rows start at any element
    ("bf16_long_fewest_slabs", 5, 65537, torch.bfloat16, 0),    # 16 slabs of 4096 (18 in registers) and one column
    ("bf16_long_registers_and_lds", 5, 110592, torch.bfloat16, 0),   # 27 whole slabs, no columns left over
    ("bf16_long_one_slab_twice", 5, 147456 + 4093, torch.bfloat16, 0),
    ("f32_long_odd_stride", 4, 55299, torch.float32, 3),
    ("f32_long_many_slabs_twice", 3, 151937, torch.float32, 0),
    ("f32_512_threads", 5, 12001, torch.float32, 0),
]

# Logits and target together just above 256 MB, where the kernels pass the caches by: each kernel of each type.
LARGE_CASES = [   # name, rows, vocabulary, dtype
    ("f32_256_threads", 8200, 4099, torch.float32),
    ("f32_512_threads", 2800, 12001, torch.float32),
    ("f32_1024_threads", 1100, 32000, torch.float32),
    ("f32_1024_threads_unaligned_rows", 1100, 32001, torch.float32),
    ("f32_long_18_slabs", 680, 50001, torch.float32),
    ("f32_long_one_part_twice", 450, 75001, torch.float32),
    ("bf16_256_threads", 4200, 16001, torch.bfloat16),
    ("bf16_512_threads", 2100, 32003, torch.bfloat16),
    ("bf16_1024_threads", 1110, 61003, torch.bfloat16),
    ("bf16_long_18_slabs", 600, 113001, torch.bfloat16),
    ("bf16_long_one_part_twice", 450, 151936, torch.bfloat16),
    ("bf16_long_one_part_twice_unaligned_rows", 450, 151937, torch.bfloat16),
]


@pytest.mark.gpu
@pytest.mark.parametrize("seed,name,n,v,dtype,pad", [(500 + i, *c) for i, c in enumerate(CASES)], ids=[c[0] for c in CASES])
def test_loss_backward_matches_oracle(seed, name, n, v, dtype, pad):
    from paper_2603_18567_amd import binding as B
    print(f"case {name}: rows={n} vocab={v} dtype={dtype} stride_pad={pad} seed={seed}", flush=True)
    z, p, g = make(n, v, dtype, seed=seed, stride_pad=pad)
    ref = logsoftmax_loss_bwd(z[:, :v].float().numpy(), p[:, :v].float().numpy(), g.numpy())
    dev = torch.device("cuda:0")
    zd, pd, gd = z.to(dev), p.to(dev), g.to(dev)
    p_before = pd.clone()
    B.ttt_loss_bwd_inplace(zd[:, :v], pd[:, :v], gd)
    torch.cuda.synchronize()
    got = zd[:, :v].float().cpu().numpy().astype(np.float64)
    assert np.isfinite(got).all()
    err = np.abs(got - ref).max()
    # every element is the difference of the two terms p*g and pi*s: the error is relative to them
    # (a one-entry vocabulary makes them cancel exactly: the reference is identically zero)
    terms = np.abs(p[:, :v].double().numpy() * g.double().numpy()[:, None]).max()
    bound = TOL[dtype] * max(np.abs(ref).max(), terms, 1e-30)
    assert err <= bound, f"max abs err {err:.3e} > {bound:.3e}"
    if n > 2:
        assert np.all(got[1] == 0.0), "a row with g = 0 must become exactly zero"
    assert torch.equal(pd, p_before), "the target must not be written"
    if pad:
        assert torch.equal(zd[:, v:].cpu(), z[:, v:]), "columns past the vocabulary must not be touched"


@pytest.mark.gpu
@pytest.mark.parametrize("name,n,v,dtype", LARGE_CASES, ids=[c[0] for c in LARGE_CASES])
def test_loss_backward_of_large_tensors(name, n, v, dtype):
    """Every element of every row against the gradient in fp64 torch operations, three rows against the oracle too;
    the bound is that of the cases above, row by row."""
    from paper_2603_18567_amd import binding as B
    print(f"case {name}: rows={n} vocab={v} dtype={dtype}", flush=True)
    assert 2 * n * v * dtype.itemsize > 256 << 20
    gen = torch.Generator(device="cuda:0").manual_seed(v)
    z = (torch.randn(n, v, generator=gen, device="cuda:0") * 3).to(dtype)
    p = torch.rand(n, v, generator=gen, device="cuda:0").pow_(6)
    p = p.div_(p.sum(1, keepdim=True)).to(dtype)
    g = torch.randn(n, generator=gen, device="cuda:0")
    got = z.clone()
    p_before = p.clone()
    B.ttt_loss_bwd_inplace(got, p, g)
    torch.cuda.synchronize()
    assert torch.equal(p, p_before), "the target must not be written"
    for rows in torch.arange(n).split(200):
        rows = slice(int(rows[0]), int(rows[-1]) + 1)
        p64, g64 = p[rows].double(), g[rows].double()[:, None]
        pg = p64 * g64
        ref = torch.softmax(z[rows].double(), 1) * (g64 * p64.sum(1, keepdim=True)) - pg
        bound = TOL[dtype] * torch.maximum(ref.abs().amax(1), pg.abs().amax(1))
        err = (got[rows].double() - ref).abs().amax(1)
        assert bool((err <= bound).all()), (rows, float((err / bound).max()))   # (a NaN fails as well)
    for r in (0, n // 2, n - 1):
        ref = logsoftmax_loss_bwd(z[r:r + 1].float().cpu().numpy(), p[r:r + 1].float().cpu().numpy(), g[r:r + 1].cpu().numpy())
        err = np.abs(got[r:r + 1].float().cpu().numpy() - ref).max()
        assert err <= TOL[dtype] * max(np.abs(ref).max(), float((p[r].float() * g[r]).abs().max()))


@pytest.mark.gpu
@pytest.mark.parametrize("v,dtype", [(2000, torch.float32), (30001, torch.float32), (70001, torch.float32), (151937, torch.bfloat16)])
def test_loss_backward_extreme_rows(v, dtype):
    """Logits that grow along the row (every vector raises the running maximum), fall along it, are masked
    with -inf except for a few, start with -inf, or lie at the type's ends of the usual range."""
    from paper_2603_18567_amd import binding as B
    _, p, g = make(5, v, dtype, seed=77)
    z = torch.zeros(5, v)
    z[0] = torch.linspace(-60, 60, v)
    z[1] = torch.linspace(60, -60, v)
    z[2] = float("-inf")
    z[2, [0, v // 3, v - 1]] = torch.tensor([1.0, 2.0, 3.0])
    z[3, : v // 2] = float("-inf")
    z[4] = torch.where(torch.arange(v) % 7 == 0, 3.0e4, -3.0e4)
    z = z.to(dtype)
    ref = logsoftmax_loss_bwd(z.float().numpy(), p.float().numpy(), g.numpy())
    dev = torch.device("cuda:0")
    zd = z.to(dev)
    B.ttt_loss_bwd_inplace(zd, p.to(dev), g.to(dev))
    torch.cuda.synchronize()
    got = zd.float().cpu().numpy().astype(np.float64)
    assert np.isfinite(got).all()
    # as above, row by row; the exponent z log2(e) is rounded at |z| = 60 and 3e4 before the maximum is
    # subtracted: 2^-24 * |z| * log2(e) * ln 2 relative in exp(z - max), 3.6e-6 at 60 (at 3e4 all terms that count are equal)
    terms = np.abs(p.double().numpy() * g.double().numpy()[:, None]).max(axis=1)
    bound = TOL[dtype] * np.maximum(np.abs(ref).max(axis=1), terms)
    err = np.abs(got - ref).max(axis=1)
    assert np.all(err <= bound), (err, bound)


@pytest.mark.gpu
def test_loss_backward_no_rows_and_bad_arguments():
    from paper_2603_18567_amd import binding as B
    dev = torch.device("cuda:0")
    z = torch.zeros(0, 16, device=dev)
    B.ttt_loss_bwd_inplace(z, z.clone(), torch.zeros(0, device=dev))      # no-op
    lib = B.load_library()
    assert lib.ttt_loss_bwd_inplace(None, None, None, 4, 0, 16, 16, B.TTT_F32, None) == B.TTT_ERR_INVALID_ARG
    assert lib.ttt_loss_bwd_inplace(None, None, None, 4, 16, 8, 16, B.TTT_F32, None) == B.TTT_ERR_INVALID_ARG
    assert lib.ttt_loss_bwd_inplace(None, None, None, 4, 16, 16, 16, 7, None) == B.TTT_ERR_UNSUPPORTED
    assert lib.ttt_loss_bwd_inplace(None, None, None, 4, 16, 16, 16, B.TTT_F32, None) == B.TTT_ERR_INVALID_ARG
