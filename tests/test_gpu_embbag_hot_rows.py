"""Batches whose lookups fall on a few rows: a row's run of sorted lookups then
crosses many reduction ranges, and its partial sums must not be one wave's work
alone.  Against float64 on both sides of the runs that a block's waves share
(runs of 32 ranges, of 64 lookups or, in the largest batch, 256), and by
time: all lookups on one row take at most three times the time of the
same lookups over 300 rows (2.2 times with ranges of 256 and a wave per run;
6.8 times with ranges of 64 and a wave per run)."""
import pytest
import torch

from tests._util import DEV

# dtype, dim, pool, lookups of each row (in bags of 5, a row's bags in a row)
MANY = [31 * 64, 32 * 64, 5, 33 * 64, 34 * 64 - 5, 1, 200 * 64, 3, 3000, 100, 700 * 64]
CASES = [("bf16", 128, "sum", [400_000]), ("f32", 256, "sum", [5000, 300_000, 7]), ("f32", 64, "mean", MANY),
         ("bf16", 32, "sum", MANY), ("f32", 8, "sum", MANY), ("bf16", 96, "mean", MANY),
         ("bf16", 64, "sum", [1_400_000, 8_100, 8_300, 900_000, 40])]


def _batch(counts, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    idx = torch.repeat_interleave(torch.arange(len(counts), device=DEV), torch.tensor(counts, device=DEV))
    nnz = idx.numel()
    B = (nnz + 4) // 5
    offsets = (torch.arange(B + 1, device=DEV) * 5).clamp_(max=nnz).to(torch.int32)
    row_base = torch.tensor([0, len(counts)], dtype=torch.int64, device=DEV)
    return g, idx, B, offsets, row_base


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,d,pool,counts", CASES)
def test_sums(dtype, d, pool, counts):
    from paper_2512_09200_amd import api
    print(f"[embbag-hot] {dtype} d={d} {pool} rows={len(counts)} nnz={sum(counts)}", flush=True)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    g, idx, B, offsets, row_base = _batch(counts, d)
    E = torch.randn((len(counts), d), generator=g, device=DEV).to(dt)
    dX = torch.randn((B, 1, d), generator=g, device=DEV).to(dt)
    E0 = E.double()
    r = api.lattice_embbag_bwd(E, row_base, offsets, idx.to(torch.int32), 1, B, dX, lr=0.25, pool=pool,
                               max_rows=len(counts))
    torch.cuda.synchronize()
    lens = (offsets[1:] - offsets[:-1]).double()
    x = dX[:, 0].double() / (lens[:, None] if pool == "mean" else 1.0)
    x = x.repeat_interleave(lens.long(), 0)
    ref = torch.zeros((len(counts), d), dtype=torch.float64, device=DEV).index_add_(0, idx, x)
    mag = torch.zeros_like(ref).index_add_(0, idx, x.abs())
    U = int(r["num_unique"])
    assert U == len(counts) and torch.equal(r["unique_rows"][:U].long(), torch.arange(U, device=DEV))
    # a partial sum has 256 terms at most, a stream the run's partial sums at most; 2^-23 also covers 1 / length
    n = torch.tensor(counts, dtype=torch.float64, device=DEV)[:, None]
    bound = (torch.minimum(n, 256 + n / 64 + 8) + 2) * 2.0 ** -23 * mag
    got = r["grad_rows"][:U].double()
    assert bool(((got - ref).abs() <= bound).all()), float(((got - ref).abs() / bound).max())
    upd = E0 - 0.25 * got
    assert bool(((E.double() - upd).abs() <= (2.0 ** -8 if dtype == "bf16" else 2.0 ** -22) * (E0.abs() + got.abs())).all())


@pytest.mark.gpu
def test_time_of_one_hot_row():
    from paper_2512_09200_amd import api
    t, nnz, d = {}, 960_000, 128
    for rows in (1, 300):
        g, idx, B, offsets, row_base = _batch([nnz // rows] * rows, rows)
        idx = idx[torch.randperm(nnz, generator=g, device=DEV)].to(torch.int32)
        E = torch.zeros((rows, d), dtype=torch.bfloat16, device=DEV)
        dX = torch.randn((B, 1, d), generator=g, device=DEV).to(torch.bfloat16)
        r = api.lattice_embbag_bwd(E, row_base, offsets, idx, 1, B, dX, lr=0.1, max_rows=rows)
        t[rows] = 1e9
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(10):
                api.lattice_embbag_bwd_noalloc(E, row_base, offsets, idx, 1, B, dX, r, lr=0.1, max_rows=rows)
            b.record()
            torch.cuda.synchronize()
            t[rows] = min(t[rows], a.elapsed_time(b) * 100)
    print(f"[embbag-hot] us: {t}", flush=True)
    assert t[1] <= 3.0 * t[300], t
