"""The sparse gradient on both sides of the sizes where its work split changes:
reduction ranges of 64 up to 2^21 lookups and of 256 above, run bookkeeping
with group sums above 4096 tiles of 4096 keys.  Bookkeeping equals torch's
stable sort exactly; every row gradient lies within the fp32 bound of its sum
in float64, and the SGD update is one rounding of it."""
import pytest
import torch

from tests._util import DEV

LIM = 1 << 21
CASES = [  # lookups, features, rows, d, table dtype, pool
    (LIM, 3, 4001, 64, torch.float32, "sum"), (LIM + 1, 3, 4001, 64, torch.float32, "sum"),
    (LIM - 77, 2, 300_000, 128, torch.bfloat16, "sum"), (LIM + 4097, 2, 300_000, 128, torch.bfloat16, "mean"),
    (LIM + 63, 5, 900, 32, torch.bfloat16, "sum"), (LIM + 255, 2, 5000, 256, torch.bfloat16, "sum"),
    (4096 * 4096, 2, 700_000, 8, torch.float32, "sum"), (4096 * 4096 + 1, 2, 700_000, 8, torch.float32, "sum"),
]


@pytest.mark.gpu
@pytest.mark.parametrize("nnz,F,rows,d,dtype,pool", CASES)
def test_sparse_gradient(nnz, F, rows, d, dtype, pool):
    from paper_2512_09200_amd import api
    print(f"[embbag-ranges] nnz={nnz} F={F} rows={rows} d={d} {dtype} {pool}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(nnz)
    B = 512
    cuts = torch.sort(torch.randint(0, nnz + 1, (F * B - 1,), generator=g, device=DEV)).values
    offsets = torch.cat([cuts.new_zeros(1), cuts, cuts.new_full((1,), nnz)])
    lens = offsets[1:] - offsets[:-1]
    bag = torch.repeat_interleave(torch.arange(F * B, device=DEV), lens, output_size=nnz)
    u = torch.rand(nnz, generator=g, device=DEV)
    idx = ((u * u * u) * rows).long().clamp_(max=rows - 1)     # hot rows: runs over many ranges
    row = idx + (bag // B) * rows
    E = (torch.randn((F * rows, d), generator=g, device=DEV) * 0.1).to(dtype)
    dX = (torch.randn((B, F, d), generator=g, device=DEV)).to(dtype)
    row_base = torch.arange(F + 1, dtype=torch.int64, device=DEV) * rows
    E0 = E.clone()
    out = api.lattice_embbag_bwd(E, row_base, offsets.to(torch.int32), idx.to(torch.int32), F, B, dX, lr=0.5,
                                 pool=pool, max_rows=rows)
    torch.cuda.synchronize()
    srt, perm = torch.sort(row, stable=True)
    uniq, counts = torch.unique_consecutive(srt, return_counts=True)
    U = uniq.numel()
    assert int(out["num_unique"]) == U
    assert torch.equal(out["unique_rows"][:U].long(), uniq)
    assert torch.equal(out["seg_offsets"][1:U + 1].long(), torch.cumsum(counts, 0))
    assert int(out["seg_offsets"][0]) == 0
    assert torch.equal(out["sorted_bags"].long(), bag[perm])
    # sums in float64, and of absolute values for the bound
    G = torch.zeros((U, d), dtype=torch.float64, device=DEV)
    A = torch.zeros_like(G)
    seg = torch.repeat_interleave(torch.arange(U, device=DEV), counts, output_size=nnz)
    flat = dX.transpose(0, 1).reshape(F * B, d)
    for i in range(0, nnz, 1 << 21):
        b = bag[perm[i:i + (1 << 21)]]
        t = flat[b].double()
        if pool == "mean":
            t = t / lens[b].double()[:, None]
        G.index_add_(0, seg[i:i + (1 << 21)], t)
        A.index_add_(0, seg[i:i + (1 << 21)], t.abs())
    # any order of K fp32 additions, and (mean) two roundings per term
    bound = (counts.double()[:, None] + 3) * 2.0 ** -24 * A + 1e-37
    assert bool(((out["grad_rows"][:U].double() - G).abs() <= bound).all())
    want = (E0[uniq].float() - 0.5 * out["grad_rows"][:U])
    us = 2.0 ** -8 if dtype == torch.bfloat16 else 2.0 ** -23
    assert bool(((E[uniq].float() - want).abs() <= us * want.abs() + 2.0 ** -23 * (want.abs() + E0[uniq].float().abs())).all())
    E[uniq] = E0[uniq]
    assert torch.equal(E, E0)
