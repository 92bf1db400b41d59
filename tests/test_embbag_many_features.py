"""The sparse gradient with so many features that short reduction ranges would
not fit the allocation-free entry point's array: that entry point accepts a
batch exactly when the workspace query says that it fits, and sums it in the
same order as the workspace entry point (bit-identical outputs)."""
from ctypes import byref

import pytest
import torch

from paper_2512_09200_amd import _abi as A
from tests._util import DEV

LIMIT = 256 << 20
OK, UNSUPPORTED = 0, 2


def _jagged(F, nnz, p=0x10000, B=16):
    return A.lattice_jagged(num_features=F, batch=B, offsets=p, indices=p, nnz=nnz)


def _workspace(lib, dim, F, nnz):
    t = A.lattice_tables(data=None, dtype=A.BF16, dim=dim, total_rows=1000, row_base=None, max_rows=0)
    return int(lib.lattice_embbag_bwd_workspace(byref(t), byref(_jagged(F, nnz))))


@pytest.mark.parametrize("dim", [8, 128, 256])
def test_workspace_is_monotone(dim):
    lib = A.load()
    for F in (20_000, 24_000, 28_000, 29_500, 32_000):
        sizes = [_workspace(lib, dim, F, n) for n in
                 [1, 64, 1000] + [(1 << 17) * q + r for q in range(1, 40) for r in (-1, 0, 1)]]
        assert all(a <= b for a, b in zip(sizes, sizes[1:])), (F, sizes)


# placeholder pointers must never reach a GPU: an accepted call ends at the
# first HIP call where none is visible
@pytest.mark.skipif(torch.cuda.device_count() > 0, reason="placeholder pointers")
@pytest.mark.parametrize("dim", [8, 128, 256])
def test_accepted_exactly_where_the_query_fits(dim):
    lib = A.load()
    p = 0x10000
    t = A.lattice_tables(data=p, dtype=A.BF16, dim=dim, total_rows=10_000_000, row_base=p, max_rows=0)
    out = A.lattice_sparse_grad(unique_rows=p, seg_offsets=p, sorted_bags=p, num_unique=p, grad_rows=p)
    seen = set()
    for F in list(range(18_000, 33_000, 500)) + [64]:
        for nnz in (1000, 500_000, 1 << 21, (1 << 21) + 1, 6_000_000, 17_000_000):
            st = lib.lattice_embbag_bwd_noalloc(byref(t), byref(_jagged(F, nnz, B=1)), A.POOL_SUM, p, A.BF16, F, 0,
                                                byref(out), 0.0, None)
            assert st != OK
            fits = _workspace(lib, dim, F, nnz) <= LIMIT
            assert (st != UNSUPPORTED) == fits, (F, nnz, st, lib.lattice_last_error())
            seen.add(fits)
    assert seen == {True, False}


@pytest.mark.gpu
def test_long_ranges_of_a_small_batch():
    from paper_2512_09200_amd import api
    lib = A.load()
    dim, B, rows, nnz0 = 256, 2, 3, 1_500_000
    # the most features the array takes; short ranges would need more (the
    # query then covers any smaller batch: the array's size)
    F = max(f for f in range(20_000, 32_000, 100) if _workspace(lib, dim, f, nnz0) <= LIMIT)
    assert _workspace(lib, dim, F, nnz0) == LIMIT
    print(f"[embbag-many] F={F} dim={dim} nnz={nnz0}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(3)
    lens = torch.randint(0, 30, (F * B,), generator=g, device=DEV)
    lens[F] += 200_000                                   # runs over many ranges
    lens[-1] += max(0, nnz0 - int(lens.sum()))
    nnz = int(lens.sum())
    assert nnz <= 1 << 21 and _workspace(lib, dim, F, nnz) == LIMIT
    offsets = torch.zeros(F * B + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(lens, 0, out=offsets[1:])
    bag = torch.repeat_interleave(torch.arange(F * B, device=DEV), lens, output_size=nnz)
    idx = torch.randint(0, rows, (nnz,), generator=g, device=DEV)
    row = idx + (bag // B) * rows
    dX = torch.randn((B, F, dim), generator=g, device=DEV).to(torch.bfloat16)
    E0 = torch.randn((F * rows, dim), generator=g, device=DEV).to(torch.bfloat16)
    rb = torch.arange(F + 1, dtype=torch.int64, device=DEV) * rows
    o32, i32 = offsets.to(torch.int32), idx.to(torch.int32)
    E1, E2 = E0.clone(), E0.clone()
    ref = api.lattice_embbag_bwd(E1, rb, o32, i32, F, B, dX, lr=0.5, max_rows=rows)
    out = dict(unique_rows=torch.full((nnz,), -7, dtype=torch.int32, device=DEV),
               seg_offsets=torch.full((nnz + 1,), -7, dtype=torch.int32, device=DEV),
               sorted_bags=torch.full((nnz,), -7, dtype=torch.int32, device=DEV),
               num_unique=torch.full((1,), -7, dtype=torch.int32, device=DEV),
               grad_rows=torch.full((nnz, dim), float("nan"), device=DEV))
    api.lattice_embbag_bwd_noalloc(E2, rb, o32, i32, F, B, dX, out, lr=0.5, max_rows=rows)
    torch.cuda.synchronize()
    srt, perm = torch.sort(row, stable=True)
    uniq, counts = torch.unique_consecutive(srt, return_counts=True)
    U = uniq.numel()
    for r in (ref, out):
        assert int(r["num_unique"]) == U
        assert torch.equal(r["unique_rows"][:U].long(), uniq)
        assert torch.equal(r["seg_offsets"][1:U + 1].long(), torch.cumsum(counts, 0))
        assert torch.equal(r["sorted_bags"].long(), bag[perm])
    assert torch.equal(out["grad_rows"][:U], ref["grad_rows"][:U]) and torch.equal(E1, E2)
    G = torch.zeros((U, dim), dtype=torch.float64, device=DEV)
    M = torch.zeros_like(G)
    seg = torch.repeat_interleave(torch.arange(U, device=DEV), counts, output_size=nnz)
    flat = dX.transpose(0, 1).reshape(F * B, dim)
    for i in range(0, nnz, 1 << 19):
        t = flat[bag[perm[i:i + (1 << 19)]]].double()
        G.index_add_(0, seg[i:i + (1 << 19)], t)
        M.index_add_(0, seg[i:i + (1 << 19)], t.abs())
    # any order of K fp32 additions
    assert bool(((ref["grad_rows"][:U].double() - G).abs() <= counts.double()[:, None] * 2.0 ** -24 * M + 1e-37).all())
    E0[uniq] = (E0[uniq].float() - 0.5 * ref["grad_rows"][:U]).to(torch.bfloat16)
    assert torch.equal(E1, E0)
