"""The sort's preparation around the sizes where its work is divided
differently: blocks of 256 bags over one to 256 features, few bags with much to
clear, and (more than 2^26 = F * F * B) the separate launch for the segments'
first tiles, with one and with several features per thread.  The bookkeeping
equals torch's stable sort exactly."""
import pytest
import torch

from tests._util import DEV

CASES = [(1, 1), (3, 1), (300, 1), (257, 3), (70, 255), (5, 256), (9, 257), (1000, 64), (1000, 68), (2100, 40), (8300, 1)]


@pytest.mark.gpu
@pytest.mark.parametrize("F,B", CASES)
def test_bookkeeping(F, B):
    from paper_2512_09200_amd import api
    print(f"[sort-prep] F={F} B={B}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(F * 1000 + B)
    rows, d = 37, 8
    lens = torch.randint(0, 7, (F, B), generator=g, device=DEV)
    lens[torch.rand(F, generator=g, device=DEV) < 0.3] = 0          # features without lookups
    lens[F // 2, B // 2] = 20_000                                   # and one of several sort tiles
    offsets = torch.zeros(F * B + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(lens.reshape(-1), 0, out=offsets[1:])
    nnz = int(offsets[-1])
    bag = torch.repeat_interleave(torch.arange(F * B, device=DEV), lens.reshape(-1), output_size=nnz)
    idx = torch.randint(0, rows, (nnz,), generator=g, device=DEV)
    row = idx + (bag // B) * rows
    E = torch.zeros((F * rows, d), device=DEV)
    dX = torch.ones((B, F, d), device=DEV)
    row_base = torch.arange(F + 1, dtype=torch.int64, device=DEV) * rows
    for _ in range(2):  # the second call finds the first one's scratch contents
        out = api.lattice_embbag_bwd(E, row_base, offsets.to(torch.int32), idx.to(torch.int32), F, B, dX, lr=0.0,
                                     max_rows=rows)
        torch.cuda.synchronize()
        srt, perm = torch.sort(row, stable=True)
        uniq, counts = torch.unique_consecutive(srt, return_counts=True)
        U = uniq.numel()
        assert int(out["num_unique"]) == U
        assert torch.equal(out["unique_rows"][:U].long(), uniq)
        assert torch.equal(out["seg_offsets"][1:U + 1].long(), torch.cumsum(counts, 0))
        assert torch.equal(out["sorted_bags"].long(), bag[perm])
        # sums of ones: whole numbers below 2^24, exact in fp32
        assert torch.equal(out["grad_rows"][:U], counts.float()[:, None].expand(U, d))
