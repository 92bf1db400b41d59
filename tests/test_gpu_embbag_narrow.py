"""Table rows narrower than a wave's 256 bytes leave lanes idle.  The sparse
gradient of rows of 64 and 128 bytes moves half and a quarter of the bytes of
256-byte rows for the same lookups: it equals the wide rows' column by column,
bit for bit (each column is summed alone, in the same order), and it takes no
longer (with loads under a lane condition the rows were fetched one at a time:
1.4 times as long)."""
import pytest
import torch

from tests._util import DEV

F, B, PER, ROWS = 96, 8192, 8, 1000


def _call(d, idx, offsets, row_base, dX, lr):
    from paper_2512_09200_amd import api
    E = torch.zeros((F * ROWS, d), dtype=torch.bfloat16, device=DEV)
    g = dX[:, :, :d].contiguous()
    r = api.lattice_embbag_bwd(E, row_base, offsets, idx, F, B, g, lr=lr, max_rows=ROWS)

    def run():
        api.lattice_embbag_bwd_noalloc(E, row_base, offsets, idx, F, B, g, r, lr=lr, max_rows=ROWS)
    return r, E, run


@pytest.mark.gpu
def test_narrow_rows():
    g = torch.Generator(device=DEV).manual_seed(5)
    nnz = F * B * PER
    idx = torch.randint(0, ROWS, (nnz,), generator=g, device=DEV, dtype=torch.int32)
    offsets = torch.arange(F * B + 1, dtype=torch.int32, device=DEV) * PER
    row_base = torch.arange(F + 1, dtype=torch.int64, device=DEV) * ROWS
    dX = torch.randn((B, F, 128), generator=g, device=DEV).to(torch.bfloat16)
    wide, wE, wrun = _call(128, idx, offsets, row_base, dX, 0.5)
    U = int(wide["num_unique"])

    def time(run):
        best = 1e9
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            torch.cuda.synchronize()
            a.record()
            for _ in range(10):
                run()
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b))
        return best

    ref, t = (wide["grad_rows"][:U].clone(), wE.clone()), {}
    for d in (32, 64):
        narrow, nE, run = _call(d, idx, offsets, row_base, dX, 0.5)
        assert torch.equal(narrow["grad_rows"][:U], ref[0][:, :d]) and torch.equal(nE, ref[1][:, :d])
        t[d] = time(run)
    t[128] = time(wrun)
    print(f"[embbag-narrow] {t}", flush=True)
    assert max(t[32], t[64]) <= 1.2 * t[128], t
