"""A step forks its sort to the side stream before the interaction in small
batches and after it in large ones (above 2^21 lookups): both, and batches on
either side of the line, give the bits of a step on one stream, also when steps
follow one another without a wait."""
import pytest
import torch

from tests._util import DEV

LINE = 1 << 21


def _model(nnz, inter, B=2048, F=8, d=64, rows=5000):
    from paper_2512_09200_amd import api
    g = torch.Generator(device=DEV).manual_seed(nnz % 1000)
    bags = F * B
    lens = torch.full((bags,), nnz // bags, device=DEV)
    lens[:nnz % bags] += 1
    offsets = torch.zeros(bags + 1, dtype=torch.int32, device=DEV)
    offsets[1:] = torch.cumsum(lens, 0)
    idx = torch.randint(0, rows, (nnz,), generator=g, device=DEV, dtype=torch.int32)
    n, k = F + 1, 32 if inter == "fm" else 0
    rnd = lambda *s, scale=0.1: (scale * torch.randn(s, generator=g, device=DEV)).to(torch.bfloat16)

    def layers(dims):
        return [dict(W=rnd(o, i), b=torch.zeros(o, device=DEV), dW=torch.zeros((o, i), device=DEV),
                     db=torch.zeros(o, device=DEV)) for i, o in zip(dims, dims[1:])]
    E0 = rnd(F * rows, d, scale=0.01)
    x = dict(dense=rnd(B, 13, scale=1.0), labels=(torch.rand((B, 4), generator=g, device=DEV) < 0.3).float(),
             mask=torch.ones((B, 4), dtype=torch.uint8, device=DEV))
    W, bottom = rnd(n, k) if k else None, layers([13, 32, d])
    top = layers([d + (n * k if k else n * (n - 1) // 2), 64, 32, 4])

    def run(side):
        E, dW = E0.clone(), torch.zeros((n, k), device=DEV) if k else None
        row_base = torch.arange(F + 1, dtype=torch.int64, device=DEV) * rows
        m = api.StepModel(tables=E, row_base=row_base, num_features=F, dense_in=13, bottom=bottom, top=top,
                          interact=inter, fm_W=W, fm_dW=dW, max_rows=rows)
        lay = api.lattice_step_plan(m, B, nnz, 0.05)
        ws = torch.zeros(lay.total_bytes, dtype=torch.uint8, device=DEV)
        for _ in range(3):
            api.lattice_step(m, offsets, idx, x["dense"], x["labels"], x["mask"], ws, 0.05, nnz_capacity=nnz, side=side)
        torch.cuda.synchronize()
        v = api.step_views(m, ws, lay, B, 4, nnz)
        u = int(v["num_unique"])
        out = [E, v["logits"], v["loss"], v["unique_rows"][:u], v["seg_offsets"][:u + 1], v["sorted_bags"]]
        return [t.clone() for t in out + [L[q] for L in bottom + top for q in ("dW", "db")] + ([dW] if k else [])]
    return run


@pytest.mark.gpu
@pytest.mark.parametrize("inter", ["fm", "dot"])
@pytest.mark.parametrize("nnz", [LINE - 1, LINE, LINE + 1, LINE + 300_000])
def test_side_stream_gives_the_bits_of_one_stream(nnz, inter):
    from paper_2512_09200_amd import api
    print(f"[sort-fork] nnz={nnz} {inter}", flush=True)
    run = _model(nnz, inter)
    a, b = run(api.SideStream()), run(None)
    assert all(torch.isfinite(t.float()).all() for t in a)
    for i, (p, q) in enumerate(zip(a, b)):
        assert torch.equal(p, q), i
