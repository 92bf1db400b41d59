"""Both sides of the lines between the scalar and the fp32 MFMA interaction
kernels, against float64 within the rounding bounds of their sums; and calls
that the MFMA kernels run several times slower than the scalar ones (a few rows
in whole 32 x 32 tiles) take the scalar kernels' time."""
import pytest
import torch

from tests._util import DEV

E32, SHAPES = 2.0 ** -24, [
    # n, d, rank (0: DOT); forward and backward each fall on both sides
    (2, 256, 0), (12, 32, 0), (12, 64, 0), (13, 48, 0), (18, 96, 0), (19, 32, 0), (19, 16, 0), (24, 16, 0), (25, 16, 0),
    (33, 16, 0), (37, 16, 0), (34, 32, 0), (35, 32, 0), (48, 16, 0), (49, 16, 0), (65, 96, 0),
    (2, 256, 16), (9, 64, 16), (40, 32, 17), (39, 64, 16), (43, 64, 16), (65, 128, 4), (65, 128, 5), (64, 128, 8),
    (16, 32, 32), (20, 256, 12), (20, 256, 16), (33, 48, 33), (97, 64, 17), (13, 256, 48), (1, 16, 64),
]


@pytest.mark.gpu
@pytest.mark.parametrize("n,d,k", SHAPES)
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16], ids=["f32", "bf16"])
def test_both_sides(dtype, n, d, k):
    from paper_2512_09200_amd import api
    kind, us = ("fm" if k else "dot"), (2.0 ** -8 if dtype == torch.bfloat16 else 0.0)
    print(f"[interact-route] {kind} {dtype} n={n} d={d} k={k}", flush=True)
    B = 21
    g = torch.Generator(device=DEV).manual_seed(n * 1000 + d + k)
    w = n * k if k else n * (n - 1) // 2
    X, dO = (torch.randn(s, generator=g, device=DEV).to(dtype) for s in ((B, n, d), (B, d + w)))
    W = torch.randn((n, k), generator=g, device=DEV).to(dtype) if k else None
    out, dX = torch.zeros_like(dO), torch.zeros_like(X)
    dW = torch.zeros((n, k), device=DEV) if k else None
    ws = api.lattice_interact_fwd(kind, X, out, True, fm_W=W)
    api.lattice_interact_bwd(kind, X, dO, dX, True, fm_W=W, fm_dW=dW, ws=ws if k else None)
    torch.cuda.synchronize()
    x, G = X.double(), dO[:, d:].double()
    T = lambda t: t.transpose(1, 2).contiguous()

    def check(name, got, ref, err):
        bound = err + us * (ref.abs() + err) + 1e-37
        worst = float(((got.double() - ref).abs() / bound).max()) if ref.numel() else 0.0
        print(f"  {name}: worst |x-r|/bound={worst:.3f}", flush=True)
        assert worst <= 1.0

    assert torch.equal(out[:, :d], X[:, 0])
    if not k:
        i, j = torch.triu_indices(n, n, 1, device=DEV)
        check("out", out[:, d:], (x @ T(x))[:, i, j], (d + 3) * E32 * (x.abs() @ T(x.abs()))[:, i, j])
        S = torch.zeros((B, n, n), dtype=torch.float64, device=DEV)
        S[:, i, j] = G
        S = S + T(S)
        ref, mag = S @ x, S.abs() @ x.abs()
        terms = n
    else:
        G = G.reshape(B, n, k)
        wd = W.double()
        P, dP = T(x) @ wd, T(x) @ G
        # stored at the storage type after an fp32 sum over the rows
        eP = (n + 3) * E32 * (T(x.abs()) @ wd.abs())
        edP = (n + 3) * E32 * (T(x.abs()) @ G.abs())
        eP, edP = eP + us * (P.abs() + eP), edP + us * (dP.abs() + edP)
        hi, hd = P.abs() + eP, dP.abs() + edP
        check("out", out[:, d:], (x @ P).reshape(B, -1),
              (x.abs() @ eP + (d + 3) * E32 * (x.abs() @ hi)).reshape(B, -1))
        ref = G @ T(P) + wd @ T(dP)
        mag = G.abs() @ T(hi) + wd.abs() @ T(hd)
        terms = 2 * k
        pre = G.abs() @ T(eP) + wd.abs() @ T(edP)
        rw = (x @ dP).sum(0)
        got = dW.double()
        ew = (x.abs() @ edP).sum(0) + (B * d + 3) * E32 * (x.abs() @ hd).sum(0) + 1e-37
        assert float(((got - rw).abs() / ew).max()) <= 1.0
    ref[:, 0] += dO[:, :d].double()
    mag[:, 0] += dO[:, :d].double().abs()
    check("dX", dX, ref, (terms + 4) * E32 * mag + (pre if k else 0.0))


@pytest.mark.gpu
@pytest.mark.parametrize("n,d,k,fwd,limit", [(9, 64, 8, True, 40), (2, 128, 16, True, 60), (2, 256, 0, False, 30),
                                             (33, 16, 0, False, 40)])
def test_small_shapes_keep_their_time(n, d, k, fwd, limit):
    """fp32, 8192 samples: 17, 23, 13 and 28 us with the scalar kernels, 71, 102,
    56 and 49 with the MFMA kernels; limit in between."""
    from paper_2512_09200_amd import api
    B, kind = 8192, "fm" if k else "dot"
    w = d + (n * k if k else n * (n - 1) // 2)
    X, o = torch.randn((B, n, d), device=DEV), torch.randn((B, w), device=DEV)
    W = torch.randn((n, k), device=DEV) if k else None
    dX = torch.zeros_like(X)

    def run():
        if fwd:
            api.lattice_interact_fwd(kind, X, o, True, fm_W=W)
        else:
            api.lattice_interact_bwd(kind, X, o, dX, True)
    best = 1e9
    for _ in range(6):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        torch.cuda.synchronize()
        a.record()
        for _ in range(50):
            run()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) / 50 * 1e3)
    print(f"[interact-route] {kind} n={n} d={d} k={k} {'forward' if fwd else 'backward'} {best:.1f} us", flush=True)
    assert best < limit
