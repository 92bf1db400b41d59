"""fp32 products of at most 32 k (input layers of few features, input gradients
of few heads), which multiply only the k they have: edges of the 8-k slices and
of the path against float64, and a 13-wide layer takes less time than a 64-wide
one (both are one step of the general kernel)."""
import numpy as np
import pytest
import torch

from tests._util import DEV, _np64, assert_product


@pytest.mark.gpu
@pytest.mark.parametrize("K,N", [(1, 70), (7, 33), (8, 64), (9, 65), (31, 32), (32, 31), (33, 1), (65, 8), (40, 32)])
def test_layer(K, N):
    from paper_2512_09200_amd import api
    print(f"[gemm-f32-short] K={K} N={N}", flush=True)
    B, ld = 131, K + 3
    g = torch.Generator(device=DEV).manual_seed(K)
    x = torch.full((B, ld), float("nan"), device=DEV)[:, :K]
    x.copy_(torch.randn((B, K), device=DEV, generator=g))
    W = torch.randn((N, K), device=DEV, generator=g) / np.sqrt(K)
    b = 0.1 * torch.randn(N, device=DEV, generator=g)
    L = [dict(W=W, b=b, dW=torch.full((N, K), 7.0, device=DEV), db=torch.full((N,), 7.0, device=DEV))]
    y = torch.empty((B, N), device=DEV)
    api.lattice_mlp_heads_fwd(L, x, [y], True)
    gout = torch.randn((B, N), device=DEV, generator=g)
    d_in = torch.empty((B, K), device=DEV)
    api.lattice_mlp_heads_bwd(L, x, [y], gout, True, d_in=d_in)
    torch.cuda.synchronize()
    X, Wn, bn, G = _np64(x), _np64(W), _np64(b), _np64(gout) * (_np64(y) > 0)
    assert_product("forward", y, np.maximum(X @ Wn.T + bn, 0), np.abs(X) @ np.abs(Wn).T + np.abs(bn), K + 1, t=np.inf)
    assert_product("dW", L[0]["dW"], G.T @ X, np.abs(G).T @ np.abs(X), B, t=np.inf)
    assert_product("d_in", d_in, G @ Wn, np.abs(G) @ np.abs(Wn), N, t=np.inf)


@pytest.mark.gpu
def test_narrow_input_takes_less_time():
    from paper_2512_09200_amd import api
    t = {}
    for K in (13, 64):
        x, W = torch.randn((30000, K), device=DEV), torch.randn((1024, K), device=DEV)
        L, y = [dict(W=W, b=torch.zeros(1024, device=DEV))], torch.zeros((30000, 1024), device=DEV)
        t[K] = 1e9
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            torch.cuda.synchronize()
            a.record()
            for _ in range(20):
                api.lattice_mlp_heads_fwd(L, x, [y], True)
            b.record()
            torch.cuda.synchronize()
            t[K] = min(t[K], a.elapsed_time(b))
    print(f"[gemm-f32-short] {t}", flush=True)
    assert t[13] <= 0.87 * t[64], t
