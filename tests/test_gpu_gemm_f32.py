"""fp32 GEMM edges through the C ABI: one ReLU layer forward and backward
(forward, input gradient with the ReLU mask, weight gradient with the bias
gradient as its row sums) at sizes around the 64-row, 64-k tiles, on both
sides of the batch from which the weight gradient splits K (512), with rows
not aligned to 16 bytes and with NaN between them, and with a row stride so
large (2^23 elements) that the loads go by pointer.  Every product is within
the fp32 accumulation bound of the float64 product of the same operands."""
import numpy as np
import pytest
import torch

from tests._util import DEV, _np64, assert_product

SHAPES = [  # batch, inputs, outputs, row stride of the input
    (1, 1, 1, 1), (63, 64, 65, 64), (64, 63, 64, 63), (65, 129, 63, 131), (130, 13, 64, 16), (511, 65, 130, 67),
    (512, 64, 8, 64), (513, 300, 70, 300), (2049, 71, 300, 75), (1024, 415, 512, 416), (5, 70, 66, 1 << 23),
]


@pytest.mark.gpu
@pytest.mark.parametrize("B,K,N,ld", SHAPES)
def test_f32_layer(B, K, N, ld):
    from paper_2512_09200_amd import api
    print(f"[gemm-f32] B={B} K={K} N={N} ld={ld}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(B * 1000 + K)
    x = torch.full((B, ld), float("nan"), device=DEV)[:, :K] if ld < 1 << 20 else \
        torch.empty((B, ld), device=DEV)[:, :K]
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
    # ReLU is 1-Lipschitz: the bound of the pre-activation holds for its output
    assert_product("forward", y, np.maximum(X @ Wn.T + bn, 0), np.abs(X) @ np.abs(Wn).T + np.abs(bn), K + 1,
                   t=np.inf)
    assert_product("dW", L[0]["dW"], G.T @ X, np.abs(G).T @ np.abs(X), B, t=np.inf)
    assert_product("db", L[0]["db"], G.sum(0), np.abs(G).sum(0), B, t=np.inf)
    assert_product("d_in", d_in, G @ Wn, np.abs(G) @ np.abs(Wn), N, t=np.inf)
