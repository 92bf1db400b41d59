"""Non-finite values through the interactions: an infinite embedding value
reaches exactly the outputs it belongs to, as an infinity, whatever padding a
kernel adds to the rank or the rows, and slot 0 is copied bit for bit."""
import pytest
import torch

from tests._util import DEV


def _pattern(t):
    t = t.double()
    return torch.where(t.isnan(), 2.0, torch.where(t.isinf(), t.sign(), 0.5))


@pytest.mark.gpu
@pytest.mark.parametrize("k", [1, 8, 16, 17, 40])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16], ids=["f32", "bf16"])
def test_fm_infinity(dtype, k):
    """All other operands are positive, so that every sum an infinite X[1, 4, 7]
    enters is +inf in exact arithmetic and none is NaN."""
    from paper_2512_09200_amd import api
    print(f"[nonfinite] fm {dtype} k={k}", flush=True)
    B, n, d = 3, 10, 32
    g = torch.Generator(device=DEV).manual_seed(k)
    X, W, dO = ((torch.rand(shape, generator=g, device=DEV) + 0.1).to(dtype)
                for shape in ((B, n, d), (n, k), (B, d + n * k)))
    X[1, 4, 7] = float("inf")
    out, dX, dW = torch.zeros_like(dO), torch.zeros_like(X), torch.zeros((n, k), device=DEV)
    ws = api.lattice_interact_fwd("fm", X, out, True, fm_W=W)
    api.lattice_interact_bwd("fm", X, dO, dX, True, fm_W=W, fm_dW=dW, ws=ws)
    torch.cuda.synchronize()
    x, w, G = X.double(), W.double(), dO[:, d:].double().view(B, n, k)
    P, dP = x.transpose(1, 2).contiguous() @ w, x.transpose(1, 2).contiguous() @ G
    assert torch.equal(_pattern(out), _pattern(torch.cat([x[:, 0], (x @ P).view(B, -1)], 1)))
    assert torch.equal(_pattern(dX), _pattern(G @ P.transpose(1, 2).contiguous() + w @ dP.transpose(1, 2).contiguous()))
    assert torch.equal(_pattern(dW), _pattern((x @ dP).sum(0)))


@pytest.mark.gpu
@pytest.mark.parametrize("kind,n,d", [("dot", 9, 32), ("dot", 40, 256), ("fm", 9, 32), ("dot", 9, 64)])
def test_slot0_is_a_copy(kind, n, d):
    """Every bf16 bit pattern, NaNs with and without the quiet bit among them."""
    from paper_2512_09200_amd import api
    print(f"[nonfinite] slot 0 {kind} n={n} d={d}", flush=True)
    B, k = 65536 // d, 16
    X = torch.ones((B, n, d), dtype=torch.bfloat16, device=DEV)
    X[:, 0] = torch.arange(65536, device=DEV).to(torch.int16).view(torch.bfloat16).view(B, d)
    out = torch.zeros((B, d + (n * (n - 1) // 2 if kind == "dot" else n * k)), dtype=torch.bfloat16, device=DEV)
    W = torch.ones((n, k), dtype=torch.bfloat16, device=DEV) if kind == "fm" else None
    api.lattice_interact_fwd(kind, X, out, True, fm_W=W)
    torch.cuda.synchronize()
    assert torch.equal(out[:, :d].contiguous().view(torch.int16), X[:, 0].contiguous().view(torch.int16))
