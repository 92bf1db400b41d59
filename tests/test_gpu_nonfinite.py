"""Non-finite values through the interactions: an infinite embedding value
reaches exactly the outputs it belongs to, as an infinity, whatever padding a
kernel adds to the rank or the rows."""
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
