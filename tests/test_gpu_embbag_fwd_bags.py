"""The pooled lookup on both sides of the 65,536 bags from which a wave takes 16
of them instead of 4: short and empty bags, waves over two and more features,
a batch that is no multiple of 16, every row width class, both types and pools.
Against the float64 sums of the same rows, within the fp32 bound of any order
and one rounding to the storage type; other slots stay as they are."""
import pytest
import torch

from tests._util import DEV


@pytest.mark.gpu
@pytest.mark.parametrize("F,B", [(7, 9361), (7, 9363), (13, 5041), (13, 5043), (6000, 11), (5, 40_001)])
@pytest.mark.parametrize("dtype,d,pool", [(torch.bfloat16, 128, "sum"), (torch.bfloat16, 96, "mean"), (torch.float32, 32, "mean"),
                                          (torch.float32, 64, "sum"), (torch.bfloat16, 256, "sum"), (torch.float32, 256, "mean"),
                                          (torch.bfloat16, 8, "mean")])
def test_pooled_lookup(F, B, dtype, d, pool):
    from paper_2512_09200_amd import api
    print(f"[embbag-fwd-bags] F={F} B={B} d={d} {dtype} {pool}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(F + d)
    rows = 29
    lens = torch.randint(-1, 4, (F * B,), generator=g, device=DEV).clamp_(min=0)
    lens[torch.rand(F * B, generator=g, device=DEV) < 0.001] = 75        # more than a chunk of a wave
    offsets = torch.zeros(F * B + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(lens, 0, out=offsets[1:])
    nnz = int(offsets[-1])
    bag = torch.repeat_interleave(torch.arange(F * B, device=DEV), lens, output_size=nnz)
    idx = torch.randint(0, rows, (nnz,), generator=g, device=DEV)
    E = torch.randn((F * rows, d), generator=g, device=DEV).to(dtype)
    X = torch.full((B, F + 1, d), 7.0, dtype=dtype, device=DEV)
    api.lattice_embbag_fwd(E, torch.arange(F + 1, dtype=torch.int64, device=DEV) * rows, offsets.to(torch.int32),
                           idx.to(torch.int32), F, B, X, first_slot=1, pool=pool)
    torch.cuda.synchronize()
    assert bool((X[:, 0] == 7.0).all())
    e = E[idx + (bag // B) * rows].double()
    ref = torch.zeros((F * B, d), dtype=torch.float64, device=DEV).index_add_(0, bag, e)
    mag = torch.zeros_like(ref).index_add_(0, bag, e.abs())
    n = lens.double()[:, None]
    if pool == "mean":
        ref, mag = ref / n.clamp(min=1), mag / n.clamp(min=1)
    acc = (n + 3) * 2.0 ** -24 * mag
    us = 2.0 ** -8 if dtype == torch.bfloat16 else 0.0
    bound = acc + us * (ref.abs() + acc)
    got = X[:, 1:].transpose(0, 1).reshape(F * B, d).double()
    assert bool(((got - ref).abs() <= bound).all())
    assert bool((got[lens == 0] == 0).all())
