"""The sparse gradient's workspace serves every batch of at most the lookups it
is planned for: its size never decreases with the lookups, although small
batches use shorter reduction ranges (more partial sums per lookup)."""
import ctypes
from ctypes import byref

import pytest

from paper_2512_09200_amd import _abi as A


@pytest.mark.parametrize("dim,F", [(8, 1), (64, 26), (128, 64), (256, 3000)])
def test_workspace_is_monotone(dim, F):
    lib = A.load()
    t = A.lattice_tables(data=None, dtype=A.BF16, dim=dim, total_rows=1000, row_base=None, max_rows=0)

    def size(nnz):
        j = A.lattice_jagged(num_features=F, batch=16, offsets=None, indices=None, nnz=nnz)
        return int(lib.lattice_embbag_bwd_workspace(byref(t), byref(j)))

    lim = 1 << 21
    sizes = [size(n) for n in (0, 1, 63, 64, 65, 4096, lim - 64, lim - 1, lim, lim + 1, lim + 256, 2 * lim, 4 * lim - 1,
                               4 * lim, 4 * lim + 1, 5 * lim, 2 ** 30)]
    assert all(a <= b for a, b in zip(sizes, sizes[1:])), sizes
    assert ctypes.sizeof(ctypes.c_size_t) == 8 and sizes[0] > 0
