"""The batch walk (widths without a variant of their own, operands off 16
bytes) at the edges of its lane counts and tiles, with rows that cross
batches and slices, and with more columns than its 24-bit row offsets hold.
Same rule as tests/parity.py."""
import numpy as np
import pytest

import paper_2205_11622_amd as slnr
from tests.gpu_util import check_A_rows, check_Y, fused, make_problem, power_law_lengths, unfused, upload

pytestmark = pytest.mark.gpu

# 1-3 (no four floats in a row), the last width of each lane count and the first
# of the next (16, 32, 64, 128, 256 floats), widths of two and three tiles, two
# launches of 512 columns and a third of one column
WIDTHS = [(1, 1), (2, 3), (3, 2), (4, 5), (15, 17), (20, 33), (33, 31), (65, 63), (66, 130),
          (129, 127), (255, 257), (257, 255), (260, 259), (515, 513), (7, 1025)]


@pytest.mark.parametrize("K,L", WIDTHS)
def test_edge_widths(gpu, K, L):
    n = power_law_lengths(700, seed=K, cap=900)
    n[3], n[650] = 5000, 1500  # rows over several slices
    p = make_problem(n, 311, K, L, seed=L, dups=True, unsorted=True, dense="normal")
    d = upload(p)
    check_A_rows(p, fused(d), what="fused")
    Y, A = unfused(d)
    check_Y(p, Y)
    check_A_rows(p, A, what="unfused")


def test_slices_of_several_batches(gpu):
    # one resident grid of at most 8192 waves: slices of 600 items and more
    n = np.full(40_000, 110)
    n[::7] = 0
    n[5], n[20_000] = 900_000, 40_000
    p = make_problem(n, 977, 5, 6, seed=3, dups=True)
    d = upload(p)
    try:
        slnr.sparselnr_set_grid_factor(1)
        check_A_rows(p, fused(d), what="fused")
    finally:
        slnr.sparselnr_set_grid_factor(0)


def test_more_columns_than_24_bits(gpu):
    import torch
    M, N, K, L = (1 << 24) + 77, 300, 3, 5
    p = make_problem(np.full(N, 20), M, 1, 1, seed=9, dups=True)
    p.colidx[:40] = M - 1 - np.arange(40)
    g = torch.Generator(device=gpu).manual_seed(1)
    C, D, E = (torch.randn(r, c, device=gpu, generator=g) for r, c in ((N, K), (M, K), (M, L)))
    csr = [torch.from_numpy(a).to(gpu) for a in (p.rowptr, p.colidx, p.vals)]
    A = slnr.sparselnr_fused_sddmm_spmm(*csr, C, D, E)
    j = csr[1].long()
    y = csr[2].double() * (C.double().repeat_interleave(20, 0) * D[j].double()).sum(1)
    t = y[:, None] * E[j].double()
    ref, scale = t.view(N, 20, L).sum(1), t.abs().view(N, 20, L).sum(1)
    # 20 terms of 3-term dot products, each rounded at most 30 times
    assert bool(((A.double() - ref).abs() <= 30 * 2.0 ** -24 * 4 * scale).all())
