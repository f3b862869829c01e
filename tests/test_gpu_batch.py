"""The batch walk (nearly every width, any alignment) at the edges of its lane
counts and tiles, with rows that cross batches and slices, with infinities, with
more columns than its 24-bit row offsets hold and up to the limits of its counters;
the sizes at which fixed-width kernels take over.  Same rule as tests/parity.py."""
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


def gathered(csr, n, C, D, E):
    """A and its scale in fp64 for rows of n nonzeros each."""
    j = csr[1].long()
    t = C.double().repeat_interleave(n, 0) * D[j].double()
    e = E[j].double() * csr[2].double()[:, None]
    one = lambda y, x: (y[:, None] * x).view(-1, n, E.shape[1]).sum(1)  # noqa: E731
    return one(t.sum(1), e), one(t.abs().sum(1), e.abs())


def run_large(gpu, N, n, M, K, L):
    import torch
    p = make_problem(np.full(N, n), M, 1, 1, seed=9, dups=True)
    p.colidx[:40] = M - 1 - np.arange(40)
    g = torch.Generator(device=gpu).manual_seed(1)
    C, D, E = (torch.randn(r, c, device=gpu, generator=g) for r, c in ((N, K), (M, K), (M, L)))
    csr = [torch.from_numpy(a).to(gpu) for a in (p.rowptr, p.colidx, p.vals)]
    ref, scale = gathered(csr, n, C, D, E)
    for factor in (0, 1, 8):
        try:
            slnr.sparselnr_set_grid_factor(factor)
            A = slnr.sparselnr_fused_sddmm_spmm(*csr, C, D, E)
        finally:
            slnr.sparselnr_set_grid_factor(0)
        # n terms of K-term dot products: each rounded at most K + n + 2 times, the
        # sums of a tree far less; 2^-24 a rounding
        err = (A.double() - ref).abs().amax(1)
        assert bool((err <= (K + n + 2) * 2.0 ** -24 * scale.amax(1)).all()), factor


@pytest.mark.parametrize("n", [20, 3])
def test_more_columns_than_24_bits(gpu, n):
    run_large(gpu, 300, n, (1 << 24) + 77, 3, 5)


# the sizes from which K = L = 64 and 128 keep kernels of their own and one column below
# them, and the rows up to which 512 columns do and one row above them
@pytest.mark.parametrize("K,L,M,N", [(64, 64, 1 << 21, 3000), (64, 64, (1 << 21) - 1, 3000), (128, 128, 1 << 20, 3000),
                                     (128, 128, (1 << 20) - 1, 3000), (512, 512, 5000, 6144), (512, 512, 5000, 6145)])
def test_kernels_chosen_by_size(gpu, K, L, M, N):
    run_large(gpu, N, 21, M, K, L)


# wide rows, whose slices several waves share: three and five parts, hub rows over
# many slices, rows that begin in one slice and end in the parts of a later one
@pytest.mark.parametrize("K,L,N,mean", [(128, 128, 70_001, 30), (5, 260, 150_000, 40), (96, 3, 330_007, 12),
                                        (3, 96, 400_000, 20)])
def test_parts(gpu, K, L, N, mean):
    import torch
    n = power_law_lengths(N, seed=L, cap=4000)
    n = n * mean * N // int(n.sum())
    n[[7, N // 3, N - 1]] = 300_000, 20_000, 9_000
    n[N // 2:N // 2 + 5000] = 0
    p = make_problem(n, 4099, K, L, seed=K, dups=True, dense="normal")
    d = upload(p)
    check_A_rows(p, fused(d), what="fused")
    Y, A = unfused(d)
    check_Y(p, Y)
    check_A_rows(p, A, what="unfused")
    A = torch.full_like(A, float("nan"))
    slnr.sparselnr_fused_sddmm_spmm_noalloc(*(d[k] for k in ("rowptr", "colidx", "vals", "C", "D", "E")), A)
    check_A_rows(p, A, what="noalloc")


# widths of more than one launch (512 columns) whose last launch has 257 to 259 columns, and
# one beside them: 65 float4 columns, which tiles of 64 would leave one lane over
@pytest.mark.parametrize("L", [769, 770, 771, 772, 1283])
def test_tiles_of_the_last_launch(gpu, L):
    # slices of 700 items, so most of them have a row that goes on in a second batch
    n = np.full(40_000, 110)
    n[5], n[20_000] = 90_000, 4_000
    p = make_problem(n, 211, 3, L, seed=L, dups=True)
    d = upload(p)
    rows = np.concatenate([np.arange(0, 40_000, 23), [5, 20_000]])
    try:
        slnr.sparselnr_set_grid_factor(1)
        check_A_rows(p, fused(d), rows=rows, what="fused")
        check_A_rows(p, unfused(d)[1], rows=rows, what="unfused")
    finally:
        slnr.sparselnr_set_grid_factor(0)


# every ragged width of a tile, one and two tiles of K, one and two launches of L
@pytest.mark.parametrize("K,L", [(5, 6), (6, 7), (7, 5), (9, 67), (130, 3), (3, 130), (66, 259), (259, 66), (515, 769)])
def test_infinities_and_nan(gpu, K, L):
    """Where a sum is infinite or not a number in 64 bits it is so in the result, and nowhere else."""
    import torch
    n = np.tile([1, 3, 17, 40, 130, 0, 7], 40)
    p = make_problem(n, 97, K, L, seed=L, dups=True, dense="normal")
    row = np.repeat(np.arange(p.N), n)
    for what in "CDE":  # one value in a row of the operand, its column another in each row
        q = make_problem(n, 97, K, L, seed=L, dups=True, dense="normal")
        X = getattr(q, what)
        for r in range(0, X.shape[0], 3 if what == "C" else 8):
            X[r, (r * 5 + 1) % X.shape[1]] = (np.inf, -np.inf, np.nan)[r % 7 % 3]
        d = upload(q)
        with np.errstate(invalid="ignore"):
            Y = q.vals * (q.C[row].astype(float) * q.D[q.colidx]).sum(1)
            A = np.zeros((q.N, L))
            np.add.at(A, row, Y[:, None] * q.E[q.colidx])
        got_Y, got_u = unfused(d)
        for got, ref in ((fused(d), A), (got_u, A), (got_Y, Y)):
            got, ref = got.cpu(), torch.from_numpy(ref)
            ends = ~torch.isfinite(ref)
            assert ends.any() or (what == "E" and ref.dim() == 1)  # the SDDMM does not read E
            assert torch.equal(torch.isfinite(got), ~ends), what
            assert torch.equal(got[ends].isnan(), ref[ends].isnan()), what
            inf = ref.isinf()
            assert torch.equal(got[inf].double(), ref[inf]), what


def test_rows_up_to_the_index_limit(gpu):
    # N + nnz = 2^31 - 1, the nonzeros in the last rows
    import torch
    N, n = (1 << 31) - 9, 8
    rowptr = torch.zeros(N + 1, dtype=torch.int32, device=gpu)
    rowptr[N - 5:] = torch.tensor([0, 3, 3, 4, 7, n], dtype=torch.int32, device=gpu)
    col = torch.arange(n, dtype=torch.int32, device=gpu) % 3
    vals = torch.arange(1, n + 1, dtype=torch.float32, device=gpu)
    C = torch.zeros(N, 1, device=gpu)
    C[N - 4:] = torch.tensor([[2.], [3.], [5.], [7.]], device=gpu)
    D = torch.tensor([[1.], [2.], [4.]], device=gpu)
    C[N - 5] = 1
    row = torch.tensor([0, 0, 0, 2, 3, 3, 3, 4], device=gpu)
    Yref = vals * C[N - 5:][row, 0] * D[col.long(), 0]
    Aref = torch.zeros(5, device=gpu).index_add_(0, row, Yref * D[col.long(), 0])
    assert torch.equal(slnr.sparselnr_sddmm(rowptr, col, vals, C, D), Yref)  # small whole numbers: exact
    A = torch.full((N, 1), float("nan"), device=gpu)
    slnr.sparselnr_fused_sddmm_spmm(rowptr, col, vals, C, D, D, A)
    assert torch.equal(A[N - 5:, 0], Aref)
    assert int(torch.count_nonzero(A[:N - 5])) == 0
    del A, C, rowptr
    torch.cuda.empty_cache()


def test_nonzeros_up_to_the_index_limit(gpu):
    import torch
    n = (1 << 31) - 2
    rowptr = torch.tensor([0, n], dtype=torch.int32, device=gpu)
    col = torch.zeros(n, dtype=torch.int32, device=gpu)
    col[-1] = 1
    vals = torch.ones(n, device=gpu)
    C, D = torch.full((1, 1), 2., device=gpu), torch.tensor([[1.], [3.]], device=gpu)
    Y = slnr.sparselnr_sddmm(rowptr, col, vals, C, D)
    assert bool((Y[:-1] == 2).all()) and float(Y[-1]) == 6
    E = torch.tensor([[0.], [5.]], device=gpu)  # the last nonzero alone counts
    assert float(slnr.sparselnr_spmm(rowptr, col, Y, E)) == 30
    del col, vals, Y
    torch.cuda.empty_cache()


# rows of at most four nonzeros, one a lane group: full and ragged groups, windows with a
# longer row among them, rows that go on in the next batch of 512 or in the next slice
@pytest.mark.parametrize("longest", [1, 3, 4, 5])
@pytest.mark.parametrize("K,L", [(16, 16), (32, 32), (5, 30), (3, 2), (16, 64), (64, 16), (300, 20)])
def test_rows_of_a_few_nonzeros(gpu, K, L, longest):
    rng = np.random.default_rng(longest)
    n = rng.integers(0, longest + 1, 30_011)
    n[:130] = longest            # windows of 64 rows without an empty one
    n[200:1000:9] = 0
    n[2000:2063] = 0             # one row in a window, then five
    n[2064:2128] = 0
    n[[2064, 2070, 2071, 2100, 2127]] = longest
    n[9000] = 700
    p = make_problem(n, 1213, K, L, seed=K, dups=True, unsorted=True, dense="normal")
    d = upload(p)
    try:
        for factor in (0, 1):
            slnr.sparselnr_set_grid_factor(factor)
            check_A_rows(p, fused(d), what="fused")
            Y, A = unfused(d)
            check_Y(p, Y)
            check_A_rows(p, A, what="unfused")
    finally:
        slnr.sparselnr_set_grid_factor(0)


def test_rows_of_a_few_nonzeros_over_batches(gpu):
    # slices of many batches: a row is cut by every third batch's end
    p = make_problem(np.tile([3, 0, 4, 2], 350_000), 4096, 16, 16, seed=2, dups=True)
    d = upload(p)
    try:
        slnr.sparselnr_set_grid_factor(1)
        A, (Y, Au) = fused(d), unfused(d)
        rows = np.arange(0, p.N, 7)
        check_A_rows(p, A, rows=rows, what="fused")
        check_Y(p, Y, rows=rows)
        check_A_rows(p, Au, rows=rows, what="unfused")
    finally:
        slnr.sparselnr_set_grid_factor(0)


@pytest.mark.parametrize("L", [16, 32, 64, 96])
def test_long_sums_add_small_terms_first(gpu, L):
    """A row's first nonzero in each lane group is 1, the others 2^-25, which added to 1 one by
    one leave it as it is.  The four of a burst summed first make 2^-23 and count, but for
    the three beside the 1: at most a quarter of the small terms is lost, not all."""
    import torch
    n, N = 256, 40_000  # rows that neither slices nor batches of 512 split
    groups = 64 // max(4, min(64, 1 << ((L + 3) // 4 - 1).bit_length()))
    vals = torch.full((N, n), 2.0 ** -25, device=gpu)
    vals[:, :groups] = 1
    rowptr = torch.arange(N + 1, dtype=torch.int32, device=gpu) * n
    col = torch.zeros(N * n, dtype=torch.int32, device=gpu)
    E, one = torch.ones(1, L, device=gpu), torch.ones(N, 1, device=gpu)
    small = (n - groups) * 2.0 ** -25
    for A in (slnr.sparselnr_spmm(rowptr, col, vals.view(-1), E),
              slnr.sparselnr_fused_sddmm_spmm(rowptr, col, vals.view(-1), one, one[:1], E)):
        err = (A.double() - (groups + small)).abs().max()
        assert float(err) <= small / 4 + 2.0 ** -24 * groups, groups  # and the rounding of the sum itself
