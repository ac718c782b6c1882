"""The MFMA instances whose tile is a whole row (tile_slices 1): every factor of a short row in one launch."""
import numpy as np
import pytest

import kron_inputs

torch = pytest.importorskip("torch")          # before the library is loaded: both then use torch's HIP runtime
import paper_2401_10187_amd as km  # noqa: E402

# (dtype, rows, P, N): fewer rows than compute units, more than one round of workgroups, no multiple of them
CASES = [("float32", 5, 64, 2), ("float32", 1367, 64, 2), ("float32", 256, 32, 3), ("float32", 700, 32, 3),
         ("float32", 230, 128, 2), ("float32", 700, 128, 2), ("float64", 1, 16, 3), ("float64", 3, 16, 3),
         ("float64", 4, 16, 3), ("float64", 2101, 16, 3),
         ("float64", 3, 32, 2), ("float64", 4099, 32, 2)]


def _plan(dtype, M, P, N):
    return km.plan(M, [P] * N, [P] * N, dtype)


def test_one_launch_without_workspace_that_reaches_every_row():
    for dtype, M, P, N in CASES:
        (st,) = _plan(dtype, M, P, N)
        assert st["kernel"] == km.KM_KERNEL_MFMA and st["num_factors"] == N and st["tile_slices"] == 1
        assert st["grid"] <= M <= st["grid"] * st["tiles_per_wg"]
        assert km.workspace_size(M, [P] * N, [P] * N, dtype) == 0
    # a row that fills a compute unit's LDS: not where the last round of 256 workgroups would be mostly idle
    for M in (100, 300, 520):
        assert len(_plan("float32", M, 128, 2)) == 2


# rows that are several rounds of workgroups, with a walk that leaves a remainder
ORDERED = [("float32", 1000, 32, 3), ("float32", 4000, 32, 3), ("float32", 5000, 64, 2), ("float32", 700, 128, 2),
           ("float64", 5000, 16, 3), ("float64", 20000, 32, 2)]


@pytest.fixture
def tile_order(request):
    old = km.get_option(km.KM_OPT_TILE_ORDER)
    km.set_option(km.KM_OPT_TILE_ORDER, request.param)
    yield request.param
    km.set_option(km.KM_OPT_TILE_ORDER, old)


@pytest.mark.parametrize("tile_order", [0, 2, 3], indirect=True)
def test_the_grid_fits_the_tile_order(tile_order):
    """Contiguous ranges (order 0) and ranges inside an XCD's eighth (3) are dealt in runs of tiles_per_wg, so
    the grid has to be the number of such runs; tiles strided by the grid (2) take any grid that reaches them all."""
    for dtype, M, P, N in ORDERED:
        (st,) = _plan(dtype, M, P, N)
        grid, walk = st["grid"], st["tiles_per_wg"]
        if st["tile_order"] == 2:
            assert tile_order == 2 or M % 8 or -(-M // walk) % 8, (dtype, M, P, N)
            assert grid <= M <= grid * walk
        else:
            assert st["tile_order"] == tile_order and grid == -(-M // walk), (dtype, M, P, N, grid, walk)


@pytest.mark.gpu
@pytest.mark.parametrize("tile_order", [0, 2, 3], indirect=True)
@pytest.mark.parametrize("dtype,M,P,N", ORDERED, ids=str)
def test_every_tile_order_gives_the_same_bits(dtype, M, P, N, tile_order):
    """The order deals out rows, it does not change one: results are those of the planner's own order, bit for bit."""
    X, Fs = kron_inputs.make_problem(M, [(P, P)] * N, dtype, seed=67)
    Xd, Fd = torch.from_numpy(X).cuda(), [torch.from_numpy(F).cuda() for F in Fs]
    print("mfma_rows order %d %s M=%d %d^%d" % (tile_order, dtype, M, P, N), flush=True)
    got = km.kronmatmul(Xd, Fd)
    km.set_option(km.KM_OPT_TILE_ORDER, -1)
    assert torch.equal(got, km.kronmatmul(Xd, Fd))


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,M,P,N", CASES, ids=str)
def test_matches_the_reference(dtype, M, P, N):
    """1e-5 (fp32), 1e-12 (fp64) of the largest value (sums of P terms per factor: at most (P + 1) N u of the
    product of absolute values), and bit for bit on small integers."""
    import oracle
    torch = pytest.importorskip("torch")
    tol = 1e-5 if dtype == "float32" else 1e-12
    for kinds, exact in ((dict(x="uniform", f="normal"), False), (dict(x="int2", f="int1"), True)):
        X, Fs = kron_inputs.make_problem(M, [(P, P)] * N, dtype, seed=65, **kinds)
        print("mfma_rows %s M=%d %d^%d" % (dtype, M, P, N), flush=True)
        Y = km.kronmatmul(torch.from_numpy(X).cuda(), [torch.from_numpy(F).cuda() for F in Fs])
        torch.cuda.synchronize()
        ref, got = oracle.kron_matmul(X, Fs), Y.cpu().numpy()
        if exact:
            assert np.array_equal(got, ref)
        else:
            assert np.abs(got - ref).max() <= tol * np.abs(ref).max()


# rows of 32^3 floats, which have a kernel of their own: the fewest that take it, a row more than compute units, walks of several
ROW32 = [96, 257, 1030]


def test_rows_of_32_cubed_are_one_launch_from_96_on():
    for M in ROW32:
        (st,) = _plan("float32", M, 32, 3)
        assert st["block"] == 1024 and st["tile_slices"] == 1 and st["grid"] <= M <= st["grid"] * st["tiles_per_wg"]
    assert len(_plan("float32", 95, 32, 3)) > 1


@pytest.mark.gpu
@pytest.mark.parametrize("M", ROW32)
def test_rows_of_32_cubed_match_and_keep_apart(M):
    """1e-5 of the largest value (sums of 32 terms per factor, three of them: at most 99 u of the product of absolute
    values), bit for bit on small integers; what is not finite stays in its row."""
    import oracle
    for kinds, exact in ((dict(x="uniform", f="normal"), False), (dict(x="int2", f="int1"), True)):
        X, Fs = kron_inputs.make_problem(M, [(32, 32)] * 3, "float32", seed=83, **kinds)
        print("rows of 32^3, M=%d" % M, flush=True)
        Fd = [torch.from_numpy(F).cuda() for F in Fs]
        got = km.kronmatmul(torch.from_numpy(X).cuda(), Fd)
        ref = oracle.kron_matmul(X, Fs)
        if exact:
            assert np.array_equal(got.cpu().numpy(), ref)
        else:
            assert np.abs(got.cpu().numpy() - ref).max() <= 1e-5 * np.abs(ref).max()
            X[5, 77] = X[M - 1, 0] = np.inf
            bad = km.kronmatmul(torch.from_numpy(X).cuda(), Fd)
            rest = [r for r in range(M) if r not in (5, M - 1)]
            assert torch.equal(bad[rest], got[rest]) and not torch.isfinite(bad[[5, M - 1]]).any()
