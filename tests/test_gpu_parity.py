"""GPU parity: the HIP library (through its C-ABI) against the CPU oracle on the same seeded inputs.

Bars (written out here): bit-exact when inputs are small integers (every partial sum is exactly
representable); otherwise max|Y_gpu - Y_ref| / max|Y_ref| <= 1e-5 for fp32 and 1e-12 for fp64, with
Y_ref from the wide-accumulator oracle.  A second, per-element bound is also checked:
|Y_gpu - Y_ref| <= 2 u (sum_i P_i + N) * (|X| (x)|F_i|), the standard forward error of the chained dot
products, evaluated by running the oracle on absolute values.
"""
import numpy as np
import pytest

import kron_inputs
import oracle

torch = pytest.importorskip("torch")
import paper_2401_10187_amd as km  # noqa: E402

pytestmark = pytest.mark.gpu

REL_TOL = {np.dtype("float32"): 1e-5, np.dtype("float64"): 1e-12}
UNIT = {np.dtype("float32"): 2.0 ** -24, np.dtype("float64"): 2.0 ** -53}


@pytest.fixture(scope="module", autouse=True)
def _device():
    if not torch.cuda.is_available():
        pytest.fail("gpu-marked tests need a GPU (torch.cuda.is_available() is False)")
    km.lib()   # fails loudly if the HIP library has not been built
    yield
    km.release()


class options:
    """Temporarily restrict the planner (kernel families bit mask, fusion depth)."""

    def __init__(self, kernels=None, max_fuse=None, tile=None, threads=None, tiles_per_wg=None, pair=None,
                 order=None, instance=None, keep_mib=None):
        self.new = {km.KM_OPT_KERNELS: kernels, km.KM_OPT_MAX_FUSE: max_fuse, km.KM_OPT_PREFER_TILE: tile,
                    km.KM_OPT_PREFER_THREADS: threads, km.KM_OPT_TILES_PER_WG: tiles_per_wg,
                    km.KM_OPT_PAIR_INTERLEAVE: pair, km.KM_OPT_TILE_ORDER: order,
                    km.KM_OPT_PREFER_INSTANCE: instance, km.KM_OPT_KEEP_MIB: keep_mib}

    def __enter__(self):
        self.old = {k: km.get_option(k) for k in self.new}
        for k, v in self.new.items():
            if v is not None:
                km.set_option(k, v)

    def __exit__(self, *exc):
        for k, v in self.old.items():
            km.set_option(k, v)


def run_gpu(X, Fs, use_ws=False):
    Xd = torch.from_numpy(X).cuda()
    Fd = [torch.from_numpy(F).cuda() for F in Fs]
    ws = None
    if use_ws:
        nbytes = km.workspace_size(X.shape[0], [F.shape[0] for F in Fs], [F.shape[1] for F in Fs], X.dtype)
        ws = torch.empty(max(nbytes, 1), dtype=torch.uint8, device="cuda")
    Y = km.kronmatmul(Xd, Fd, workspace=ws)
    torch.cuda.synchronize()
    assert torch.equal(Xd.cpu(), torch.from_numpy(X)), "X was modified"
    return Y.cpu().numpy()


def assert_close(got, X, Fs, exact=False):
    ref = oracle.kron_matmul(X, Fs)
    assert got.shape == ref.shape and got.dtype == ref.dtype
    if exact:
        assert np.array_equal(got, ref)
        return
    scale = float(np.abs(ref).max())
    err = float(np.abs(got.astype(np.float64) - ref.astype(np.float64)).max())
    assert err <= REL_TOL[ref.dtype] * scale, (err, scale)
    bound = oracle.kron_matmul(np.abs(X), [np.abs(F) for F in Fs]).astype(np.float64)
    n_terms = sum(F.shape[0] for F in Fs) + len(Fs)
    slack = 2 * UNIT[ref.dtype] * n_terms * bound + np.finfo(np.float64).tiny
    assert np.all(np.abs(got.astype(np.float64) - ref.astype(np.float64)) <= slack)


# shapes that span several tiles, ragged tails and the degenerate cases
SMALL_CASES = [
    ("float32", 16, [(8, 8)] * 3),                       # config 1
    ("float32", 5, [(8, 8)] * 4),
    ("float32", 3, [(8, 8)] * 2),
    ("float32", 2, [(8, 8)]),
    ("float32", 3, [(4, 4)] * 5),
    ("float32", 7, [(3, 5), (4, 2), (6, 6), (2, 3)]),    # distinct rectangular factors
    ("float64", 4, [(5, 2), (5, 2), (5, 2)]),
    ("float32", 2, [(1, 3), (7, 1), (2, 2)]),            # P = 1 and Q = 1
    ("float32", 1, [(130, 70)]),                         # N = 1, ragged everything
    ("float64", 3, [(33, 17), (2, 65)]),
    ("float32", 9, [(16, 32)] * 3),                      # growing intermediates
    ("float32", 4, [(32, 16)] * 3),                      # shrinking intermediates
    ("float32", 6, [(32, 32)] * 3),
    ("float32", 2, [(16, 16)] * 4),
    ("float64", 2, [(128, 128)] * 2),
    ("float64", 3, [(16, 16)] * 3),
    ("float32", 2, [(64, 64)] * 2),
    ("float64", 1, [(8, 8)] * 5),
    ("float32", 1, [(2, 2)] * 11),                       # many tiny factors, M = 1
    ("float32", 5, [(8, 8), (8, 8), (8, 8), (32, 32), (32, 32)]),
    ("float32", 2, [(128, 128)] * 2),
    ("float64", 2, [(64, 64)] * 2),
    ("float64", 2, [(32, 32)] * 3),
    ("float32", 3, [(16, 16)] * 5),
    ("float64", 1, [(16, 16)] * 4),
    # very small factors: several factors per LDS pass, tile length chosen at launch
    ("float32", 3, [(3, 3)] * 7),
    ("float32", 2, [(6, 6)] * 4),
    ("float32", 3, [(5, 5)] * 4),
    ("float32", 1, [(5, 5), (5, 5), (5, 5), (2, 2)]),
    ("float32", 20, [(2, 2)] * 7),
    ("float32", 5, [(4, 4)] * 7),
    ("float32", 4, [(2, 2)] * 12),
    ("float64", 2, [(2, 2)] * 10),
    ("float64", 3, [(4, 4)] * 5),
    ("float64", 5, [(4, 4)] * 7),
    ("float64", 2, [(8, 8)] * 4),
    ("float32", 7, [(4, 4), (4, 4), (2, 2), (2, 2), (2, 2), (3, 3)]),
    ("float64", 3, [(3, 3)] * 8),
    ("float64", 2, [(5, 5)] * 5),
    ("float64", 2, [(6, 6)] * 5),
    ("float64", 1, [(6, 6)] * 3 + [(3, 3)] * 2),
    # rows of K = P^2: one whole row per tile of the single-factor MFMA instances
    ("float32", 70, [(16, 16)] * 2),
    ("float32", 33, [(32, 32)] * 2),
    ("float32", 9, [(64, 64)] * 2),
    ("float64", 21, [(16, 16)] * 2),
    ("float64", 10, [(32, 32)] * 2),
    ("float64", 5, [(64, 64)] * 2),
    # rectangular small factors, growing and shrinking rows
    ("float32", 5, [(2, 4)] * 7),
    ("float32", 5, [(4, 2)] * 7),
    ("float64", 3, [(4, 8)] * 4),
    ("float64", 3, [(8, 4)] * 5),
    ("float32", 1100, [(2, 4)] * 4),
    ("float32", 4, [(4, 8), (4, 8), (8, 4), (8, 4), (2, 4)]),
    # rows of exactly P*P elements: the pair kernel that takes rows as its slow index, ragged last tile
    ("float32", 1000, [(32, 32)] * 2),
    ("float32", 77, [(16, 32)] * 2),
    ("float32", 1, [(32, 32)] * 2),
    ("float32", 3, [(7, 7)] * 5),
    ("float64", 2, [(7, 7)] * 5),
    ("float32", 2, [(9, 9)] * 4),
    ("float64", 3, [(9, 9)] * 4),
    ("float32", 5, [(10, 10)] * 4),
    ("float64", 1, [(10, 10)] * 4),
    ("float32", 2, [(12, 12)] * 4),
    ("float64", 3, [(12, 12)] * 3),
    # P and Q multiples of 16 without compiled instances: the run-time-shape MFMA kernel (ragged last
    # unit, slices of a unit in different rows, 3/4/5 column blocks, partial last column group, several
    # LDS chunks with a short last one)
    ("float32", 3, [(48, 48)] * 2),
    ("float32", 5, [(96, 96)] * 2),
    ("float32", 2, [(80, 112), (48, 80)]),
    ("float64", 3, [(48, 48)] * 2),
    ("float64", 2, [(112, 80), (96, 48)]),
    ("float32", 7, [(144, 16)]),
    ("float32", 301, [(48, 96)]),
    ("float64", 67, [(80, 160)]),
    ("float32", 2, [(48, 48)] * 3),
    ("float32", 3, [(8, 8), (48, 48), (8, 8), (8, 8)]),
    # the same kernel on shapes it pads to multiples of 16 with zeros (P a whole number of 16-byte
    # vectors, Q anything): narrow units for slices of up to 128 bytes, factors read element by element
    # when Q is not a whole number of vectors, output runs that start off 64-byte boundaries
    ("float32", 3, [(20, 20)] * 3),
    ("float32", 5, [(36, 36)] * 2),
    ("float32", 2, [(24, 28), (28, 20)]),
    ("float32", 7, [(20, 15)] * 3),
    ("float32", 1, [(100, 100)] * 2),
    ("float32", 3, [(36, 50), (52, 33)]),
    ("float32", 300, [(32, 20)]),
    ("float32", 2, [(16, 80)] * 2),
    ("float64", 3, [(14, 14)] * 3),
    ("float64", 2, [(40, 40)] * 2),
    ("float64", 5, [(30, 30)] * 2),
    ("float64", 3, [(16, 48), (44, 41)]),
    ("float64", 129, [(90, 90)]),
    # ... and on slices that do not start on 16-byte boundaries (a unit fetched as one contiguous run):
    # odd P, P = 2 mod 4, narrow and wide units, ragged last unit, more slices than one unit per row
    ("float32", 3, [(13, 13)] * 4),
    ("float32", 5, [(22, 22)] * 3),
    ("float32", 2, [(33, 40), (50, 33)]),
    ("float32", 700, [(19, 19)]),
    ("float32", 1, [(63, 63)] * 2),
    ("float64", 3, [(15, 15)] * 3),
    ("float64", 2, [(27, 27)] * 2),
    ("float64", 301, [(31, 20)]),
    ("float64", 4, [(11, 11)] * 4),
    # ... and on such slices of several 256-byte chunks (a chunk row starts anywhere inside a 16-byte
    # vector): ragged last unit, last chunks of 1 to 15 elements, X that ends inside a vector
    ("float32", 3, [(65, 65)] * 2),
    ("float32", 1, [(99, 70), (67, 33)]),
    ("float32", 130, [(127, 20)]),
    ("float32", 1, [(65, 16)]),
    ("float32", 7, [(129, 24)]),
    ("float64", 2, [(33, 33)] * 3),
    ("float64", 5, [(45, 37), (35, 50)]),
    ("float64", 200, [(81, 17)]),
    ("float64", 1, [(33, 16)]),
    # whole short rows in one launch: four super-stages, tiles up to the whole LDS, several rows per tile
    ("float32", 3, [(2, 2)] * 15),
    ("float64", 2, [(3, 3)] * 9),
    ("float32", 2, [(7, 7)] * 5),
    ("float32", 3, [(14, 14)] * 4),
    ("float64", 1100, [(5, 5)] * 4),
    ("float32", 1030, [(7, 7)] * 4),
    ("float32", 1100, [(11, 11)] * 3),
    ("float32", 3, [(2, 4)] * 7),
    ("float64", 1100, [(4, 8)] * 3),
    ("float32", 2, [(8, 4)] * 5),
    ("float64", 1030, [(12, 12)] * 3),
    # tiles of several whole rows with rectangular factors: output rows longer or shorter than the input rows
    ("float32", 1100, [(4, 8)]),
    ("float32", 1500, [(2, 4)] * 2),
    ("float32", 1030, [(8, 4)] * 2),
    ("float32", 2050, [(4, 2)] * 3),
    ("float32", 1025, [(4, 8)] * 3),
    # neighbouring runs of different small shapes fused into one launch
    ("float32", 5, [(4, 4)] * 5 + [(2, 2)] * 4),
    ("float32", 3, [(3, 3)] + [(4, 4)] * 2 + [(2, 2)] * 4),
    ("float64", 4, [(8, 8)] * 2 + [(4, 4)] * 2),
    ("float32", 1100, [(5, 5)] * 2 + [(2, 2)]),
    ("float32", 7, [(2, 2)] + [(5, 5)] * 2 + [(9, 9)]),
    ("float64", 2, [(7, 7)] + [(2, 2)] * 4 + [(4, 4)] * 2),
]


@pytest.mark.parametrize("dtype,M,shapes", SMALL_CASES, ids=lambda v: str(v).replace(" ", ""))
@pytest.mark.parametrize("mode", ["auto", "unfused", "generic"])
def test_small_float(dtype, M, shapes, mode):
    kw = {"auto": {}, "unfused": {"max_fuse": 1}, "generic": {"kernels": 0}}[mode]
    X, Fs = kron_inputs.make_problem(M, shapes, dtype, "uniform", "normal", seed=len(shapes) * 100 + M)
    with options(**kw):
        got = run_gpu(X, Fs, use_ws=(mode == "unfused"))
    assert_close(got, X, Fs)


@pytest.mark.parametrize("dtype,M,shapes", SMALL_CASES, ids=lambda v: str(v).replace(" ", ""))
def test_small_integer_bit_exact(dtype, M, shapes):
    width = int(np.prod([max(p, 1) for p, _ in shapes], dtype=np.int64))
    fdist = "int2" if 2 * 2 ** len(shapes) * width < 2 ** 24 else "int1"
    if 2 * width >= 2 ** 24 and dtype == "float32":
        pytest.skip("sums not exactly representable in fp32")
    X, Fs = kron_inputs.make_problem(M, shapes, dtype, "int2", fdist, seed=7)
    assert_close(run_gpu(X, Fs), X, Fs, exact=True)


@pytest.mark.parametrize("dtype,M,shapes", [("float32", 5, [(48, 80), (96, 48)]), ("float64", 3, [(48, 48)] * 2),
                                            ("float32", 3, [(20, 20)] * 2), ("float64", 2, [(14, 40), (40, 14)]),
                                            ("float32", 3, [(13, 13)] * 4), ("float64", 2, [(15, 22), (27, 15)]),
                                            ("float32", 4, [(8, 8)] * 3), ("float32", 3, [(32, 32)] * 3),
                                            ("float64", 2, [(5, 3), (16, 16), (7, 9)])],
                         ids=lambda v: str(v).replace(" ", ""))
def test_factors_need_only_their_elements_alignment(dtype, M, shapes):
    """X and Y must start on 16-byte boundaries, factors need not: each factor here starts one element
    into its allocation."""
    X, Fs = kron_inputs.make_problem(M, shapes, dtype, seed=41)
    Xd = torch.from_numpy(X).cuda()
    Fd = []
    for F in Fs:
        buf = torch.empty(F.size + 1, dtype=Xd.dtype, device="cuda")
        view = buf[1:].view(F.shape)
        view.copy_(torch.from_numpy(F))
        assert view.data_ptr() % 16 != 0 and view.is_contiguous()
        Fd.append(view)
    Y = km.kronmatmul(Xd, Fd)
    torch.cuda.synchronize()
    assert_close(Y.cpu().numpy(), X, Fs)


# every compiled instance and launch mode, forced through the tuning options, on mid-size inputs
def _random_problems(count, seed, pool=(1, 2, 2, 3, 4, 4, 5, 6, 7, 8, 8, 9, 12, 16, 16, 17, 32, 32, 33, 64),
                     max_m=40):
    """Seeded random problems: any mix of factor shapes (runs of equal shapes are likely, so fused
    groups, single launches and the generic kernel all occur), rows of at most 2^17 elements."""
    rng = np.random.default_rng(seed)
    pool = list(pool)
    out = []
    while len(out) < count:
        n = int(rng.integers(1, 7))
        shapes = []
        while len(shapes) < n:
            p, q = int(rng.choice(pool)), int(rng.choice(pool))
            if rng.random() < 0.6:
                q = p
            shapes += [(p, q)] * int(min(n - len(shapes), rng.integers(1, 4)))
        widths = [int(np.prod([s[0] for s in shapes], dtype=np.int64))]
        for p, q in reversed(shapes):
            widths.append(widths[-1] // p * q)
        if max(widths) > 2 ** 17:
            continue
        out.append(("float32" if rng.random() < 0.6 else "float64", int(rng.integers(1, max_m + 1)), shapes))
    return out


@pytest.mark.parametrize("dtype,M,shapes", _random_problems(48, 2024), ids=lambda v: str(v).replace(" ", ""))
def test_random_shapes(dtype, M, shapes):
    X, Fs = kron_inputs.make_problem(M, shapes, dtype, seed=300 + M + len(shapes))
    assert_close(run_gpu(X, Fs), X, Fs)
    Xi, Fi = kron_inputs.make_problem(M, shapes, dtype, x="int2", f="int1", seed=400 + M)
    if 2.0 * np.prod([s[0] for s in shapes], dtype=np.float64) < (2 ** 24 if dtype == "float32" else 2 ** 53):
        assert_close(run_gpu(Xi, Fi, use_ws=True), Xi, Fi, exact=True)


@pytest.mark.parametrize("dtype,M,shapes", _random_problems(32, 31, pool=(2, 2, 2, 4, 4, 4, 8, 8, 5, 3, 20, 36, 40, 14, 48, 100),
                                                          max_m=600), ids=lambda v: str(v).replace(" ", ""))
def test_random_shapes_of_mixed_small_and_padded_factors(dtype, M, shapes):
    """Random problems from the shapes the per-stage small-factor instances and the zero-padding MFMA
    kernel take, with up to 600 rows so that the planner finds enough workgroups to fuse."""
    X, Fs = kron_inputs.make_problem(M, shapes, dtype, seed=500 + M + len(shapes))
    assert_close(run_gpu(X, Fs), X, Fs)
    Xi, Fi = kron_inputs.make_problem(M, shapes, dtype, x="int2", f="int1", seed=600 + M)
    if 2.0 * np.prod([s[0] for s in shapes], dtype=np.float64) < (2 ** 24 if dtype == "float32" else 2 ** 53):
        assert_close(run_gpu(Xi, Fi, use_ws=True), Xi, Fi, exact=True)


def _random_short_row_problems(count, seed):
    """Seeded random problems with many short rows (M of 1024 to 6000, rows of at most 4096 elements)."""
    rng = np.random.default_rng(seed)
    out = []
    while len(out) < count:
        p = int(rng.choice([2, 3, 4, 5, 6, 7, 8, 9, 10, 12, 16, 32]))
        n = int(rng.integers(1, 7))
        if p ** n > 4096:
            continue
        shapes = [(p, p)] * n
        if rng.random() < 0.3:                      # a second family in front
            p2 = int(rng.choice([2, 3, 4, 5]))
            if p2 * p ** n <= 4096:
                shapes = [(p2, p2)] + shapes
        out.append(("float32" if rng.random() < 0.6 else "float64", int(rng.integers(1024, 6001)), shapes))
    return out


@pytest.mark.parametrize("dtype,M,shapes", _random_short_row_problems(24, 7), ids=lambda v: str(v).replace(" ", ""))
def test_random_short_row_shapes(dtype, M, shapes):
    X, Fs = kron_inputs.make_problem(M, shapes, dtype, x="int2", f="int1", seed=500 + M)
    assert_close(run_gpu(X, Fs), X, Fs, exact=True)
    X, Fs = kron_inputs.make_problem(M, shapes, dtype, seed=600 + M)
    assert_close(run_gpu(X, Fs, use_ws=True), X, Fs)


FORCED = [
    ("float32", 64, [(32, 32)] * 3, dict(tile=16, threads=256, tiles_per_wg=1, pair=1)),
    ("float32", 64, [(32, 32)] * 3, dict(tile=16, threads=256, tiles_per_wg=4, pair=1)),
    ("float32", 64, [(32, 32)] * 3, dict(tile=16, threads=256, tiles_per_wg=4, pair=0)),
    ("float32", 16, [(32, 32)] * 3, dict(tile=32, threads=512, tiles_per_wg=3)),
    ("float32", 16, [(32, 32)] * 3, dict(tile=32, threads=1024, tiles_per_wg=2)),
    ("float32", 16, [(32, 32)] * 3, dict(max_fuse=1, tile=128)),
    ("float32", 16, [(32, 32)] * 3, dict(max_fuse=1, tile=256, tiles_per_wg=5)),
    ("float32", 32, [(16, 32)] * 3, dict(tile=16, tiles_per_wg=2, pair=1)),
    ("float32", 4, [(16, 32)] * 4, dict(tile=32, tiles_per_wg=2)),
    ("float32", 8, [(16, 32)] * 3, dict(max_fuse=1, tile=128)),
    ("float64", 8, [(128, 128)] * 2, dict(tiles_per_wg=7)),
    ("float64", 8, [(128, 128)] * 2, dict(tiles_per_wg=7, order=0)),
    ("float32", 16, [(32, 32)] * 3, dict(tile=32, threads=256, tiles_per_wg=3, order=0)),
    ("float32", 16, [(32, 32)] * 3, dict(tile=32, threads=256, tiles_per_wg=3, order=2)),
    ("float32", 4, [(16, 32)] * 4, dict(tile=32, tiles_per_wg=5, order=0)),
    ("float64", 8, [(128, 128)] * 2, dict(tiles_per_wg=1)),
    ("float64", 8, [(128, 128)] * 2, dict(tiles_per_wg=5, order=3)),
    ("float64", 8, [(128, 128)] * 2, dict(tile=32, threads=256)),
    ("float64", 8, [(128, 128)] * 2, dict(tile=32, threads=512, tiles_per_wg=3)),
    ("float32", 16, [(32, 32)] * 3, dict(tile=32, threads=256, tiles_per_wg=4, order=3)),
    ("float32", 16, [(32, 32)] * 3, dict(tile=32, threads=256, tiles_per_wg=3, order=3)),   # grid not a multiple of 8: falls back to 2
    ("float32", 8, [(16, 32)] * 4, dict(tile=32, tiles_per_wg=2, order=3)),
    ("float32", 8, [(8, 8)] * 6, dict(tile=32, threads=256)),
    ("float32", 8, [(8, 8)] * 6, dict(tile=32, threads=1024)),
    ("float32", 8, [(8, 8)] * 6, dict(tile=16, threads=256)),
    ("float32", 8, [(8, 8)] * 6, dict(tile=8, threads=128)),
    ("float32", 8, [(8, 8)] * 6, dict(tile=1)),
    ("float32", 8, [(8, 8)] * 6, dict(max_fuse=2, tile=256)),
    ("float32", 8, [(8, 8)] * 6, dict(max_fuse=2, tile=64)),
    ("float32", 8, [(8, 8)] * 6, dict(max_fuse=2, tile=8)),
    ("float32", 8, [(8, 8)] * 6, dict(max_fuse=1, tile=2048)),
    ("float32", 8, [(8, 8)] * 6, dict(max_fuse=1, tile=64)),
    ("float32", 8, [(8, 8)] * 6, dict(max_fuse=1, tile=8)),
    ("float32", 8, [(8, 8)] * 6, dict(max_fuse=1, kernels=8 | 1)),      # shuffle family only
    ("float32", 3, [(8, 8)] * 5, dict(max_fuse=1, kernels=8 | 1)),
]


@pytest.mark.parametrize("dtype,M,shapes,opts", FORCED, ids=lambda v: str(v).replace(" ", ""))
def test_forced_instances(dtype, M, shapes, opts):
    P = [s[0] for s in shapes]
    Q = [s[1] for s in shapes]
    with options(**opts):
        steps = km.plan(M, P, Q, dtype)
        if "tile" in opts:
            assert any(st["tile_slices"] == opts["tile"] for st in steps), steps
        X, Fs = kron_inputs.make_problem(M, shapes, dtype, "uniform", "normal", seed=17)
        got = run_gpu(X, Fs)
        assert_close(got, X, Fs)
        Xi, Fi = kron_inputs.make_problem(M, shapes, dtype, "int2", "int1", seed=18)
        assert_close(run_gpu(Xi, Fi), Xi, Fi, exact=True)


EVERY_INSTANCE = [
    ("float32", 8, [(8, 8)] * 6), ("float64", 4, [(8, 8)] * 5),
    ("float32", 16, [(32, 32)] * 3), ("float32", 32, [(32, 32)] * 4), ("float64", 4, [(32, 32)] * 3),
    ("float32", 4, [(16, 32)] * 4),
    ("float32", 8, [(16, 16)] * 4), ("float64", 8, [(16, 16)] * 4),
    ("float32", 8, [(64, 64)] * 3), ("float64", 8, [(64, 64)] * 3),
    ("float32", 4, [(128, 128)] * 2), ("float64", 8, [(128, 128)] * 2),
    ("float32", 8, [(48, 48)] * 3), ("float64", 4, [(48, 48)] * 3),
    ("float32", 2, [(96, 96)] * 3), ("float32", 2, [(80, 80)] * 3), ("float32", 2, [(112, 112)] * 3), ("float32", 1, [(144, 144)] * 3),
    ("float64", 2, [(80, 80)] * 3), ("float64", 1, [(96, 96)] * 3), ("float64", 1, [(112, 112)] * 3), ("float64", 1, [(144, 144)] * 3),
    ("float32", 1, [(160, 160)] * 3), ("float32", 1, [(192, 192)] * 3), ("float32", 1, [(256, 256)] * 3),
    ("float64", 1, [(160, 160)] * 3), ("float64", 1, [(192, 192)] * 3),
    ("float32", 2, [(2, 2)] * 14), ("float64", 2, [(2, 2)] * 13),
    ("float32", 3, [(3, 3)] * 9), ("float64", 3, [(3, 3)] * 9),
    ("float32", 4, [(4, 4)] * 8), ("float64", 4, [(4, 4)] * 7), ("float64", 64, [(4, 4)] * 7),
    ("float32", 2, [(5, 5)] * 6), ("float64", 2, [(5, 5)] * 6), ("float32", 300, [(5, 5)] * 6), ("float32", 300, [(5, 5)] * 8), ("float32", 300, [(4, 4)] * 7),
    ("float32", 2, [(6, 6)] * 6), ("float64", 2, [(6, 6)] * 6),
    ("float32", 2, [(7, 7)] * 5), ("float64", 2, [(7, 7)] * 5),
    ("float32", 2, [(9, 9)] * 5), ("float64", 2, [(9, 9)] * 4),
    ("float32", 2, [(10, 10)] * 5), ("float64", 2, [(10, 10)] * 4),
    ("float32", 2, [(12, 12)] * 4), ("float64", 2, [(12, 12)] * 4),
    ("float32", 3, [(11, 11)] * 4), ("float64", 3, [(11, 11)] * 4), ("float32", 3, [(13, 13)] * 4), ("float64", 3, [(13, 13)] * 4),
    ("float32", 2, [(14, 14)] * 4), ("float64", 2, [(14, 14)] * 4), ("float32", 2, [(15, 15)] * 4), ("float64", 2, [(15, 15)] * 4),
    # short rows, for the instances with short tiles
    ("float32", 16, [(8, 8)] * 3), ("float32", 5, [(8, 8)] * 4), ("float32", 3, [(8, 8)] * 2), ("float32", 2, [(8, 8)]),
    ("float32", 6, [(32, 32)] * 2), ("float32", 8, [(16, 32)] * 3), ("float32", 5, [(16, 16)] * 2),
    ("float64", 5, [(16, 16)] * 3), ("float64", 3, [(32, 32)] * 2), ("float32", 3, [(64, 64)] * 2),
    ("float32", 1100, [(8, 8)] * 2), ("float32", 1100, [(8, 8)]), ("float64", 3, [(8, 8)] * 3),
    ("float32", 2, [(2, 2)] * 9), ("float64", 2, [(4, 4)] * 4), ("float32", 2, [(4, 4)] * 5),
    ("float64", 2, [(2, 2)] * 9), ("float64", 2, [(9, 9)] * 3), ("float64", 2, [(10, 10)] * 3),
    ("float32", 9, [(16, 32)] * 2),
    # rectangular factors on the matrix cores
    ("float32", 4, [(32, 16)] * 3), ("float32", 4, [(64, 16)] * 3), ("float32", 4, [(64, 32)] * 3),
    ("float32", 8, [(32, 64)] * 3), ("float32", 8, [(16, 64)] * 4), ("float32", 4, [(128, 64)] * 2),
    ("float32", 8, [(64, 128)] * 3), ("float32", 4, [(128, 32)] * 2), ("float32", 16, [(32, 128)] * 3),
    ("float64", 4, [(32, 16)] * 3), ("float64", 4, [(16, 32)] * 4), ("float64", 4, [(64, 32)] * 3),
    ("float64", 4, [(32, 64)] * 3),
    # rectangular small factors
    ("float32", 3, [(2, 4)] * 6), ("float32", 3, [(4, 2)] * 6), ("float32", 3, [(4, 8)] * 4), ("float32", 3, [(8, 4)] * 5),
    ("float64", 3, [(2, 4)] * 6), ("float64", 3, [(4, 2)] * 6), ("float64", 3, [(4, 8)] * 4), ("float64", 3, [(8, 4)] * 4),
    ("float32", 2, [(2, 4)] * 2), ("float32", 2, [(4, 2)]), ("float64", 2, [(4, 8)]), ("float32", 2, [(8, 4)] * 2),
    # six 2x2 factors in one launch
    ("float32", 2, [(2, 2)] * 6), ("float64", 2, [(2, 2)] * 6),
    # whole short rows in one launch: up to twelve 2x2, seven 3x3 or 4x4 factors
    ("float32", 3, [(2, 2)] * 12), ("float32", 3, [(2, 2)] * 11), ("float32", 3, [(2, 2)] * 10), ("float32", 3, [(2, 2)] * 8),
    ("float32", 3, [(2, 2)] * 7), ("float32", 3, [(2, 2)] * 5), ("float32", 3, [(2, 2)] * 4),
    ("float64", 3, [(2, 2)] * 12), ("float64", 3, [(2, 2)] * 11), ("float64", 3, [(2, 2)] * 10), ("float64", 3, [(2, 2)] * 8),
    ("float64", 3, [(2, 2)] * 7), ("float64", 3, [(2, 2)] * 5), ("float64", 3, [(2, 2)] * 4),
    ("float32", 3, [(4, 4)] * 7), ("float32", 3, [(4, 4)] * 6), ("float32", 3, [(4, 4)] * 5),
    ("float64", 3, [(4, 4)] * 6), ("float64", 3, [(4, 4)] * 5),
    ("float32", 3, [(3, 3)] * 7), ("float32", 3, [(3, 3)] * 6), ("float32", 3, [(3, 3)] * 5),
    ("float64", 3, [(3, 3)] * 7), ("float64", 3, [(3, 3)] * 6), ("float64", 3, [(3, 3)] * 5),
    # one launch for a single short row, and two shapes whose groupings name the remaining instances
    ("float32", 1, [(4, 4)] * 7), ("float32", 1, [(5, 5)] * 3), ("float32", 1, [(6, 6)] * 3), ("float64", 1, [(6, 6)] * 3),
    ("float64", 1, [(6, 6)] * 2), ("float32", 1, [(9, 9)] * 3), ("float32", 64, [(8, 8)] * 4), ("float64", 64, [(32, 32)] * 3),
    ("float64", 64, [(8, 8)] * 6),
    # rows of 6^7 elements, for the 6x6 instances with fixed tiles of 48, 288 and 16 slices
    ("float32", 24, [(6, 6)] * 7), ("float64", 12, [(6, 6)] * 7),
    # neighbouring runs of different small shapes in one launch (a factor shape per stage): whole rows as
    # tiles, several tiles per row behind other factors, many short rows per tile
    ("float32", 300, [(4, 4)] * 5 + [(2, 2)] * 4), ("float32", 300, [(4, 4)] * 4 + [(2, 2)] * 4),
    ("float32", 300, [(2, 2)] * 8 + [(4, 4)] * 2), ("float32", 300, [(8, 8)] * 2 + [(4, 4)] * 2),
    ("float32", 300, [(4, 4)] * 2 + [(8, 8)] * 2), ("float64", 300, [(4, 4)] * 4 + [(2, 2)] * 4),
    ("float64", 300, [(8, 8)] * 2 + [(4, 4)] * 2),
    ("float32", 300, [(6, 6)] * 2 + [(4, 4)] * 2 + [(2, 2)] * 4),
    ("float32", 300, [(6, 6)] * 2 + [(4, 4)] * 2 + [(2, 2)] * 3),
    ("float32", 300, [(6, 6)] * 2 + [(2, 2)] * 4 + [(4, 4)] * 2),
    ("float32", 300, [(6, 6)] * 2 + [(8, 8)] * 2 + [(2, 2)] * 3),
    ("float32", 300, [(6, 6)] * 2 + [(2, 2)] * 3 + [(8, 8)] * 2), ("float32", 300, [(6, 6)] * 3 + [(5, 5)] * 2 + [(2, 2)]),
    ("float32", 300, [(6, 6)] * 3 + [(2, 2)] + [(5, 5)] * 2), ("float32", 300, [(7, 7)] * 3 + [(3, 3)] * 2 + [(2, 2)] * 2),
    ("float64", 300, [(6, 6)] * 2 + [(4, 4)] * 2 + [(2, 2)] * 4),
    ("float64", 300, [(6, 6)] * 2 + [(2, 2)] * 4 + [(4, 4)] * 2),
    ("float64", 300, [(6, 6)] * 3 + [(5, 5)] * 2 + [(2, 2)]),
    ("float32", 1100, [(4, 4)] * 2 + [(2, 2)] * 3), ("float32", 1100, [(5, 5)] * 2 + [(2, 2)]), ("float64", 1100, [(5, 5)] * 2 + [(2, 2)]),
    # whole short rows in one launch (four super-stages)
    ("float32", 300, [(13, 13)] * 4), ("float32", 300, [(12, 12)] * 4), ("float32", 300, [(14, 14)] * 4),
    ("float32", 300, [(11, 11)] * 4), ("float32", 300, [(10, 10)] * 4), ("float32", 300, [(9, 9)] * 4),
    ("float64", 300, [(11, 11)] * 4), ("float64", 300, [(10, 10)] * 4), ("float64", 300, [(9, 9)] * 4),
    ("float32", 300, [(8, 8)] * 4), ("float32", 300, [(7, 7)] * 5), ("float32", 300, [(7, 7)] * 4),
    ("float32", 300, [(6, 6)] * 5), ("float32", 300, [(5, 5)] * 6), ("float32", 300, [(5, 5)] * 5),
    ("float32", 300, [(3, 3)] * 9), ("float32", 300, [(3, 3)] * 8), ("float32", 300, [(2, 2)] * 15),
    ("float32", 300, [(2, 2)] * 14), ("float32", 300, [(2, 2)] * 13), ("float64", 300, [(8, 8)] * 4),
    ("float64", 300, [(7, 7)] * 5), ("float64", 300, [(7, 7)] * 4), ("float64", 300, [(6, 6)] * 5),
    ("float64", 300, [(6, 6)] * 4), ("float64", 300, [(5, 5)] * 6), ("float64", 300, [(5, 5)] * 5),
    ("float64", 300, [(5, 5)] * 4), ("float64", 300, [(3, 3)] * 9), ("float64", 300, [(3, 3)] * 8),
    ("float64", 300, [(2, 2)] * 14), ("float64", 300, [(2, 2)] * 13),
    ("float32", 300, [(6, 6)] * 4), ("float32", 300, [(11, 11)] * 3), ("float32", 300, [(12, 12)] * 3),
    ("float32", 300, [(13, 13)] * 3), ("float32", 300, [(14, 14)] * 3), ("float32", 300, [(15, 15)] * 3),
    ("float64", 300, [(11, 11)] * 3), ("float64", 300, [(12, 12)] * 3), ("float64", 300, [(13, 13)] * 3),
    ("float64", 300, [(14, 14)] * 3), ("float64", 300, [(15, 15)] * 3),
    ("float32", 300, [(2, 4)] * 6), ("float32", 300, [(2, 4)] * 7), ("float32", 300, [(4, 2)] * 6), ("float32", 300, [(4, 2)] * 7),
    ("float32", 300, [(4, 8)] * 4), ("float32", 300, [(4, 8)] * 5), ("float32", 300, [(8, 4)] * 4), ("float32", 300, [(8, 4)] * 5),
    ("float64", 300, [(2, 4)]), ("float64", 300, [(4, 2)]), ("float64", 300, [(4, 8)] * 3), ("float64", 300, [(8, 4)] * 3),
    ("float64", 300, [(2, 4)] * 6), ("float64", 300, [(2, 4)] * 7), ("float64", 300, [(4, 2)] * 6), ("float64", 300, [(4, 2)] * 7),
    ("float64", 300, [(4, 8)] * 4), ("float64", 300, [(4, 8)] * 5), ("float64", 300, [(8, 4)] * 4),
]
FUSE_LIMITS = (16, 15, 14, 13, 12, 11, 10, 9, 8, 7, 6, 5, 4, 3, 2, 1)


def test_every_instance_is_reached_by_some_shape_of_the_list():
    """The list above reaches every compiled instance (planning only)."""
    n = km.get_option(km.KM_OPT_INSTANCE_COUNT)
    reached = set()
    for dtype, M, shapes in EVERY_INSTANCE:
        P, Q = [s[0] for s in shapes], [s[1] for s in shapes]
        for k in range(n):
            for fuse in FUSE_LIMITS:
                with options(instance=k + 1, max_fuse=fuse, kernels=15):
                    if any(st["variant"] == k for st in km.plan(M, P, Q, dtype)):
                        reached.add(k)
    assert reached == set(range(n))


@pytest.mark.parametrize("dtype,M,shapes", EVERY_INSTANCE, ids=lambda v: str(v).replace(" ", ""))
def test_every_compiled_instance_that_fits(dtype, M, shapes):
    """Each compiled kernel instance in turn is made the planner's first choice; wherever it fits the
    shape (the plan then names it) the result is checked, integer inputs bit for bit.  Every family's
    instances fit at least one of the shapes."""
    P, Q = [s[0] for s in shapes], [s[1] for s in shapes]
    X, Fs = kron_inputs.make_problem(M, shapes, dtype, seed=91)
    exact = 2.0 * np.prod(P, dtype=np.float64) < (2 ** 24 if dtype == "float32" else 2 ** 53)
    Xi, Fi = kron_inputs.make_problem(M, shapes, dtype, x="int2", f="int1", seed=92)
    used = set()
    for k in range(km.get_option(km.KM_OPT_INSTANCE_COUNT)):
        for fuse in FUSE_LIMITS:                         # the grouping must also ask for its number of factors
            with options(instance=k + 1, max_fuse=fuse, kernels=15):
                if k in used or not any(st["variant"] == k for st in km.plan(M, P, Q, dtype)):
                    continue
                used.add(k)
                assert_close(run_gpu(X, Fs), X, Fs)
                if exact:
                    assert_close(run_gpu(Xi, Fi, use_ws=True), Xi, Fi, exact=True)
    assert used


def test_config1_integer_and_float():
    """fp32, M=16, three 8x8 factors: the float variant and the {-2..2} bit-exact variant."""
    X, Fs = kron_inputs.make_config("c1_f32_m16_8x8x3", seed=1)
    assert_close(run_gpu(X, Fs), X, Fs)
    X, Fs = kron_inputs.make_config("c1_f32_m16_8x8x3", seed=1, x="int2", f="int2")
    assert_close(run_gpu(X, Fs), X, Fs, exact=True)
    assert np.array_equal(run_gpu(X, Fs), oracle.kron_bruteforce(X, Fs))


def test_identity_factors_return_x_bit_exact():
    X = kron_inputs.draw((6, 8 * 8 * 8 * 8), "float32", "uniform", 3, 0)
    Fs = [np.eye(8, dtype=np.float32)] * 4
    assert np.array_equal(run_gpu(X, Fs), X)


def test_empty_rows_and_library_workspace_reuse():
    Fs = [np.ones((8, 8), np.float32)] * 3
    Y = km.kronmatmul(torch.empty((0, 512), device="cuda"), [torch.from_numpy(F).cuda() for F in Fs])
    assert tuple(Y.shape) == (0, 512)
    # a small problem after a larger one reuses the cached workspace; a larger one regrows it
    for M in (2, 64, 3):
        X, Fs = kron_inputs.make_problem(M, [(8, 8)] * 4, "float32", seed=M)
        assert_close(run_gpu(X, Fs), X, Fs)


def test_prepared_call_repeats_without_marshalling():
    """A prepared call only crosses the C-ABI; repeated with new contents of X it gives what a fresh
    call gives, with and without a caller workspace."""
    shapes = [(8, 8)] * 4
    X, Fs = kron_inputs.make_problem(16, shapes, "float32", seed=41)
    Xd = torch.from_numpy(X).cuda()
    Fd = [torch.from_numpy(F).cuda() for F in Fs]
    ws = torch.empty(max(km.workspace_size(16, [8] * 4, [8] * 4, "float32"), 1), dtype=torch.uint8, device="cuda")
    for workspace in (None, ws):
        call = km.Prepared(Xd, Fd, workspace=workspace)
        for seed in (41, 42, 43):
            Xn, _ = kron_inputs.make_problem(16, shapes, "float32", seed=seed)
            Xd.copy_(torch.from_numpy(Xn).cuda())
            Y = call()
            torch.cuda.synchronize()
            assert_close(Y.cpu().numpy(), Xn, Fs)
            assert torch.equal(Y, km.kronmatmul(Xd, Fd))


@pytest.mark.parametrize("dtype,M,shapes", [
    ("float32", 16, [(8, 8)] * 3),
    ("float32", 7, [(3, 5), (4, 2), (6, 6), (2, 3)]),
    ("float32", 9, [(16, 32)] * 3),
    ("float64", 2, [(128, 128)] * 2),
    ("float32", 5, [(8, 8), (8, 8), (32, 32), (32, 32)]),
    ("float64", 3, [(33, 17), (2, 65)]),
], ids=lambda v: str(v).replace(" ", ""))
def test_transposed_factors(dtype, M, shapes):
    """Factors handed over transposed (Q x P arrays) give the result of the plain form; the oracle is
    fed the untransposed factors.  Library and caller workspace, and a prepared call."""
    X, Fs = kron_inputs.make_problem(M, shapes, dtype, seed=51)
    Xd = torch.from_numpy(X).cuda()
    Ft = [torch.from_numpy(np.ascontiguousarray(F.T)).cuda() for F in Fs]
    Y = km.kronmatmul(Xd, Ft, transposed=True)
    torch.cuda.synchronize()
    assert_close(Y.cpu().numpy(), X, Fs)
    P, Q = [s[0] for s in shapes], [s[1] for s in shapes]
    ws = torch.empty(max(km.workspace_size(M, P, Q, dtype, transposed=True), 1), dtype=torch.uint8, device="cuda")
    Y2 = km.kronmatmul(Xd, Ft, workspace=ws, transposed=True)
    Y3 = km.Prepared(Xd, Ft, workspace=ws, transposed=True)()
    torch.cuda.synchronize()
    assert torch.equal(Y, Y2) and torch.equal(Y, Y3)
    assert torch.equal(Y, km.kronmatmul(Xd, [torch.from_numpy(F).cuda() for F in Fs]))
    small = torch.empty(max(ws.numel() - 256, 1), dtype=torch.uint8, device="cuda")
    with pytest.raises(km.KronMatmulError):
        km.kronmatmul(Xd, Ft, workspace=small, transposed=True)


def test_transposed_form_is_the_gradient_of_the_plain_form():
    """d/dX of sum(Y * G) with Y = X (F1 (x) F2 (x) F3) is G (F1^T (x) F2^T (x) F3^T): handing the
    factors of the forward pass to the transposed entry point as they are gives that product (its
    shapes are then Q x P).  Checked against the oracle applied to the transposes."""
    shapes = [(4, 6), (8, 8), (5, 3)]
    _, Fs = kron_inputs.make_problem(1, shapes, "float64", seed=61)
    G = kron_inputs.draw((6, 6 * 8 * 3), "float64", "normal", 62, 0)
    Fd = [torch.from_numpy(F).cuda() for F in Fs]
    dX = km.kronmatmul(torch.from_numpy(G).cuda(), Fd, transposed=True)      # stored P x Q = transpose of Q x P
    torch.cuda.synchronize()
    assert dX.shape == (6, 4 * 8 * 5)
    assert_close(dX.cpu().numpy(), G, [np.ascontiguousarray(F.T) for F in Fs])


def test_profiled_call_reports_each_launch():
    X, Fs = kron_inputs.make_problem(8, [(8, 8)] * 4, "float32", seed=5)
    steps = km.plan(8, [8] * 4, [8] * 4, "float32")
    km.set_option(km.KM_OPT_PROFILE, 1)
    try:
        got = run_gpu(X, Fs)
        ms = km.last_profile()
    finally:
        km.set_option(km.KM_OPT_PROFILE, 0)
    assert len(ms) == len(steps) and all(t > 0 for t in ms)
    assert_close(got, X, Fs)


def test_caller_stream_is_used():
    X, Fs = kron_inputs.make_problem(32, [(8, 8)] * 4, "float32", seed=9)
    Xd = torch.from_numpy(X).cuda()
    Fd = [torch.from_numpy(F).cuda() for F in Fs]
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        Y = km.kronmatmul(Xd, Fd)
    side.synchronize()
    ref = oracle.kron_matmul(X, Fs)
    assert np.abs(Y.cpu().numpy() - ref).max() <= 1e-5 * np.abs(ref).max()


# ------------------------------------------------------------------ full-size workloads
# Checked on sampled rows (rows are independent, so the oracle computes exactly those rows) plus
# properties that hold at any size.

FULL = ["c2_f32_m1024_8x8x6", "c3_f32_m1024_32x32x4", "c4_f64_m16_128x128x3", "c5_f32_m256_16x32x4"]


def _sample_rows(M):
    rng = np.random.default_rng(M)
    rows = {0, 1, M // 2, M - 2, M - 1} | set(int(r) for r in rng.integers(0, M, 3))
    return sorted(rows)


@pytest.mark.parametrize("name", FULL)
def test_full_size_sampled_rows(name):
    X, Fs = kron_inputs.make_config(name, seed=2)
    Xd = torch.from_numpy(X).cuda()
    Fd = [torch.from_numpy(F).cuda() for F in Fs]
    Y = km.kronmatmul(Xd, Fd)
    torch.cuda.synchronize()
    rows = _sample_rows(X.shape[0])
    got = Y[rows].cpu().numpy()
    assert_close(got, X[rows], Fs)
    # second call into the same Y gives the same bits (no dependence on stale contents)
    Y2 = km.kronmatmul(Xd, Fd, Y=torch.full_like(Y, float("nan")))
    torch.cuda.synchronize()
    assert torch.equal(Y, Y2)
    del Y, Y2, Xd
    torch.cuda.empty_cache()


@pytest.mark.parametrize("name", FULL)
def test_full_size_every_element(name):
    """The measured workloads at full size, in the launch configuration the benchmark times (default
    plan, caller's workspace), every element of Y against the oracle, in slabs of rows."""
    X, Fs = kron_inputs.make_config(name, seed=3)
    M = X.shape[0]
    P, Q = [F.shape[0] for F in Fs], [F.shape[1] for F in Fs]
    Xd = torch.from_numpy(X).cuda()
    Fd = [torch.from_numpy(F).cuda() for F in Fs]
    ws = torch.empty(max(km.workspace_size(M, P, Q, X.dtype), 1), dtype=torch.uint8, device="cuda")
    Y = km.kronmatmul(Xd, Fd, workspace=ws)
    torch.cuda.synchronize()
    for r0 in range(0, M, 64):
        assert_close(Y[r0:r0 + 64].cpu().numpy(), X[r0:r0 + 64], Fs)
    del Y, Xd, ws
    torch.cuda.empty_cache()


@pytest.mark.parametrize("dtype,M,shapes", [
    ("float32", 64, [(8, 8)] * 6),          # small-factor kernel, 64 MiB intermediate
    ("float32", 64, [(64, 64)] * 3),        # fp32 MFMA launches that leave digits in place, 64 MiB
    ("float64", 4, [(128, 128)] * 3),       # fp64 MFMA instances, 64 MiB
    ("float32", 16, [(32, 32)] * 4),        # pair kernel, 64 MiB
    ("float32", 64, [(80, 80)] * 3),        # single-factor fp32 MFMA instances, 125 MiB
    ("float32", 32, [(100, 100)] * 3),      # run-time-shape MFMA kernel, 122 MiB
    ("float64", 128, [(40, 40)] * 3),       # the same, 62 MiB
    ("float32", 64, [(4, 4)] * 9),          # several small factors per LDS pass, 64 MiB
    ("float64", 48, [(3, 3)] * 11),         # the same on rows of odd length (element-sized stores), 65 MiB
], ids=lambda v: str(v).replace(" ", ""))
def test_intermediates_kept_in_cache_change_no_result(dtype, M, shapes):
    """Intermediates of 48 to 320 MiB are written with ordinary stores so that they stay in the
    last-level cache for the next launch, others (and every final result) with non-temporal ones: the
    two forms of each kernel give the same bits, and sampled rows match the oracle."""
    X, Fs = kron_inputs.make_problem(M, shapes, dtype, seed=77)
    Xd = torch.from_numpy(X).cuda()
    Fd = [torch.from_numpy(F).cuda() for F in Fs]
    assert km.get_option(km.KM_OPT_KEEP_MIB) == 320
    assert len(km.plan(M, [p for p, _ in shapes], [q for _, q in shapes], dtype)) > 1
    Y = km.kronmatmul(Xd, Fd)
    with options(keep_mib=0):
        Y0 = km.kronmatmul(Xd, Fd)
    with options(keep_mib=1 << 20):
        Y1 = km.kronmatmul(Xd, Fd)
    torch.cuda.synchronize()
    assert torch.equal(Y, Y0) and torch.equal(Y, Y1)
    rows = _sample_rows(M)[:4]
    assert_close(Y[rows].cpu().numpy(), X[rows], Fs)
    del Y, Y0, Y1, Xd
    torch.cuda.empty_cache()


@pytest.mark.parametrize("case", kron_inputs.TABLE4, ids=lambda c: "id%d_m%d_%s" % (c[0], c[1], "_".join(
    "%dx%d" % s for s in dict.fromkeys(c[2]))))
@pytest.mark.parametrize("dtype", ["float32", "float64"])
def test_table4_shapes_at_full_size(case, dtype):
    """Every problem size of the paper's Table 4 (odd M, M = 1, distinct and rectangular factors, N up
    to 11), with synthetic values, in both precisions: all rows where the oracle needs under about
    2e9 multiply-adds, sampled rows otherwise; then the integer variant bit for bit."""
    _, M, shapes = case
    X, Fs = kron_inputs.make_problem(M, shapes, dtype, seed=100 + case[0])
    width, macs = X.shape[1], 0
    for p, q in reversed(shapes):
        macs += width * q
        width = width // p * q
    rows = list(range(M)) if M * macs <= 2e9 else _sample_rows(M)
    Xd = torch.from_numpy(X).cuda()
    Y = km.kronmatmul(Xd, [torch.from_numpy(F).cuda() for F in Fs])
    torch.cuda.synchronize()
    assert_close(Y[rows].cpu().numpy(), X[rows], Fs)
    Xi, Fi = kron_inputs.make_problem(M, shapes, dtype, x="int2", f="int1", seed=200 + case[0])
    bound = 2.0 * np.prod([s[0] for s in shapes], dtype=np.float64)
    if bound < (2 ** 24 if dtype == "float32" else 2 ** 53):      # every partial sum exactly representable
        Yi = km.kronmatmul(torch.from_numpy(Xi).cuda(), [torch.from_numpy(F).cuda() for F in Fi])
        torch.cuda.synchronize()
        assert_close(Yi[rows].cpu().numpy(), Xi[rows], Fi, exact=True)
    del Y, Xd
    torch.cuda.empty_cache()


@pytest.mark.parametrize("name", FULL)
def test_full_size_integer_rows_bit_exact(name):
    X, Fs = kron_inputs.make_config(name, seed=4, x="int2", f="int1")
    Xd = torch.from_numpy(X).cuda()
    Y = km.kronmatmul(Xd, [torch.from_numpy(F).cuda() for F in Fs])
    torch.cuda.synchronize()
    rows = _sample_rows(X.shape[0])
    assert_close(Y[rows].cpu().numpy(), X[rows], Fs, exact=True)
    del Y, Xd
    torch.cuda.empty_cache()


@pytest.mark.parametrize("name", FULL)
def test_full_size_all_ones_factors_give_row_sums(name):
    """All-ones factors: every output of a row is that row's sum (exact for small-integer X)."""
    c = kron_inputs.CONFIGS[name]
    X, _ = kron_inputs.make_config(name, seed=6, x="int1")
    Fs = [np.ones(s, dtype=c["dtype"]) for s in c["shapes"]]
    Xd = torch.from_numpy(X).cuda()
    Y = km.kronmatmul(Xd, [torch.from_numpy(F).cuda() for F in Fs])
    torch.cuda.synchronize()
    sums = torch.from_numpy(X.sum(axis=1, dtype=np.float64).astype(c["dtype"])).cuda()
    assert bool((Y == sums[:, None]).all())
    del Y, Xd
    torch.cuda.empty_cache()


@pytest.mark.parametrize("name", ["c2_f32_m1024_8x8x6", "c3_f32_m1024_32x32x4", "c4_f64_m16_128x128x3"])
def test_full_size_permutation_factors_move_columns_bit_exact(name):
    """Permutation-matrix factors: Y is a known column permutation of X, bit for bit, for float X."""
    c = kron_inputs.CONFIGS[name]
    X, _ = kron_inputs.make_config(name, seed=8)
    rng = np.random.default_rng(8)
    sig, Fs = [], []
    for p, q in c["shapes"]:
        s = rng.permutation(p)
        F = np.zeros((p, q), dtype=c["dtype"])
        F[np.arange(p), s] = 1
        sig.append(s)
        Fs.append(F)
    Xd = torch.from_numpy(X).cuda()
    Y = km.kronmatmul(Xd, [torch.from_numpy(F).cuda() for F in Fs])
    torch.cuda.synchronize()
    # destination column of every source column: digits (p1..pN) -> (sigma1(p1)..sigmaN(pN))
    dest = np.zeros(1, dtype=np.int64)
    for s, (p, _) in zip(sig, c["shapes"]):
        dest = (dest[:, None] * p + s[None, :]).reshape(-1)
    want = torch.empty_like(Xd)
    want[:, torch.from_numpy(dest).cuda()] = Xd
    assert torch.equal(Y, want)
    del Y, Xd, want
    torch.cuda.empty_cache()


@pytest.mark.parametrize("kernels,variant", [(1, -1), (None, -8)])
def test_rows_beyond_32_bit_offsets_use_the_generic_kernel_and_stay_exact(kernels, variant):
    """Maximum sizes: one row of 8^10 floats (4 GiB) is past the 32-bit in-row offsets of the tiled
    kernels, so every factor takes the generic kernel with 64-bit indexing or, by default, the one with a
    slice per lane (variant -8).  Cyclic-shift factors
    (F[p][(p+1) % 8] = 1) make Y an exactly known column permutation of X, checked bit for bit on
    sampled columns: output digits (q_1..q_10) come from input digits ((q_i - 1) % 8)."""
    n, P = 10, 8
    old = km.get_option(km.KM_OPT_KERNELS)
    try:
        if kernels is not None:
            km.set_option(km.KM_OPT_KERNELS, kernels)
        _cyclic_shifts_of_one_row(n, P, variant)
    finally:
        km.set_option(km.KM_OPT_KERNELS, old)


def _cyclic_shifts_of_one_row(n, P, variant):
    steps = km.plan(1, [P] * n, [P] * n, "float32")
    assert all(st["variant"] == variant for st in steps)
    K = P ** n
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1234)
    Xd = torch.rand((1, K), dtype=torch.float32, device="cuda", generator=gen)
    F = np.zeros((P, P), dtype=np.float32)
    F[np.arange(P), (np.arange(P) + 1) % P] = 1
    Fd = [torch.from_numpy(F).cuda() for _ in range(n)]
    Y = km.kronmatmul(Xd, Fd)
    torch.cuda.synchronize()
    rng = np.random.default_rng(99)
    cols = np.unique(np.concatenate([rng.integers(0, K, 200000), [0, 1, K - 1, K - 2, K // 2, 2 ** 31 // 4, 2 ** 31 // 4 + 1]]))
    src = np.zeros_like(cols)
    rem = cols.copy()
    for i in range(n):                       # peel digits from the fastest
        q = rem % P
        rem //= P
        src += ((q - 1) % P) * P ** i
    got = Y[0, torch.from_numpy(cols).cuda()].cpu().numpy()
    want = Xd[0, torch.from_numpy(src).cuda()].cpu().numpy()
    assert np.array_equal(got, want)
    del Y, Xd
    torch.cuda.empty_cache()
    km.release()


def test_rows_beyond_32_bit_offsets_on_the_run_time_shape_mfma_kernel():
    """One row of 16^8 floats (16 GiB): the compiled 16x16 instances address inside a row with 32-bit
    offsets and are not planned, the run-time-shape MFMA kernel (64-bit indexing, slices counted
    through all rows) takes every factor.  Cyclic-shift factors make Y an exactly known column
    permutation of X, checked bit for bit on sampled columns, among them the ones around 2^31 and 2^32
    bytes."""
    n, P = 8, 16
    steps = km.plan(1, [P] * n, [P] * n, "float32")
    assert all(st["kernel"] == km.KM_KERNEL_MFMA_ANY for st in steps)
    K = P ** n
    gen = torch.Generator(device="cuda")
    gen.manual_seed(4321)
    Xd = torch.rand((1, K), dtype=torch.float32, device="cuda", generator=gen)
    F = np.zeros((P, P), dtype=np.float32)
    F[np.arange(P), (np.arange(P) + 1) % P] = 1
    Fd = [torch.from_numpy(F).cuda() for _ in range(n)]
    Y = km.kronmatmul(Xd, Fd)
    torch.cuda.synchronize()
    rng = np.random.default_rng(98)
    special = [0, 1, K - 1, K - 2, K // 2, 2 ** 31 // 4 - 1, 2 ** 31 // 4, 2 ** 32 // 4 - 1, 2 ** 32 // 4, 2 ** 32 // 4 + 1]
    cols = np.unique(np.concatenate([rng.integers(0, K, 200000), special])).astype(np.int64)
    src = np.zeros_like(cols)
    rem = cols.copy()
    for i in range(n):                       # peel digits from the fastest
        q = rem % P
        rem //= P
        src += ((q - 1) % P) * P ** i
    got = Y[0, torch.from_numpy(cols).cuda()].cpu().numpy()
    want = Xd[0, torch.from_numpy(src).cuda()].cpu().numpy()
    assert np.array_equal(got, want)
    del Y, Xd
    torch.cuda.empty_cache()
    km.release()


@pytest.mark.parametrize("dtype,M,shapes", [
    ("float32", 4099, [(4, 4)] * 4),          # ragged last tile
    ("float32", 2048, [(2, 2)] * 8),
    ("float64", 1500, [(6, 6)] * 3),
    ("float32", 3001, [(3, 3)] * 4),          # rows that are not 16-byte aligned
    ("float64", 1024, [(8, 8)] * 3),
    ("float32", 1025, [(5, 5)] * 2 + [(7, 7)] * 2),
    ("float32", 1030, [(12, 12)] * 2),
], ids=lambda v: str(v).replace(" ", ""))
def test_many_short_rows_share_a_tile(dtype, M, shapes):
    """Rows much shorter than a tile: several whole rows per tile (the T_M of section 4), the last
    tile ragged.  All rows are compared."""
    P, Q = [s[0] for s in shapes], [s[1] for s in shapes]
    with options(kernels=7):                             # the tiled families (not the whole-row kernel)
        assert any(st["tile_rows"] > 1 for st in km.plan(M, P, Q, dtype))
        X, Fs = kron_inputs.make_problem(M, shapes, dtype, seed=81)
        assert_close(run_gpu(X, Fs), X, Fs)
        Xi, Fi = kron_inputs.make_problem(M, shapes, dtype, x="int2", f="int1", seed=82)
        assert_close(run_gpu(Xi, Fi, use_ws=True), Xi, Fi, exact=True)


def test_more_rows_than_a_launch_has_workgroups():
    """Maximum sizes along M: 2^24 + 5 rows of 4 elements.  One row per workgroup would need more
    work-items than a launch may hold.  The planner puts many rows into each tile; restricted to the
    generic kernel it caps the grid and the kernel strides over its tiles.  Every row must be right
    either way, the last ones included."""
    M, shapes = (1 << 24) + 5, [(2, 2), (2, 2)]
    X, Fs = kron_inputs.make_problem(M, shapes, "float32", x="int2", f="int2", seed=71)
    want = oracle.kron_matmul(X, Fs)
    Xd = torch.from_numpy(X).cuda()
    Fd = [torch.from_numpy(F).cuda() for F in Fs]
    steps = km.plan(M, [2, 2], [2, 2], "float32")
    assert all(st["grid"] * st["block"] < 2 ** 32 for st in steps) and any(st["tile_rows"] > 1 for st in steps)
    Y = km.kronmatmul(Xd, Fd)
    torch.cuda.synchronize()
    assert np.array_equal(Y.cpu().numpy(), want)
    with options(kernels=1):
        steps = km.plan(M, [2, 2], [2, 2], "float32")
        assert all(st["kernel"] == km.KM_KERNEL_GENERIC and st["grid"] < M and st["grid"] * st["block"] < 2 ** 32
                   for st in steps)
        Y = km.kronmatmul(Xd, Fd)
        torch.cuda.synchronize()
    assert np.array_equal(Y.cpu().numpy(), want)
    del Y, Xd
    torch.cuda.empty_cache()
    km.release()


def test_graph_capture_and_replay_matches_eager():
    """Iterative callers (the small-M, many-calls pattern of the paper's Gaussian-process case study)
    can capture kronmatmul_ws in a HIP graph: it allocates nothing and synchronises nothing.  Replays
    are interleaved with eager work and each one is checked against the eager result."""
    X, Fs = kron_inputs.make_problem(16, [(8, 8)] * 5, "float32", seed=21)
    P = [8] * 5
    Xd = torch.from_numpy(X).cuda()
    Fd = [torch.from_numpy(F).cuda() for F in Fs]
    Yd = torch.empty_like(Xd)
    ws = torch.empty(max(km.workspace_size(16, P, P, "float32"), 1), dtype=torch.uint8, device="cuda")
    km.prepare(16, P, P, "float32")                      # sets kernel attributes, outside capture; launches nothing
    g = torch.cuda.CUDAGraph()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        with torch.cuda.graph(g, stream=side):
            km.kronmatmul(Xd, Fd, Y=Yd, workspace=ws)
    torch.cuda.current_stream().wait_stream(side)
    for rep in range(4):
        Xn, _ = kron_inputs.make_problem(16, [(8, 8)] * 5, "float32", seed=30 + rep)
        Xd.copy_(torch.from_numpy(Xn).cuda())
        Yd.fill_(float("nan"))
        g.replay()
        torch.cuda.synchronize()
        got = Yd.cpu().numpy()
        eager = km.kronmatmul(Xd, Fd, workspace=ws)
        torch.cuda.synchronize()
        assert np.array_equal(got, eager.cpu().numpy())
        assert_close(got, Xn, Fs)


TUNED = [
    ("float32", 16, [(8, 8)] * 4),
    ("float32", 64, [(8, 8)] * 5),
    ("float32", 8, [(32, 32)] * 3),
    ("float32", 8, [(16, 32)] * 3),
    ("float64", 2, [(128, 128)] * 2),
    ("float32", 6, [(4, 4)] * 7),
    ("float64", 4, [(8, 8)] * 4),
    ("float32", 5, [(3, 5), (7, 2), (8, 8), (8, 8)]),
    ("float32", 40, [(4, 4)] * 4 + [(2, 2)] * 4),        # runs of different small shapes: per-stage instances compete
    ("float64", 24, [(20, 20)] * 2 + [(40, 40)]),        # the run-time-shape MFMA kernel against the generic one
]


@pytest.mark.parametrize("dtype,M,shapes", TUNED, ids=lambda v: str(v).replace(" ", ""))
def test_tuned_plan_matches_the_oracle(dtype, M, shapes):
    """The autotuner times every instance that fits (each tile length and tile walk it may launch
    with) and installs the fastest plan: the result must still be the oracle's, the reported plan
    must be the installed one, and it must not be slower than the cost-model plan it was measured
    against."""
    P, Q = [s[0] for s in shapes], [s[1] for s in shapes]
    kept, model = km.tune(M, P, Q, dtype)
    assert 0 < kept <= model
    steps = km.plan(M, P, Q, dtype)
    assert sum(st["num_factors"] for st in steps) == len(shapes)
    X, Fs = kron_inputs.make_problem(M, shapes, dtype, seed=77)
    assert_close(run_gpu(X, Fs, use_ws=True), X, Fs)
    assert km.plan(M, P, Q, dtype) == steps              # a run does not replace the measured plan
    Xi, Fi = kron_inputs.make_problem(M, shapes, dtype, x="int2", f="int1", seed=78)
    assert_close(run_gpu(Xi, Fi), Xi, Fi, exact=True)
    km.release()                                          # forget the measured plans


# The cost model's plan against the autotuner's on the measured workloads and on the Table 4 sizes that
# are not launch-bound.  Exceptions (shape: reason) are listed in the design notes; none at present.
PLANNER_CHECK = ([(c["dtype"], c["M"], c["shapes"]) for c in kron_inputs.CONFIGS.values()]
                 + [("float32", t[1], t[2]) for t in kron_inputs.TABLE4 if t[0] in (17, 18, 19, 24, 25, 26, 27, 28)]
                 + [("float64", t[1], t[2]) for t in kron_inputs.TABLE4 if t[0] in (25, 28)]
                 + [("float32", 1024, [(p, p)] * n) for p, n in ((3, 11), (5, 8), (7, 6), (9, 5))]      # rows of odd length
                 + [("float32", 1024, [(48, 48)] * 3), ("float32", 256, [(80, 80)] * 3), ("float32", 256, [(112, 112)] * 3),
                    ("float64", 64, [(96, 96)] * 3), ("float32", 2048, [(160, 160)] * 2)]                                 # other multiples of 16
                 + [("float32", 1024, [(36, 36)] * 3), ("float32", 512, [(20, 20)] * 4)]                # padded to multiples of 16
                 + [("float32", 1024, [(4, 4)] * 5 + [(2, 2)] * 4), ("float32", 4096, [(8, 8)] * 2 + [(4, 4)] * 2)])   # mixed small shapes


@pytest.mark.parametrize("dtype,M,shapes", PLANNER_CHECK, ids=lambda v: str(v).replace(" ", "")[:40])
def test_cost_model_plan_is_close_to_the_tuned_plan(dtype, M, shapes):
    """The planner's rules were fitted to measurements; this holds them to the autotuner on the device
    at hand: the cost-model plan may be at most 10 % (and at least 2 us) slower than the plan the tuner
    keeps, both timed by the tuner as whole launch sequences in alternation."""
    P, Q = [s[0] for s in shapes], [s[1] for s in shapes]
    try:
        kept, model = km.tune(M, P, Q, dtype)
        assert model <= max(1.10 * kept, kept + 0.002), (kept, model, km.plan(M, P, Q, dtype))
    finally:
        km.release()
        torch.cuda.empty_cache()


def test_concurrent_callers_on_their_own_streams_and_workspaces():
    """Entry points are thread-safe with respect to each other: four host threads, each with its own
    stream, workspace and problem (profiling switched on, so that the shared event pool grows under
    them), call kronmatmul_ws repeatedly; every result must be the oracle's."""
    import threading
    problems = [("float32", 16, [(8, 8)] * 5), ("float64", 3, [(16, 16)] * 3),
                ("float32", 6, [(32, 32)] * 3), ("float32", 5, [(48, 80), (96, 48)])]
    data, errors = [], []
    for k, (dtype, M, shapes) in enumerate(problems):
        X, Fs = kron_inputs.make_problem(M, shapes, dtype, seed=300 + k)
        P, Q = [s[0] for s in shapes], [s[1] for s in shapes]
        Xd = torch.from_numpy(X).cuda()
        Fd = [torch.from_numpy(F).cuda() for F in Fs]
        ws = torch.empty(max(km.workspace_size(M, P, Q, dtype), 1), dtype=torch.uint8, device="cuda")
        Yd = torch.empty((M, int(np.prod(Q))), dtype=Xd.dtype, device="cuda")
        km.prepare(M, P, Q, dtype)
        data.append((X, Fs, Xd, Fd, ws, Yd, torch.cuda.Stream()))
    torch.cuda.synchronize()

    def worker(item):
        try:
            X, Fs, Xd, Fd, ws, Yd, stream = item
            call = km.Prepared(Xd, Fd, Y=Yd, workspace=ws)
            for _ in range(25):
                call(stream.cuda_stream)
            stream.synchronize()
        except Exception as exc:          # noqa: BLE001 - reported in the main thread
            errors.append(exc)

    km.set_option(km.KM_OPT_PROFILE, 1)
    try:
        threads = [threading.Thread(target=worker, args=(item,)) for item in data]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
    finally:
        km.set_option(km.KM_OPT_PROFILE, 0)
    torch.cuda.synchronize()
    assert not errors, errors
    for X, Fs, _Xd, _Fd, _ws, Yd, _stream in data:
        assert_close(Yd.cpu().numpy(), X, Fs)
    km.release()


def test_clock_probe_reports_both_clocks():
    """The probe sleeps for the asked time and reports how far the shader clock and the constant
    100 MHz clock advanced; next to a Kron-Matmul on another stream it neither disturbs the result
    nor fails to end."""
    ticks = torch.zeros(2, dtype=torch.int64, device="cuda")
    side = torch.cuda.Stream()
    X, Fs = kron_inputs.make_problem(64, [(8, 8)] * 4, "float32", seed=5)
    torch.cuda.synchronize()
    km.clock_probe(ticks, 300, side)
    Y = run_gpu(X, Fs)
    torch.cuda.synchronize()
    shader, wall = ticks.tolist()
    assert 300 * 100 <= wall < 3 * 300 * 100             # at least the asked time, and not much more
    assert 300.0 < 100.0 * shader / wall < 3000.0        # MHz
    assert_close(Y, X, Fs)


ROWS_CASES = [
    ("float32", 5, [(3, 5), (5, 3), (7, 2), (2, 7)]),
    ("float64", 5, [(3, 5), (5, 3), (7, 2), (2, 7)]),
    ("float32", 1, [(5, 5), (5, 5), (5, 5), (2, 2)]),                 # Table 4, id 20
    ("float64", 1, [(5, 5), (5, 5), (2, 2), (25, 25)]),               # Table 4, id 21
    ("float32", 10, [(52, 50), (65, 20)]),                            # Table 4, id 6
    ("float32", 7, [(2, 3)] * 8),                                     # eight factors, rows growing 256 -> 6561
    ("float64", 3, [(9, 1), (4, 6), (1, 5)]),                         # one-column and one-row factors
    ("float32", 70001, [(3, 2), (2, 3)]),                             # more rows than workgroups
    ("float32", 33, [(32, 32), (64, 3)]),                             # slices a multiple of 32 words apart
    ("float32", 4, [(1, 1), (6, 6), (6, 6)]),
]


@pytest.mark.parametrize("dtype,M,shapes", ROWS_CASES, ids=lambda v: str(v).replace(" ", ""))
def test_whole_row_kernel_matches_the_oracle(dtype, M, shapes):
    """Every factor in one launch with the row resident in LDS (any factor shapes): forced wherever
    the row fits, against the oracle, integer inputs bit for bit."""
    P, Q = [s[0] for s in shapes], [s[1] for s in shapes]
    with options(instance=km.get_option(km.KM_OPT_INSTANCE_COUNT) + 1):
        steps = km.plan(M, P, Q, dtype)
        assert len(steps) == 1 and steps[0]["kernel"] == km.KM_KERNEL_ROWS and steps[0]["num_factors"] == len(shapes)
        assert steps[0]["variant"] == -1, "the general form, not the one on the matrix cores"
        assert km.workspace_size(M, P, Q, dtype) == 0
        X, Fs = kron_inputs.make_problem(M, shapes, dtype, seed=41)
        assert_close(run_gpu(X, Fs), X, Fs)
        Xi, Fi = kron_inputs.make_problem(M, shapes, dtype, x="int2", f="int1", seed=42)
        assert_close(run_gpu(Xi, Fi, use_ws=True), Xi, Fi, exact=True)


def test_whole_row_kernel_is_planned_for_small_mixed_shapes_only():
    """Distinct small factors on a few rows take the one-launch kernel; rows that do not fit LDS,
    more than eight factors and work-heavy rows do not."""
    assert [st["kernel"] for st in km.plan(5, [3, 5, 7, 2], [5, 3, 2, 7], "float32")] == [km.KM_KERNEL_ROWS]
    assert [st["kernel"] for st in km.plan(1, [5, 5, 5, 2], [5, 5, 5, 2], "float32")] == [km.KM_KERNEL_ROWS]
    assert all(st["kernel"] != km.KM_KERNEL_ROWS for st in km.plan(16, [6] * 5, [6] * 5, "float32"))
    assert all(st["kernel"] != km.KM_KERNEL_ROWS for st in km.plan(4, [30, 31, 32], [30, 31, 32], "float32"))
    with options(instance=km.get_option(km.KM_OPT_INSTANCE_COUNT) + 1):
        assert all(st["kernel"] != km.KM_KERNEL_ROWS for st in km.plan(4, [30, 31, 32], [30, 31, 32], "float32"))
        assert all(st["kernel"] != km.KM_KERNEL_ROWS for st in km.plan(4, [2] * 9, [2] * 9, "float32"))
