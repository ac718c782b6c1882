"""The run-time-shape MFMA kernel with the factor in registers (plan steps of that family with variant -3)."""
import numpy as np
import pytest

import kron_inputs

torch = pytest.importorskip("torch")          # before the library is loaded: both then use torch's HIP runtime
import paper_2401_10187_amd as km  # noqa: E402

PAD = -3


def _plan(dtype, M, shapes):
    return km.plan(M, [p for p, _ in shapes], [q for _, q in shapes], dtype)


# (dtype, rows, factors): contractions at the ends of the compiled classes (32, 64, 96, 128), slices that are whole
# 16-byte vectors and not, one to eight column blocks, rows shorter than a tile, of one slice and longer, ragged ends
CASES = [
    ("float32", 1300, [(20, 20)] * 3), ("float32", 30001, [(31, 17)]), ("float32", 3000, [(32, 8), (33, 33)]),
    ("float32", 1100, [(60, 64), (64, 63)]), ("float32", 9, [(65, 65)] * 2 + [(13, 13)]), ("float32", 1050, [(96, 80), (40, 96)]),
    ("float32", 1030, [(97, 97), (9, 13)]), ("float32", 6, [(127, 128), (128, 127), (2, 2)]), ("float32", 5, [(100, 100)] * 3),
    ("float32", 70001, [(20, 15)]), ("float32", 333, [(128, 113)]), ("float32", 1100, [(50, 33), (22, 28)]),
    ("float64", 1300, [(20, 20)] * 3), ("float64", 1111, [(31, 33), (32, 17), (16, 17)]), ("float64", 1025, [(33, 33)] * 2),
    ("float64", 1030, [(64, 48), (45, 63)]), ("float64", 40, [(96, 65), (66, 96)]), ("float64", 40, [(97, 100), (100, 113)]),
    ("float64", 4, [(128, 127), (127, 128), (3, 3)]), ("float64", 50001, [(14, 15)]), ("float64", 3, [(100, 100)] * 2 + [(7, 7)]),
]


def test_the_list_takes_the_kernel_and_its_launches_fit():
    """Grids are whole eighths (one part of the tiles per XCD), workgroups at most 1024 threads, LDS at most 96 KB."""
    for dtype, M, shapes in CASES:
        steps = [s for s in _plan(dtype, M, shapes) if s["variant"] == PAD]
        assert steps, (dtype, M, shapes)
        for s in steps:
            assert s["kernel"] == km.KM_KERNEL_MFMA_ANY and s["num_factors"] == 1
            assert s["grid"] % 8 == 0 and s["grid"] > 0 and s["block"] <= 1024 and s["lds_bytes"] <= 96 * 1024


@pytest.fixture
def options():
    """Sets planner options by name and puts the old values back."""
    old = {}

    def set_(**values):
        for name, value in values.items():
            key = getattr(km, "KM_OPT_" + name.upper())
            old.setdefault(key, km.get_option(key))
            km.set_option(key, value)
    yield set_
    for key, value in old.items():
        km.set_option(key, value)


def _forms(dtype, M, shapes):
    return [s["variant"] for s in _plan(dtype, M, shapes)]


def test_chunked_form_where_it_needs_fewer_rounds():
    """654 x 80x80^2 fp64 is three rounds of the register form's workgroups and one of the chunked form's; few tiles,
    slices that are no whole vectors and wavefronts that fill the SIMDs evenly stay with the register form."""
    assert _forms("float64", 654, [(80, 80)] * 2) == [-1, -1]
    assert _forms("float32", 1586, [(48, 48)] * 2) == [-1, -1]
    assert _forms("float64", 240, [(80, 80)] * 2) == [PAD, PAD]
    rng = np.random.default_rng(12)
    chunked = 0
    for _ in range(4000):
        dtype = "float32" if rng.random() < 0.5 else "float64"
        P, Q, M = int(rng.integers(17, 129)), int(rng.integers(8, 129)), int(10 ** rng.uniform(0, 5))
        for s in _plan(dtype, M, [(P, Q)] * 2):
            if s["kernel"] != km.KM_KERNEL_MFMA_ANY:
                continue
            slices, tall = M * s["k_in"] // P, Q <= 48 and P > 32      # (tall: its tile may be too long for the register form)
            if s["variant"] == -1 and not tall:
                chunked += 1
                assert P * (4 if dtype == "float32" else 8) % 16 == 0 and (Q + 15) // 16 not in (4, 7, 8) and slices > 256 * 16
    assert chunked > 20


def test_options_prefer_a_form_by_its_tile_or_workgroup(options):
    options(kernels=39)
    assert _forms("float64", 654, [(80, 80)] * 2) == [-1, -1]
    options(prefer_threads=320)                           # five column blocks, a wavefront each
    assert _forms("float64", 654, [(80, 80)] * 2) == [PAD, PAD]
    options(prefer_threads=256)
    assert _forms("float64", 10, [(80, 80)] * 2) == [-1, -1]
    options(prefer_threads=0, prefer_tile=128)
    assert _forms("float32", 10, [(50, 60)] * 2) == [-1, -1]
    options(prefer_tile=64)
    assert _forms("float32", 10, [(50, 60)] * 2) == [PAD, PAD]


# every compiled form of the chunked kernel: slices of half a chunk (narrow) and longer ones; whole 16-byte vectors,
# others of one chunk, others of several; one to five column blocks
CHUNKED = [("float32", P, Q) for P in (20, 13, 40, 50, 66) for Q in (16, 31, 40, 63, 78)] + \
          [("float64", P, Q) for P in (16, 13, 20, 25, 35) for Q in (15, 32, 40, 63, 78)] + \
          [("float32", 20, 200), ("float32", 13, 160), ("float32", 33, 200), ("float64", 13, 160), ("float64", 25, 200), ("float64", 144, 100)]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,P,Q", CHUNKED, ids=str)
def test_chunked_form_matches_the_reference(options, dtype, P, Q):
    """1407 slices in rows of 3: whole units and a ragged one.  Bars as below."""
    import oracle
    M, shapes = 469, [(3, 2), (P, Q)]
    narrow = P * (4 if dtype == "float32" else 8) <= 128
    options(kernels=39, max_fuse=1, prefer_tile=256 if narrow else 128, prefer_threads=256)
    first = _plan(dtype, M, shapes)[0]
    assert first["kernel"] == km.KM_KERNEL_MFMA_ANY and first["variant"] == -1 and first["tile_slices"] == (256 if narrow else 128)
    for kinds, exact in ((dict(x="uniform", f="normal"), False), (dict(x="int2", f="int1"), True)):
        X, Fs = kron_inputs.make_problem(M, shapes, dtype, seed=69, **kinds)
        print("chunked %s %dx%d" % (dtype, P, Q), flush=True)
        got = km.kronmatmul(torch.from_numpy(X).cuda(), [torch.from_numpy(F).cuda() for F in Fs]).cpu().numpy()
        ref = oracle.kron_matmul(X, Fs)
        if exact:
            assert np.array_equal(got, ref)
        else:
            assert np.abs(got - ref).max() <= (1e-5 if dtype == "float32" else 1e-12) * np.abs(ref).max()


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,M,shapes", CASES, ids=lambda v: str(v).replace(" ", ""))
def test_matches_the_reference(dtype, M, shapes):
    """Relative to the largest value 1e-5 in fp32 and 1e-12 in fp64 (a chain of dot products of lengths P_i is off by
    at most (sum P_i + N) u of the product of absolute values); bit for bit on small integers."""
    import oracle
    torch = pytest.importorskip("torch")
    tol = 1e-5 if dtype == "float32" else 1e-12
    exact_too = 2.0 * np.prod([p for p, _ in shapes], dtype=np.float64) < (2 ** 24 if dtype == "float32" else 2 ** 53)
    for kinds, exact in ((dict(x="uniform", f="normal"), False), (dict(x="int2", f="int1"), True)):
        if exact and not exact_too:
            continue
        X, Fs = kron_inputs.make_problem(M, shapes, dtype, seed=63, **kinds)
        print("mfma_pad %s M=%d %s" % (dtype, M, shapes), flush=True)
        Y = km.kronmatmul(torch.from_numpy(X).cuda(), [torch.from_numpy(F).cuda() for F in Fs])
        torch.cuda.synchronize()
        ref, got = oracle.kron_matmul(X, Fs), Y.cpu().numpy()
        if exact:
            assert np.array_equal(got, ref)
        else:
            assert np.abs(got - ref).max() <= tol * np.abs(ref).max()


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,P", [("float32", 21), ("float32", 50), ("float64", 33), ("float64", 97)])
def test_nothing_leaks_between_slices(dtype, P):
    """A contraction length that is no multiple of 4 reads past its slice: an infinity there must not turn a
    neighbour into NaN, and what the last, ragged tile holds past the end must not either."""
    torch = pytest.importorskip("torch")
    M = 1027
    X, Fs = kron_inputs.make_problem(M, [(P, P)], dtype, seed=64)
    assert _plan(dtype, M, [(P, P)])[0]["variant"] == PAD
    F = [torch.from_numpy(Fs[0]).cuda()]
    clean = km.kronmatmul(torch.from_numpy(X).cuda(), F)
    X[7, 0] = X[M - 1, P - 1] = np.inf
    got = km.kronmatmul(torch.from_numpy(X).cuda(), F)
    rest = [r for r in range(M) if r not in (7, M - 1)]
    assert torch.equal(got[rest], clean[rest])
    assert torch.isinf(got[7]).all() and torch.isinf(got[M - 1]).all()
