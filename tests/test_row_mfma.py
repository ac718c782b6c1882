"""The whole-row kernel on the matrix cores (plan steps of the whole-row family with variant -2): every factor of
a short row in one launch, for problems of few rows."""
import numpy as np
import pytest

import kron_inputs
import paper_2401_10187_amd as km

ROW_MFMA = -2


def _plan(dtype, M, shapes):
    return km.plan(M, [p for p, _ in shapes], [q for _, q in shapes], dtype)


def test_planned_only_where_its_limits_hold():
    """Up to 1024 rows and eight factors, both row buffers (slices of a multiple of 8 elements padded by 4)
    within 60 KB; a single launch without workspace."""
    rng = np.random.default_rng(11)
    seen = 0
    for _ in range(6000):
        dtype = "float32" if rng.random() < 0.5 else "float64"
        shapes = [(int(rng.integers(1, 140)), int(rng.integers(1, 140))) for _ in range(int(rng.integers(1, 5)))]
        M = int(rng.integers(1, 3000))
        if np.prod([p for p, _ in shapes]) > 1 << 20:
            continue
        steps = _plan(dtype, M, shapes)
        if steps[0]["variant"] != ROW_MFMA:
            assert all(s["variant"] != ROW_MFMA for s in steps)
            continue
        seen += 1
        es = 4 if dtype == "float32" else 8
        w = k_in = int(np.prod([p for p, _ in shapes]))
        need = 0
        for p, q in reversed(shapes):
            need = max(need, w // p * (p + (4 if p % 8 == 0 else 0)))
            w = w // p * q
        st = steps[0]
        assert len(steps) == 1 and st["num_factors"] == len(shapes) and st["kernel"] == km.KM_KERNEL_ROWS
        assert st["k_in"] == k_in and st["k_out"] == w and st["grid"] == M <= 1024 and st["block"] in (256, 1024)
        assert 2 * max(need, w) * es <= st["lds_bytes"] <= 60 * 1024
        assert km.workspace_size(M, [p for p, _ in shapes], [q for _, q in shapes], dtype) == 0
    assert seen > 100


@pytest.mark.parametrize("dtype,M,shapes", [("float32", 257, [(16, 16)] * 2), ("float32", 487, [(16, 16)] * 2), ("float32", 1024, [(16, 16)] * 2),
                                            ("float64", 793, [(16, 16)] * 2), ("float64", 1000, [(16, 16)] * 2), ("float64", 257, [(2, 2)] * 2),
                                            ("float64", 512, [(2, 2)] * 2), ("float64", 400, [(4, 4)] * 3), ("float64", 300, [(2, 4)] * 3),
                                            ("float64", 300, [(4, 2)] * 3),
                                            # tiled launches would need more than the static array, or have up to 256 rows
                                            ("float64", 793, [(37, 5), (76, 81)]), ("float64", 850, [(37, 5), (76, 81)]),
                                            ("float32", 6, [(52, 122), (6, 3), (2, 18)]), ("float32", 2, [(85, 124), (5, 54)])], ids=str)
def test_tiled_launches_are_weighed_against_the_whole_row_plan_that_they_stand_in_for(dtype, M, shapes):
    """The general whole-row kernel loses to tiled launches here, or generic launches are cheap; the one on the matrix cores
    is the plan all the same: one launch, no workspace."""
    assert [s["variant"] for s in _plan(dtype, M, shapes)] == [ROW_MFMA]
    assert km.workspace_size(M, [p for p, _ in shapes], [q for _, q in shapes], dtype) == 0


def test_the_general_form_can_be_asked_for():
    """The option that takes the whole-row kernel wherever it fits means the general form, also where the planner
    would take this one."""
    old = km.get_option(km.KM_OPT_PREFER_INSTANCE)
    for dtype, M, shapes in (("float32", 10, [(52, 50), (65, 20)]), ("float64", 3, [(9, 1), (4, 6), (1, 5)]),
                             ("float32", 33, [(32, 32), (64, 3)]), ("float32", 4, [(1, 1), (6, 6), (6, 6)])):
        assert _plan(dtype, M, shapes)[0]["variant"] == ROW_MFMA
        km.set_option(km.KM_OPT_PREFER_INSTANCE, km.get_option(km.KM_OPT_INSTANCE_COUNT) + 1)
        try:
            (st,) = _plan(dtype, M, shapes)
            assert st["kernel"] == km.KM_KERNEL_ROWS and st["variant"] == -1
        finally:
            km.set_option(km.KM_OPT_PREFER_INSTANCE, old)


def test_taken_where_it_is_the_faster_one():
    """On either side of the line, as measured: against the FMA form 5.0 us here and 19.9 there (300 x (32x32, 64x3)),
    10.4 and 8.5 (37 x (9x4, 15x14, 4x44)); against tiled launches 7.6 and 9.3 (200 x 50x50^2), 21.3 and 14.1
    (265 x (104x100, 52x40)), 11.0 and 9.1 (5 x 61x61^2 fp64)."""
    for dtype, M, shapes, taken in (("float32", 300, [(32, 32), (64, 3)], True), ("float32", 37, [(9, 4), (15, 14), (4, 44)], False),
                                    ("float32", 200, [(50, 50)] * 2, True), ("float32", 265, [(104, 100), (52, 40)], False),
                                    ("float64", 5, [(61, 61)] * 2, False)):
        assert (_plan(dtype, M, shapes)[0]["variant"] == ROW_MFMA) == taken, (dtype, M, shapes)


CASES = [
    ("float32", 10, [(52, 50), (65, 20)]), ("float64", 10, [(52, 50), (65, 20)]),
    ("float32", 3, [(80, 80), (80, 80)]), ("float64", 2, [(40, 33), (79, 48)]),      # contractions of one round of the operand registers
    ("float32", 5, [(81, 33), (65, 20)]), ("float64", 3, [(7, 9), (161, 20)]), ("float32", 20, [(3, 5), (200, 100)]),   # two, three
    ("float32", 4, [(128, 16), (9, 40)]), ("float64", 37, [(8, 25), (91, 8)]),
    ("float32", 5, [(16, 16), (17, 17)]), ("float64", 5, [(15, 16), (18, 31)]),      # around one chunk of 16
    ("float32", 300, [(32, 32), (64, 3)]), ("float32", 1, [(33, 70), (21, 1)]),      # few columns, one column
    ("float32", 77, [(14, 40), (77, 39)]), ("float64", 90, [(30, 30), (30, 30)]),
    ("float32", 1024, [(36, 36), (36, 36)]), ("float32", 1000, [(50, 50), (50, 50)]),   # the most rows
    ("float32", 25, [(20, 26), (10, 16), (12, 4)]), ("float64", 50, [(17, 17), (17, 17), (9, 9)]),
    ("float32", 7, [(1, 19), (37, 1), (41, 23)]),                                    # P = 1, rows of odd length
]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,M,shapes", CASES, ids=lambda v: str(v).replace(" ", ""))
def test_matches_the_reference(dtype, M, shapes):
    """Against the CPU reference: relative to the largest value 1e-5 in fp32 and 1e-12 in fp64 (a chain of dot
    products of lengths P_i is off by at most (sum P_i + N) u of the product of absolute values), and bit for
    bit where every partial sum is a small integer."""
    import oracle
    torch = pytest.importorskip("torch")
    assert _plan(dtype, M, shapes)[0]["variant"] == ROW_MFMA
    tol = 1e-5 if dtype == "float32" else 1e-12
    for kinds, exact in ((dict(x="uniform", f="normal"), False), (dict(x="int2", f="int1"), True)):
        X, Fs = kron_inputs.make_problem(M, shapes, dtype, seed=61, **kinds)
        print("row_mfma %s M=%d %s" % (dtype, M, shapes), flush=True)
        Y = km.kronmatmul(torch.from_numpy(X).cuda(), [torch.from_numpy(F).cuda() for F in Fs])
        torch.cuda.synchronize()
        ref = oracle.kron_matmul(X, Fs)
        got = Y.cpu().numpy()
        if exact:
            assert np.array_equal(got, ref)
        else:
            assert np.abs(got - ref).max() <= tol * np.abs(ref).max()


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["float32", "float64"])
def test_nothing_leaks_between_slices_and_subnormals_stay(dtype):
    """Contraction lengths that are no multiple of 4 read past their slice: an infinity there must not turn a
    neighbour into NaN.  Identity factors return rows of subnormal numbers bit for bit."""
    torch = pytest.importorskip("torch")
    shapes = [(21, 21), (37, 37)]
    assert _plan(dtype, 6, shapes)[0]["variant"] == ROW_MFMA
    X, Fs = kron_inputs.make_problem(6, shapes, dtype, seed=62)
    bad = X.copy()
    bad[2, 5 * 37] = np.inf                                   # first element of slice 5 of row 2: right behind slice 4
    # the first factor applied mixes elements of one slice only; the identity keeps the others apart afterwards ...
    got = km.kronmatmul(torch.from_numpy(bad).cuda(), [torch.from_numpy(F).cuda() for F in (np.ones((21, 21), dtype), Fs[1])])
    rest = [r for r in range(6) if r != 2]
    clean = km.kronmatmul(torch.from_numpy(X).cuda(), [torch.from_numpy(F).cuda() for F in (np.ones((21, 21), dtype), Fs[1])])
    assert torch.equal(got[rest], clean[rest])
    assert torch.isinf(got[2]).all()                          # ... and inf * f + finite sums are infinities, never NaN
    tiny = (X * (2.0 ** -140 if dtype == "float32" else 2.0 ** -1060)).astype(dtype)
    assert 0 < np.abs(tiny[tiny != 0]).min() < np.finfo(dtype).tiny
    got = km.kronmatmul(torch.from_numpy(tiny).cuda(), [torch.from_numpy(np.eye(p, dtype=dtype)).cuda() for p, _ in shapes])
    assert np.array_equal(got.cpu().numpy(), tiny)
