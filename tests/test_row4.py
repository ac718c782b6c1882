"""Whole rows of 4^7 floats, 4x4 factors or two 2x2 ones in the place of each, in one launch (plan step variant -6)."""
import numpy as np
import pytest

import kron_inputs

torch = pytest.importorskip("torch")          # before the library is loaded: both then use torch's HIP runtime
import paper_2401_10187_amd as km  # noqa: E402

ROW4 = -6
FOUR, TWO = (4, 4), (2, 2)
# (rows, factors): 4x4 and 2x2 at every digit, one row, fewer rows than workgroups, one more, walks of several
CASES = [(1, [FOUR] * 7), (511, [FOUR] * 7), (513, [FOUR] * 7), (1, [TWO] * 14), (514, [TWO] * 14), (1100, [FOUR] * 5 + [TWO] * 4),
         (3, [FOUR] * 6 + [TWO] * 2), (5, [FOUR] * 3 + [TWO] * 8), (2, [FOUR] + [TWO] * 12)]


def _plan(M, shapes, dtype="float32"):
    return km.plan(M, [p for p, _ in shapes], [q for _, q in shapes], dtype)


def test_one_launch_for_rows_of_seven_two_bit_digits():
    for M, shapes in CASES:
        (st,) = _plan(M, shapes)
        assert st["kernel"] == km.KM_KERNEL_FUSED and st["variant"] == ROW4 and st["num_factors"] == len(shapes)
        assert st["grid"] == min(M, 512) and M <= st["grid"] * st["tiles_per_wg"]
        assert km.workspace_size(M, [p for p, _ in shapes], [q for _, q in shapes], "float32") == 0
    # 2x2 factors before 4x4 ones, one that straddles digits, other lengths, other types, other shapes
    for M, shapes, dtype in ((9, [TWO, FOUR, TWO] + [FOUR] * 5, "float32"), (9, [TWO] * 2 + [FOUR] * 6, "float32"), (9, [FOUR] * 6, "float32"), (9, [FOUR] * 7, "float64"),
                             (9, [FOUR] * 6 + [(4, 2)], "float32"), (9, [FOUR] * 5 + [(16, 16)], "float32")):
        assert all(s["variant"] != ROW4 for s in _plan(M, shapes, dtype)), (M, shapes, dtype)


@pytest.mark.parametrize("option,value", [("MAX_FUSE", 6), ("KERNELS", 53), ("TILE_ORDER", 2), ("PREFER_TILE", 1), ("PREFER_INSTANCE", 1)])
def test_options_that_ask_for_other_kernels_get_them(option, value):
    key = getattr(km, "KM_OPT_" + option)
    old = km.get_option(key)
    km.set_option(key, value)
    try:
        assert all(s["variant"] != ROW4 for s in _plan(64, [FOUR] * 7))
    finally:
        km.set_option(key, old)


@pytest.mark.gpu
@pytest.mark.parametrize("M,shapes", CASES, ids=lambda v: str(v).replace(" ", ""))
def test_matches_the_reference(M, shapes):
    """1e-5 of the largest value (sums of P terms per factor: at most (P + 1) N u of the product of absolute values), bit for
    bit on small integers; every factor another one, so that a digit given the wrong one shows."""
    import oracle
    for kinds, exact in ((dict(x="uniform", f="normal"), False), (dict(x="int2", f="int1"), True)):
        X, Fs = kron_inputs.make_problem(M, shapes, "float32", seed=84, **kinds)
        print("rows of 4^7, M=%d %s" % (M, shapes), flush=True)
        Xd, Fd = torch.from_numpy(X).cuda(), [torch.from_numpy(F).cuda() for F in Fs]
        Y = km.kronmatmul(Xd, Fd)
        ref, got = oracle.kron_matmul(X, Fs), Y.cpu().numpy()
        if exact:
            assert np.array_equal(got, ref)
            continue
        assert np.abs(got - ref).max() <= 1e-5 * np.abs(ref).max()
        assert torch.equal(km.kronmatmul(Xd, [F.t().contiguous() for F in Fd], transposed=True), Y)
        if M > 2:
            X[M - 1, 0], X[1, 16383] = np.inf, np.nan
            bad = km.kronmatmul(torch.from_numpy(X).cuda(), Fd)
            rest = [r for r in range(M) if r not in (1, M - 1)]
            assert torch.equal(bad[rest], Y[rest]) and not torch.isfinite(bad[[1, M - 1]]).any()


@pytest.mark.gpu
@pytest.mark.parametrize("shapes", [[FOUR] * 7, [TWO] * 14, [FOUR] * 3 + [TWO] * 8], ids=str)
def test_factors_are_applied_last_to_first(shapes):
    """Scaling by powers of two changes no rounding as long as nothing overflows: of two neighbours the later one makes values small
    and the earlier one large again, so any other order of the two is infinite."""
    X, Fs = kron_inputs.make_problem(3, shapes, "float32", "uniform", "normal", seed=91)
    Xd, Fd = torch.from_numpy(X).cuda(), [torch.from_numpy(F).cuda() for F in Fs]
    assert [s["variant"] for s in _plan(3, shapes)] == [ROW4]
    want = km.kronmatmul(Xd, Fd) * 2.0 ** 60
    for i in range(len(Fd) - 1):
        scaled = list(Fd)
        scaled[i], scaled[i + 1] = Fd[i] * 2.0 ** 80, Fd[i + 1] * 2.0 ** -80
        assert torch.equal(km.kronmatmul(Xd * 2.0 ** 60, scaled), want), i
