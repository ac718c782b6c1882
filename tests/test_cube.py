"""Rows of 5^6, 5^8, 3^9 and 3^12 floats on tiles of three groups of digits (plan steps with variant -7)."""
import numpy as np
import pytest

import kron_inputs

torch = pytest.importorskip("torch")          # before the library is loaded: both then use torch's HIP runtime
import paper_2401_10187_amd as km  # noqa: E402

CUBE = -7
# (rows, P, N): one row, fewer tiles than workgroups, numbers of them that split by 8 and do not, walks of several with a
# remainder, one workgroup per compute unit
CASES = [(1, 5, 6), (511, 5, 6), (512, 5, 6), (1037, 5, 6), (2, 5, 8), (21, 5, 8), (165, 5, 8),
         (1, 3, 9), (515, 3, 9), (1030, 3, 9), (2, 3, 12), (20, 3, 12), (153, 3, 12)]


def _plan(M, shapes, dtype="float32"):
    return km.plan(M, [p for p, _ in shapes], [q for _, q in shapes], dtype)


def test_three_groups_are_one_launch_and_four_are_two():
    for M, P, N in CASES:
        steps = _plan(M, [(P, P)] * N)
        G = 2 if P == 5 else 3
        assert len(steps) == N // G - 2 and sum(s["num_factors"] for s in steps) == N
        for s in steps:
            tiles = M * (P ** N // P ** (3 * G))
            assert s["kernel"] == km.KM_KERNEL_FUSED and s["variant"] == CUBE and s["k_in"] == s["k_out"] == P ** N
            assert s["grid"] <= tiles <= s["grid"] * s["tiles_per_wg"] and (s["grid"] % 8 == 0 or s["grid"] == tiles)
        assert km.workspace_size(M, [P] * N, [P] * N, "float32") == (0 if len(steps) == 1 else (M * P ** N * 4 + 255) // 256 * 256)
    for M, shapes, dtype in ((9, [(5, 5)] * 7, "float32"), (9, [(5, 5)] * 6, "float64"), (9, [(5, 5)] * 5 + [(5, 3)], "float32"),
                             (9, [(5, 5)] * 5 + [(3, 3)], "float32"), (1, [(5, 5)] * 8, "float32"), (9, [(3, 3)] * 8, "float32")):
        assert all(s["variant"] != CUBE for s in _plan(M, shapes, dtype)), (M, shapes, dtype)


@pytest.mark.parametrize("option,value", [("MAX_FUSE", 4), ("KERNELS", 53), ("TILE_ORDER", 2), ("PREFER_TILE", 5), ("PREFER_THREADS", 256)])
def test_options_that_ask_for_other_kernels_get_them(option, value):
    key = getattr(km, "KM_OPT_" + option)
    old = km.get_option(key)
    km.set_option(key, value)
    try:
        assert all(s["variant"] != CUBE for s in _plan(64, [(5, 5)] * 8))
    finally:
        km.set_option(key, old)


@pytest.mark.gpu
@pytest.mark.parametrize("M,P,N", CASES, ids=str)
def test_matches_the_reference(M, P, N):
    """1e-5 of the largest value (sums of P terms per factor: at most (P + 1) N u of the product of absolute values), bit for bit
    on small integers; every factor another one; what is not finite stays in its row, and stores keep to Y."""
    import oracle
    for kinds, exact in ((dict(x="uniform", f="normal"), False), (dict(x="int2", f="int1"), True)):
        X, Fs = kron_inputs.make_problem(M, [(P, P)] * N, "float32", seed=85, **kinds)
        print("cube M=%d %d^%d" % (M, P, N), flush=True)
        Fd = [torch.from_numpy(F).cuda() for F in Fs]
        frame = torch.full((X.size + 2048,), -7.0, device="cuda")
        Y = frame[1024:1024 + X.size].view(X.shape)
        km.kronmatmul(torch.from_numpy(X).cuda(), Fd, Y=Y)
        assert (frame[:1024] == -7).all() and (frame[1024 + X.size:] == -7).all()
        got, rows = Y.cpu().numpy(), sorted({0, M // 2, M - 1, *range(0, M, max(1, M // 24))})
        ref = oracle.kron_matmul(X[rows], Fs)
        if exact:
            if 2.0 * P ** N < 2 ** 24:
                assert np.array_equal(got[rows], ref)
            continue
        assert np.abs(got[rows] - ref).max() <= 1e-5 * np.abs(ref).max()
        if M > 3:
            X[M - 1, -1], X[1, 7] = np.inf, np.nan
            bad = km.kronmatmul(torch.from_numpy(X).cuda(), Fd)
            rest = [r for r in range(M) if r not in (1, M - 1)]
            assert torch.equal(bad[rest], Y[rest]) and not torch.isfinite(bad[[1, M - 1]]).any()


@pytest.mark.gpu
@pytest.mark.parametrize("M,P,N", [(3, 5, 6), (3, 5, 8), (3, 3, 9), (2, 3, 12)], ids=str)
def test_factors_are_applied_last_to_first(M, P, N):
    """Scaling by powers of two changes no rounding as long as nothing overflows: of two neighbours the later one makes values small
    and the earlier one large again, so any other order of the two is infinite."""
    X, Fs = kron_inputs.make_problem(M, [(P, P)] * N, "float32", "uniform", "normal", seed=92)
    Xd, Fd = torch.from_numpy(X).cuda(), [torch.from_numpy(F).cuda() for F in Fs]
    assert {s["variant"] for s in _plan(M, [(P, P)] * N)} == {CUBE}
    want = km.kronmatmul(Xd, Fd) * 2.0 ** 60
    for i in range(N - 1):
        scaled = list(Fd)
        scaled[i], scaled[i + 1] = Fd[i] * 2.0 ** 80, Fd[i + 1] * 2.0 ** -80
        assert torch.equal(km.kronmatmul(Xd * 2.0 ** 60, scaled), want), i
