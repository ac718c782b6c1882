"""Problems whose faster plan is launches that share a workspace and whose other plan is one launch without any: calls that bring no
such workspace run the one launch."""
import ctypes

import pytest

import kron_inputs

torch = pytest.importorskip("torch")          # before the library is loaded: both then use torch's HIP runtime
import paper_2401_10187_amd as km  # noqa: E402

# (type, rows, factors): the one launch is the general whole-row kernel's, or that of the one on the matrix cores
CASES = [("float32", 9363, [(74, 14), (18, 5)]), ("float32", 1254, [(7, 2), (51, 23)]), ("float64", 957, [(17, 112), (10, 31), (5, 1)])]


def _ws_call(X, Fs, Y, ws, nbytes, transposed=False):
    """Status of the C entry point with the caller's workspace (address and size as given)."""
    n = len(Fs)
    shapes = [tuple(F.shape)[::-1] if transposed else tuple(F.shape) for F in Fs]
    p, q = ((ctypes.c_int * n)(*[s[i] for s in shapes]) for i in (0, 1))
    f = (ctypes.c_void_p * n)(*[F.data_ptr() for F in Fs])
    entry = km.lib().kronmatmul_transposed_ws if transposed else km.lib().kronmatmul_ws
    return entry(X.shape[0], n, p, q, X.data_ptr(), f, Y.data_ptr(), km.KM_F32 if X.dtype == torch.float32 else km.KM_F64, ws, nbytes,
                 torch.cuda.current_stream().cuda_stream)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,M,shapes", CASES, ids=str)
def test_calls_without_the_workspace_run_one_launch(dtype, M, shapes):
    """1e-5 (fp32), 1e-12 (fp64) of the largest value, as in the tests of either plan's kernels."""
    import oracle
    P, Q = [p for p, _ in shapes], [q for _, q in shapes]
    need = km.workspace_size(M, P, Q, dtype)
    launches = len(km.plan(M, P, Q, dtype))
    assert need > 0 and launches > 1
    X, Fs = kron_inputs.make_problem(M, shapes, dtype, "uniform", "normal", seed=88)
    ref = oracle.kron_matmul(X, Fs)
    Xd, Fd = torch.from_numpy(X).cuda(), [torch.from_numpy(F).cuda() for F in Fs]
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    Y = torch.empty(ref.shape, dtype=Xd.dtype, device="cuda")

    def right():
        return abs(Y.cpu().numpy() - ref).max() <= (1e-5 if dtype == "float32" else 1e-12) * abs(ref).max()

    km.set_option(km.KM_OPT_PROFILE, 1)
    try:
        for call, want in ((lambda: km.kronmatmul(Xd, Fd, Y=Y), 1), (lambda: km.Prepared(Xd, Fd, Y=Y)(), 1),
                           (lambda: km.kronmatmul(Xd, Fd, Y=Y, workspace=ws), launches),
                           (lambda: km.kronmatmul(Xd, Fd, Y=Y, workspace=ws[:need - 256]), 1),
                           (lambda: km.kronmatmul(Xd, [F.t().contiguous() for F in Fd], Y=Y, transposed=True), launches)):
            Y.zero_()
            call()
            assert right() and len(km.last_profile()) == want
        # what a plan without a workspace never looked at: none, one that overlaps X, one on no boundary
        for at, size in ((None, 0), (Xd.data_ptr(), need), (ws.data_ptr() + 1, need)):
            Y.zero_()
            assert _ws_call(Xd, Fd, Y, at, size) == km.KM_OK
            assert right() and len(km.last_profile()) == 1
    finally:
        km.set_option(km.KM_OPT_PROFILE, 0)
    Y.zero_()
    km.kronmatmul(Xd, Fd, Y=Y, static=True)
    assert right()
    copies = sum((p * q * Xd.element_size() + 255) // 256 * 256 for p, q in shapes)
    Ft, small = [F.t().contiguous() for F in Fd], torch.empty(copies, dtype=torch.uint8, device="cuda")
    Y.zero_()
    assert _ws_call(Xd, Ft, Y, small.data_ptr(), copies, transposed=True) == km.KM_OK
    assert right()


@pytest.mark.gpu
def test_two_streams_side_by_side():
    """Plain calls of such a problem on two streams at once share nothing."""
    dtype, M, shapes = CASES[0]
    probs = [kron_inputs.make_problem(M, shapes, dtype, "int2", "int1", seed=s) for s in (89, 90)]
    dev = [(torch.from_numpy(X).cuda(), [torch.from_numpy(F).cuda() for F in Fs]) for X, Fs in probs]
    want = [km.kronmatmul(X, Fs) for X, Fs in dev]
    side = [torch.cuda.Stream() for _ in dev]
    torch.cuda.synchronize()
    for _ in range(20):
        got = []
        for s, (X, Fs) in zip(side, dev):
            with torch.cuda.stream(s):
                got.append(km.kronmatmul(X, Fs))
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(got, want))
