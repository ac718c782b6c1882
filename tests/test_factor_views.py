"""Factors that start at odd elements of a larger tensor, and factors handed over transposed, on every kernel that
loads them with wide or buffer loads: the same bits as from factors of their own."""
import pytest

import kron_inputs

torch = pytest.importorskip("torch")
import paper_2401_10187_amd as km  # noqa: E402

# (dtype, rows, factors, family and variant of the first launch: None where it is a compiled instance)
CASES = [("float32", 10, [(52, 50), (65, 20)], (km.KM_KERNEL_ROWS, -2)), ("float64", 5, [(23, 31), (33, 9)], (km.KM_KERNEL_ROWS, -2)),
         ("float32", 1100, [(60, 64), (64, 63)], (km.KM_KERNEL_MFMA_ANY, -3)), ("float64", 1025, [(33, 33)] * 2, (km.KM_KERNEL_MFMA_ANY, -3)),
         ("float32", 700, [(144, 100)], (km.KM_KERNEL_MFMA_ANY, -1)), ("float64", 654, [(80, 80)] * 2, (km.KM_KERNEL_MFMA_ANY, -1)),
         ("float32", 300, [(64, 64)] * 2, None), ("float32", 250, [(32, 32)] * 3, None), ("float64", 300, [(16, 16)] * 3, None)]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,M,shapes,kernel", CASES, ids=lambda v: str(v).replace(" ", ""))
def test_views_and_transposed_factors_give_the_same_bits(dtype, M, shapes, kernel):
    first = km.plan(M, [p for p, _ in shapes], [q for _, q in shapes], dtype)[0]
    if kernel is None:
        assert first["kernel"] == km.KM_KERNEL_MFMA and first["num_factors"] == len(shapes)
    else:
        assert (first["kernel"], first["variant"]) == kernel
    X, Fs = kron_inputs.make_problem(M, shapes, dtype, seed=71)
    Xd, Fd = torch.from_numpy(X).cuda(), [torch.from_numpy(F).cuda() for F in Fs]
    print("factor views %s M=%d %s" % (dtype, M, shapes), flush=True)
    want = km.kronmatmul(Xd, Fd)
    views = []
    for F in Fd:
        base = torch.full((F.numel() + 3,), float("nan"), dtype=F.dtype, device="cuda")
        views.append(base[1:1 + F.numel()].view(F.shape))
        views[-1].copy_(F)
        assert views[-1].data_ptr() % 16 == F.element_size()
    assert torch.equal(km.kronmatmul(Xd, views), want)
    assert torch.equal(km.kronmatmul(Xd, [F.t().contiguous() for F in Fd], transposed=True), want)
