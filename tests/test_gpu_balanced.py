"""FP32 plans from 2^24 items on whose shape has no symmetric form run the
balanced shape's passes (and so does the inverse of every non-square shape):
the same bits as the balanced plan's, within the FP32 bound (1e-6 rel-L2) of
the FP64 oracle, with the shape's own stage hooks still there."""
import numpy as np
import pytest

import oracle
from paper_2609_06449_amd import inputs, paco

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu
TOL = 1e-6


def _call(fn, xd):
    out, ws = torch.empty_like(xd), torch.empty_like(xd)
    fn(xd.data_ptr(), out.data_ptr(), ws.data_ptr(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    return out


def _best(k):
    l1 = 13 if k == 28 else k // 2
    return 1 << l1, 1 << (k - l1)


def _dev(x):
    return torch.from_numpy(x).to("cuda")


@pytest.mark.parametrize("N1,N2,p,b,mixed", [(1024, 1 << 14, 16, 4, False), (1 << 14, 1024, 64, 16, True),
                                             (2048, 1 << 13, 8, 2, False), (1 << 8, 1 << 16, 16, 16, False),
                                             (2048, 1 << 14, 128, 16, True), (1 << 15, 1 << 10, 2, 8, True)])
def test_runs_the_balanced_passes(N1, N2, p, b, mixed):
    N, k = N1 * N2, (N1 * N2).bit_length() - 1
    x = inputs.normal(N, seed=k + N1)
    xd = _dev(x)
    plan = paco.Plan(N1, N2, p, b, mixed=mixed)
    best = paco.Plan(*_best(k), 2, 2)
    assert plan.launches == 3 and "executes sym[" in plan.description and best.has_split == 2
    y = _call(plan.execute, xd)
    assert torch.equal(y, _call(best.execute, xd))
    z = _call(plan.execute_inverse, xd)
    buf = xd.clone()
    ws = torch.empty_like(buf)
    plan.execute(buf.data_ptr(), buf.data_ptr(), ws.data_ptr(), torch.cuda.current_stream().cuda_stream)
    assert torch.equal(buf, y)
    if k == 24:
        assert oracle.rel_l2(y.cpu().numpy(), oracle.fft_radix2(x, threads=oracle.cpu_threads())) <= TOL
    back = _call(plan.execute_inverse, y)
    assert oracle.rel_l2(back.cpu().numpy(), x) <= 2 * TOL
    assert oracle.rel_l2(_call(plan.execute, z).cpu().numpy(), x) <= 2 * TOL


@pytest.mark.parametrize("N1,N2", [(1 << 13, 4096), (1 << 14, 4096), (4096, 1 << 15), (1 << 13, 1 << 14)])
def test_inverse_of_non_square_symmetric_shapes(N1, N2):
    k = (N1 * N2).bit_length() - 1
    plan = paco.Plan(N1, N2, 64, 2)
    best = paco.Plan(*_best(k), 2, 2)
    x = inputs.normal(N1 * N2, seed=k)
    y = _call(plan.execute, _dev(x))
    back = _call(plan.execute_inverse, y)
    assert torch.equal(back, _call(best.execute_inverse, y))
    assert oracle.rel_l2(back.cpu().numpy(), x) <= 2 * TOL


def test_2p28_square_and_wide_agree():
    x = torch.view_as_complex(torch.randn(1 << 28, 2, device="cuda", generator=torch.Generator("cuda").manual_seed(3)))
    square, wide = paco.Plan(1 << 14, 1 << 14, 256, 4), paco.Plan(1 << 13, 1 << 15, 128, 2)
    assert square.has_split == 2 and "executes sym[" in square.description and "executes" not in wide.description
    y = _call(square.execute, x)
    assert torch.equal(y, _call(wide.execute, x))
    back = _call(square.execute_inverse, y)
    assert torch.equal(back, _call(wide.execute_inverse, y))
    assert ((back - x).norm() / x.norm()).item() <= 2 * TOL
    del y, back, x
    torch.cuda.empty_cache()


def test_stage_hooks_and_options_keep_the_shape():
    plan = paco.Plan(1 << 14, 1024, 64, 4, mixed=True)
    assert plan.has_split == 1
    xd = _dev(inputs.normal(1 << 24, seed=5))
    t = torch.empty_like(xd)
    z = torch.empty_like(xd)
    s = torch.cuda.current_stream().cuda_stream
    plan.execute_stage(1, xd.data_ptr(), t.data_ptr(), s, paco.PACO_SPLIT)
    plan.execute_stage(2, t.data_ptr(), z.data_ptr(), s, paco.PACO_SPLIT)
    plan.execute_stage(3, z.data_ptr(), z.data_ptr(), s)
    y = _call(plan.execute, xd)
    assert oracle.rel_l2(z.cpu().numpy(), y.cpu().numpy().astype(np.complex128)) <= TOL
    for flags in (paco.PACO_PLAN_NO_SYM, paco.PACO_PLAN_NO_SPLIT):
        assert "executes" not in paco.Plan(1 << 14, 1024, 64, 4, mixed=True, flags=flags).description
    assert "executes" not in paco.Plan(1024, 1 << 14, 16, 4, paco.PACO_C64_MFMA_BF16X6).description
