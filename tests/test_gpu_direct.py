"""The direct form (FP32, N <= 2^23: one workgroup up to 2^14 items, two column
passes above) on the GPU: every length of its range against the FP64 oracle,
forward and inverse, in place, the same bits for every shape, base and slab
count of a length, the batched kernel's same bits (partly filled tasks, both
queue modes), and replays of a captured graph.  Tolerance: 1e-6 rel-L2, the
FP32 bound of every transform of the library."""
import numpy as np
import pytest

import oracle
from paper_2609_06449_amd import inputs, paco

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu
TOL = 1e-6


def _stream() -> int:
    return torch.cuda.current_stream().cuda_stream


def _dev(x):
    return torch.from_numpy(np.ascontiguousarray(x.astype(np.complex64).ravel())).to("cuda")


def _call(fn, xd, out=None):
    out = torch.empty_like(xd) if out is None else out
    ws = torch.empty_like(xd)
    fn(xd.data_ptr(), out.data_ptr(), ws.data_ptr(), _stream())
    torch.cuda.synchronize()
    return out.cpu().numpy()


def _bits(y):
    return y.view(np.uint64)


def _balanced(k):
    l1 = (k + 1) // 2
    return 1 << l1, 1 << (k - l1)


@pytest.mark.parametrize("k", range(2, 24))
def test_every_length_forward_inverse_in_place(k):
    N1, N2 = _balanced(k)
    plan = paco.Plan(N1, N2, 2, 2)
    assert plan.launches == (1 if k <= 14 else 2) and " direct[" in plan.description, plan.description
    x = inputs.loguniform(N1 * N2, seed=100 + k)
    xd = _dev(x)
    y = _call(plan.execute, xd)
    assert oracle.rel_l2(y, oracle.dft(x.astype(np.complex128))) <= TOL
    z = _call(plan.execute_inverse, xd)
    assert oracle.rel_l2(z, oracle.idft(x)) <= TOL
    buf = xd.clone()
    assert np.array_equal(_bits(_call(plan.execute, buf, out=buf)), _bits(y))
    buf = xd.clone()
    assert np.array_equal(_bits(_call(plan.execute_inverse, buf, out=buf)), _bits(z))


@pytest.mark.parametrize("k,shapes", [
    (6, [(2, 32, 2, 2, False), (32, 2, 2, 2, False), (16, 4, 2, 8, True), (8, 8, 8, 8, False)]),
    (13, [(2, 4096, 2, 2, False), (2048, 4, 4, 2, False), (128, 64, 4, 16, True)]),
    (14, [(16, 1024, 2, 4, False), (128, 128, 16, 16, True)]),
    (17, [(2, 1 << 16, 2, 2, False), (512, 256, 4, 2, False), (64, 2048, 4, 16, True)]),
    (22, [(64, 1 << 16, 16, 4, False), (2048, 2048, 64, 2, False), (4096, 1024, 16, 4, False)]),
    (23, [(4096, 2048, 16, 16, True), (1 << 13, 1024, 16, 2, False)]),
])
def test_same_bits_for_every_shape_base_and_slab_count(k, shapes):
    x = _dev(inputs.normal(1 << k, seed=200 + k))
    ref = _call(paco.Plan(*_balanced(k), 2, 2).execute, x)
    for N1, N2, p, b, mixed in shapes:
        plan = paco.Plan(N1, N2, p, b, mixed=mixed)
        assert " direct[" in plan.description, plan.description
        assert np.array_equal(_bits(_call(plan.execute, x)), _bits(ref)), (N1, N2, p, b)


def test_options_and_split_shapes_keep_their_plans():
    for flags in (paco.PACO_PLAN_PAPER_LAYOUT, paco.PACO_PLAN_GENERIC, paco.PACO_PLAN_NO_SPLIT, paco.PACO_PLAN_NO_SYM):
        assert " direct[" not in paco.Plan(64, 64, 4, 4, flags=flags).description
    assert " direct[" not in paco.Plan(64, 64, 4, 4, groups1=1).description
    assert " direct[" not in paco.Plan(4096, 64, 4, 4).description
    assert " direct[" not in paco.Plan(64, 64, 4, 4, paco.PACO_C64_MFMA_FP16X3).description
    assert " direct[" not in paco.Plan(4096, 4096, 4, 2).description


@pytest.mark.parametrize("queue", [0, paco.PACO_BATCH_ONE_QUEUE])
def test_batched_bits_equal_single_bits_for_every_length(queue):
    # several transforms of every length, in an order that mixes them: tasks
    # of short transforms are partly filled and their members lie apart
    sizes = [1 << k for k in range(2, 21)] + [1 << k for k in range(13, 1, -1)] + [4] * 3 + [64] * 5 + [1 << 14]
    plan = paco.BatchPlan(sizes, flags=paco.PACO_BATCH_NO_TUNE | queue)
    x = _dev(inputs.batch_inputs(sizes, seed=31))
    y = _call(plan.execute, x)
    assert plan.errors() == 0
    single = {}
    for i, n in enumerate(sizes):
        a, c = plan.offsets[i], plan.offsets[i + 1]
        if n not in single:
            single[n] = paco.Plan(*_balanced(n.bit_length() - 1), 2, 2)
        assert np.array_equal(_bits(y[a:c]), _bits(_call(single[n].execute, x[a:c].clone()))), (i, n)


def test_batch_of_few_large_transforms_uses_every_xcd():
    # one large transform would run on one XCD with a queue per XCD
    assert "shared queue" in paco.BatchPlan([1 << 20], flags=paco.PACO_BATCH_NO_TUNE).description
    assert "one per XCD" in paco.BatchPlan([1 << 16] * 64, flags=paco.PACO_BATCH_NO_TUNE).description


def test_graph_replays_equal_eager():
    for k in (12, 14, 18):
        N1, N2 = _balanced(k)
        plan = paco.Plan(N1, N2, 2, 2)
        x = _dev(inputs.normal(1 << k, seed=300 + k))
        out, ws = torch.empty_like(x), torch.empty_like(x)
        eager = _call(plan.execute, x)
        g = torch.cuda.CUDAGraph()
        s = torch.cuda.Stream()
        s.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(s):
            with torch.cuda.graph(g, stream=s):
                plan.execute(x.data_ptr(), out.data_ptr(), ws.data_ptr(), s.cuda_stream)
        torch.cuda.current_stream().wait_stream(s)
        for rep in range(3):
            out.zero_()
            ws.fill_(float(rep + 1))
            torch.cuda.synchronize()
            g.replay()
            torch.cuda.synchronize()
            assert np.array_equal(_bits(out.cpu().numpy()), _bits(eager)), (k, rep)


def test_torch_calls_run_on_the_current_stream():
    from paper_2609_06449_amd import torch_api as ta
    streams = [torch.cuda.current_stream(), torch.cuda.Stream(), torch.cuda.Stream()]
    assert len({s.cuda_stream for s in streams}) == 3
    x = _dev(inputs.normal(1 << 13, seed=400))
    for s in streams:
        with torch.cuda.stream(s):
            assert ta._stream() == s.cuda_stream == torch.cuda.current_stream().cuda_stream
            # ordered behind the stream's own work: the copy is slow, the transform reads its result
            big = torch.zeros(1 << 26, dtype=torch.float32, device="cuda")
            y = x.clone()
            big.add_(1.0)
            y.mul_(big[0])
            out = ta.fft(y, 128, 64, 4, 2)
        torch.cuda.synchronize()
        assert oracle.rel_l2(out.cpu().numpy(), oracle.dft(x.cpu().numpy())) <= TOL


@pytest.mark.parametrize("dt,tol", [(paco.PACO_C64_MFMA_FP16X3, 1e-6), (paco.PACO_C64_MFMA_BF16X3, 3e-5),
                                    (paco.PACO_C64_MFMA_BF16X6, 1e-6)])
@pytest.mark.parametrize("N1,N2,p,b,mixed", [(128, 128, 4, 2, False), (128, 2048, 8, 2, False), (2048, 128, 4, 16, True),
                                             (512, 512, 16, 8, False), (1024, 256, 8, 4, False), (2048, 2048, 64, 4, True)])
def test_split_forms_in_two_passes(N1, N2, p, b, mixed, dt, tol):
    # the bounds of the split forms' other plans, on wide-range inputs
    x = inputs.loguniform(N1 * N2, seed=N1 + 3 * N2)
    plan = paco.Plan(N1, N2, p, b, dt, mixed=mixed)
    assert plan.launches == 2 and " direct[" in plan.description, plan.description
    xd = _dev(x)
    y = _call(plan.execute, xd)
    assert oracle.rel_l2(y, oracle.dft(x.astype(np.complex128))) <= tol
    assert oracle.rel_l2(_call(plan.execute_inverse, xd), oracle.idft(x)) <= tol
    buf = xd.clone()
    assert np.array_equal(_bits(_call(plan.execute, buf, out=buf)), _bits(y))


@pytest.mark.parametrize("N1,N2", [(64, 2048), (4096, 128), (128, 4096)])
def test_split_forms_outside_the_two_passes_sides(N1, N2):
    assert " direct[" not in paco.Plan(N1, N2, 4, 2, paco.PACO_C64_MFMA_BF16X6).description
