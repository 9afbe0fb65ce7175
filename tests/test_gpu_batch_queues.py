"""The batched form's three launches, each on lists that are sure to run it
(asserted from the plan's description): the plain launch of 256 threads (sizes
up to 2^12) and of 512 (up to 2^14), with full and partly filled tasks; the
persistent kernel with a work queue per XCD (full-width tiles, plain stores),
whose bits are also those of the shared queue.  Every transform has the bits of
the single plan; in place, repeated, and replayed from a graph the same."""
import re

import numpy as np
import pytest

import oracle
from paper_2609_06449_amd import inputs, paco

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu
TOL = 1e-6
NO_TUNE = paco.PACO_BATCH_NO_TUNE


def _stream() -> int:
    return torch.cuda.current_stream().cuda_stream


def _sizes(counts, seed):
    sizes = [1 << k for k, c in counts.items() for _ in range(c)]
    np.random.default_rng(seed).shuffle(sizes)
    return [int(n) for n in sizes]


def _input(total, seed):
    return torch.from_numpy(inputs.normal(total, seed=seed)).to("cuda")


def _single_calls(plan, x):
    """The transforms as a loop of single calls of the plans it reports."""
    y, ws, singles = torch.empty_like(x), torch.empty_like(x), {}
    for i, n in enumerate(plan.sizes):
        if n not in singles:
            singles[n] = paco.Plan(*plan.transform_plan(i))
        o = 8 * plan.offsets[i]
        singles[n].execute(x.data_ptr() + o, y.data_ptr() + o, ws.data_ptr() + o, _stream())
    torch.cuda.synchronize()
    return y


def _check(plan, seed):
    """Bits of single calls, one transform of each size against the oracle, in
    place, three launches more on dirty buffers, and graph replays."""
    x = _input(plan.total, seed)
    out, ws = torch.empty_like(x), torch.empty_like(x)
    plan.execute(x.data_ptr(), out.data_ptr(), ws.data_ptr(), _stream())
    torch.cuda.synchronize()
    y = out.clone()
    assert torch.equal(y, _single_calls(plan, x))
    for n in sorted(set(plan.sizes)):
        i = plan.sizes.index(n)
        a, b = plan.offsets[i], plan.offsets[i + 1]
        assert oracle.rel_l2(y[a:b].cpu().numpy(), oracle.dft(x[a:b].cpu().numpy().astype(np.complex128))) <= TOL, n
    for rep in range(3):
        out.fill_(float(rep + 1))
        ws.fill_(float(rep + 2))
        plan.execute(x.data_ptr(), out.data_ptr(), ws.data_ptr(), _stream())
        torch.cuda.synchronize()
        assert torch.equal(out, y), rep
    buf = x.clone()
    plan.execute(buf.data_ptr(), buf.data_ptr(), ws.data_ptr(), _stream())
    torch.cuda.synchronize()
    assert torch.equal(buf, y)
    g, s = torch.cuda.CUDAGraph(), torch.cuda.Stream()
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
        assert torch.equal(out, y), rep
        plan.execute(x.data_ptr(), out.data_ptr(), ws.data_ptr(), _stream())  # eager between the replays
        torch.cuda.synchronize()
        assert torch.equal(out, y), rep
    assert plan.errors() == 0
    return x, y


def _tasks(plan, threads):
    """Tasks of a plain launch of `threads`-thread workgroups (one each)."""
    m = re.search(r"(\d+) tasks, 1 task list \(one workgroup per task\), grid (\d+) x (\d+),", plan.description)
    assert m and int(m.group(1)) == int(m.group(2)) and int(m.group(3)) == threads, plan.description
    return int(m.group(1))


def _full_tasks(counts, threads):
    """Tasks when every one holds all it can: 16 items per thread, or one transform per thread below 2^4."""
    return sum(-(-c // (threads if k < 4 else max(1, 16 * threads >> k))) for k, c in counts.items())


# more items than the resident workgroups hold at once: tasks are as full as they get, the last of a size partly
@pytest.mark.parametrize("threads,counts", [
    (256, {2: 1027, 3: 515, 4: 1025, 5: 700, 6: 513, 7: 300, 8: 129, 9: 77, 10: 41, 11: 23, 12: 1100}),
    (512, {2: 513, 4: 700, 7: 129, 10: 33, 11: 17, 12: 501, 13: 301, 14: 37}),
])
def test_plain_launch_with_full_tasks(threads, counts):
    plan = paco.BatchPlan(_sizes(counts, 1), flags=NO_TUNE)
    assert _tasks(plan, threads) == _full_tasks(counts, threads) < len(plan.sizes)
    _check(plan, seed=51)


# fewer: tasks of a few transforms each
@pytest.mark.parametrize("threads,counts", [
    (256, {2: 5, 3: 1, 4: 3, 6: 40, 8: 9, 9: 2, 11: 1, 12: 2}),
    (256, {3: 1}), (256, {12: 3}), (256, {2: 2000}),
    (512, {2: 7, 5: 33, 9: 3, 13: 2}), (512, {14: 5}), (512, {4: 300, 14: 1}),
])
def test_plain_launch_with_partly_filled_tasks(threads, counts):
    plan = paco.BatchPlan(_sizes(counts, 2), flags=NO_TUNE)
    assert _tasks(plan, threads) >= _full_tasks(counts, threads)
    _check(plan, seed=52)


PER_XCD = {2: 9, 3: 17, 5: 65, 8: 33, 10: 9, 12: 7, 13: 17, 14: 9, 15: 8, 16: 9, 17: 8, 18: 9, 19: 8, 20: 8}


def test_queue_per_xcd_and_shared_queue():
    sizes = _sizes(PER_XCD, 3)
    plan = paco.BatchPlan(sizes, flags=NO_TUNE)
    assert "8 queues (one per XCD)" in plan.description, plan.description
    x, y = _check(plan, seed=53)
    shared = paco.BatchPlan(sizes, flags=NO_TUNE | paco.PACO_BATCH_ONE_QUEUE)
    assert "shared queue" in shared.description, shared.description
    out, ws = torch.empty_like(x), torch.empty_like(x)
    for _ in range(2):
        out.zero_()
        shared.execute(x.data_ptr(), out.data_ptr(), ws.data_ptr(), _stream())
        torch.cuda.synchronize()
        assert torch.equal(out, y)
    assert shared.errors() == 0


@pytest.mark.parametrize("gap", [0, 1, 10**6])
def test_queue_per_xcd_for_any_gap(gap):
    # 0: a job's successor right behind it, so that its tiles wait; 10^6: last of all
    sizes = _sizes({10: 9, 14: 3, 15: 17, 16: 16, 18: 8, 20: 8}, 4)
    plan = paco.BatchPlan(sizes, flags=NO_TUNE | paco.PACO_BATCH_SET_GAP, gap=gap)
    assert "one per XCD" in plan.description, plan.description
    x = _input(plan.total, 54)
    out, ws = torch.empty_like(x), torch.empty_like(x)
    for _ in range(2):
        plan.execute(x.data_ptr(), out.data_ptr(), ws.data_ptr(), _stream())
    torch.cuda.synchronize()
    assert torch.equal(out, _single_calls(plan, x))
    assert plan.errors() == 0


def test_queue_per_xcd_wait_limit_forced_from_the_host():
    """A poll limit of one: waits give up while their producers still run, the
    launch ends all the same, and another plan on the same buffers is right."""
    sizes = [1 << 20] * 8 + [1 << 16] * 16
    hasty = paco.BatchPlan(sizes, flags=NO_TUNE | paco.PACO_BATCH_SET_GAP, gap=0, spin_limit=1)
    patient = paco.BatchPlan(sizes, flags=NO_TUNE)
    assert "one per XCD" in hasty.description and "one per XCD" in patient.description
    x = _input(hasty.total, 55)
    out, ws = torch.empty_like(x), torch.empty_like(x)
    for _ in range(3):
        hasty.execute(x.data_ptr(), out.data_ptr(), ws.data_ptr(), _stream())
        torch.cuda.synchronize()              # the launch finished
        if hasty.errors():
            break
    assert hasty.errors() > 0
    patient.execute(x.data_ptr(), out.data_ptr(), ws.data_ptr(), _stream())
    torch.cuda.synchronize()
    assert torch.equal(out, _single_calls(patient, x))
    assert patient.errors() == 0
