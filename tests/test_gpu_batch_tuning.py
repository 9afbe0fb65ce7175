"""The batched form's tuning: which files and lines are trusted, and that a
transform has the bits of the single plan with the (N1, N2, p, b) that the
batch plan reports for it, whatever the tuner picked."""
import re

import numpy as np
import pytest

import oracle
from paper_2609_06449_amd import inputs, paco

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu
NO_TUNE = paco.PACO_BATCH_NO_TUNE
TOL = 1e-6  # the FP32 bound of every transform of the library
MANY = [1 << 17] * 64  # a queue per XCD


def _key(path) -> str:
    keys = [ln for ln in open(path).read().splitlines() if ln.startswith("key ")]
    assert len(keys) == 1, keys
    return keys[0]


@pytest.fixture(scope="module")
def key(tmp_path_factory):
    """The key line of a file written on this device."""
    path = str(tmp_path_factory.mktemp("tune") / "fresh.txt")
    paco.BatchPlan([64], tune_cache_path=path).close()
    return _key(path)


def test_file_of_another_format_is_ignored_and_rewritten(tmp_path, key):
    # right device, the format of the three-phase kernel, and a split that is a
    # candidate of the present one too
    stale = re.sub(r"format=\d+", "format=1", key)
    assert stale != key
    path = str(tmp_path / "tune.txt")
    with open(path, "w") as f:
        f.write(stale + "\n17 8 9 1 0 1\n")
    plan = paco.BatchPlan(MANY, tune_cache_path=path, flags=NO_TUNE)
    assert plan.transform_plan(0)[:2] == (512, 256)  # the default, not the file's
    assert _key(path) == stale                       # without tuning the file stays
    paco.BatchPlan(MANY, tune_cache_path=path).close()
    assert _key(path) == key
    lines = [ln for ln in open(path).read().splitlines() if ln and not ln.startswith(("#", "key "))]
    assert [ln.split()[0] for ln in lines] == ["17"] and len(lines[0].split()) < 6, lines


def _lines(path):
    return sorted(ln.split() for ln in open(path).read().splitlines() if ln and not ln.startswith(("#", "key ")))


def test_lines_hold_for_the_queue_mode_they_were_timed_in(tmp_path, key):
    path = str(tmp_path / "tune.txt")
    few, many = [1 << 18], [1 << 18] * 64
    for lines, want_few, want_many in ((["18 10 8 1 0"], 512, 1024), (["18 10 8 1 1"], 1024, 512),
                                       (["18 10 8 1 1", "18 8 10 1 0"], 1024, 256)):
        with open(path, "w") as f:
            f.write("\n".join([key] + lines) + "\n")
        for sizes, flags, mode, want in ((few, 0, "shared queue", want_few), (many, 0, "one per XCD", want_many),
                                         (many, paco.PACO_BATCH_ONE_QUEUE, "shared queue", want_few)):
            plan = paco.BatchPlan(sizes, tune_cache_path=path, flags=NO_TUNE | flags)
            assert mode in plan.description and plan.transform_plan(0)[0] == want, (lines, mode)


def test_tuning_runs_in_the_batchs_queue_mode(tmp_path, key):
    path = str(tmp_path / "tune.txt")
    shared = paco.BatchPlan([1 << 18, 1 << 17, 1 << 10], tune_cache_path=path)
    assert "shared queue" in shared.description
    first = _lines(path)
    assert [(ln[0], ln[4]) for ln in first] == [("10", "0"), ("17", "1"), ("18", "1")]
    many = paco.BatchPlan([1 << 18] * 64 + [1 << 10], tune_cache_path=path)   # 2^18 is tuned anew
    assert "one per XCD" in many.description
    both = _lines(path)
    assert [(ln[0], ln[4]) for ln in both] == [("10", "0"), ("17", "1"), ("18", "0"), ("18", "1")]
    assert all(ln in both for ln in first)
    assert _key(path) == key


def _stream() -> int:
    return torch.cuda.current_stream().cuda_stream


def _run(execute, xd):
    out, ws = torch.empty_like(xd), torch.empty_like(xd)
    execute(xd.data_ptr(), out.data_ptr(), ws.data_ptr(), _stream())
    torch.cuda.synchronize()
    return out


SPLITS = [(7, 8), (8, 7), (8, 8), (8, 9), (9, 8), (8, 10), (9, 9), (10, 8), (9, 10), (10, 9), (10, 10)]


@pytest.mark.parametrize("l1,l2", SPLITS)
@pytest.mark.parametrize("flags", [0, paco.PACO_BATCH_ONE_QUEUE])
def test_every_choice_of_the_tuner_has_the_single_plans_bits(tmp_path, key, l1, l2, flags):
    path = str(tmp_path / "tune.txt")
    with open(path, "w") as f:
        f.write(f"{key}\n{l1 + l2} {l1} {l2} 1 {int(bool(flags))}\n")
    plan = paco.BatchPlan([1 << (l1 + l2)] * 16, tune_cache_path=path, flags=NO_TUNE | flags)
    assert plan.transform_plan(0)[:2] == (1 << l1, 1 << l2)
    assert ("shared queue" if flags else "one per XCD") in plan.description
    x = torch.from_numpy(inputs.normal(plan.total, seed=10 * l1 + l2)).to("cuda")
    y = _run(plan.execute, x)
    single = paco.Plan(*plan.transform_plan(0))
    for i in range(16):
        a, b = plan.offsets[i], plan.offsets[i + 1]
        assert torch.equal(y[a:b], _run(single.execute, x[a:b].clone())), i
    ref = oracle.dft(x[:1 << (l1 + l2)].cpu().numpy().astype(np.complex128))
    assert oracle.rel_l2(y[:1 << (l1 + l2)].cpu().numpy(), ref) <= TOL
    back = _run(single.execute_inverse, y[:1 << (l1 + l2)].clone()).cpu().numpy()
    assert oracle.rel_l2(back, x[:1 << (l1 + l2)].cpu().numpy()) <= 2 * TOL
    assert plan.errors() == 0


def test_tuned_batch_has_the_single_plans_bits(tmp_path):
    sizes = [1 << k for k in (20, 19, 18, 17, 16, 15, 14, 10)] * 8
    plan = paco.BatchPlan(sizes, tune_cache_path=str(tmp_path / "tune.txt"))
    print(plan.description, flush=True)
    x = torch.from_numpy(inputs.normal(plan.total, seed=7)).to("cuda")
    y = _run(plan.execute, x)
    for i, n in enumerate(sizes):
        a, b = plan.offsets[i], plan.offsets[i + 1]
        if n >= 1 << 13:
            assert torch.equal(y[a:b], _run(paco.Plan(*plan.transform_plan(i)).execute, x[a:b].clone())), (i, n)


@pytest.mark.parametrize("k,l1", [(15, 6), (16, 7), (16, 9), (17, 7), (17, 10), (18, 7)])
def test_other_splits_are_no_choice(tmp_path, key, k, l1):
    path = str(tmp_path / "tune.txt")
    with open(path, "w") as f:
        f.write(f"{key}\n{k} {l1} {k - l1} 1 0\n")
    plan = paco.BatchPlan([1 << k] * 16, tune_cache_path=path, flags=NO_TUNE)
    assert plan.transform_plan(0)[0] == 1 << (k + 1) // 2
    # the single plan of that shape runs the balanced split
    x = torch.from_numpy(inputs.normal(1 << k, seed=k)).to("cuda")
    a, b = paco.Plan(1 << l1, 1 << (k - l1), 2, 2), paco.Plan(*plan.transform_plan(0))
    assert torch.equal(_run(a.execute, x), _run(b.execute, x))
