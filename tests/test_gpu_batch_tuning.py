"""The batched form's tuning cache: which files and lines are trusted."""
import re

import pytest

from paper_2609_06449_amd import paco

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu
NO_TUNE = paco.PACO_BATCH_NO_TUNE
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
