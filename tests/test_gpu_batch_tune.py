"""What a batch's autotuning times and records: the parts whose product takes a
tile shape, and nothing where there is none."""
import os

import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    return t


def jobs(torch, shapes):
    g = torch.Generator(device="cuda")
    g.manual_seed(2)
    r = lambda a, b: torch.randn((a, b), generator=g, device="cuda")
    return [(r(m, d), r(n, d), k) for m, n, d, k in shapes]


def tuned(torch, tmp_path, name, shapes):
    """The grouped keys that a tuned batch adds to its cache file, with its
    results compared with an untuned handle's."""
    import paper_1309_5478_amd as knn
    js = jobs(torch, shapes)
    path = str(tmp_path / name)
    os.environ["KNN_AUTOTUNE_CACHE"] = path
    try:
        a = knn.Handle(0).batch_search(js, flags=knn.FLAG_AUTOTUNE)
        torch.cuda.synchronize()
    finally:
        del os.environ["KNN_AUTOTUNE_CACHE"]
    b = knn.Handle(0).batch_search(js)
    for (x, i), (y, j) in zip(a, b):
        assert torch.equal(x, y) and torch.equal(i, j)
    if not os.path.exists(path):
        return set()
    return {line.split('"')[1] for line in open(path) if '"grouped|' in line}


PIPED = [(300, 30011, 128, 9), (1024, 70001, 64, 3), (200, 5000, 96, 16)]   # (the last: stored rows)
TILED = [(200, 90000, 32, 5), (90, 100000, 32, 12), (77, 70000, 17, 2)]     # (d = 17: a launch of its own)


def test_nothing_to_choose_records_nothing(torch, tmp_path):
    assert tuned(torch, tmp_path, "piped.json", PIPED) == set()


def test_key_is_of_the_tiled_parts(torch, tmp_path):
    """The parts that were timed give the key, whatever other jobs the batch has."""
    alone = tuned(torch, tmp_path, "tiled.json", TILED)
    assert len(alone) >= 1
    both = tuned(torch, tmp_path, "both.json", PIPED + TILED)
    assert both <= alone, (both, alone)


def test_only_own_launches(torch, tmp_path):
    assert len(tuned(torch, tmp_path, "own.json", [(200, 90000, 33, 4)])) >= 1
