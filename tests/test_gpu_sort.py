"""The point sort of the tree build at the edges of its tiles and merge groups.

Sorted keys and the permutation are whole numbers and have to be those of a
stable sort by key: one partial or whole tile (1024 points), the first merge
(1025), a whole and an overfull group of eight tiles (8192, 8193), two merge
launches, with distinct keys, many equal keys and all keys equal; then a
rebuild from moved points, which merges the displaced points into the rest."""
import numpy as np
import pytest
import torch

from paper_2512_09478_amd import Plan

pytestmark = pytest.mark.gpu


def positions(n, ties, seed):
    rng = np.random.default_rng(seed)
    if ties == "all":
        x = np.full((n, 3), 0.375)
    elif ties == "many":   # points on an 8^3 lattice: runs of equal keys across tiles
        x = rng.integers(0, 8, (n, 3)) / 8.0 + 1 / 16
    else:
        x = rng.random((n, 3))
    return x.astype(np.float32).astype(np.float64)


def morton(x):
    k = np.minimum((x * 2.0 ** 21).astype(np.uint64), np.uint64(2 ** 21 - 1))
    key = np.zeros(len(x), dtype=np.uint64)
    for b in range(21):
        for d in range(3):
            key |= ((k[:, d] >> np.uint64(b)) & np.uint64(1)) << np.uint64(3 * b + 2 - d)
    return key


def check(plan, x):
    t = plan.tree()
    key = morton(x)
    perm = np.lexsort((np.arange(len(x)), key))
    assert np.array_equal(np.asarray(t["perm"]), perm)
    assert np.array_equal(np.asarray(t["keys"]).astype(np.uint64), key[perm])


@pytest.mark.parametrize("ties", ["none", "many", "all"])
@pytest.mark.parametrize("n", [2, 63, 1023, 1024, 1025, 8191, 8192, 8193, 65536, 65537, 70001])
def test_sort(n, ties):
    print(f"sort n={n} ties={ties}", flush=True)
    x = positions(n, ties, n)
    plan = Plan(torch.from_numpy(x).cuda(), p=3, leaf_size=64, max_depth=8, root=((0.0, 0.0, 0.0), 1.0))
    check(plan, x)
    rng = np.random.default_rng(n + 1)
    few = rng.random(n) < 0.05   # displaced points, some onto others
    x2 = x.copy()
    x2[few] = positions(n, "none", n + 2)[few]
    plan.rebuild(torch.from_numpy(x2).cuda())
    check(plan, x2)
