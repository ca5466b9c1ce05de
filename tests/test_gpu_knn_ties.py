"""Neighbour lists of centres on an integer lattice, against brute force.

Squared distances are small integers, exact in any order of operations, so the
lists are known to the entry: many equal distances (ties by index), coincident
centres (distance 0), one cell, one row, one query more or less than a wave."""
import numpy as np
import pytest

import oracle  # noqa: F401  (the path of the shared inputs)
from tests.test_gpu_gsr import _splats

pytestmark = pytest.mark.gpu


class _Scene:
    def __init__(self, means):
        n = means.shape[0]
        rng = np.random.default_rng(7)
        self.n, self.means = n, means.astype(np.float32)
        self.scales = np.full((n, 3), 0.1, np.float32)
        self.quats = np.tile(np.float32([1, 0, 0, 0]), (n, 1))
        self.opacities, self.betas = np.full(n, 0.5, np.float32), np.full(n, 2.0, np.float32)
        self.sh = rng.normal(size=(n, 1, 3)).astype(np.float32)


def _means(kind, n):
    rng = np.random.default_rng([420, n])
    m = rng.integers(0, 13, (n, 3)).astype(np.float64)
    if kind == "row":
        m[:, 1:] = 3.0
        m[:, 0] = rng.integers(0, 200, n)
    elif kind == "same":
        m[:] = 2.0
    return m


@pytest.mark.parametrize("k", [2, 3, 7, 15, 16])
@pytest.mark.parametrize("kind,n", [("cube", 17), ("cube", 64), ("cube", 257), ("cube", 4000), ("row", 1500),
                                    ("same", 300)])
def test_lattice_lists_are_exact(kind, n, k):
    from paper_2411_09156_amd.gsr import knn
    means = _means(kind, n)
    nb = knn(_splats(_Scene(means)), k)
    got = nb["knn"].cpu().numpy().astype(np.int64).reshape(n, k)
    d2 = ((means[:, None] - means[None]) ** 2).sum(-1)
    np.fill_diagonal(d2, -1.0)
    np.testing.assert_array_equal(got, np.argsort(d2, axis=1, kind="stable")[:, :k])
    # the inverse lists: entries by the splat they name, in entry order, and their places
    order = nb["order"].cpu().numpy().astype(np.int64)
    named = got[order].ravel()
    entries = np.argsort(named, kind="stable")
    np.testing.assert_array_equal(nb["inv_entries"].cpu().numpy().astype(np.int64), entries)
    slot = np.empty(n * k, np.int64)
    slot[entries] = np.arange(n * k)
    np.testing.assert_array_equal(nb["inv_slot"].cpu().numpy().astype(np.int64), slot)
