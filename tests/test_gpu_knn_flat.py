"""Neighbour lists of centres on lines and planes and of clusters with far outliers, whose
queries go through many shells of a grid that is flat or mostly empty, against brute force.
Centres on an integer lattice: squared distances are exact, the lists known to the entry."""
import numpy as np
import pytest

from tests.gpu_util import log
from tests.test_gpu_gsr import _splats
from tests.test_gpu_knn_ties import _Scene

pytestmark = pytest.mark.gpu


def _means(axes, n, outliers):
    """n centres that vary along `axes` only, all but `outliers` of them close together."""
    rng = np.random.default_rng([421, n, len(axes), outliers])
    m = np.full((n, 3), 3.0)
    for a in axes:
        m[:, a] = rng.integers(0, 9, n)
        m[:outliers, a] = rng.integers(-700, 700, outliers)
    return m[rng.permutation(n)]


@pytest.mark.parametrize("k", [2, 16])
@pytest.mark.parametrize("axes", ["x", "y", "z", "xy", "xz", "yz", "xyz"])
@pytest.mark.parametrize("n,outliers", [(900, 0), (900, 20), (70, 60)])
def test_lists_of_flat_and_sparse_centres_are_exact(axes, n, outliers, k):
    from paper_2411_09156_amd.gsr import knn
    log(f"[gpu] knn along {axes}, {n} centres, {outliers} far off, k={k}")
    means = _means(["xyz".index(a) for a in axes], n, outliers)
    got = knn(_splats(_Scene(means)), k)["knn"].cpu().numpy().astype(np.int64).reshape(n, k)
    d2 = ((means[:, None] - means[None]) ** 2).sum(-1)
    np.fill_diagonal(d2, -1.0)
    np.testing.assert_array_equal(got, np.argsort(d2, axis=1, kind="stable")[:, :k])
