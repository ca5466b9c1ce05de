"""The oracle's regulariser on padded neighbour lists (negative entries): a padding slot
names no splat, so losses, margins and gradients are those of the list without it, and
g* is the slot in the list as given."""
import numpy as np
import pytest

import oracle
from tests.test_oracle_gsr import _random


@pytest.mark.parametrize("n,k", [(1, 16), (2, 5), (9, 16), (15, 16)])
@pytest.mark.parametrize("spread", [False, True])
def test_padded_lists_equal_the_cut_lists(n, k, spread):
    rng = np.random.default_rng([n, k])
    sc = _random(rng, n, spread=0.2)
    xi = rng.standard_normal((n, 3))
    cut = oracle.knn(sc.means, n)
    at = np.sort(rng.permutation(np.arange(1, k))[:n - 1]) if spread else np.arange(1, n)
    at = np.concatenate([[0], at]).astype(int)
    lists = np.full((n, k), -1, np.int32)
    lists[:, at] = cut
    want = oracle.gsr(sc, oracle.Settings(), cut, xi, w_sdf=0.7, w_nor=0.4)
    got = oracle.gsr(sc, oracle.Settings(), lists, xi, w_sdf=0.7, w_nor=0.4)
    np.testing.assert_array_equal(got["gstar"], at[want["gstar"]])
    for key in ("l_sdf", "l_nor", "margins"):
        np.testing.assert_array_equal(got[key], want[key], err_msg=key)
    for key, v in want["grads"].items():
        # the samples' shares are added thread by thread, in an order that may differ
        np.testing.assert_allclose(got["grads"][key], v, rtol=1e-12, atol=1e-12 * max(np.abs(v).max(), 1.0), err_msg=key)
        assert np.abs(v).max() > 0 or n == 1
