"""Regulariser under masks that leave whole waves, parts of a wave or nothing on: each
sample's losses are those of the unmasked call to the bit, and the gradients are those of
the samples that are on (the sums of their calls one half at a time)."""
import numpy as np
import pytest

from tests.gpu_util import log, norm_errors
from tests.test_gpu_gsr import _scene, _splats

pytestmark = pytest.mark.gpu

KEYS = ("mean", "scale", "quat", "opacity", "beta")


def _masks(n, order):
    rng = np.random.default_rng([440, n])
    block = np.zeros(n, bool)
    block[order[:n // 3]] = True  # a run in the order the samples are taken in
    one = np.zeros(n, bool)
    one[order[n // 2]] = True
    return dict(none=np.zeros(n, bool), block=block, one=one, few=rng.random(n) < 0.05, half=rng.random(n) < 0.5)


@pytest.mark.parametrize("n,k", [(1, 16), (9, 16), (63, 5), (1000, 16), (3001, 7)])
@pytest.mark.parametrize("name", ["none", "block", "one", "few", "half"])
def test_masked_calls(name, n, k):
    import torch
    from paper_2411_09156_amd import RasterSettings
    from paper_2411_09156_amd.gsr import gsr, knn
    log(f"[gpu] gsr mask {name} n={n} k={k}")
    sp = _splats(_scene("cube", n, 6))
    nb = knn(sp, k)
    xi = torch.as_tensor(np.random.default_rng([441, n]).standard_normal((3, n)).astype(np.float32), device="cuda")
    mask = _masks(n, nb["order"].cpu().numpy().astype(np.int64))[name]

    def call(m, grads=True):
        g = {key: torch.zeros_like(getattr(sp, key)) for key in KEYS} if grads else None
        m = None if m is None else torch.as_tensor(m.astype(np.uint8), device="cuda")
        out = gsr(sp, RasterSettings(), nb, xi, mask=m, w_sdf=0.6, w_nor=0.4, grads=g)
        return out["sample_out"].cpu().numpy(), {key: v.cpu().numpy().astype(np.float64) for key, v in (g or {}).items()}

    every, all_grads = call(None)
    got, grads = call(mask)
    want = np.where(mask[:, None], every, np.float32([0, 0, -1, 0]))
    np.testing.assert_array_equal(got, want)
    np.testing.assert_array_equal(call(mask, grads=False)[0], want)
    rest = call(~mask)[1]
    for key in KEYS:
        assert np.isfinite(grads[key]).all()
        if not mask.any():
            assert (grads[key] == 0).all()
        # float32 sums of some k terms a splat, split in two: 1e-5 of the largest
        scale = np.abs(all_grads[key]).max() + np.abs(grads[key]).max()
        np.testing.assert_allclose(grads[key] + rest[key], all_grads[key], rtol=0, atol=1e-5 * scale)
    einf, _ = norm_errors(grads["mean"], all_grads["mean"])
    assert mask.all() or n == 1 or einf > 1e-6
