"""The autotuner times each renderer once: candidates that differ only in a batch their
kernels do not read would be chosen between by noise."""
import ctypes

from paper_2411_09156_amd import _lib


def test_no_two_candidates_run_the_same_kernels():
    lib = _lib.load()
    seen = []
    for k in range(lib.gesr_autotune_candidate(-1, None)):
        c = _lib.Settings()
        assert lib.gesr_autotune_candidate(k, ctypes.byref(c)) == 0
        if c.tile_w == 0:  # a digit width, tried with the chosen renderer
            seen.append(("radix", c.radix_bits))
        else:
            # the adjoints that stage 128 records: four waves on 16x16, and 32x16
            both = (c.tile_w, c.tile_h, c.variant) in ((16, 16, 1), (32, 16, 0))
            seen.append((c.tile_w, c.tile_h, c.variant, c.batch >= 128 if both else None))
    assert len(set(seen)) == len(seen), seen
