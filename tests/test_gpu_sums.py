"""Sums over slab partials: written and added, at slab counts on both sides of where a thread adds all slabs of its outputs."""
from dataclasses import replace

import numpy as np
import pytest

import gen

pytestmark = pytest.mark.gpu


# slabs of a block's weight gradients: 1 to 3 tiles one to five, 24 and 37 tiles nine to eleven, 64 sixteen or more; at 90 and more
# the large-M kernel takes them (multiples of eight); float32: 8 to 16
@pytest.mark.parametrize("dtype,tiles", [(1, 1), (1, 3), (1, 24), (1, 37), (1, 64), (1, 130), (0, 7), (0, 24)])
def test_added_gradients_are_twice_the_written_ones(dtype, tiles):
    from slide_harness import GpuSlide
    cfg = replace(gen.CONFIGS["small"][0], layers=2)
    ds, ws, ls = gen.SEEDS["small"]
    prm = {k: gen.to_bf16_grid(v) for k, v in gen.make_params(cfg, ws, perturbed=True).items()}
    X = gen.to_bf16_grid(gen.make_pixels(cfg, tiles, ds, workers=8))
    lab = gen.make_label(cfg, ls)
    print(f"case sums dtype={dtype} n={tiles}", flush=True)
    g = GpuSlide(cfg, prm, dtype, tiles)
    once = g.step(X, lab)["grads"]
    twice = g.step(X, lab, accumulate=True)["grads"]
    for k, v in once.items():   # g + g is exact
        assert np.isfinite(v).all()
        np.testing.assert_array_equal(twice[k], 2.0 * v, err_msg=k)
