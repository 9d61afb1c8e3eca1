"""Sums over slab partials, at slab counts on both sides of where a thread adds all slabs of its outputs: the weight gradients of the
blocks against the oracle (a slab too few or too many is off by about one over their number), and added gradients against written
ones."""
from dataclasses import replace

import numpy as np
import pytest

import gen

pytestmark = pytest.mark.gpu


# Slabs of the weight gradients, one thread up to 8: bf16, 1 tile two, from 3 tiles on five (the last block, of which only QKV has
# all rows, 5 at 3 tiles and 19 from 24 on), at 130 tiles the large-M kernel's multiples of eight; float32, QKV 7 at 4 tiles, 8 at
# 5, 10 at 6, 22 at 24.  The larger bags without the oracle (test_gpu_whole_and_chunks.py holds their gradients to another cut)
@pytest.mark.parametrize("dtype,tiles", [(1, 1), (1, 3), (1, 24), (1, 64), (1, 130), (0, 4), (0, 5), (0, 6), (0, 24)])
def test_gradients_written_and_added(dtype, tiles):
    from oracle import slide_oracle as so
    from slide_harness import GpuSlide, rel_l2
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
    if tiles <= 24:
        ref = so.slide_step(prm, X.astype(np.float64), lab, cfg)["grads"]
        errs = {k: rel_l2(once[k], v) for k, v in ref.items() if k[0] == "l" and k[1].isdigit() and k.endswith(".W")}
        assert len(errs) == 8, list(ref)
        print("worst:", sorted(errs.items(), key=lambda kv: -kv[1])[:4], flush=True)
        assert max(errs.values()) <= (2e-2 if dtype else 1e-4), errs   # the bounds of the parity tests of the step
