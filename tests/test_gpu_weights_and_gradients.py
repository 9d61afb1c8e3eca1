"""Weight copies and weight gradients at the sizes where their tiles and slabs change (needs an MI355X)."""
from dataclasses import replace

import numpy as np
import pytest

import gen

pytestmark = pytest.mark.gpu


# Weight copies by 64 x 64 tiles of matrices that are no multiple of 64 (96, 288, 32), LayerNorm rows of half a wavefront and of
# one and a half.  Tolerances: those of every parity test.  (Not 32 features in bf16: their few hundred roundings, 2e-3 of the features, reach the
# aggregator's gradients conditioned 18-fold, 5e-2.)
@pytest.mark.parametrize("dim,dtype,tol", [(96, 1, 2e-2), (32, 0, 1e-4), (96, 0, 1e-4)])
def test_step_of_widths_beside_the_tiles(dim, dtype, tol):
    from oracle import slide_oracle as so
    from slide_harness import GpuSlide, compare_step
    cfg = replace(gen.CONFIGS["tiny"][0], dim=dim, heads=dim // 32)
    ds, ws, ls = gen.SEEDS["tiny"]
    prm = gen.make_params(cfg, ws, perturbed=True)
    X = gen.make_pixels(cfg, 16, ds)
    if dtype == 1:
        prm, X = {k: gen.to_bf16_grid(v) for k, v in prm.items()}, gen.to_bf16_grid(X)
    lab = gen.make_label(cfg, ls)
    print(f"case width {dim} n=16 dtype={dtype} label={lab}", flush=True)
    out = GpuSlide(cfg, prm, dtype, 16).step(X, lab)
    ref = so.slide_step(prm, X.astype(np.float64), lab, cfg)
    _, pool_same = so.pool_bwd(so.pool_fwd(prm, out["H"], lab, cfg)[4])
    errs, bad, kappa = compare_step(out, ref, tol, cfg, None, pool_same)
    print(f"kappa={kappa:.1f} worst:", sorted(errs.items(), key=lambda kv: -kv[1])[:6], flush=True)
    assert not bad, bad


# A block's weight gradients whole and in chunks (of 4,096 rows and more, where the forward's bits are the same) are the same terms in other
# slabs.  ViT-B: 432 tiles of 128 x 128, 11,820 rows take four slabs (two rounds of workgroups), 8,668 and 5,910 two, 4,334 two; ViT-S: 108 tiles,
# 33,490 rows nine slabs, 16,745 nine, 49,250 the large-M kernel.
@pytest.mark.parametrize("name,tiles,chunk", [("full", 60, 30), ("full", 44, 22), ("small", 170, 85), ("small", 250, 125)])
def test_weight_gradients_in_other_slabs(name, tiles, chunk):
    from slide_harness import GpuSlide, rel_l2
    cfg = replace(gen.CONFIGS[name][0], layers=2)
    ds, ws, ls = gen.SEEDS[name]
    prm = {k: gen.to_bf16_grid(v) for k, v in gen.make_params(cfg, ws, perturbed=True).items()}
    X = gen.to_bf16_grid(gen.make_pixels(cfg, tiles, ds, workers=8))
    label = gen.make_label(cfg, ls)
    print(f"case weight gradients {name} whole {tiles}, chunks of {chunk}", flush=True)
    g = GpuSlide(cfg, prm, 1, tiles)
    whole, parts = g.step(X, label), g.step_chunked(X, label, chunk)
    errs = {k: rel_l2(parts["grads"][k], v) for k, v in whole["grads"].items()}
    print("worst:", sorted(errs.items(), key=lambda kv: -kv[1])[:4], flush=True)
    # float32 sums of n <= 49,250 terms in two orders: 2 sqrt(n) 2^-24 = 2.7e-5 of the terms' norm
    assert max(errs.values()) < 2.7e-5
