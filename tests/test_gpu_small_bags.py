"""Whole steps at the bag sizes where the choice of kernel changes: a few tiles to a few dozen, ViT-S and ViT-B widths
with two blocks, against the CPU oracle (needs an MI355X)."""
from dataclasses import replace

import numpy as np
import pytest

import gen

pytestmark = pytest.mark.gpu

BF16_TOL = 2e-2   # the bound of every bf16 parity test of the step (test_gpu_parity.py)


# token rows = 197 x tiles (of two tiles the gate gradients are one difference of two feature rows, no sum to average
# its rounding).  5: every GEMM on 64 x 64 tiles, a last tile of 25 rows; 13: 64 x 64 and 64 x 128 tiles,
# 2561 = 40 * 64 + 1 rows; 20: 3940 rows, below the 4096 from which biases start the accumulators, QKV (279 tiles of 128 x 128) and the
# GELU derivative on 128 x 128, GELU on 64 x 128; 33: 6501 rows, QKV on 128 x 128, GELU on 256 x 192, its derivative on 64 x 128, the others
# on 64 x 64.  ViT-B width: contractions of 3072.
@pytest.mark.parametrize("name,tiles", [("small", 5), ("small", 13), ("small", 20), ("small", 33), ("full", 4)])
def test_bf16_step_small_bags(name, tiles):
    from oracle import slide_oracle as so
    from slide_harness import GpuSlide, compare_step
    cfg = replace(gen.CONFIGS[name][0], layers=2)
    ds, ws, ls = gen.SEEDS[name]
    prm = {k: gen.to_bf16_grid(v) for k, v in gen.make_params(cfg, ws, perturbed=True).items()}
    X = gen.to_bf16_grid(gen.make_pixels(cfg, tiles, ds))
    lab = gen.make_label(cfg, ls)
    print(f"case {name} layers=2 n={tiles} dtype=1 label={lab}", flush=True)
    out = GpuSlide(cfg, prm, 1, tiles).step(X, lab)
    ref = so.slide_step(prm, X.astype(np.float64), lab, cfg)
    _, pool_same = so.pool_bwd(so.pool_fwd(prm, out["H"], lab, cfg)[4])
    errs, bad, kappa = compare_step(out, ref, BF16_TOL, cfg, None, pool_same)
    print(f"kappa={kappa:.1f} worst:", sorted(errs.items(), key=lambda kv: -kv[1])[:6], flush=True)
    assert not bad, bad


# float32: 5 tiles = 985 rows (64 x 64 tiles with a last one of 25 rows, slabs of a few 32-row steps, four wavefronts per
# head), 45 tiles: eight wavefronts per head in both directions; ViT-B width: contractions of 3072
@pytest.mark.parametrize("name,tiles", [("small", 5), ("small", 45), ("full", 3)])
def test_fp32_step_small_bags(name, tiles):
    from oracle import slide_oracle as so
    from slide_harness import GpuSlide, compare_step
    cfg = replace(gen.CONFIGS[name][0], layers=2)
    ds, ws, ls = gen.SEEDS[name]
    prm = gen.make_params(cfg, ws, perturbed=True)
    X = gen.make_pixels(cfg, tiles, ds)
    lab = gen.make_label(cfg, ls)
    print(f"case {name} layers=2 n={tiles} dtype=0 label={lab}", flush=True)
    out = GpuSlide(cfg, prm, 0, tiles).step(X, lab)
    ref = so.slide_step(prm, X.astype(np.float64), lab, cfg)
    _, pool_same = so.pool_bwd(so.pool_fwd(prm, out["H"], lab, cfg)[4])
    errs, bad, kappa = compare_step(out, ref, 1e-4, cfg, None, pool_same)   # the bound of every fp32 parity test
    print(f"kappa={kappa:.1f} worst:", sorted(errs.items(), key=lambda kv: -kv[1])[:6], flush=True)
    assert not bad, bad


# position rows, class token and patch bias stay float32 on the way into the sum: a patch whose product is -100 plus a little
# meets a position of 100 plus a little, and only what is left over carries the signal (bf16 numbers near 100 are 0.5 apart)
@pytest.mark.parametrize("name,tiles", [("tiny", 16), ("tiny", 250), ("small", 5)])
def test_position_rows_are_added_in_float32(name, tiles):
    from oracle import slide_oracle as so
    from slide_harness import GpuSlide, compare_step
    cfg = replace(gen.CONFIGS[name][0], layers=2)
    ds, ws, ls = gen.SEEDS[name]
    prm = {k: gen.to_bf16_grid(v) for k, v in gen.make_params(cfg, ws, perturbed=True).items()}
    prm["pe.W"][:, 0] = -100.0
    pos = 25.0 * prm["pos"]
    pos[1:] += 100.0
    prm["pos"] = pos.astype(np.float32).astype(np.float64)
    X = gen.to_bf16_grid(gen.make_pixels(cfg, tiles, ds))
    X[:, 0, ::cfg.patch, ::cfg.patch] = 1.0
    lab = gen.make_label(cfg, ls)
    print(f"case position rows {name} layers=2 n={tiles}", flush=True)
    # no pixel gradient: that of the pixel with equal weights is -100 times a sum that LayerNorm makes zero
    out = GpuSlide(cfg, prm, 1, tiles).step(X, lab, want_pixel_grad=False)
    ref = so.slide_step(prm, X.astype(np.float64), lab, cfg, want_pixel_grad=False)
    _, pool_same = so.pool_bwd(so.pool_fwd(prm, out["H"], lab, cfg)[4])
    errs, bad, kappa = compare_step(out, ref, BF16_TOL, cfg, None, pool_same)
    print(f"kappa={kappa:.1f} worst:", sorted(errs.items(), key=lambda kv: -kv[1])[:6], flush=True)
    assert not bad, bad
