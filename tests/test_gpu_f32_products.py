"""float32 products as bf16 terms (gemm_f32.hip) at the sizes where the kernel changes, and operands that have no such terms
(needs an MI355X)."""
from dataclasses import replace

import numpy as np
import pytest

import gen

pytestmark = pytest.mark.gpu


# token rows = 197 x tiles, two blocks of ViT-S width.  1: 32 x 32 blocks with K over eight wavefronts (N = 384), K over four groups (N = 1152,
# 1536), a last tile of 5 rows, and the CLS rows alone; 13: two groups for QKV (738 workgroups) and the first MLP matrix's one group (984); 18: 64 x 128
# for the first MLP matrix (672), 128 x 128 weight gradients in 14 slabs whose last is short.
@pytest.mark.parametrize("tiles", [1, 13, 18])
def test_fp32_step_where_the_kernel_changes(tiles):
    from oracle import slide_oracle as so
    from slide_harness import GpuSlide, compare_step
    cfg = replace(gen.CONFIGS["small"][0], layers=2)
    ds, ws, ls = gen.SEEDS["small"]
    prm = gen.make_params(cfg, ws, perturbed=True)
    X = gen.make_pixels(cfg, tiles, ds)
    lab = gen.make_label(cfg, ls)
    print(f"case f32 products layers=2 n={tiles} dtype=0 label={lab}", flush=True)
    out = GpuSlide(cfg, prm, 0, tiles).step(X, lab)
    ref = so.slide_step(prm, X.astype(np.float64), lab, cfg)
    _, pool_same = so.pool_bwd(so.pool_fwd(prm, out["H"], lab, cfg)[4])
    errs, bad, kappa = compare_step(out, ref, 1e-4, cfg, None, pool_same)   # the bound of every fp32 parity test
    print(f"kappa={kappa:.1f} worst:", sorted(errs.items(), key=lambda kv: -kv[1])[:6], flush=True)
    assert not bad, bad


# Weights near the largest float: a pixel of 2 times 3e38 is infinite (no number where two such meet with other signs), as in
# float32 products, and is so in the rows of its tile only.  The others' products are finite: pixels that meet a zero weight stay.
@pytest.mark.parametrize("tiles", [1, 40])
def test_products_that_are_infinite(tiles):
    from slide_harness import GpuSlide
    cfg = replace(gen.CONFIGS["small"][0], layers=0)
    ds, ws, _ = gen.SEEDS["small"]
    prm = gen.make_params(cfg, ws, perturbed=True)
    prm["pe.W"] = np.zeros_like(prm["pe.W"])
    prm["pe.W"][:, 0] = 3e38     # the first channel's first pixel of every patch
    prm["pe.W"][:, 1] = np.where(np.arange(cfg.dim) % 2, 1e-3, -2e-3)
    prm["pos"] *= 0.0
    prm["pe.b"] *= 0.0
    X = np.zeros((tiles, 3, cfg.tile, cfg.tile), np.float32)
    X[:, 0, ::cfg.patch, 1::cfg.patch] = 1.5          # finite products everywhere
    X[0, 0, 0, 0] = 2.0                               # 6e38 in the first patch of the first tile
    X[0, 0, 0, cfg.patch] = np.inf
    X[0, 0, 0, 2 * cfg.patch] = np.nan
    g = GpuSlide(cfg, prm, 0, tiles)
    g.lib.encoder_fwd_tiles(g.to_dev(X), tiles, g.torch.zeros((tiles, cfg.dim), device=g.dev), 1)
    g.torch.cuda.synchronize()
    # the stream behind the patch embedding is the arena's tensor of n T rows that holds 1.5 W[:, 1] on its patch rows
    rows = g.arena[: g.arena.numel() // 4 * 4].view(g.torch.float32)
    want = (np.float32(1.5) * prm["pe.W"][:, 1].astype(np.float32))
    T = cfg.tokens
    key = g.torch.from_numpy(want).to(g.dev)
    last = None
    for off in range(0, rows.numel() - cfg.dim, 64):   # allocations are aligned to 64 floats, rows are 384 of them
        if bool((rows[off:off + cfg.dim] == key).all()):
            last = off
            break
    assert last is not None
    x = rows[last:last + cfg.dim * (T - 4)].reshape(-1, cfg.dim)   # the fourth patch row of the first tile and on
    assert bool((x == key).all())
    first = rows[last - 3 * cfg.dim:last].reshape(3, cfg.dim).cpu().numpy()
    assert np.isposinf(first[0]).all() and np.isposinf(first[1]).all() and np.isnan(first[2]).all()


def _embedding(cfg, prm, X):
    """Patch rows of the stream behind the patch embedding (float32), and the patches and results in float64."""
    from slide_harness import GpuSlide
    tiles, P, g2 = X.shape[0], cfg.patch, cfg.grid ** 2
    g = GpuSlide(cfg, prm, 0, tiles)
    torch = g.torch
    px = g.to_dev(X)
    g.lib.encoder_fwd_tiles(px, tiles, torch.zeros((tiles, cfg.dim), device=g.dev), 1)
    torch.cuda.synchronize()
    # the arena's tensor whose first row is class token and position
    mem = g.arena[:g.arena.numel() // 256 * 256].view(torch.float32)
    key = torch.from_numpy(prm["cls"].reshape(-1) + prm["pos"][0]).to(g.dev)
    near = (mem.view(-1, 64) == key[:64]).all(1).nonzero().flatten().tolist()
    near = [o * 64 for o in near if bool((mem[o * 64:o * 64 + cfg.dim] == key).all())]
    got = mem[near[0]:near[0] + tiles * cfg.tokens * cfg.dim].view(tiles, cfg.tokens, cfg.dim)[:, 1:].double().cpu().numpy().reshape(-1, cfg.dim)
    p = X.astype(np.float64).reshape(tiles, 3, cfg.grid, P, cfg.grid, P).transpose(0, 2, 4, 1, 3, 5).reshape(tiles * g2, -1)
    with np.errstate(invalid="ignore"):
        want = p @ prm["pe.W"].astype(np.float64).T + prm["pe.b"] + np.tile(prm["pos"][1:], (tiles, 1))
    return got, p, want


# A row's products are off by 2^-24 each, its 768 additions by as much of a partial sum: 2 sqrt(768) 2^-24 = 3.3e-6 of the terms' norm
def _worst(cfg, prm, got, p, want):
    norm = np.sqrt((p ** 2) @ (prm["pe.W"].astype(np.float64) ** 2).T) + np.abs(want)
    err = (np.abs(got - want) / norm).max()
    print("worst", err, flush=True)
    return err


# One operand that is no finite number, in a column of each group of wavefronts that K is dealt to (two groups: columns 0 .. 31, 64 .. 95, ...
# are the first one's; four: 0 .. 31, 128 .. 159, ...), in blocks of 64 rows of their own, dense weights: its row has what float32
# products give, every other row what it has anyway.  Patch embedding of ViT-S, K = 768: 1 tile takes 32 x 32 blocks, 5 four groups, 20
# two, 65 one, 70 the 64 x 128 tiles.
@pytest.mark.parametrize("tiles", [1, 5, 20, 65, 70])
def test_rows_beside_one_that_is_not_finite(tiles):
    cfg = replace(gen.CONFIGS["small"][0], layers=0)
    ds, ws, _ = gen.SEEDS["small"]
    prm = gen.make_params(cfg, ws, perturbed=True)
    X = gen.make_pixels(cfg, tiles, ds)
    P, g2, bad = cfg.patch, cfg.grid ** 2, {}
    for i, col in enumerate([0, 33, 40, 70, 100, 135, 200, 767][:max(3, tiles)]):
        row = 5 + 64 * i   # of the patch matrix; a patch is [3][P][P]
        n, j, (c, y, x) = row // g2, row % g2, np.unravel_index(col, (3, P, P))
        X[n, c, j // cfg.grid * P + y, j % cfg.grid * P + x] = bad[row] = (np.inf, np.nan, -np.inf)[i % 3]
    print(f"case rows beside one that is not finite n={tiles}", flush=True)
    got, p, want = _embedding(cfg, prm, X)
    for row in bad:
        w = prm["pe.W"][:, int(np.flatnonzero(~np.isfinite(p[row]))[0])]
        assert np.array_equal(got[row], bad[row] * np.sign(w), equal_nan=True), (row, got[row][:4])
    rest = np.setdiff1d(np.arange(tiles * g2), list(bad))
    assert _worst(cfg, prm, got[rest], p[rest], want[rest]) < 4e-6


# First operands of about 2^-120, whose trailing bits no bf16 number holds as they are, and of about 2^84, which are infinite when scaled
@pytest.mark.parametrize("tiles", [1, 5, 20, 65, 70])
@pytest.mark.parametrize("power", [-120, 84])
def test_operands_at_the_ends_of_the_range(tiles, power):
    cfg = replace(gen.CONFIGS["small"][0], layers=0)
    ds, ws, _ = gen.SEEDS["small"]
    prm = gen.make_params(cfg, ws, perturbed=True)
    prm["pe.W"] = prm["pe.W"] * np.float32(64)
    prm["pe.b"] = np.zeros_like(prm["pe.b"])
    prm["pos"][1:] = 0
    X = np.ldexp(gen.make_pixels(cfg, tiles, ds), power)
    print(f"case operands at the ends of the range n={tiles} 2^{power}", flush=True)
    assert _worst(cfg, prm, *_embedding(cfg, prm, X)) < 4e-6


# Positive operands, whose products' errors a bias would line up: what is left out of a product has either sign, and what the matrix core's
# additions pull downwards cancels where several groups of wavefronts share K (1e-9 of the result is left) and is 2e-8 of it over 48 steps in one
# group.  Limit: half as much again (terms cut off instead of rounded: 4e-8 in several groups, 1.9e-7 in one).
@pytest.mark.parametrize("tiles", [1, 5, 20, 65, 70])
def test_positive_operands_have_no_bias(tiles):
    cfg = replace(gen.CONFIGS["small"][0], layers=0)
    ds, ws, _ = gen.SEEDS["small"]
    prm = gen.make_params(cfg, ws, perturbed=True)
    prm["pe.W"] = np.abs(prm["pe.W"])
    prm["pe.b"] = np.zeros_like(prm["pe.b"])
    prm["pos"][1:] = 0
    X = np.abs(gen.make_pixels(cfg, tiles, ds))
    print(f"case positive operands n={tiles}", flush=True)
    got, p, want = _embedding(cfg, prm, X)
    bias = float((got - want).sum() / want.sum())
    print("bias", bias, flush=True)
    assert abs(bias) < 3e-8
    assert _worst(cfg, prm, got, p, want) < 4e-6
