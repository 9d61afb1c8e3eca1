"""The forward LayerNorm of 384 and 768 columns to the last bit: what fuses with what is written out in the kernels and must not change
from one of them to the next or over time, since a float32 bit decides roundings to bf16 all the way down (needs an MI355X)."""
from dataclasses import replace

import numpy as np
import pytest

import gen

pytestmark = pytest.mark.gpu

f32, f64 = np.float32, np.float64


def _fma(a, b, c):   # a product of two floats is exact in 64 bits
    return (f64(a) * f64(b) + f64(c)).astype(f32)


def _layernorm(x, gam, bet, eps):
    """Rows as 16 lanes take them: lane l has columns (l + 16 k) * 8 .. + 7; sums in that order, then over the lanes by halves."""
    D = x.shape[1]
    v = x.reshape(-1, D // 128, 16, 8).transpose(0, 2, 1, 3).reshape(-1, 16, D // 16)

    def total(s):
        for o in (8, 4, 2, 1):
            s = s[:, :o] + s[:, o:2 * o]
        return s

    s = np.zeros(v.shape[:2], f32)
    for i in range(v.shape[2]):
        s = s + v[:, :, i]
    v = _fma(total(s)[:, :, None], f32(-1) / f32(D), v)          # the mean's product is not rounded
    q = _fma(v[:, :, 0], v[:, :, 0], v[:, :, 1] * v[:, :, 1])
    for i in range(2, v.shape[2]):
        q = _fma(v[:, :, i], v[:, :, i], q)
    rstd = f32(1) / np.sqrt(_fma(total(q), f32(1) / f32(D), f32(eps)))
    u = (v * rstd[:, :, None]).astype(f32).reshape(-1, 16, D // 128, 8).transpose(0, 2, 1, 3).reshape(-1, D)
    return gen.to_bf16_grid(_fma(u, gam.astype(f32), bet.astype(f32)))


# Rows whose mean is twelve times their deviation, where a rounded mean shows: a few hundred of the results differ then.  The class
# token, patch bias and patch weights are zero, so that the rows are those of the position table in every tile.
@pytest.mark.parametrize("name", ["small", "full"])
def test_forward_layernorm_bits(name):
    from slide_harness import GpuSlide
    cfg = replace(gen.CONFIGS[name][0], layers=1)
    ds, ws, _ = gen.SEEDS[name]
    prm = gen.make_params(cfg, ws, perturbed=True)
    for k in ("pe.W", "pe.b", "cls"):
        prm[k] = np.zeros_like(prm[k])
    rows = gen.to_bf16_grid(12.0 + np.random.Generator(np.random.PCG64(5)).standard_normal(prm["pos"].shape))
    prm["pos"] = rows
    print(f"case layernorm bits D={cfg.dim}", flush=True)
    g = GpuSlide(cfg, prm, 1, 2)
    px = g.to_dev(gen.make_pixels(cfg, 2, ds))
    g.lib.encoder_fwd_tiles(px, 2, g.torch.zeros((2, cfg.dim), device=g.dev), 1)
    g.torch.cuda.synchronize()
    want = _layernorm(rows.astype(f32), prm["l0.ln1.g"], prm["l0.ln1.b"], cfg.ln_eps)
    want = g.torch.from_numpy(np.concatenate([want, want])).to(g.dev)
    # the block's first LayerNorm output is a bf16 tensor of the arena (tensors begin at multiples of 256 bytes)
    mem = g.arena[:g.arena.numel() // 256 * 256].view(g.torch.bfloat16)
    heads = mem.view(-1, 128).float()
    near = ((heads - want[0, :128]).abs().amax(1) < 0.1).nonzero().flatten().tolist()
    found = [mem[o * 128:o * 128 + want.numel()].view_as(want).float() for o in near if o * 128 + want.numel() <= mem.numel()]
    found = [u for u in found if float((u - want).abs().max()) < 0.1]
    assert len(found) == 1
    assert int((found[0] != want).sum()) == 0
