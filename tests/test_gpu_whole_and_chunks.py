"""A slide gives the same results whole and in chunks: which kernel takes a call depends on its number of rows, what a tile's
rows come to does not (needs an MI355X)."""
from dataclasses import replace

import numpy as np
import pytest

import gen

pytestmark = pytest.mark.gpu


def _slide(tiles):
    cfg = replace(gen.CONFIGS["small"][0], layers=2)   # ViT-S blocks
    ds, ws, ls = gen.SEEDS["small"]
    prm = {k: gen.to_bf16_grid(v) for k, v in gen.make_params(cfg, ws, perturbed=True).items()}
    return cfg, prm, gen.to_bf16_grid(gen.make_pixels(cfg, tiles, ds, workers=8)), gen.make_label(cfg, ls)


# 400 rows of the CLS lane take its 64 x 64 form with a LayerNorm launch, 200 the 32 x 32 form with the LayerNorm on the way in;
# 33 and 3 rows: one block of 32 rows and one row more, a few rows.  The last features go to an address that is a multiple of 4 only.
def test_features_by_either_form_of_the_cls_lane():
    import torch
    from slide_harness import GpuSlide
    cfg, prm, X, _ = _slide(436)
    print("case features 436 = 400 + 33 + 3, 200 + 200", flush=True)
    g = GpuSlide(cfg, prm, 1, 436)
    px = g.to_dev(X)

    def feats(lo, hi, shift=0):
        buf = torch.zeros((hi - lo) * cfg.dim + 4, device=g.dev)
        f = buf[shift:shift + (hi - lo) * cfg.dim].view(hi - lo, cfg.dim)
        g.lib.encoder_fwd_tiles(px[lo:hi], hi - lo, f, 0)
        torch.cuda.synchronize()
        return f.cpu().numpy()

    whole = feats(0, 400)
    assert np.isfinite(whole).all() and np.abs(whole).max() > 0.1
    assert np.array_equal(whole, np.concatenate([feats(0, 200), feats(200, 400, 1)]))
    assert np.array_equal(feats(400, 433), feats(400, 433, 1))
    assert np.array_equal(feats(433, 436), feats(433, 436, 1))


# From 4,096 rows on an encoder GEMM runs on 256 x 192 tiles or on smaller ones, whichever fill the chip, and 21 ViT-S tiles are
# 4,137 rows: both kernels take part on both sides here (and both forms of the CLS lane at 500).  Features and pixel gradients
# belong to one tile, so they have to agree to the last bit; the other gradients are the same terms added in another order.
@pytest.mark.parametrize("tiles,chunk", [(48, 24), (100, 26), (170, 43), (500, 300)])
def test_step_whole_and_in_chunks(tiles, chunk):
    from slide_harness import GpuSlide, rel_l2
    cfg, prm, X, label = _slide(tiles)
    print(f"case whole {tiles}, chunks of {chunk}", flush=True)
    g = GpuSlide(cfg, prm, 1, tiles)
    whole, parts = g.step(X, label), g.step_chunked(X, label, chunk)
    for k in ("H", "G", "dX"):
        assert np.isfinite(whole[k]).all() and np.abs(whole[k]).max() > 0
        assert np.array_equal(whole[k], parts[k]), (k, rel_l2(parts[k], whole[k]))
    errs = {k: rel_l2(parts["grads"][k], v) for k, v in whole["grads"].items()}
    print("worst:", sorted(errs.items(), key=lambda kv: -kv[1])[:4], flush=True)
    # float32 sums of n <= 98,500 terms in two orders: 2 sqrt(n) 2^-24 = 3.7e-5 of the terms' norm
    assert max(errs.values()) < 4e-5
