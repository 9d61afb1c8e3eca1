"""MLP half of a block as one kernel: the same bits as the two GEMM launches, on both sides of the lines that pick it.

On 256 compute units its 128-row workgroups come in rounds of 256.  The kernel is taken where the last round leaves at most 0.42
of the units idle over all rounds (backward 0.35): forwards that no backward follows from 149 workgroups on but for 257 to 296, backwards
from 167 on but for 257 to 332.  Otherwise, and in a step's own forward, two GEMMs run.  A step in chunks runs both kinds of forward, so
what belongs to one tile has to agree with the whole step to the last bit; parameter gradients are the same terms added in another
order."""
import numpy as np
import pytest
import torch

from paper_2403_04865_amd import SlideConfig, SlideLib

pytestmark = pytest.mark.gpu


def _run(n, chunk, recompute, ratio, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    lib = SlideLib(SlideConfig(224, 16, 384, 2, 6, ratio, 128, 1, dtype=1, recompute=recompute))
    p = torch.randn(lib.slide_param_count(), device="cuda", generator=g).clamp_(-2, 2).mul_(0.05)
    for name, off, length in lib.param_layout():
        if name.endswith(".g"):
            p[off:off + length] += 1.0
    x = torch.randn((n, 3, 224, 224), device="cuda", generator=g).to(torch.bfloat16)
    grads, dpix = torch.zeros_like(p), torch.zeros_like(x)
    loss, logits, alpha = (torch.zeros(k, device="cuda") for k in (1, 1, n))
    nbytes = lib.slide_chunked_arena_bytes(n, chunk) if chunk else lib.slide_arena_bytes(n)
    arena = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    lib.slide_bind(p, grads, arena)
    if chunk:
        lib.slide_step_chunked(x, n, chunk, 1, 0, loss, logits, alpha, dpix)
    else:
        lib.slide_step_fwd(x, n, 1, loss, logits, alpha)
        lib.slide_step_bwd(0, dpix)
    torch.cuda.synchronize()
    return [t.float().cpu().numpy() for t in (loss, logits, alpha, dpix, grads)]


# 197 rows per tile.  97 tiles: 150 workgroups, the first count above the forward's line (a ragged last one); 109: 168, above the
# backward's; 130: 201, with chunks below both lines; 167: 258, a round and two, where neither takes it, in chunks of which it takes
# some; 193 and 217: 298 and 334, the second round full enough for the forward and for both; 333: 513, a third round of one workgroup,
# in chunks of 167 and 166 tiles (258 and 256 workgroups) and of 84 and 81, which it does not take.
# MLP ratios 1, 2 and 3: 6, 12 and 18 steps of 64 hidden columns instead of 24.
@pytest.mark.parametrize("n,chunk,recompute,ratio", [
    (97, 49, 0, 4), (109, 55, 0, 4), (130, 65, 1, 4), (167, 84, 0, 4), (167, 97, 1, 4), (193, 97, 1, 4), (217, 109, 1, 4),
    (333, 167, 1, 4), (333, 84, 1, 4),
    (97, 49, 1, 1), (333, 84, 0, 1), (333, 84, 1, 2), (217, 109, 1, 3)])
def test_same_bits_as_two_launches(n, chunk, recompute, ratio):
    print(f"case {n} tiles, chunks of {chunk}, recompute {recompute}, ratio {ratio}", flush=True)
    whole, parts = _run(n, 0, recompute, ratio, n), _run(n, chunk, recompute, ratio, n)
    for a, b in zip(whole[:4], parts[:4]):
        assert np.isfinite(a).all() and np.abs(a).max() > 0
        np.testing.assert_array_equal(a, b)
    # float32 sums of at most 66,000 terms in two orders: 2 sqrt(n) 2^-24 = 3.1e-5 of the terms' norm
    assert np.linalg.norm(whole[4] - parts[4]) <= 3.1e-5 * np.linalg.norm(whole[4])
