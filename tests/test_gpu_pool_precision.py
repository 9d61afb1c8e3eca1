"""Softmax weights of the aggregator's matrix-core forward to float32 (needs an MI355X)."""
import pytest

pytestmark = pytest.mark.gpu


# 256 gate units below 32,768 rows, where the shift of the softmax is the largest logit: fewer blocks of rows than workgroups, a last block
# of one row, several blocks per workgroup, the last row count of this path.  Features and weights on the bf16 grid, so that the gates'
# operands are exact.  Logits differ by 0.1 at most, so their own errors and that of the exponential's argument are a tenth of 2^-24; the
# exponential, the sum and the quotient are roundings of 2^-24 / sqrt(3) each: 2^-24 in all, and half of that to spare.
@pytest.mark.parametrize("rows", [4097, 8192, 16384 + 1, 32767])
def test_softmax_weights_of_256_gate_units(rows):
    import torch
    from paper_2403_04865_amd import SlideConfig, SlideLib
    D, Mh = 384, 256
    print(f"case softmax weights N={rows}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(3)
    lib = SlideLib(SlideConfig(224, 16, D, 0, D // 64, 4, Mh, 1, dtype=1))
    prm = (torch.randn(lib.slide_param_count(), device="cuda", generator=g).clamp_(-2, 2) * 0.02).bfloat16().float()
    H = (torch.randn(D, device="cuda", generator=g) + 0.25 * torch.randn((rows, D), device="cuda", generator=g)).bfloat16().float()
    alpha, loss, logits = torch.zeros(rows, device="cuda"), torch.zeros(1, device="cuda"), torch.zeros(1, device="cuda")
    p = {n: prm[o:o + l].double() for n, o, l in lib.param_layout()}
    h = H.double()
    a = (torch.tanh(h @ p["mil.V.W"].view(Mh, D).T + p["mil.V.b"])
         * torch.sigmoid(h @ p["mil.U.W"].view(Mh, D).T + p["mil.U.b"])) @ p["mil.w"]
    want = torch.softmax(a, 0)
    nbytes = lib.slide_pool_arena_bytes(rows)
    arena = torch.empty(nbytes + 256, dtype=torch.uint8, device="cuda")
    o = (-arena.data_ptr()) % 256
    lib.slide_bind(prm, torch.zeros_like(prm), arena[o:o + nbytes])
    for call in (lambda: lib.mil_pool_fwd(H, rows, 0, loss, logits, alpha),
                 lambda: lib.mil_pool_fwd_static(prm, H, rows, 0, loss, logits, alpha)):
        alpha.zero_()
        call()
        torch.cuda.synchronize()
        err = ((alpha.double() - want).norm() / want.norm()).item()
        print("error", err, "spread of the logits", (a.max() - a.min()).item(), flush=True)
        assert err < 1.5 * 2 ** -24
