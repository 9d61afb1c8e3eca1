"""Aggregator over long bags where its kernels change: the float32 gate gradients and G as bf16 terms (pool_f32.hip), the forward whose
weights stream (pool_mfma.hip), against float64 (needs an MI355X)."""
import pytest

pytestmark = pytest.mark.gpu


def _step(D, Mh, N, dtype, C=1, w_inf=False, seed=7):
    import torch
    from paper_2403_04865_amd import SlideConfig, SlideLib
    print(f"case long bag D={D} Mh={Mh} N={N} C={C} dtype={dtype} inf={w_inf}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(seed)
    lib = SlideLib(SlideConfig(32, 16, D, 0, D // 64, 4, Mh, C, dtype=dtype))
    layout = lib.param_layout()
    prm = torch.randn(lib.slide_param_count(), device="cuda", generator=g) * 0.06
    at = {n: (o, l) for n, o, l in layout if n.startswith(("mil.", "head."))}
    if w_inf:   # a gate unit that is saturated for every row: t = +-1, its own gradient zero, the others' as they were
        o, _ = at["mil.V.W"]
        prm[o + 3 * D:o + 4 * D] = 0.0
        prm[o + 3 * D + 5] = float("inf")
    H = torch.randn(D, device="cuda", generator=g) + 0.25 * torch.randn((N, D), device="cuda", generator=g)
    H[:, 5] = H[:, 5].abs() + 0.01
    grads, G, alpha = torch.zeros_like(prm), torch.zeros_like(H), torch.zeros(N, device="cuda")
    loss, logits = torch.zeros(1, device="cuda"), torch.zeros(C, device="cuda")
    nbytes = lib.slide_pool_arena_bytes(N)
    arena = torch.empty(nbytes + 256, dtype=torch.uint8, device="cuda")
    o = (-arena.data_ptr()) % 256
    lib.slide_bind(prm, grads, arena[o:o + nbytes])
    lib.mil_pool_fwd(H, N, 0, loss, logits, alpha)
    lib.mil_pool_bwd(H, N, 0, G, 0)
    torch.cuda.synchronize()
    p = {n: prm[o:o + l].double().requires_grad_(True) for n, (o, l) in at.items()}
    h = H.double().requires_grad_(True)
    a = (torch.tanh(h @ p["mil.V.W"].view(Mh, D).T + p["mil.V.b"])
         * torch.sigmoid(h @ p["mil.U.W"].view(Mh, D).T + p["mil.U.b"])) @ p["mil.w"]
    al = torch.softmax(a, 0)
    y = p["head.W"].view(C, D) @ (al @ h) + p["head.b"]
    ref = torch.nn.functional.softplus(y[0]) if C == 1 else -torch.log_softmax(y, 0)[0]
    ref.backward()
    pairs = {n: (grads[o:o + l].double(), p[n].grad) for n, (o, l) in at.items()}
    pairs["G"] = (G.double(), h.grad)
    pairs["alpha"] = (alpha.double(), al.detach())
    pairs["loss"] = (loss[0].double(), ref.detach())
    return pairs


def _rel(x, r):
    return ((x - r).norm() / r.norm()).item()


# The backward goes by tiles where the gates make more than 128 of 64 rows x 64 units: the row count just below and just above (a last panel of
# one row), last panels of 33 and 63 rows and none short, and widths that leave the last 128 features of G short (D = 192).
# Tolerance: the bound of every float32 parity test.
@pytest.mark.parametrize("D,Mh,N", [(768, 128, 4096), (768, 128, 4097), (768, 256, 4096 + 33), (192, 64, 16384 + 63), (384, 192, 6016)])
def test_float32_gradients_of_long_bags(D, Mh, N):
    errs = {n: _rel(*v) for n, v in _step(D, Mh, N, 0, C=3).items()}
    print(errs, flush=True)
    assert all(e < 1e-4 for e in errs.values()), errs


# A weight that is infinite has no bf16 terms: such blocks are taken in float32 products, and only its own feature column of G has no number
def test_float32_gradients_with_an_infinite_weight():
    import torch
    pairs = _step(192, 64, 16384 + 5, 0, w_inf=True)
    for n, (x, r) in pairs.items():
        same = torch.isfinite(r)
        assert torch.equal(torch.isfinite(x), same), n
        assert _rel(x[same], r[same]) < 1e-4, n


# Forward with streaming weights: one block, blocks with a last row of one, one and two rounds of workgroups, a ragged end.  Tolerance: the bound
# of every bf16 parity test (the gates' operands are rounded to bf16).
@pytest.mark.parametrize("Mh,N", [(128, 512), (128, 16384 + 1), (256, 8192 + 31), (256, 40000)])
def test_streaming_forward(Mh, N):
    errs = {n: _rel(*v) for n, v in _step(768, Mh, N, 1).items()}
    print(errs, flush=True)
    assert all(e < 2e-2 for e in errs.values()), errs
