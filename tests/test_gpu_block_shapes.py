"""The block's products at the edges of their tile choice, against float64 products of the same
bfloat16 operands: shapes on both sides of the 64, 128 and 256 tiles (forward) and of the two
weight-gradient tiles with their splits. Q is compared with the rounded product of the stored
norm output, y with h plus the product of the stored SwiGLU output, the weight gradients with
sums over all tokens of operands recomputed in float64.

Bounds: an entry of a bfloat16 output differs by the float32 sum's error (below 2^-16 of the sum
of |terms|) and one rounding (2^-8 of the value); float32 outputs by the sum's error alone. dW2
sums bfloat16 operands exactly as stored: its error is the float32 sum's."""
import numpy as np
import pytest
import torch

from paper_2506_12541_amd import bsa as gb

pytestmark = pytest.mark.gpu

# batch, n, heads, d, F: tiles of the Q/K/V, output and SwiGLU products
CASES = [
    (1, 256, 4, 32, 128),      # 64 tiles everywhere, the smallest block
    (1, 1024, 8, 64, 384),     # 64 tiles, F not a multiple of 256
    (2, 2048, 8, 64, 2048),    # 128 tiles for Q/K/V and SwiGLU, 64 for the others
    (3, 4096, 4, 32, 640),     # 12288 rows of 128 channels: weight gradients of one small tile
    (4, 4096, 8, 64, 1152),    # 256 tiles for Q/K/V and SwiGLU, 128 for the others
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
def test_block_products(case):
    B, n, H, d, F = case
    C, M = H * d, B * n
    print(f"block products {case}", flush=True)
    gen = torch.Generator("cuda").manual_seed(n + F)
    rn = lambda *s: torch.randn(s, generator=gen, device="cuda")
    l = 8 if d == 32 else 16
    p = gb.Params(batch=B, n=n, heads=H, head_dim=d, ball_size=256, cmp_block=l, slc_block=2 * l, topk=4, group_size=l)
    W = {"g1": 1 + 0.1 * rn(C), "wqkv": rn(3 * C, C) / C ** 0.5, "wg": rn(3, C) / C ** 0.5, "wo": rn(C, C) / C ** 0.5,
         "g2": 1 + 0.1 * rn(C), "w1": rn(F, C) / C ** 0.5, "w3": rn(F, C) / C ** 0.5, "w2": rn(C, F) / F ** 0.5}
    phi = [{"w1": (0.02 * rn(l * d, d)).bfloat16().float(), "b1": 0.02 * rn(d), "w2": 0.02 * rn(d, d), "b2": 0.02 * rn(d)}
           for _ in range(2)]
    x, dy = rn(B, n, C), rn(B, n, C)
    y, sv = gb.block_forward(p, F, W, *phi, x)
    g = gb.block_backward(p, F, W, *phi, x, sv, dy)
    r64 = lambda t: t.bfloat16().double()

    def near(got, ref, mag, ulp):
        err = (got.double() - ref).abs()
        assert bool((err <= 2.0 ** -16 * mag + ulp * ref.abs()).all()), float((err / (mag + ref.abs())).max())

    merge = lambda t: t.transpose(1, 2).reshape(M, C)
    xn1, xn2, a, h = sv.xn1.double().view(M, C), sv.xn2.double().view(M, C), sv.a.double().view(M, F), sv.h.double().view(M, C)
    wq, wo, w1, w3, w2 = (r64(W[k]) for k in ("wqkv", "wo", "w1", "w3", "w2"))
    ref, mag = xn1 @ wq.t(), xn1.abs() @ wq.abs().t()
    for i, t in enumerate((sv.q, sv.k, sv.v)):
        near(merge(t), ref[:, i * C:(i + 1) * C], mag[:, i * C:(i + 1) * C], 2.0 ** -8)
    o = merge(sv.o).double()
    near(sv.h.view(M, C), x.double().view(M, C) + o @ wo.t(), x.double().view(M, C).abs() + o.abs() @ wo.abs().t(), 0)
    uw = sv.uw.view(M, 2 * F)
    near(uw[:, :F], xn2 @ w1.t(), xn2.abs() @ w1.abs().t(), 2.0 ** -8)
    near(uw[:, F:], xn2 @ w3.t(), xn2.abs() @ w3.abs().t(), 2.0 ** -8)
    u, w = uw[:, :F].double(), uw[:, F:].double()
    near(sv.a.view(M, F), torch.nn.functional.silu(u) * w, torch.zeros_like(u), 2.0 ** -8 + 2.0 ** -16)
    near(y.view(M, C), h + a @ w2.t(), h.abs() + a.abs() @ w2.abs().t(), 0)
    # backward of the SwiGLU sublayer: dy rounded, du and dw rounded
    dyr = r64(dy.view(M, C))
    near(g["dW"]["w2"], dyr.t() @ a, dyr.abs().t() @ a.abs(), 0)
    da, s = dyr @ w2, torch.sigmoid(u)
    du, dw = r64((da * w * s * (1 + u * (1 - s))).float()), r64((da * u * s).float())
    # a rounding of du (dw) may fall the other way: one more bfloat16 step of every term
    for name, t in (("w1", du), ("w3", dw)):
        ref, mag = t.t() @ xn2, t.abs().t() @ xn2.abs()
        err = (g["dW"][name].double() - ref).abs()
        assert bool((err <= (2.0 ** -16 + 2.0 ** -8) * mag).all()), name
        assert float(err.norm() / ref.norm()) < 1e-3, name
    assert np.isfinite(float(g["dx"].double().norm()))


def test_swiglu_far_negative():
    """silu(u) w for u down to about -200, where exp(-u) leaves float32's range: within one
    bfloat16 rounding and float32's relative error, except where sigmoid(u) is below float32's
    smallest normal number 2^-126 (that times |u w|, below 2^15 here)."""
    B, n, H, d, F = 1, 256, 4, 32, 128
    C, l = H * d, 8
    print("swiglu far negative", flush=True)
    gen = torch.Generator("cuda").manual_seed(11)
    rn = lambda *s: torch.randn(s, generator=gen, device="cuda")
    p = gb.Params(batch=B, n=n, heads=H, head_dim=d, ball_size=256, cmp_block=l, slc_block=2 * l, topk=4, group_size=l,
                  kv_pool=gb.BSA_POOL_MEAN)
    W = {"g1": 1 + 0.1 * rn(C), "wqkv": rn(3 * C, C) / C ** 0.5, "wg": rn(3, C) / C ** 0.5, "wo": rn(C, C) / C ** 0.5,
         "g2": 1 + 0.1 * rn(C), "w1": 50 * rn(F, C) / C ** 0.5, "w3": rn(F, C) / C ** 0.5, "w2": rn(C, F) / F ** 0.5}
    phi = {"w1": rn(l * d, d), "b1": rn(d), "w2": rn(d, d), "b2": rn(d)}
    _, sv = gb.block_forward(p, F, W, phi, phi, rn(B, n, C))
    uw = sv.uw.view(B * n, 2 * F).double()
    u, w = uw[:, :F], uw[:, F:]
    assert float(u.min()) < -100 and float((u * w).abs().max()) < 2.0 ** 15
    ref = torch.nn.functional.silu(u) * w
    err = (sv.a.view(B * n, F).double() - ref).abs()
    assert bool((err <= (2.0 ** -8 + 2.0 ** -16) * ref.abs() + 2.0 ** -111).all()), float(err[u < -80].max())
