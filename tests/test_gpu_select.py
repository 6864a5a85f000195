"""Group top-k on inputs whose scores are whole numbers (exact in float32), so the selected
blocks must equal the float64 oracle's bit for bit: many tied scores, keys that differ little
from a large common vector (candidate lists overflow and groups are scanned exactly), equal
keys, zero queries, one key far longer than the rest; every list width, block ratio and head
dim of the kernel, from one partly filled key tile to several, for bf16 layers and (head dim
32) the float32 layers' scores from bf16 parts."""
import numpy as np
import pytest
import torch

from oracle import bsa as ob
from paper_2506_12541_amd import bsa as gb

pytestmark = pytest.mark.gpu

# n, ball, l, l', k*, g, d
SHAPES = [
    (256, 64, 16, 16, 4, 16, 64),      # 16 compressed keys
    (1024, 64, 8, 16, 3, 8, 32),       # one full tile
    (2048, 128, 16, 64, 16, 16, 64),   # four keys per block
    (4096, 256, 8, 16, 8, 8, 32),      # several tiles
    (8192, 256, 16, 32, 16, 16, 64),
    (4096, 64, 16, 16, 16, 16, 32),    # one key per block
    (2048, 256, 16, 32, 13, 1, 64),    # per-token selection
]


def _keys(kind, rng, nc, d):
    k = rng.integers(-1, 2, (nc, d)).astype(np.float64)
    if kind == "common":
        k += 64
    elif kind == "equal":
        k[:] = k[0]
    elif kind == "outlier":
        k[nc // 3] *= 128
    return k


@pytest.mark.parametrize("padded", [False, True])
@pytest.mark.parametrize("kind", ["ties", "common", "equal", "zero_q", "outlier"])
@pytest.mark.parametrize("shape,f32", [(s, False) for s in SHAPES] + [(s, True) for s in SHAPES if s[-1] == 32],
                         ids=lambda s: "-".join(map(str, s)) if isinstance(s, tuple) else ("f32" if s else "bf16"))
def test_select_whole_numbers(shape, f32, kind, padded):
    n, m, l, ls, kk, g, d = shape
    print(f"select {shape} f32={f32} {kind} padded={padded}", flush=True)
    rng = np.random.default_rng([n, d, g, len(kind)])
    B, H = 2, 2
    q = rng.integers(-3, 4, (B, H, n, d)).astype(np.float64)
    if kind == "zero_q":
        q[:, :, : n // 2] = 0
    k = np.stack([[np.repeat(_keys(kind, rng, n // l, d), l, axis=0) for _ in range(H)] for _ in range(B)])
    valid = np.ones((B, n), bool)
    if padded:   # scattered dummies, and whole blocks and groups without a real token
        valid = rng.random((B, n)) < 0.8
        valid[:, n // 4:n // 4 + 4 * ls] = False
        valid[:, -max(ls, g):] = False
    p = gb.Params(batch=B, n=n, heads=H, head_dim=d, ball_size=m, cmp_block=l, slc_block=ls, topk=kk, group_size=g,
                  kv_pool=gb.BSA_POOL_MEAN, dtype=gb.BSA_F32 if f32 else gb.BSA_BF16)
    dev = lambda a, t: torch.from_numpy(a).to("cuda").to(t)
    qd, kd = dev(q, p.torch_dtype), dev(k, p.torch_dtype)
    gate = torch.zeros((B, n, 3), device="cuda")
    _, saved = gb.forward(p, qd, kd, kd, dev(valid, torch.uint8) if padded else None, gate, None, None)
    sel = saved.sel_idx.cpu().numpy()
    P = ob.Params(ball=m, cmp_block=l, slc_block=ls, topk=kk, group=g, kv_pool="mean")
    for b in range(B):
        for h in range(H):
            kc, _ = ob.compress(k[b, h], valid[b], None, P)
            scores = ob.group_block_scores(q[b, h], kc, valid[b], P)
            assert np.array_equal(sel[b, h], ob.topk_blocks(scores, kk)), (b, h)
