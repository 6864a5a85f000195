"""Group top-k on inputs whose scores are whole numbers (exact in float32), so the selected
blocks must equal the float64 oracle's bit for bit: many tied scores, keys that differ little
from a large common vector, equal keys (the filter is skipped and every block scored), zero
queries, one key far longer than the rest; every list width, block ratio and head dim of the
kernel, from one partly filled key tile to several, for bf16 layers and (head dim 32) float32
ones. Then scores that are equal in float32 only, and real values against float64 scores."""
import numpy as np
import pytest
import torch

from oracle import bsa as ob
from paper_2506_12541_amd import _lib, bsa as gb

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


@pytest.mark.parametrize("many", [False, True], ids=["listed", "overflow"])
@pytest.mark.parametrize("f32,d,g", [(False, 64, 16), (False, 32, 8), (False, 64, 1), (True, 32, 8)])
def test_equal_float32_scores_rank_by_block(f32, d, g, many):
    """Scores that differ by less than float32 holds rank by block index. Keys score 1 or
    1 + 2^-30, the larger ones in the higher blocks: every float32 sum of the products 1 and
    2^-30 is 1. `many`: all blocks tie so (candidate lists overflow), else k* + 4 of them."""
    n, m, l, ls, kk, B, H = 4096, 256, 16, 32, 8, 1, 2
    print(f"equal float32 scores f32={f32} d={d} g={g} many={many}", flush=True)
    nblk = n // ls
    tied = np.arange(nblk) if many else np.arange(nblk - 5 * (kk + 4), nblk, 5)
    k = np.zeros((nblk, d))
    k[:, 0] = 0.25
    k[tied, 0] = 1.0
    k[tied[len(tied) // 2:], 1] = 2.0 ** -30
    k = np.broadcast_to(np.repeat(k, ls, axis=0), (B, H, n, d))
    q = np.zeros((B, H, n, d))
    q[..., :2] = 1.0
    p = gb.Params(batch=B, n=n, heads=H, head_dim=d, ball_size=m, cmp_block=l, slc_block=ls, topk=kk, group_size=g,
                  kv_pool=gb.BSA_POOL_MEAN, dtype=gb.BSA_F32 if f32 else gb.BSA_BF16)
    qd, kd = (torch.from_numpy(np.ascontiguousarray(a)).to("cuda").to(p.torch_dtype) for a in (q, k))
    _, saved = gb.forward(p, qd, kd, kd, None, torch.zeros((B, n, 3), device="cuda"), None, None)
    score = np.full(nblk, 0.25)
    score[tied] = 1.0
    scores = np.broadcast_to(score, (n // g, nblk)).copy()
    scores[np.arange(n // g)[:, None] * g // m == np.arange(nblk)[None] * ls // m] = -np.inf
    want = ob.topk_blocks(scores, kk)
    for h in range(H):
        assert np.array_equal(saved.sel_idx[0, h].cpu().numpy(), want), h


@pytest.mark.parametrize("bad", [float("nan"), float("inf"), -float("inf")])
@pytest.mark.parametrize("shape,f32", [(SHAPES[1], False), (SHAPES[2], False), (SHAPES[4], False), (SHAPES[6], False),
                                       (SHAPES[3], True)],
                         ids=lambda s: "-".join(map(str, s)) if isinstance(s, tuple) else ("f32" if s else "bf16"))
def test_select_non_finite(shape, f32, bad):
    """A block with a value that is not finite in one of its keys is never selected, whatever the
    query, and a group whose pooled query is not finite selects nothing (products of three parts
    turn an infinity into NaN); every other group selects as the oracle does without that block."""
    n, m, l, ls, kk, g, d = shape
    print(f"select non-finite {shape} f32={f32} {bad}", flush=True)
    rng = np.random.default_rng([n, d, g])
    H, r = 2, ls // l
    q = rng.integers(-3, 4, (1, H, n, d)).astype(np.float64)
    kc = rng.integers(-1, 2, (H, n // l, d)).astype(np.float64)
    P = ob.Params(ball=m, cmp_block=l, slc_block=ls, topk=kk, group=g, kv_pool="mean")
    want, valid = [], np.ones(n, bool)
    blk, grp = [3, n // ls - 2], n // g // 2
    for h in range(H):
        scores = ob.group_block_scores(q[0, h], kc[h], valid, P)
        scores[:, blk] = -np.inf
        scores[grp] = -np.inf
        want.append(ob.topk_blocks(scores, kk))
    k = np.repeat(kc, l, axis=1)[None]
    k[:, :, blk[0] * ls, 5] = bad
    k[:, :, blk[1] * ls + (r - 1) * l, d - 1] = bad
    q[:, :, grp * g, 7] = bad
    p = gb.Params(batch=1, n=n, heads=H, head_dim=d, ball_size=m, cmp_block=l, slc_block=ls, topk=kk, group_size=g,
                  kv_pool=gb.BSA_POOL_MEAN, dtype=gb.BSA_F32 if f32 else gb.BSA_BF16)
    qd, kd = (torch.from_numpy(np.ascontiguousarray(a)).to("cuda").to(p.torch_dtype) for a in (q, k))
    _, saved = gb.forward(p, qd, kd, kd, None, torch.zeros((1, n, 3), device="cuda"), None, None)
    for h in range(H):
        assert np.array_equal(saved.sel_idx[0, h].cpu().numpy(), want[h]), h


# n, ball, l, l', k*, g, d
REAL = [
    (4096, 256, 8, 16, 8, 8, 32),
    (8192, 256, 16, 32, 16, 16, 64),
    (8192, 512, 16, 64, 16, 32, 64),
    (65536, 256, 16, 32, 16, 1, 64),
]


@pytest.mark.parametrize("kind", ["normal", "common", "far common", "binades", "cancel"])
@pytest.mark.parametrize("shape,f32", [(s, False) for s in REAL] + [(REAL[0], True)],
                         ids=lambda s: "-".join(map(str, s)) if isinstance(s, tuple) else ("f32" if s else "bf16"))
def test_select_real_values(shape, f32, kind):
    """Real-valued scores against float64 scores of the saved compressed keys and coarse queries:
    no block left out may score above a selected one by more than the two scores' float32 error.
    A score of six bf16 products errs by at most 2^-15 |q| times the sum of its keys' norms (224
    sums of at most |q||k|, each off by an ulp at most), over r for a block's mean. Keys: normal,
    with a common vector 20 and 1000 times their spread, of lengths over 40 binades, and with the
    keys of a block nearly cancelling."""
    n, m, l, ls, kk, g, d = shape
    print(f"select real {shape} f32={f32} {kind}", flush=True)
    gen = torch.Generator("cuda").manual_seed(n + d + len(kind))
    rn = lambda *s: torch.randn(s, generator=gen, device="cuda")
    B, H, r, nblk = 1, 2, ls // l, n // ls
    key = rn(B, H, n // l, d)
    if "common" in kind:
        key = key * (0.05 if kind == "common" else 0.001) + rn(B, H, 1, d)
    elif kind == "binades":
        key = key * torch.exp2(40 * torch.rand((B, H, n // l, 1), generator=gen, device="cuda") - 20)
    elif kind == "cancel":
        key = key * 0.01
        key[:, :, ::2] += 1.0
        key[:, :, 1::2] -= 1.0
    p = gb.Params(batch=B, n=n, heads=H, head_dim=d, ball_size=m, cmp_block=l, slc_block=ls, topk=kk, group_size=g,
                  kv_pool=gb.BSA_POOL_MEAN, dtype=gb.BSA_F32 if f32 else gb.BSA_BF16)
    k = key.repeat_interleave(l, 2).to(p.torch_dtype).contiguous()
    q = rn(B, H, n, d).to(p.torch_dtype)
    _, saved = gb.forward(p, q, k, k, None, torch.zeros((B, n, 3), device="cuda"), None, None)
    for h in range(H):
        kc, qc = saved.kcmp[0, h].double(), saved.qcmp[0, h].double()
        norms = kc.norm(dim=1).view(nblk, r).sum(1)
        for s in range(0, n // g, 8192):
            qs, sel = qc[s:s + 8192], saved.sel_idx[0, h, s:s + 8192].long()
            assert bool((sel >= 0).all()) and bool((sel[:, 1:] > sel[:, :-1]).all())
            sc = (qs @ kc.view(nblk, r, d).sum(1).t()) / r
            err = 2.0 ** -15 / r * qs.norm(dim=1, keepdim=True) * norms
            own = (torch.arange(s, s + qs.shape[0], device="cuda") * g // m)[:, None] == \
                (torch.arange(nblk, device="cuda") * ls // m)[None]
            taken = torch.zeros_like(own).scatter(1, sel, True)
            assert not bool((taken & own).any())
            worst = torch.where(taken, sc + err, torch.inf).amin(1)
            best_left = torch.where(taken | own, -torch.inf, sc - err).amax(1)
            assert bool((best_left <= worst).all()), (h, s, float((best_left - worst).max()))


def test_select_time_does_not_depend_on_a_common_key():
    """A component that all keys share shifts every score of a group alike: the selection takes
    the time it takes without it (bound: twice; it was over forty times when the filter's error
    bound followed the whole keys and every candidate list overflowed)."""
    p = gb.Params(batch=1, n=65536, heads=8, head_dim=64, ball_size=256, cmp_block=16, slc_block=32, topk=16,
                  group_size=16, kv_pool=gb.BSA_POOL_MEAN)
    gen = torch.Generator("cuda").manual_seed(3)
    rn = lambda *s: torch.randn(s, generator=gen, device="cuda")
    q, key, common = rn(1, 8, 65536, 64).bfloat16(), rn(1, 8, 4096, 64), rn(1, 8, 1, 64)
    gate = torch.zeros((1, 65536, 3), device="cuda")
    lib = _lib.load()
    ms, count = {}, _lib.C.c_int32()
    for scale in (0.0, 20.0):
        k = (key + scale * common).repeat_interleave(16, 2).bfloat16().contiguous()
        gb.forward(p, q, k, k, None, gate, None, None)
        times = []
        for _ in range(5):
            lib.bsa_timing_enable(1)
            gb.forward(p, q, k, k, None, gate, None, None)
            t = _lib.C.c_double()
            _lib.check(lib.bsa_timing_query(b"fwd.select", _lib.C.byref(t), _lib.C.byref(count)), "timing")
            times.append(t.value)
            lib.bsa_timing_enable(0)
        ms[scale] = min(times)
    print(f"select with and without a common key: {ms}", flush=True)
    assert ms[20.0] < 2 * ms[0.0], ms
