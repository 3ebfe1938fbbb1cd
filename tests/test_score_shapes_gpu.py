"""im_index_score on indexer keys that are given, at the sizes where it changes its form, against the oracle's functions on
the same keys: the scores must be the same fp32 numbers."""
import numpy as np
import pytest
import torch

import paper_2605_25475_amd as im
from helpers import f64
from oracle import indexmem_oracle as O

pytestmark = pytest.mark.gpu
BF = torch.bfloat16


def _check(shared, H, Hk, batch, n, n_q, mode="plain"):
    Hi, di, sets = H // 4, 16 if shared else 64, 1 if shared else Hk
    g = torch.Generator().manual_seed(1000 * n_q + n)
    rand = lambda *s: torch.randn(s, generator=g).to(BF)
    cfg = im.Config(batch=batch, n_q_heads=H, n_kv_heads=Hk, capacity=n + 3, n_idx_heads=Hi, idx_dim=di, gate_in_dim=128,
                    max_queries=n_q, head_shared=int(shared))
    h, st = im.Handle(cfg, "cuda"), im.State(cfg, "cuda")
    Uq, G, ones = (rand(Hi * di, H * 128).float() * 0.02).to(BF), rand(Hi, 128), torch.ones(di, dtype=BF)
    dev = lambda t: t.contiguous().cuda()
    keep = [dev(t) for t in (Uq, G, ones)]
    p = im.Params(keep[0], keep[1], keep[2], keep[2], keep[2], 0.0, keep[2], keep[2])
    keys, pos = rand(batch, sets, n, di), torch.stack([torch.randperm(n, generator=g) for _ in range(batch * sets)])
    pos = pos.view(batch, sets, n).to(torch.int32)
    q, xg = rand(batch, n_q, H, 128), rand(batch, n_q, 128)
    if mode == "equal-queries":
        q[:], xg[:] = q[:, :1].clone(), xg[:, :1].clone()
    # positions in no order: some queries see every key, some a part, some none
    qpos = torch.randint(-3, n + 2, (batch, n_q), generator=g, dtype=torch.int32)
    k0, q0, qpos0 = keys.clone(), q.clone(), qpos.clone()
    if mode == "non-finite":   # NaN features count as zeros (an infinity in a row makes its features NaN), a NaN gate's query not at all
        for i, bad in enumerate((float("inf"), -float("inf"), float("nan"))):
            t, s = (0, n // 2, n - 1)[i], (0, 5, n_q - 1)[i]
            keys[0, :, t], k0[0, :, t] = float("nan"), 0
            q[-1, s, i, 3 * i], q0[-1, s] = bad, 0
        xg[0, 2, 1], qpos0[0, 2] = float("nan"), -10 ** 6
    shape = lambda t: t.view((batch,) + tuple(t.shape[2:])) if shared else t
    st.Kidx[..., :n, :] = shape(dev(keys))
    st.pos[..., :n] = shape(dev(pos))
    st.len.fill_(n)
    st.n_projected.fill_(n)
    im.im_set_max_live(h, n)
    scores = torch.full(tuple(st.pos.shape), 7.0, device="cuda")
    im.im_index_score(h, p, st, dev(q), dev(xg), dev(qpos), scores)
    torch.cuda.synchronize()
    got = scores.view(batch, sets, n + 3)[..., :n].cpu().numpy().astype(np.float64)
    assert im.im_query_status(h) == 0 and bool((scores[..., n:] == 7.0).all())
    xg0 = torch.where(torch.isfinite(xg.float()), xg, torch.zeros_like(xg))
    for b in range(batch):
        qhat = O.query_feature(f64(q0[b]).reshape(n_q, -1), f64(Uq), f64(ones), Hi, di, float(np.float32(1e-6)))
        alpha = O.head_gate(f64(xg0[b]), f64(G), Hi, di)
        for u in range(sets):
            want = O.importance(qhat, alpha, qpos0[b].numpy(), f64(k0[b, u]), pos[b, u].numpy())
            wrong = int((got[b, u] != want).sum())
            assert wrong == 0, f"sequence {b}, set {u}: {wrong} of {n} scores differ"


SHORT = [   # windows that are scored in fp64: 16 keys per wave over short caches, groups of queries below 512 tiles of 256 keys
    (False, 32, 8, 1, 1, 16), (False, 32, 8, 2, 63, 17), (False, 32, 8, 1, 300, 64), (False, 28, 4, 1, 129, 128),
    (False, 64, 8, 1, 65, 33), (False, 32, 8, 4, 1025, 9), (False, 64, 8, 4, 1025, 16), (False, 16, 4, 8, 1100, 31),
    (False, 32, 8, 4, 1025, 31), (False, 28, 4, 16, 511, 32), (False, 32, 8, 4, 4097, 17),
    (True, 32, 8, 2, 64, 49), (True, 32, 8, 2, 257, 64), (True, 28, 4, 16, 2049, 33), (True, 64, 8, 16, 2100, 32),
    (True, 4, 4, 3, 70, 511),
]


@pytest.mark.parametrize("shared,H,Hk,batch,n,n_q", SHORT, ids=["-".join(map(str, c)) for c in SHORT])
def test_short_windows(shared, H, Hk, batch, n, n_q):
    for mode in ("plain", "equal-queries", "non-finite"):
        if mode != "non-finite" or (n >= 3 and n_q >= 7):
            _check(shared, H, Hk, batch, n, n_q, mode)


@pytest.mark.parametrize("H,n_q", [(4, 33000), (8, 16500)])
def test_many_queries_with_one_or_two_indexer_heads(H, n_q):
    # (their projection has 16 and 32 columns and more than 2048 tiles)
    _check(True, H, H, 1, 70, n_q)


# Past both thresholds of the form for large caches (from 128 tiles of 256 keys on a wave scans 64 keys instead of 16; above 32768
# keys it evaluates 16 instead of 4), one key around whole tiles.  Per unit 32 units of 1023 .. keys, head-shared 16
# sequences of 2047 .. keys: 32736 to 36000 keys.
LARGE = [(shared, H, n, n_q) for shared, ns in ((False, (1023, 1024, 1025, 1100)), (True, (2047, 2048, 2049, 2200)))
         for H in (32, 64) for n in ns for n_q in ((33,) if not shared else (81 if H == 32 else 49,))]


@pytest.mark.parametrize("shared,H,n,n_q", LARGE, ids=["-".join(map(str, c)) for c in LARGE])
def test_many_queries_over_large_caches(shared, H, n, n_q):
    for mode in ("plain", "equal-queries", "non-finite"):
        _check(shared, H, 8, 16 if shared else 4, n, n_q, mode)


@pytest.mark.parametrize("shared,H,n,n_q", [(False, 32, 1025, 140), (False, 64, 1100, 260), (True, 32, 2049, 300), (True, 64, 2200, 150)])
def test_query_groups_over_large_caches(shared, H, n, n_q):
    # more blocks of 16 queries than groups: records name one block of several
    for mode in ("plain", "equal-queries", "non-finite"):
        _check(shared, H, 8, 16 if shared else 4, n, n_q, mode)
