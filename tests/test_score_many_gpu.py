"""im_index_score with at least as many queries as indexer heads: bounds of all pairs on the fp16 matrix cores, fp64
for the pairs that can be a key's maximum (short windows: fp64 for all pairs).  The scores must be the oracle's fp32
numbers bit for bit, at the edges of the tiles of the form for small caches (16 queries, 64 keys) and where the
bounds decide nothing: equal queries, gates of zero, and values outside the range in which bounds are formed.
(Large caches: test_score_shapes_gpu.py.)"""
import numpy as np
import pytest
import torch

import paper_2605_25475_amd as im
from helpers import f64
from parity import LockStep, LockStepShared
from workloads import WORKLOADS

pytestmark = pytest.mark.gpu


def _scaled(**factors):
    def mod(p):
        for name, f in factors.items():
            p[name] = (p[name].float() * f).to(torch.bfloat16)
    return mod


MODES = {
    "plain": {},
    "equal-queries": {},                                            # every query is a candidate of every key
    "zero-gates": dict(params_mod=_scaled(G=0.0)),                  # every score is 0
    "tiny-gates": dict(params_mod=_scaled(G=2.0 ** -100)),          # no bound is formed: everything in fp64
    "large-norm-weights": dict(params_mod=_scaled(norm_q_w=2.0 ** 20, norm_k_w=2.0 ** 20)),
    "small-norm-weights": dict(params_mod=_scaled(norm_q_w=2.0 ** -20, norm_k_w=2.0 ** -20)),
}


@pytest.mark.parametrize("mode", sorted(MODES))
@pytest.mark.parametrize("heads", [(32, 8), (28, 4), (64, 8)], ids=["8", "7", "16"])   # indexer heads
@pytest.mark.parametrize("shared", [False, True], ids=["per-unit", "head-shared"])
def test_scores_of_many_queries_are_the_oracles(mode, heads, shared):
    for n_q, n in ((16, 1), (17, 63), (31, 64), (32, 65), (33, 257), (140, 300)):
        kw = dict(context=n, budget=n, decode_steps=n_q, batch=2, n_layers=1, n_q_heads=heads[0], n_kv_heads=heads[1])
        w = WORKLOADS["cfg1"].shared(**kw) if shared else WORKLOADS["cfg1"].scaled(**kw)
        cls, args = (LockStepShared, {}) if shared else (LockStep, dict(max_queries=n_q))
        if shared:   # (its handle takes at most `context` queries)
            w = w.scaled(context=max(n, n_q), decode_steps=0)
        ls = cls(w, capacity=max(n, n_q), **args, **MODES[mode])
        g, ref, d = ls.gpu, ls.ref, (lambda t: t.cuda())
        k, v = ls.K[:, :, :n].contiguous(), ls.V[:, :, :n].contiguous()
        pos = torch.arange(n, dtype=torch.int32).repeat(w.batch, 1).contiguous()
        q = ls.Q[:, -n_q:].contiguous()
        if mode == "equal-queries":
            q[:] = q[:, :1].clone()
        # positions in no order: some queries see every key, some a part, some none
        rng = np.random.default_rng(n_q * 1000 + n)
        qpos = torch.tensor(rng.integers(-3, n + 2, (w.batch, n_q)), dtype=torch.int32)
        if shared:
            x = ls.X[:, :n].contiguous()
            im.im_append_kv_hidden(ls.handle, ls.params, g.st, d(k), d(v), d(x), d(pos))
            ref.append_kv_hidden(f64(k), f64(v), f64(x), pos.numpy())
        else:
            im.im_append_kv(ls.handle, g.st, d(k), d(v), d(pos))
            ref.append_kv(f64(k), f64(v), pos.numpy())
        im.im_set_max_live(ls.handle, n)
        xg = q.view(w.batch, n_q, -1)
        im.im_index_score(ls.handle, ls.params, g.st, d(q), d(xg), d(qpos), g.scores)
        torch.cuda.synchronize()
        want = ref.index_score(f64(q), f64(xg), qpos.numpy())[..., :n]
        got = g.scores[..., :n].cpu().numpy().astype(np.float64)
        same = (got == want) | (np.isneginf(got) & np.isneginf(want))
        assert same.all(), f"{n_q} queries, {n} keys: {int((~same).sum())} of {same.size} scores differ"
        assert im.im_query_status(ls.handle) == 0


def _shrink(t, share, seed):
    """A share of the values becomes 2^-26 of its size: 22 bits below a row's largest value is where the exact
    product's integers end, and what they lose is added from lists."""
    g = torch.Generator().manual_seed(seed)
    small = torch.rand(t.shape, generator=g) < share
    return torch.where(small, (t.float() * 2.0 ** -26).to(torch.bfloat16), t)


# (a row lists 8 values at most: 1 to 2 a row stay below that, 8 a row put most tiles on the fp64 cores)
@pytest.mark.parametrize("share_q,share_u", [(0.0, 0.0), (0.0003, 0.0), (0.0, 0.0003), (0.0003, 0.0003), (0.002, 0.0), (0.002, 0.0005),
                                             (0.0, 0.01), (0.05, 0.0)],
                         ids=["plain", "few-q", "few-u", "few-both", "lists-q", "lists-both", "overflow-u", "overflow-q"])
@pytest.mark.parametrize("heads,n_q,shared", [((32, 8), 1089, False), ((28, 4), 1207, False), ((32, 8), 2081, True),
                                              ((24, 8), 701, False), ((40, 8), 430, False), ((64, 8), 270, False),
                                              ((26, 13), 700, False)],
                         ids=["512", "448", "128", "384", "640", "1024", "384-k3328"])   # columns of the query projection
def test_query_projection_as_an_exact_product(heads, n_q, shared, share_q, share_u):
    # row counts that are no multiple of the product's 64-row tiles; 448 columns are no multiple of its 128
    n = 40
    kw = dict(context=n_q, budget=n, decode_steps=0, batch=2, n_layers=1, n_q_heads=heads[0], n_kv_heads=heads[1])
    w = WORKLOADS["cfg1"].shared(**kw) if shared else WORKLOADS["cfg1"].scaled(**kw)

    def mod(p):
        p["Uq"] = _shrink(p["Uq"], share_u, 5)
    ls = (LockStepShared if shared else LockStep)(w, params_mod=mod)
    g, ref, d = ls.gpu, ls.ref, (lambda t: t.cuda())
    k, v = ls.K[:, :, :n].contiguous(), ls.V[:, :, :n].contiguous()
    pos = torch.arange(n, dtype=torch.int32).repeat(w.batch, 1).contiguous()
    q = _shrink(ls.Q.contiguous(), share_q, 6)
    qpos = torch.arange(n_q, dtype=torch.int32).repeat(w.batch, 1).contiguous() % (n + 3)
    if shared:
        x = ls.X[:, :n].contiguous()
        im.im_append_kv_hidden(ls.handle, ls.params, g.st, d(k), d(v), d(x), d(pos))
        ref.append_kv_hidden(f64(k), f64(v), f64(x), pos.numpy())
    else:
        im.im_append_kv(ls.handle, g.st, d(k), d(v), d(pos))
        ref.append_kv(f64(k), f64(v), pos.numpy())
    im.im_set_max_live(ls.handle, n)
    want = ref.index_score(f64(q), f64(q.view(w.batch, n_q, -1)), qpos.numpy())[..., :n]
    for _ in range(2):   # the second call finds the first one's lists
        g.scores.fill_(float("nan"))
        im.im_index_score(ls.handle, ls.params, g.st, d(q), d(q).view(w.batch, n_q, -1), d(qpos), g.scores)
        torch.cuda.synchronize()
        got = g.scores[..., :n].cpu().numpy().astype(np.float64)
        assert np.array_equal(got, want), f"{int((got != want).sum())} of {want.size} scores differ"


@pytest.mark.parametrize("n_q,n", [(33, 300), (1089, 70)], ids=["fp64-projection", "exact-product"])
@pytest.mark.parametrize("shared", [False, True], ids=["per-unit", "head-shared"])
def test_infinities_and_nan_count_as_no_similarity(shared, n_q, n):
    """A non-finite row has NaN features; ReLU takes a NaN similarity as 0, so a query or key with one scores like a
    row of zeros (which the oracle gets), and a query whose gates are NaN counts for no key."""
    kw = dict(context=max(n, n_q), budget=n, decode_steps=0, batch=2, n_layers=1)
    w = WORKLOADS["cfg1"].shared(**kw) if shared else WORKLOADS["cfg1"].scaled(**kw)
    ls = (LockStepShared if shared else LockStep)(w)
    g, ref, d = ls.gpu, ls.ref, (lambda t: t.cuda())
    k, v = ls.K[:, :, :n].contiguous(), ls.V[:, :, :n].contiguous()
    pos = torch.arange(n, dtype=torch.int32).repeat(w.batch, 1).contiguous()
    q = ls.Q[:, :n_q].contiguous()
    xg = q.view(w.batch, n_q, -1).clone()
    qpos = (torch.arange(n_q, dtype=torch.int32) % (n + 3)).repeat(w.batch, 1).contiguous()
    inf, nan = float("inf"), float("nan")
    bad = torch.tensor([inf, -inf, nan], dtype=torch.bfloat16)
    q0, k0, qpos0 = q.clone(), k.clone(), qpos.clone()
    for i, s in enumerate((0, 7, n_q - 1)):
        q[0, s, i, 5 * i] = bad[i]
        q0[0, s] = 0
    for i, t in enumerate((0, 31, n - 1)):
        k[1, :, t, 9 * i] = bad[i]
        k0[1, :, t] = 0
    xg0 = xg.clone()
    xg[1, 3, 0] = nan
    xg0[1, 3] = 0
    qpos0[1, 3] = -10 ** 6
    if shared:   # (indexer keys come from the hidden state)
        x = ls.X[:, :n].contiguous()
        x0 = x.clone()
        for i, t in enumerate((0, 31, n - 1)):
            x[1, t, 9 * i] = bad[i]
            x0[1, t] = 0
        im.im_append_kv_hidden(ls.handle, ls.params, g.st, d(k), d(v), d(x), d(pos))
        ref.append_kv_hidden(f64(k0), f64(v), f64(x0), pos.numpy())
    else:
        im.im_append_kv(ls.handle, g.st, d(k), d(v), d(pos))
        ref.append_kv(f64(k0), f64(v), pos.numpy())
    im.im_set_max_live(ls.handle, n)
    want = ref.index_score(f64(q0), f64(xg0), qpos0.numpy())[..., :n]
    for _ in range(2):
        g.scores.fill_(7.0)
        im.im_index_score(ls.handle, ls.params, g.st, d(q), d(xg), d(qpos), g.scores)
        torch.cuda.synchronize()
        got = g.scores[..., :n].cpu().numpy().astype(np.float64)
        assert np.array_equal(got, want), f"{int((got != want).sum())} of {want.size} scores differ"


@pytest.mark.parametrize("call", ["steps", "attend"])
def test_an_infinity_in_a_value_row_reaches_the_output_as_one(call):
    """P enters the product P V in three parts; a part that is zero times an infinity is not what P times it is."""
    w = WORKLOADS["cfg1"].scaled(context=200, budget=200, decode_steps=1, batch=1, n_layers=1)
    ls = LockStep(w, capacity=256)
    d = lambda t: t.contiguous().cuda()
    v = ls.V[:, :, :200].clone()
    v[0, 0, 17, 3], v[0, 1, 150, 64] = float("inf"), -float("inf")
    pos = torch.arange(201, dtype=torch.int32).repeat(1, 1)
    im.im_append_kv(ls.handle, ls.gpu.st, d(ls.K[:, :, :200]), d(v), d(pos[:, :200]))
    out = torch.zeros((1, w.n_q_heads, 128), dtype=torch.bfloat16, device="cuda")
    if call == "steps":
        im.im_decode_attn_with_readout(ls.handle, ls.params, ls.gpu.st, d(ls.Q[:, 200]), out)
    else:
        im.im_attend_step(ls.handle, ls.params, ls.gpu.st, d(ls.Q[:, 200]), d(ls.K[:, :, 200:]), d(ls.V[:, :, 200:]),
                          d(pos[0, 200:]), out)
    torch.cuda.synchronize()
    got = out.float().cpu().view(w.n_kv_heads, -1, 128)
    want = torch.zeros_like(got)
    want[0, :, 3], want[1, :, 64] = float("inf"), -float("inf")
    assert torch.equal(torch.where(torch.isfinite(got), torch.zeros_like(got), got), want)
