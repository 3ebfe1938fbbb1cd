"""The launches of the fused decode step where their split of the work changes: query heads per workgroup of the last
launch, 16-key tiles per wave of the scoring launch, and an evicted entry whose share of the attention sums does not
come out by subtraction."""
import numpy as np
import pytest
import torch

import paper_2605_25475_amd as im
from parity import LockStep, LockStepShared, assert_out_close, assert_state_close
from helpers import f64
from workloads import WORKLOADS

pytestmark = pytest.mark.gpu


def _run(shared, batch, hq, hkv, context, budget, n_recent=0):
    """One prompt eviction and three decode steps; of a large batch the oracle follows the first and last sequence."""
    w = WORKLOADS["cfg1"].scaled(n_layers=1, batch=batch, n_q_heads=hq, n_kv_heads=hkv, context=context, budget=budget,
                                 decode_steps=3, n_recent=n_recent)
    few = dict(batch_ids=[0, batch - 1]) if batch > 4 else {}
    if shared:
        LockStepShared(w.shared(), **few).run_schedule(fused_decode=True)
    else:
        LockStep(w, **few).run_schedule(fused_decode=True)


@pytest.mark.parametrize("shared", [False, True])
@pytest.mark.parametrize("batch,hq,hkv", [(16, 28, 4), (16, 64, 8), (40, 64, 8), (3, 8, 8), (33, 32, 8)],
                         ids=["2-heads", "4-heads", "8-heads", "group-1", "units-264"])
def test_query_heads_per_workgroup(shared, batch, hq, hkv):
    _run(shared, batch, hq, hkv, 45, 20)


@pytest.mark.parametrize("batch,hq,hkv,budget", [
    (1, 32, 8, 15), (1, 32, 8, 16), (1, 32, 8, 127), (1, 32, 8, 128),   # one tile a wave; splits and tiles that end at the new token
    (2, 32, 8, 1030), (2, 16, 4, 2070), (1, 64, 8, 2064),
    (4, 32, 8, 1056), (8, 16, 4, 1100), (2, 64, 8, 2100),               # two tiles (more than 1536 in all)
    (4, 32, 8, 1535), (4, 32, 8, 1536),                                 # two and four (more than 3072)
    (1, 40, 8, 3071), (1, 40, 8, 3072), (1, 36, 6, 4190), (2, 64, 8, 3100)])   # more than 8 indexer heads: one and two
def test_tiles_per_scoring_wave(batch, hq, hkv, budget):
    _run(False, batch, hq, hkv, budget + 7, budget, n_recent=3 if budget > 16 else 0)


@pytest.mark.parametrize("budget", [64, 127, 2047, 2048, 4100])
def test_tiles_per_scoring_wave_head_shared(budget):
    _run(True, 2, 32, 8, budget + 5, budget)


@pytest.mark.parametrize("batch,hq,hkv,budget", [
    (2, 32, 8, 15), (2, 32, 8, 31), (2, 32, 8, 32), (2, 64, 8, 2048),   # two tiles a wave: the new token first and last of a wave's keys
    (64, 32, 8, 783), (64, 32, 8, 784), (64, 64, 8, 784)])              # four (more than 3072 in all), the new token last and first of a tile
def test_new_token_in_a_scoring_wave_head_shared(batch, hq, hkv, budget):
    _run(True, batch, hq, hkv, budget + 5, budget, n_recent=3 if budget > 16 else 0)


@pytest.mark.parametrize("hq,hkv,n", [(16, 2, 8193), (8, 1, 9000)])
def test_more_than_64_splits(hq, hkv, n):
    """Decode steps and one step that only attends, with more splits than a wave has lanes (and more last-ranked entries than it looks at first)."""
    steps = 3
    w = WORKLOADS["cfg1"].scaled(n_layers=1, batch=1, n_q_heads=hq, n_kv_heads=hkv, context=n, budget=n, decode_steps=steps)
    ls = LockStep(w, capacity=n + 1, max_queries=4)
    d = lambda t: t.contiguous().to("cuda")
    pos = torch.arange(n + steps, dtype=torch.int32).view(1, -1)
    k, v, q, win, last = ls.K[:, :, :n], ls.V[:, :, :n], ls.Q[:, n - 4:n], slice(n - 4, n), ls.Q[:, n - 1]
    ls.gpu.step(d(k), d(v), d(pos[:, :n]), d(q), d(q).view(1, 4, -1), d(pos[:, win]), d(last), n, w.lam, w.eta)
    ls.ref.step(f64(k), f64(v), pos[:, :n].numpy(), f64(q), f64(q).reshape(1, 4, -1), pos[:, win].numpy(), f64(last), n, w.lam, w.eta)
    im.im_set_max_live(ls.handle, n + 1)
    for t in range(n, n + steps - 1):
        ls.event_fused(t, n, f"decode@{t}")
    t = n + steps - 1
    new = [ls.K[:, :, t:t + 1], ls.V[:, :, t:t + 1], pos[:, t:t + 1]]
    ls.gpu.attend_step(*(d(x) for x in new), d(ls.Q[:, t]))
    ls.ref.append_kv(f64(new[0]), f64(new[1]), new[2].numpy())
    out, res = ls.ref.decode_attn_with_readout(f64(ls.Q[:, t]))
    torch.cuda.synchronize()
    ls.compare(None, None, None, out, res, f"attend@{t}", lists=False)
    assert im.im_query_status(ls.handle) == 0


@pytest.mark.parametrize("what", ["plain", "all-the-weight", "large-value", "last-entry"])
@pytest.mark.parametrize("n", [40, 129, 300])
def test_evicted_entry_leaves_the_attention_sums(what, n):
    """A follower step names the slot.  Its entry has all of the softmax weight of every head, or a value row 12 orders above the
    others', of which no difference of fp32 sums would leave the others' digits; or it is the new token.
    Bars: those of parity.py (bf16 output, fp32 memory state)."""
    w = WORKLOADS["cfg1"].scaled(n_layers=1, batch=2, n_q_heads=32, n_kv_heads=8, context=n, budget=n, decode_steps=1)
    ls = LockStep(w, capacity=n + 1)
    slot = n // 2 if what != "last-entry" else n
    eta = w.eta
    if what == "all-the-weight":     # logits of 22 and more for every head of the unit; the others' are N(0, 1)
        q = ls.Q[:, n].float().view(w.batch, w.n_kv_heads, w.group, w.head_dim)
        ls.K[:, :, slot] = (2.0 * q.sum(2)).to(torch.bfloat16)
    if what == "large-value":        # (the memory takes the row, too: written so weakly that its readout does not show it)
        ls.V[:, :, slot] = (ls.V[:, :, slot].float() * 1e12).to(torch.bfloat16)
        eta = 1e-24
    ls.event(0, n, n, "fill")
    d = lambda t: t.to("cuda")
    k, v, q = (x.contiguous() for x in (ls.K[:, :, n:n + 1], ls.V[:, :, n:n + 1], ls.Q[:, n]))
    named = torch.full((w.batch, w.n_kv_heads), slot, dtype=torch.int32, device="cuda")
    im.im_set_max_live(ls.handle, n + 1)
    ls.gpu.follow_step(d(k), d(v), torch.full((w.batch,), n, dtype=torch.int32, device="cuda"), d(q), named, w.lam, eta, debug=True)
    torch.cuda.synchronize()
    assert im.im_query_status(ls.handle) == 0
    ls.ref.append_kv(f64(k), f64(v), np.full((w.batch, 1), n, np.int32))
    evict = [[np.array([slot]) for _ in range(w.n_kv_heads)] for _ in range(w.batch)]
    keep = ls._keep_from(evict)
    ls.ref.memory_update(evict, w.lam, eta)
    ls.ref.compact_kv(keep, evict)
    out, _ = ls.ref.decode_attn_with_readout(f64(q))
    got = f64(ls.gpu.out).reshape(w.batch, w.n_kv_heads, w.group, w.head_dim)
    st = ls.gpu.st
    for b in range(w.batch):
        for h in range(w.n_kv_heads):
            assert_out_close(f"{what} unit({b},{h})", got[b, h], out[b, h])
            assert_state_close("M", f64(st.M[b, h]), ls.ref.M[b, h])
            assert np.array_equal(f64(st.K[b, h, :n]), ls.ref.K[b, h, :n])
            assert np.array_equal(st.pos[b, h, :n].cpu().numpy(), ls.ref.pos[b, h, :n])
            assert int(st.len[b, h]) == n


def _without_the_evicted(shared, batch, hq, hkv, n, edit, tag, finite=None, eta=1e-24):
    """A follower step that names a slot, against the oracle without that entry.  edit(ls, unit_q, slot) prepares K and V (and
    returns the size of the largest logit).  The step leaves the entry's value out of the memory's readout (a tiny eta).

    Bar: a logit is an fp32 sum of 128 products, of size L in all: 16 x 2^-24 L covers its rounding in any order (the bound of a random
    walk of 128 roundings is 11), which moves a weight by as much, and the output by that and the other weights' times the largest |V|.
    Then the output is rounded to bf16, by the oracle, too (2^-7 |o| is a whole step)."""
    w = WORKLOADS["cfg1"].scaled(n_layers=1, batch=batch, n_q_heads=hq, n_kv_heads=hkv, context=n, budget=n, decode_steps=1)
    ids = dict(batch_ids=[0, batch - 1]) if batch > 4 else {}
    ls = LockStepShared(w.shared(), capacity=n + 1, **ids) if shared else LockStep(w, capacity=n + 1, **ids)
    q = ls.Q[:, n].float().view(batch, hkv, w.group, w.head_dim)
    slot = (2 * n) // 3
    largest = edit(ls, q, slot)
    ls.Q[:, n] = q.reshape(batch, hq, w.head_dim).to(torch.bfloat16)
    d = lambda t: t.contiguous().to("cuda")
    pos = torch.arange(n + 1, dtype=torch.int32).repeat(batch, 1)
    named = torch.full((batch,) if shared else (batch, hkv), slot, dtype=torch.int32, device="cuda")
    im.im_set_max_live(ls.handle, n + 1)
    ids = ls.batch_ids
    old, new = slice(0, n), slice(n, n + 1)
    if shared:
        im.im_append_kv_hidden(ls.handle, ls.params, ls.gpu.st, d(ls.K[:, :, old]), d(ls.V[:, :, old]), d(ls.X[:, old]), d(pos[:, old]))
        for s in (old, new):
            ls.ref.append_kv_hidden(f64(ls.K[ids][:, :, s]), f64(ls.V[ids][:, :, s]), f64(ls.X[ids][:, s]), pos[ids][:, s].numpy())
        evict = [np.array([slot]) for _ in ids]
        keep = [np.delete(np.arange(n + 1), slot) for _ in ids]
    else:
        im.im_append_kv(ls.handle, ls.gpu.st, d(ls.K[:, :, old]), d(ls.V[:, :, old]), d(pos[:, old]))
        for s in (old, new):
            ls.ref.append_kv(f64(ls.K[ids][:, :, s]), f64(ls.V[ids][:, :, s]), pos[ids][:, s].numpy())
        evict = [[np.array([slot]) for _ in range(hkv)] for _ in ids]
        keep = [[np.delete(np.arange(n + 1), slot) for _ in range(hkv)] for _ in ids]
    x_new = dict(x_new=d(ls.X[:, new])) if shared else {}
    ls.gpu.follow_step(d(ls.K[:, :, new]), d(ls.V[:, :, new]), d(pos[:, n]), d(ls.Q[:, n]), named, w.lam, eta, debug=True, **x_new)
    torch.cuda.synchronize()
    assert im.im_query_status(ls.handle) == 0
    with np.errstate(invalid="ignore"):
        ls.ref.memory_update(evict, w.lam, eta)
        ls.ref.compact_kv(keep, evict)
        out, _ = ls.ref.decode_attn_with_readout(f64(ls.Q[ids, n]))
    got = f64(ls.gpu.out)[ids].reshape(len(ids), hkv, w.group, w.head_dim)
    v = ls.ref.V[:, :, :n]
    atol = 32 * 2.0 ** -24 * (1 + largest) * float(np.max(np.abs(v[np.isfinite(v) & (np.abs(v) < 100)])))
    dims = np.ones(w.head_dim, bool) if finite is None else finite
    assert_out_close(tag, got[..., dims], out[..., dims], atol=atol, rtol=2.0 ** -7)
    st = ls.gpu.st
    for ib, b in enumerate(ids):   # the cache itself: the last entry has moved into the hole
        assert np.array_equal(f64(st.K[b, :, :n]), ls.ref.K[ib, :, :n])
        assert np.array_equal(f64(st.V[b, :, :n]), ls.ref.V[ib, :, :n], equal_nan=True)
    return got, out


GROUPS = [(2, 32, 8), (16, 28, 4), (16, 64, 8), (40, 64, 8)]   # 1, 2, 4, 8 query heads per workgroup of the last launch


@pytest.mark.parametrize("shared", [False, True])
@pytest.mark.parametrize("n,batch,hq,hkv", [(40, *GROUPS[0]), (300, *GROUPS[0]), (1500, *GROUPS[0])] + [(129, *g) for g in GROUPS[1:]])
@pytest.mark.parametrize("size,share", [(10, 0.3), (10, 0.97), (40, 0.6), (40, 0.99), (300, 0.9), (300, 0.99), (300, 0.9999)])
def test_evicted_entry_with_a_share_of_the_weight(shared, n, batch, hq, hkv, size, share):
    """All logits near `size`, the evicted entry's so much larger that it has about `share` of every head's weight."""
    def edit(ls, q, slot):
        g = torch.Generator().manual_seed(5)
        r = torch.randn(q.shape[0], q.shape[1], 128, generator=g)
        a = {10: 1.0, 40: 2.0, 300: 4.0}[size]
        unit = a * (r * r).sum(-1) * 128 ** -0.5          # the logit of a row r under the query a r
        q[:] = a * (r[:, :, None] + 0.02 * torch.randn(q.shape, generator=g))
        up = np.log((n - 1) * np.exp(0.5) * share / (1 - share))
        K = (size / unit)[..., None, None] * r[:, :, None] + torch.randn(ls.K.shape, generator=g) / a
        K[:, :, slot] = ((size + up) / unit)[..., None] * r
        ls.K[:] = K.to(torch.bfloat16)
        lg = torch.einsum("bhjd,bhkd->bhjk", q.to(torch.bfloat16).double(), ls.K.double()) * 128 ** -0.5
        p = torch.softmax(lg, -1)[..., slot]
        assert (abs(torch.log(p / (1 - p)) - np.log(share / (1 - share))) < 2.5).all()   # (the test is about this share)
        return float(lg.abs().max())
    _without_the_evicted(shared, batch, hq, hkv, n, edit, f"{share} of the weight at logits of {size}")


@pytest.mark.parametrize("shared", [False, True])
@pytest.mark.parametrize("n,batch,hq,hkv", [(40, *GROUPS[0]), (300, *GROUPS[0]), (1500, *GROUPS[0])] + [(129, *g) for g in GROUPS[1:]])
@pytest.mark.parametrize("large", [1e4, 1e6, 1e9])
def test_evicted_entry_with_a_channel_of_its_own(shared, n, batch, hq, hkv, large):
    """The evicted entry's value is large in one channel, a kept entry's as large in another one of the same half, at the same weight: what
    is left of the first channel has nothing to do with the largest output."""
    def edit(ls, q, slot):
        ls.K[:, :, 3] = ls.K[:, :, slot]
        ls.V[:, :, slot, 1] = large
        ls.V[:, :, 3, 0] = large
        return float((torch.einsum("bhjd,bhkd->bhjk", q, ls.K.float()) * 128 ** -0.5).abs().max())
    _without_the_evicted(shared, batch, hq, hkv, n, edit, f"channel {large}")


@pytest.mark.parametrize("shared", [False, True])
@pytest.mark.parametrize("n,batch,hq,hkv", [(300, *GROUPS[0]), (129, *GROUPS[1])])
@pytest.mark.parametrize("below,part", [(3, 60), (3, 200), (20, 25), (45, 15), (45, 200)])
def test_evicted_entry_far_below_the_largest_logit(shared, n, batch, hq, hkv, below, part):
    """The evicted entry's logit lies about `below` under the others', and its part of 32 dims is `part` times what the others have there.
    An exponent of size D is rounded by 2^-24 D, a weight by as much, and by about four roundings more: subtracted up to
    1024 / (4 + D) of the rest, that is at most 1024 x 2^-24 of the dim, and an output of 8 bits (a step is at least 2^-8 of it) is rounded
    the other way in at most one case in 64."""
    def edit(ls, q, slot):
        g = torch.Generator().manual_seed(7)
        r = torch.randn(q.shape[0], q.shape[1], 128, generator=g)
        unit = (r * r).sum(-1) * 128 ** -0.5          # the logit of a row r under the query r
        q[:] = r[:, :, None] + 0.005 * torch.randn(q.shape, generator=g)
        K = (10 / unit)[..., None, None] * r[:, :, None] + 0.3 * torch.randn(ls.K.shape, generator=g)
        K[:, :, slot] = ((10 - below) / unit)[..., None] * r
        ls.K[:] = K.to(torch.bfloat16)
        ls.V[..., ::4] = ls.V[..., ::4].abs() + 0.5
        lg = torch.einsum("bhjd,bhkd->bhjk", q.to(torch.bfloat16).double(), ls.K.double()) * 128 ** -0.5
        lg = lg[..., :n + 1]
        odds = torch.exp(torch.logsumexp(torch.cat([lg[..., :slot], lg[..., slot + 1:]], -1), -1) - lg[..., slot]).mean(-1)
        ls.V[:, :, slot, ::4] = (1.3 * part * odds)[..., None].to(torch.bfloat16)   # (the others' mean is 1.3)
        return float(lg.abs().max())
    got, out = _without_the_evicted(shared, batch, hq, hkv, n, edit, f"{part} times the rest, {below} below", eta=1e-36)
    differ = float(np.mean(got[..., ::4] != out[..., ::4]))
    assert differ <= 1 / 64, differ


@pytest.mark.parametrize("shared", [False, True])
@pytest.mark.parametrize("n,batch,hq,hkv", [(300, *GROUPS[0]), (129, *GROUPS[2])])
@pytest.mark.parametrize("bad", [float("inf"), float("nan"), 3e37])
def test_evicted_entry_that_is_not_finite(shared, n, batch, hq, hkv, bad):
    """Not finite in two channels, which the memory then holds; and a kept entry's infinity stays one."""
    def edit(ls, q, slot):
        ls.V[:, :, slot, 5] = bad
        ls.V[:, :, slot, 70] = -bad
        ls.V[:, :, 7, 9] = float("inf")
        return float((torch.einsum("bhjd,bhkd->bhjk", q, ls.K.float()) * 128 ** -0.5).abs().max())
    dims = np.ones(128, bool)
    dims[[5, 70] if bad != 3e37 else [], ] = False
    dims[9] = False
    got, _ = _without_the_evicted(shared, batch, hq, hkv, n, edit, f"value {bad}", finite=dims)
    assert np.isposinf(got[..., 9]).all()


@pytest.mark.parametrize("shared", [False, True])
def test_memory_state_keeps_its_digits(shared):
    """Twelve evictions one after another into an empty memory, against fp64, root mean square over the state.  A phi is a sum of 128 exact
    products in four parts (4.8e-8 of its size; head-shared: of each head's, then 8 are added), and every step rounds phi v, or phi^2, and
    the sum once (2^-24 / sqrt(3) = 3.4e-8 each, of a state that grows to its last size as sqrt(t)): 8e-8 for b, which sums squares, and 9e-8
    for M (head-shared, with the eight roundings of the sum over the heads: 10e-8).  Bars: a sixth more."""
    n, steps = 40, 12
    w = WORKLOADS["cfg1"].scaled(n_layers=1, batch=8, n_q_heads=32, n_kv_heads=8, context=n + steps, budget=n, decode_steps=1)
    ls = LockStepShared(w.shared(), capacity=n + 1) if shared else LockStep(w, capacity=n + 1)
    d = lambda t: t.contiguous().to("cuda")
    pos = torch.arange(n + steps, dtype=torch.int32).repeat(w.batch, 1)
    old = slice(0, n)
    if shared:
        im.im_append_kv_hidden(ls.handle, ls.params, ls.gpu.st, d(ls.K[:, :, old]), d(ls.V[:, :, old]), d(ls.X[:, old]), d(pos[:, old]))
    else:
        im.im_append_kv(ls.handle, ls.gpu.st, d(ls.K[:, :, old]), d(ls.V[:, :, old]), d(pos[:, old]))
    im.im_set_max_live(ls.handle, n + 1)
    W = f64(ls.params.Wtheta)
    M = b = 0.0
    for t in range(n, n + steps):
        e = (7 * t) % n
        ke, ve = f64(ls.gpu.st.K[:, :, e]), f64(ls.gpu.st.V[:, :, e])
        ke, ve = (ke.sum(1), ve.sum(1)) if shared else (ke, ve)
        named = torch.full((w.batch,) if shared else (w.batch, w.n_kv_heads), e, dtype=torch.int32, device="cuda")
        ls.gpu.follow_step(d(ls.K[:, :, t:t + 1]), d(ls.V[:, :, t:t + 1]), d(pos[:, t]), d(ls.Q[:, t]), named, w.lam, w.eta,
                           **(dict(x_new=d(ls.X[:, t:t + 1])) if shared else {}))
        phi = ke @ W.T
        M = w.lam * M + w.eta * phi[..., :, None] * ve[..., None, :]
        b = w.lam * b + w.eta * phi * phi
    torch.cuda.synchronize()
    assert im.im_query_status(ls.handle) == 0
    off = lambda got, want: float(np.linalg.norm(f64(got) - want) / np.linalg.norm(want))
    err = off(ls.gpu.st.M, M), off(ls.gpu.st.b, b)
    assert err[0] <= (11.5e-8 if shared else 10.5e-8) and err[1] <= 9.3e-8, err
