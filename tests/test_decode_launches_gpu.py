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
    (4, 32, 8, 1535), (4, 32, 8, 1536), (2, 64, 8, 3100)])              # two and four (more than 3072)
def test_tiles_per_scoring_wave(batch, hq, hkv, budget):
    _run(False, batch, hq, hkv, budget + 7, budget, n_recent=3 if budget > 16 else 0)


@pytest.mark.parametrize("budget", [64, 127, 2047, 2048, 4100])
def test_tiles_per_scoring_wave_head_shared(budget):
    _run(True, 2, 32, 8, budget + 5, budget)


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
