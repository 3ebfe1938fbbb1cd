"""im_topb_select around the sizes at which it changes its form (4096, 8192 and 16384 entries in registers, more from
memory): ties of scores and positions, infinities, sinks and a recent window, against a sort on the host."""
import numpy as np
import pytest
import torch

import paper_2605_25475_amd as im

pytestmark = pytest.mark.gpu


def _want(sc, pos, budget, n_sink, n_recent):
    forced = (pos < n_sink) | ((n_recent > 0) & (pos > pos.max() - n_recent))
    key = np.where(forced, np.inf, sc)
    order = np.lexsort((np.arange(len(sc)), pos, -key))   # best first: score, then low position, then low slot
    return np.sort(order[:budget]), np.sort(order[budget:])


@pytest.mark.parametrize("n", [1, 65, 1024, 1025, 4095, 4096, 4097, 8192, 8193, 16384, 16385])
def test_lists_at_the_edges_of_the_register_forms(n):
    units, n_sink, n_recent = 2, 2, 3
    cfg = im.Config(batch=1, n_q_heads=8, n_kv_heads=units, capacity=max(n, 16), n_idx_heads=2, n_sink=n_sink,
                    n_recent=n_recent, max_queries=1)
    h = im.Handle(cfg, "cuda")
    rng = np.random.default_rng(n)
    for live in (n, max(1, n - 700)):
        for ties in ("none", "scores", "both"):
            sc = rng.standard_normal((1, units, cfg.capacity)).astype(np.float32)
            pos = np.stack([rng.permutation(cfg.capacity) for _ in range(units)])[None].astype(np.int32)
            if ties != "none":
                sc = np.round(sc)
                sc[0, 1] = 0.0
                sc[..., ::7] = -np.inf
            if ties == "both":
                pos //= 5
            st = im.State(h.cfg, "cuda")
            st.len.fill_(live)
            st.pos.copy_(torch.from_numpy(pos))
            out = [torch.full(tuple(st.pos.shape), -1, dtype=torch.int32, device="cuda") for _ in range(2)]
            cnt = [torch.zeros_like(st.len) for _ in range(2)]
            im.im_set_max_live(h, n)
            for budget in sorted({min(max(b, n_sink + n_recent), cfg.capacity) for b in (5, n // 3, live - 1, n)}):
                im.im_topb_select(h, torch.from_numpy(sc).cuda(), st, budget, *out, *cnt)
                torch.cuda.synchronize()
                for u in range(units):
                    keep, evict = _want(sc[0, u, :live], pos[0, u, :live], budget, n_sink, n_recent)
                    nk, ne = int(cnt[0].flatten()[u]), int(cnt[1].flatten()[u])
                    assert (nk, ne) == (len(keep), len(evict)), (live, ties, budget, u)
                    assert np.array_equal(out[0][0, u, :nk].cpu().numpy(), keep), (live, ties, budget, u)
                    assert np.array_equal(out[1][0, u, :ne].cpu().numpy(), evict), (live, ties, budget, u)
    assert im.im_query_status(h) == 0
