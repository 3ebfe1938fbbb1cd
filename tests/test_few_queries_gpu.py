"""im_index_score with fewer queries than indexer heads where its form changes (up to 4 queries normalise their features in
the scoring launch, more in a launch of their own), on a cache filled by appends of 16 and 17 tokens (where the
length is raised by the copying launch and by one of its own)."""
import numpy as np
import pytest
import torch

import paper_2605_25475_amd as im
from helpers import f64
from parity import LockStep, LockStepShared
from workloads import WORKLOADS

pytestmark = pytest.mark.gpu


def _norm_weights(p):
    g = torch.Generator().manual_seed(3)
    for k in ("norm_q_w", "norm_k_w"):
        p[k] = (1.0 + 0.1 * torch.randn(p[k].shape, generator=g)).to(torch.bfloat16)


@pytest.mark.parametrize("n_q", [1, 4, 5, 7])
@pytest.mark.parametrize("shared", [False, True], ids=["per-unit", "head-shared"])
def test_few_queries_and_appends_at_their_limits(shared, n_q):
    n = 33
    kw = dict(context=n, budget=n, decode_steps=0, batch=2, n_layers=1)
    w = WORKLOADS["cfg1"].shared(**kw) if shared else WORKLOADS["cfg1"].scaled(**kw)
    ls = (LockStepShared if shared else LockStep)(w, capacity=n, params_mod=_norm_weights)
    g, ref, d = ls.gpu, ls.ref, (lambda t: t.contiguous().cuda())
    pos = torch.arange(n, dtype=torch.int32).repeat(w.batch, 1)
    for t0, t1 in ((0, 16), (16, 33)):
        k, v, p = ls.K[:, :, t0:t1], ls.V[:, :, t0:t1], pos[:, t0:t1]
        if shared:
            im.im_append_kv_hidden(ls.handle, ls.params, g.st, d(k), d(v), d(ls.X[:, t0:t1]), d(p))
            ref.append_kv_hidden(f64(k), f64(v), f64(ls.X[:, t0:t1]), p.numpy())
        else:
            im.im_append_kv(ls.handle, g.st, d(k), d(v), d(p))
            ref.append_kv(f64(k), f64(v), p.numpy())
    q = ls.Q[:, :n_q].contiguous()
    qpos = torch.arange(n - n_q, n, dtype=torch.int32).repeat(w.batch, 1).contiguous()
    xg = q.view(w.batch, n_q, -1)
    want = ref.index_score(f64(q), f64(xg), qpos.numpy())[..., :n]
    for _ in range(2):   # (the raw projections stay raw)
        g.scores.zero_()
        im.im_index_score(ls.handle, ls.params, g.st, d(q), d(xg), d(qpos), g.scores)
        torch.cuda.synchronize()
        assert np.array_equal(g.scores[..., :n].cpu().numpy().astype(np.float64), want)
    assert torch.equal(g.st.pos[..., :n].cpu(), pos.view(w.batch, *([1] * (g.st.pos.dim() - 2)), n).expand(g.st.pos[..., :n].shape))
    assert int(g.st.len.min()) == n and im.im_query_status(ls.handle) == 0
    if not shared:   # full: another token is refused, by the copying launch
        before = g.st.K.clone()
        im.im_append_kv(ls.handle, g.st, d(ls.K[:, :, :1]), d(ls.V[:, :, :1]), d(pos[:, :1]))
        assert im.im_query_status(ls.handle) == 1
        assert torch.equal(g.st.K, before) and int(g.st.len.max()) == n
