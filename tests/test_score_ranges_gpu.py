"""im_index_score of many queries at the ends of the number range: bounds that are infinite, or would be, and scores
that round to a negative zero.  The scores must be the oracle's fp32 numbers."""
import numpy as np
import pytest
import torch

import paper_2605_25475_amd as im
from helpers import f64
from parity import LockStep, LockStepShared
from workloads import WORKLOADS

pytestmark = pytest.mark.gpu


def _first_column(p, rows):
    """Gates that read the first value of the gate input alone: alpha_j = rows[j] x_0 / sqrt(H_idx d_idx)."""
    p["G"].zero_()
    p["G"][:, 0] = torch.tensor(rows, dtype=torch.float64).to(torch.bfloat16)


def _high(p):
    # bounds of infinity, and keys whose scale takes a score in the bounds' units beyond fp32
    p["G"] = (p["G"].float() * 2.0 ** 60).to(torch.bfloat16)
    p["norm_q_w"] = (p["norm_q_w"].float() * 2.0 ** 66).to(torch.bfloat16)
    p["norm_k_w"] = (p["norm_k_w"].float() * 2.0 ** -60).to(torch.bfloat16)


def _opposite(p):
    # heads (u, -u, w, -w) with gates (a, a, -a, -a): the linear part of the bound vanishes, S = a |u k| - a |w k|, and
    # the two parts are beyond fp32 in the bounds' units although every single factor is inside them
    U, Hi, di = p["Uq"], p["G"].shape[0], p["norm_q_w"].shape[0]
    rows = [0.0] * Hi
    for j in range(0, Hi - 3, 4):
        for s in (0, 2):
            U[(j + s + 1) * di:(j + s + 2) * di] = -U[(j + s) * di:(j + s + 1) * di]
            rows[j + s] = rows[j + s + 1] = (1.1e18 if s == 0 else -1.1e18) * (Hi * di) ** 0.5
    _first_column(p, rows)
    p["norm_q_w"].fill_(1.12e18 / di ** 0.5)
    p["norm_k_w"].fill_(15.9 / di ** 0.5)


def _negative_zero(p):
    # scores of the first 16 queries round to -0.0, the others are large and negative
    _first_column(p, [-1.0] * p["G"].shape[0])
    p["norm_q_w"].fill_(2.0 ** -40)
    p["norm_k_w"].fill_(2.0 ** -40)


MODES = {"high": _high, "opposite": _opposite, "negative-zero": _negative_zero}


@pytest.mark.parametrize("mode", sorted(MODES))
@pytest.mark.parametrize("heads", [(32, 8), (28, 4)], ids=["8", "7"])   # indexer heads
@pytest.mark.parametrize("shared", [False, True], ids=["per-unit", "head-shared"])
def test_scores_at_the_ends_of_the_range(mode, heads, shared):
    n_q, n = 400, 100   # 25 blocks of queries in 8 groups: most candidates come from the list
    kw = dict(context=n_q, budget=n, decode_steps=0, batch=2, n_layers=1, n_q_heads=heads[0], n_kv_heads=heads[1])
    w = WORKLOADS["cfg1"].shared(**kw) if shared else WORKLOADS["cfg1"].scaled(**kw)
    ls = (LockStepShared if shared else LockStep)(w, params_mod=MODES[mode])
    g, ref, d = ls.gpu, ls.ref, (lambda t: t.contiguous().cuda())
    pos = torch.arange(n, dtype=torch.int32).repeat(w.batch, 1).contiguous()
    q = ls.Q[:, :n_q].contiguous()
    xg = q.view(w.batch, n_q, -1).clone()
    if mode != "high":
        xg[:] = 0
        xg[:, :, 0] = 1.0
    if mode == "negative-zero":
        xg[:, :16, 0], xg[:, 16:, 0] = 2.0 ** -100, 2.0 ** 100
    if shared:
        im.im_append_kv_hidden(ls.handle, ls.params, g.st, d(ls.K[:, :, :n]), d(ls.V[:, :, :n]), d(ls.X[:, :n]), d(pos))
        ref.append_kv_hidden(f64(ls.K[:, :, :n]), f64(ls.V[:, :, :n]), f64(ls.X[:, :n]), pos.numpy())
    else:
        im.im_append_kv(ls.handle, g.st, d(ls.K[:, :, :n]), d(ls.V[:, :, :n]), d(pos))
        ref.append_kv(f64(ls.K[:, :, :n]), f64(ls.V[:, :, :n]), pos.numpy())
    qpos = torch.full((w.batch, n_q), n, dtype=torch.int32)
    want = ref.index_score(f64(q), f64(xg), qpos.numpy())[..., :n]
    im.im_index_score(ls.handle, ls.params, g.st, d(q), d(xg), d(qpos), g.scores)
    torch.cuda.synchronize()
    got = g.scores[..., :n].cpu().numpy().astype(np.float64)
    assert np.isfinite(want).all() and (mode == "negative-zero") == bool((want == 0).all())
    wrong = int((got != want).sum())
    assert wrong == 0, f"{wrong} of {want.size} scores differ"
