"""The memory write of a prompt against fp64: how many partial sums its evicted rows are split into must not show in
the error."""
import pytest
import torch

import paper_2605_25475_amd as im

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,kv_heads,n,shared", [(8, 8, 3072, True), (3, 8, 8300, True), (2, 4, 5300, False), (1, 1, 20000, False)])
def test_memory_of_many_splits_has_the_error_of_a_few(batch, kv_heads, n, shared):
    cfg = im.Config(batch=batch, n_q_heads=kv_heads, n_kv_heads=kv_heads, capacity=n, n_idx_heads=2, n_sink=0,
                    idx_dim=16 if shared else 64, head_shared=int(shared))
    h = im.Handle(cfg, "cuda")
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    rand = lambda *s: torch.randn(s, generator=g, device="cuda").to(torch.bfloat16)
    st = im.State(cfg, "cuda")
    st.K.copy_(rand(*st.K.shape))
    st.V.copy_(rand(*st.V.shape))
    st.len.fill_(n)
    w = (rand(128, 128).float() * 0.02).to(torch.bfloat16)
    p = im.Params(w, w, w, w, w, 0.0)   # (only Wtheta is read)
    sets = tuple(st.len.shape)
    evict = torch.arange(n, dtype=torch.int32, device="cuda").expand(sets + (n,)).contiguous()
    n_evict = torch.full(sets, n, dtype=torch.int32, device="cuda")
    im.im_memory_update(h, p, st, evict, n_evict, 1.0, 1.0)
    K, V = st.K.double(), st.V.double()
    if shared:
        K, V = K.sum(1), V.sum(1)
    phi = K @ w.double().t().contiguous()
    M, b = phi.transpose(-1, -2).contiguous() @ V, (phi * phi).sum(-2)
    rel = lambda got, want: float((got.double() - want).norm() / want.norm())
    # b: a chain of k fp32 additions of like terms errs by about 2^-24 sqrt(k) / 3 of the sum; the longest here, the
    # 32 rows of a tile, then 3 + 8 + 16 partials: 1.6e-7 at most, and an average over many of them below 1e-7.
    # M: dominated by Phi's 16 bits, 2^-17 / sqrt(3) of each product at most
    err_b, err_M = rel(st.b, b), rel(st.M, M)
    assert err_b < 1.0e-7
    assert err_M < 2.0 ** -17 / 3 ** 0.5
