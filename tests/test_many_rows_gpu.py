"""An append of more rows than one dimension of a grid has workgroups of 16 rows."""
import numpy as np
import pytest
import torch

import paper_2605_25475_amd as im
from helpers import f64
from oracle import indexmem_oracle as O

pytestmark = pytest.mark.gpu


def test_append_of_a_million_rows():
    batch, n = 8, 131072 + 16   # 65544 tiles of 16 rows
    cfg = im.Config(batch=batch, n_q_heads=1, n_kv_heads=1, capacity=n, n_idx_heads=1, idx_dim=16, gate_in_dim=128, head_shared=1)
    h, st = im.Handle(cfg, "cuda"), im.State(cfg, "cuda")
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    rand = lambda *s: torch.randn(s, generator=g, device="cuda").to(torch.bfloat16)
    x, Uk, ones = rand(batch, n, 128), rand(16, 128), torch.ones(16, dtype=torch.bfloat16, device="cuda")
    p = im.Params(Uk, Uk, Uk, Uk, Uk, 0.0, ones, ones)
    pos = torch.arange(n, dtype=torch.int32, device="cuda").repeat(batch, 1).contiguous()
    im.im_append_kv_hidden(h, p, st, None, None, x, pos)
    torch.cuda.synchronize()
    assert int(st.len.min()) == n and im.im_query_status(h) == 0
    for b, rows in ((0, slice(0, 100)), (3, slice(65530, 65600)), (7, slice(n - 100, n))):
        want = O.round_bf16(O.key_feature(f64(x[b, rows]), f64(Uk), f64(ones), float(np.float32(1e-6))))
        assert np.array_equal(f64(st.Kidx[b, rows]), want)
