"""The workspace may hold anything when a handle is created, and between the calls of one handle other handles may use the
same memory (in stream order): a call reads only what it, or one call of the same program step before it, has written."""
import ctypes as C

import pytest
import torch

import paper_2605_25475_amd as im

pytestmark = pytest.mark.gpu
CFG = dict(batch=2, n_q_heads=32, n_kv_heads=8, n_idx_heads=8)
N, N_Q = 70, 1089   # 2178 queries: their projection is an exact product with lists


def _bf(*shape, seed, scale=1.0):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return (torch.randn(shape, generator=g, device="cuda") * scale).to(torch.bfloat16)


def _params():
    ones = torch.ones(64, dtype=torch.bfloat16, device="cuda")
    return im.Params(_bf(512, 4096, seed=1, scale=0.02), _bf(8, 4096, seed=2, scale=0.02), _bf(64, 128, seed=3, scale=0.02),
                     _bf(128, 128, seed=4, scale=0.02), _bf(128, seed=5, scale=0.02), 0.0, ones, ones)


def _queries(seed):
    q = _bf(2, N_Q, 32, 128, seed=seed)
    g = torch.Generator(device="cuda")
    g.manual_seed(seed + 1)
    small = torch.rand(q.shape, generator=g, device="cuda") < 2e-4   # about one listed value per row
    return torch.where(small, (q.float() * 2.0 ** -26).to(torch.bfloat16), q).contiguous()


def _prompt(h, p, seed):
    """A state of N entries scored by N_Q queries: its scores."""
    st = im.State(h.cfg, "cuda")
    pos = torch.arange(N, dtype=torch.int32, device="cuda").repeat(2, 1).contiguous()
    k = _bf(2, 8, N, 128, seed=seed + 10)
    im.im_append_kv(h, st, k, k, pos)
    im.im_set_max_live(h, N)
    scores = torch.full((2, 8, h.cfg.capacity), 7.0, device="cuda")
    q = _queries(seed)
    qpos = (torch.arange(N_Q, dtype=torch.int32, device="cuda") % (N + 3)).repeat(2, 1).contiguous()
    im.im_index_score(h, p, st, q, q.view(2, N_Q, -1), qpos, scores)
    torch.cuda.synchronize()
    return scores[..., :N].clone()


def _handle(max_queries=N_Q, capacity=N, fill=0, block=None):
    """A handle whose workspace is filled with a pattern, or lies at the start of `block`."""
    h = im.Handle(im.Config(capacity=capacity, max_queries=max_queries, **CFG), "cuda")
    if block is None:
        h.workspace.view(torch.uint8).fill_(fill)
        return h
    h.lib.im_destroy(h.h)
    h.workspace, h.h = block, C.c_void_p()
    base = (block.data_ptr() + 255) & ~255
    assert h.lib.im_create(C.byref(h.cfg.c_struct()), base, block.data_ptr() + block.numel() - base, C.byref(h.h)) == 0
    return h


@pytest.mark.parametrize("fill", [0x01, 0x7f, 0x80, 0xff])
def test_scores_do_not_depend_on_what_the_workspace_held(fill):
    p = _params()
    want = [_prompt(_handle(), p, s) for s in (100, 200)]
    h = _handle(fill=fill)
    for s, w in zip((100, 200), want):
        assert torch.equal(_prompt(h, p, s), w)
        h.workspace[256 + 4 * 64:].fill_(fill)   # (all but the status words, which a handle clears once)


@pytest.mark.parametrize("fill", [0x01, 0xff])
def test_first_call_inside_a_capture(fill):
    """The captured call runs only at a replay: an eager call before it finds the workspace as it was created."""
    p = _params()
    want = _prompt(_handle(), p, 100)
    h = _handle(fill=fill)
    st = im.State(h.cfg, "cuda")
    k = _bf(2, 8, 1, 128, seed=9)
    pos = torch.zeros((2, 1), dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        im.im_append_kv(h, st, k, k, pos)
    assert torch.equal(_prompt(h, p, 100), want)
    for _ in range(3):
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(_prompt(h, p, 100), want)
    assert int(st.len.min()) == 3


def test_two_handles_take_turns_on_one_block():
    p = _params()

    def decode(h, steps):
        st = im.State(h.cfg, "cuda")
        k = _bf(2, 8, 40, 128, seed=20)
        im.im_append_kv(h, st, k, k, torch.arange(40, dtype=torch.int32, device="cuda").repeat(2, 1).contiguous())
        outs = []
        for t in range(steps):
            kn, q = _bf(2, 8, 1, 128, seed=30 + t), _bf(2, 32, 128, seed=60 + t)
            p1 = torch.full((2,), 40 + t, dtype=torch.int32, device="cuda")
            out = torch.empty((2, 32, 128), dtype=torch.bfloat16, device="cuda")
            im.im_decode_step(h, p, st, q, q.view(2, -1), p1, kn, kn, p1, 40, 0.9, 0.5, out)
            outs.append(out)
            yield out
        yield torch.cat([t.flatten().float() for t in outs + [st.M, st.K, st.pos]])

    want_prompt = [_prompt(_handle(), p, s) for s in (100, 200)]
    want_decode = list(decode(_handle(1, 41), 2))
    block = torch.full((max(_handle(1, 41).workspace.numel(), _handle().workspace.numel()) + 512,), 0x55, dtype=torch.uint8,
                       device="cuda")
    hp, hd = _handle(block=block), _handle(1, 41, block=block)
    run = decode(hd, 2)
    for s, w in zip((100, 200), want_prompt):
        assert torch.equal(_prompt(hp, p, s), w)
        assert torch.equal(next(run), want_decode[0 if s == 100 else 1])
    assert torch.equal(next(run), want_decode[2])
