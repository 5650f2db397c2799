"""Runs of steps that dynts_decode_loop makes in one to three launches, where they meet something else: recorded steps replayed around
them, full caches, updates owed in each of their forms, chunks without a finite logit.  Against single calls, bit for bit."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2601_18383_amd import binding
    return binding


DEV = "cuda:0"
# one tile a wave, two, and several chunks with merges of four, of eight and of 32 at a time: Nb, Hq, Hkv, d, cap
FORMS = [(3, 8, 2, 64, 200), (45, 32, 8, 128, 490), (2, 28, 4, 128, 700), (2, 8, 1, 128, 1500), (1, 32, 8, 128, 4544)]


def _normal(g, *shape, scale=1.0):
    return (torch.randn(shape, generator=g, device=DEV) * scale).to(torch.bfloat16)


def _caches(B, g, L, Nb, Hq, Hkv, d, cap, lens, count=2):
    """Caches of the same random contents."""
    caches = [B.Cache(L, Nb, Hq, Hkv, d, cap, cap - 100, 32, 16) for _ in range(count)]
    K, V, S = _normal(g, L, Nb, Hkv, cap, d), _normal(g, L, Nb, Hkv, cap, d), torch.rand((L, Nb, Hkv, cap), generator=g, device=DEV)
    for c in caches:
        c.K.copy_(K)
        c.V.copy_(V)
        c.S.copy_(S)
        c.seq_len.copy_(lens.to(DEV).expand(L, Nb))
        c.next_pos.fill_(cap)
        c.n_prompt.fill_(9)
    return caches


def _tokens(g, T, L, Nb, Hq, Hkv, d):
    return _normal(g, T, L, Nb, Hq, d, scale=1.5), _normal(g, T, L, Nb, Hkv, d), _normal(g, T, L, Nb, Hkv, d)


def _single_steps(B, cache, x, outs, active=None):
    for t in range(x[0].shape[0]):
        for l in range(x[0].shape[1]):
            B.dynts_decode_step(cache.ctx, l, x[0][t, l], x[1][t, l], x[2][t, l], outs[t, l], active=None if active is None else active[t])


def _same(a, b, L, Nb):
    assert torch.equal(a.seq_len, b.seq_len) and torch.equal(a.next_pos, b.next_pos) and torch.equal(a.status, b.status)
    for l in range(L):
        for i in range(Nb):
            n = int(a.seq_len[l, i])
            for x, y in ((a.K, b.K), (a.V, b.V), (a.S, b.S), (a.pos, b.pos)):
                assert torch.equal(x[l, i, :, :n], y[l, i, :, :n])


@pytest.mark.parametrize("Nb,Hq,Hkv,d,cap", FORMS)
def test_replays_around_runs(B, Nb, Hq, Hkv, d, cap):
    """Two steps recorded behind an eager one, replayed with an even number of eager steps between the replays: however the loop makes
    those, the replayed launches find the saved query where they look for it."""
    g = torch.Generator(device=DEV)
    g.manual_seed(cap)
    between = [4, 0, 16, 3, 6]  # steps of a loop; behind the three one by itself
    a, b = _caches(B, g, 1, Nb, Hq, Hkv, d, cap, torch.tensor(cap - 60))
    first = _tokens(g, 1, 1, Nb, Hq, Hkv, d)
    out = torch.zeros(2, 1, Nb, Hq, d, device=DEV)
    for c in (a, b):
        _single_steps(B, c, first, out)
    now = [x.clone() for x in _tokens(g, 2, 1, Nb, Hq, Hkv, d)]
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        _single_steps(B, a, now, out)
    for steps in between:
        x = _tokens(g, 2, 1, Nb, Hq, Hkv, d)
        want = torch.zeros_like(out)
        for dst, src in zip(now, x):
            dst.copy_(src)
        graph.replay()
        _single_steps(B, b, x, want)
        torch.cuda.synchronize()
        assert torch.equal(out, want)
        if steps == 0:
            continue
        x = _tokens(g, steps + steps % 2, 1, Nb, Hq, Hkv, d)
        got, want = (torch.zeros(steps + steps % 2, 1, Nb, Hq, d, device=DEV) for _ in range(2))
        B.dynts_decode_loop(a.ctx, steps, *(y[:steps] for y in x), got, a.keep_idx, a.new_len, out_step_stride=got[0].numel())
        _single_steps(B, a, [y[steps:] for y in x], got[steps:])
        _single_steps(B, b, x, want)
        torch.cuda.synchronize()
        assert torch.equal(got, want)
        _same(a, b, 1, Nb)
    graph.replay()
    _single_steps(B, b, now, out.clone())
    for c in (a, b):
        B.dynts_update_scores(c.ctx, 0)
    _same(a, b, 1, Nb)
