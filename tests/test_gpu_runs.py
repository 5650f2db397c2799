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
# one tile a wave, two, and several chunks with merges of four, of eight and of 32 at a time, to the most chunks there are: Nb, Hq, Hkv, d, cap
FORMS = [(3, 8, 2, 64, 200), (45, 32, 8, 128, 490), (2, 28, 4, 128, 700), (2, 8, 1, 128, 1500), (1, 32, 8, 128, 4544), (1, 16, 1, 64, 20000),
         (1, 4, 1, 128, 65536)]


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


@pytest.mark.parametrize("Nb,Hq,Hkv,d,cap", FORMS)
@pytest.mark.parametrize("stride", ["none", "slab"])
def test_runs_past_full_caches(B, Nb, Hq, Hkv, d, cap, stride):
    """Sequences that fill up at different steps of a run, one before it: their later steps are dropped, outputs left alone, the status
    bit set, no update owed by them."""
    g = torch.Generator(device=DEV)
    g.manual_seed(cap + 1)
    L, T = 2, 30
    lens = torch.tensor([cap - (0, 7, T - 1, 40, 19)[(i + 1) % 5] for i in range(Nb)], dtype=torch.int32)
    a, b = _caches(B, g, L, Nb, Hq, Hkv, d, cap, lens)
    active = (torch.rand((T, Nb), generator=g, device=DEV) < 0.9).to(torch.uint8)
    step = L * Nb * Hq * d if stride == "slab" else 0
    got, want = (torch.full(((T if step else 1) * L * Nb * Hq * d,), 7.0, device=DEV) for _ in range(2))
    for part in range(2):  # an update of the first is owed to the second
        x = _tokens(g, T, L, Nb, Hq, Hkv, d)
        B.dynts_decode_loop(a.ctx, T, *x, got, a.keep_idx, a.new_len, active=active, out_step_stride=step)
        _single_steps(B, b, x, want.view(-1, L, Nb, Hq, d).expand(T, L, Nb, Hq, d), active)
        assert torch.equal(got, want) and bool((got != 7.0).any())
        _same(a, b, L, Nb)
    assert int(a.status.item()) == 1
    for l in range(L):
        B.dynts_update_scores(a.ctx, l)
        B.dynts_update_scores(b.ctx, l)
    _same(a, b, L, Nb)


@pytest.mark.parametrize("Nb,Hq,Hkv,d,cap", FORMS)
@pytest.mark.parametrize("before", ["attend 0", "attend 0, attend 1", "hinted 0", "hinted 0, hinted 1", "hinted 1, attend 0"])
@pytest.mark.parametrize("trigger", [False, True])
def test_runs_behind_updates_owed_in_every_form(B, Nb, Hq, Hkv, d, cap, before, trigger):
    """A run begins behind an unfused attention (whose update may be made from its kept logits or by a pass over K) or behind an announced
    step (from its kept logits alone), on the same layer or the other one, which shares the room for them."""
    g = torch.Generator(device=DEV)
    g.manual_seed(cap + 2)
    L, T = 2, 12
    a, b = _caches(B, g, L, Nb, Hq, Hkv, d, cap, torch.tensor(cap - 40))
    one = _tokens(g, 1, L, Nb, Hq, Hkv, d)
    out = torch.zeros(L, Nb, Hq, d, device=DEV)
    for c in (a, b):
        for what in before.split(", "):
            kind, l = what.split()
            l = int(l)
            if kind == "attend":
                B.dynts_decode_attend(c.ctx, l, one[0][0, l], out[l])
            else:
                B.dynts_hint_trigger(c.ctx, l)
                B.dynts_decode_step(c.ctx, l, one[0][0, l], one[1][0, l], one[2][0, l], out[l])
    x = _tokens(g, T, L, Nb, Hq, Hkv, d)
    got, want = (torch.zeros(T, L, Nb, Hq, d, device=DEV) for _ in range(2))
    flags = torch.tensor([0] * (T - 1) + [int(trigger)], dtype=torch.uint8)
    B.dynts_decode_loop(a.ctx, T, *x, got, a.keep_idx, a.new_len, evict_steps=flags, out_step_stride=got[0].numel())
    _single_steps(B, b, [y[:T - 1] for y in x], want)
    for l in range(L):
        if trigger:
            B.dynts_hint_trigger(b.ctx, l)
        B.dynts_decode_step(b.ctx, l, x[0][-1, l], x[1][-1, l], x[2][-1, l], want[-1, l])
        if trigger:
            B.dynts_select_evict(b.ctx, l, b.keep_idx, b.new_len, b.cfg.budget)
            B.dynts_compact(b.ctx, l, b.keep_idx, b.new_len)
    assert torch.equal(got, want)
    _same(a, b, L, Nb)
    for l in range(L):
        B.dynts_update_scores(a.ctx, l)
        B.dynts_update_scores(b.ctx, l)
    _same(a, b, L, Nb)
    assert int(a.status.item()) == 0


# merges of four, of eight and of 32 chunks of 256 slots at a time: the slots of the first group, and more, have no finite logit
@pytest.mark.parametrize("Hq,Hkv,d,cap,dead", [(8, 2, 128, 1600, 1024), (8, 2, 64, 1600, 1300), (8, 1, 128, 2700, 2048), (8, 2, 128, 8900, 8192)])
@pytest.mark.parametrize("paged", [False, True])
def test_chunks_whose_logits_are_all_minus_infinity(B, Hq, Hkv, d, cap, dead, paged):
    """They weigh nothing, the new tokens' among them: every other slot has a logit of zero, so the outputs are the mean of their V rows
    (sums of fp32: 1e-5), and each gains 1 / their number from each of the group's heads (an exponential and a reciprocal: 1e-6 of it)."""
    g = torch.Generator(device=DEV)
    g.manual_seed(cap)
    T, n0 = 5, cap - 40
    big = torch.tensor(3e38).bfloat16()
    K0 = torch.zeros((1, Hkv, n0, d), dtype=torch.bfloat16, device=DEV)
    K0[:, :, :dead] = -big
    V0 = _normal(g, 1, Hkv, n0, d)
    q, k = big.expand(T, 1, 1, Hq, d).contiguous().to(DEV), (-big).expand(T, 1, 1, Hkv, d).contiguous().to(DEV)
    v = _normal(g, T, 1, 1, Hkv, d)
    a, b = ((B.PagedCache if paged else B.Cache)(1, 1, Hq, Hkv, d, cap, cap - 80, 32, 16) for _ in range(2))
    for c in (a, b):
        B.dynts_prefill(c.ctx, 0, K0, V0, torch.tensor([n0], dtype=torch.int32, device=DEV))
        c.n_prompt.fill_(0)
        c.S.zero_()
    want = V0[0, :, dead:].double().mean(1).repeat_interleave(Hq // Hkv, 0)
    got, single = (torch.zeros(T, 1, 1, Hq, d, device=DEV) for _ in range(2))
    B.dynts_decode_loop(a.ctx, T, q, k, v, got, a.keep_idx, a.new_len, out_step_stride=got[0].numel())
    _single_steps(B, b, (q, k, v), single)
    alone, lse = torch.zeros(1, Hq, d, device=DEV), torch.zeros(1, Hq, device=DEV)
    for c in (a, b):
        B.dynts_update_scores(c.ctx, 0)
    gain = torch.zeros(Hkv, n0 + T, dtype=torch.float64, device=DEV)
    gain[:, dead:n0] = T * (Hq // Hkv) / (n0 - dead)
    for c in (a, b):
        assert float((c.S[0, 0, :, :n0 + T].double() - gain).abs().max()) <= 1e-6 * float(gain.max())
    B.dynts_decode_attend(b.ctx, 0, q[0, 0], alone, lse=lse)
    for x in (got, single, alone):
        assert float((x.double().view(-1, Hq, d) - want).abs().max()) <= 1e-5
    assert float((lse.double() - np.log(n0 - dead)).abs().max()) <= 1e-5


@pytest.mark.parametrize("Nb,Hq,Hkv,d,cap", FORMS[2:])
@pytest.mark.parametrize("room", ["none", "part", "all"])
def test_loops_with_and_without_room_for_runs(B, Nb, Hq, Hkv, d, cap, room):
    """A workspace that ends before, inside and behind the room for the partials of runs: the same bits, and nothing written behind it."""
    g = torch.Generator(device=DEV)
    g.manual_seed(cap + 3)
    T = 20
    a, b = _caches(B, g, 1, Nb, Hq, Hkv, d, cap, torch.tensor(cap - 50))
    need, full = B.dynts_workspace_bytes(a.cfg), B.dynts_ctx_workspace_bytes(a.ctx)
    size = {"none": need, "part": (need + full) // 2, "all": full}[room]
    space = torch.zeros(full + 4096, dtype=torch.uint8, device=DEV)
    space[size:] = 0xA5
    B.dynts_bind(a.ctx, a.K, a.V, a.S, a.pos, a.seq_len, a.next_pos, a.n_prompt, space[:size], a.status)
    x = _tokens(g, T, 1, Nb, Hq, Hkv, d)
    got, want = (torch.zeros(T, 1, Nb, Hq, d, device=DEV) for _ in range(2))
    B.dynts_decode_loop(a.ctx, T, *x, got, a.keep_idx, a.new_len, out_step_stride=got[0].numel())
    _single_steps(B, b, x, want)
    assert torch.equal(got, want) and bool((space[size:] == 0xA5).all())
    assert bool(space[need:size].any()) == (room == "all")  # (that is where a run leaves its partials)
    _same(a, b, 1, Nb)
