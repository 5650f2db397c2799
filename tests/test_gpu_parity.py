"""GPU parity: the HIP path, called through the C ABI, against the float64 oracle on the same
seeded synthetic inputs."""
import numpy as np
import pytest
import torch

from oracle import dynts_oracle as orc
from paper_2601_18383_amd import configs, synth
from tests.helpers import SideBySide, assert_close, f64, i32

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2601_18383_amd import binding
    return binding


def _bf16(rng, *shape, scale=1.0):
    return torch.from_numpy(rng.standard_normal(shape).astype(np.float32) * scale).to(torch.bfloat16)


def _pair(B, Nb, Hq, Hkv, d, M_max, budget, window, E, mode, external=False, scale=0.0, launch_shape=None):
    cap = M_max + budget + window + E
    cache = B.Cache(1, Nb, Hq, Hkv, d, cap, budget, window, E, softmax_scale=scale, external_scores=external,
                    launch_shape=launch_shape)
    o = orc.OracleLayer(Nb, Hq, Hkv, d, cap, budget, window, E,
                        softmax_scale=scale if scale else None, external_scores=external)
    return SideBySide(B, cache, 0, o, mode), cap


@pytest.mark.parametrize("mode", ["unfused", "fused", "step", "step+hint", "fused+hint", "step+hintall"])
@pytest.mark.parametrize("d,Hq,Hkv", [(64, 8, 2), (128, 28, 4), (128, 6, 6), (128, 16, 1)])
def test_trajectory_small(B, mode, d, Hq, Hkv):
    """Several tiles, a ragged tail, ragged prompts, several evictions, a sequence that finishes early."""
    rng = np.random.default_rng(100 + d + Hq)
    Nb, M_max, budget, window, E, T = 3, 37, 150, 19, 13, 260
    sbs, cap = _pair(B, Nb, Hq, Hkv, d, M_max, budget, window, E, mode)
    m = [37, 5, 20]
    sbs.prefill(_bf16(rng, Nb, Hkv, M_max, d), _bf16(rng, Nb, Hkv, M_max, d), m)
    last = [T, 90, T]
    for t in range(1, T + 1):
        active = np.array([t <= last[b] for b in range(Nb)], np.uint8)
        q = _bf16(rng, Nb, Hq, d, scale=1.5)
        k = _bf16(rng, Nb, Hkv, d)
        v = _bf16(rng, Nb, Hkv, d)
        sbs.step(q, k, v, active=active, check_scores=(t % 5 == 0 or mode == "unfused"))
    sbs.check_scores()
    sbs.check_state()
    assert sbs.evictions >= 5
    assert int(sbs.c.status.item()) == 0
    # the finished sequence was left alone
    assert int(sbs.c.seq_len[0, 1].item()) == sbs.o.seq_len[1]


@pytest.mark.parametrize("hint", ["", "+hint"])
@pytest.mark.parametrize("waves", [4, 8])
@pytest.mark.parametrize("d,Hq,Hkv", [(64, 8, 2), (128, 28, 4)])
def test_trajectory_single_workgroup(B, d, Hq, Hkv, waves, hint):
    """One workgroup per (sequence, KV head), 4 or 8 waves: every wave walks a ragged range of slots behind its
    first tile, the launch shape of the large workloads, here at a size the oracle replays step by step."""
    rng = np.random.default_rng(500 + d + Hq)
    Nb, M_max, budget, window, E, T = 2, 41, 330, 23, 57, 560
    sbs, cap = _pair(B, Nb, Hq, Hkv, d, M_max, budget, window, E, "step" + hint, launch_shape=(1, waves))
    sbs.prefill(_bf16(rng, Nb, Hkv, M_max, d), _bf16(rng, Nb, Hkv, M_max, d), [41, 7])
    for t in range(1, T + 1):
        sbs.step(_bf16(rng, Nb, Hq, d, scale=1.5), _bf16(rng, Nb, Hkv, d), _bf16(rng, Nb, Hkv, d),
                 check_scores=(t % 11 == 0))
    sbs.check_scores()
    sbs.check_state()
    assert sbs.evictions >= 3 and int(sbs.c.status.item()) == 0


@pytest.mark.parametrize("mode", ["fused", "step"])
def test_trajectory_paper_shaped_schedule(B, mode):
    """The paper's own budget shape (Sec. 6.1, inference settings) in small: a wide local window, and a
    trigger that keeps 0.4 of the other tokens, so one trigger evicts many rows at once and
    budget + window is not a multiple of the period."""
    rng = np.random.default_rng(4242)
    Nb, Hq, Hkv, d = 2, 28, 4, 128
    M_max, total, window = 21, 250, 100
    budget = int(round(0.4 * (total - window)))
    E, T = total - window - budget, 640
    sbs, cap = _pair(B, Nb, Hq, Hkv, d, M_max, budget, window, E, mode)
    sbs.prefill(_bf16(rng, Nb, Hkv, M_max, d), _bf16(rng, Nb, Hkv, M_max, d), [21, 9])
    lens = []
    for t in range(1, T + 1):
        sbs.step(_bf16(rng, Nb, Hq, d, scale=1.5), _bf16(rng, Nb, Hkv, d), _bf16(rng, Nb, Hkv, d),
                 check_scores=(t % 45 == 0))
        lens.append(int(sbs.o.seq_len[0]))
    sbs.check_scores()
    sbs.check_state()
    assert sbs.evictions == (T - total) // E + 1
    assert max(lens) == 21 + total - 1 and min(lens[total:]) == 21 + budget + window
    assert int(sbs.c.status.item()) == 0


def test_cfg1_full_trajectory(B):
    """Config 1 end to end: 512 steps, 22 evictions, planted critical keys."""
    wl = configs.get("cfg1")
    gen = synth.Synth(wl, "cpu")
    cache = B.Cache.for_workload(wl)
    o = orc.OracleLayer(wl.batch, wl.n_q_heads, wl.n_kv_heads, wl.head_dim, wl.capacity, wl.budget,
                        wl.window, wl.evict_every)
    sbs = SideBySide(B, cache, 0, o, "step")
    K0, V0 = gen.prompt_kv(0)
    sbs.prefill(K0, V0, [wl.prompt] * wl.batch)
    T = wl.steps[0]
    steps = torch.arange(1, T + 1)
    q = gen.q(0, steps)
    k, v = gen.kv(0, steps)
    crit = gen.critical(0, steps)
    for t in range(1, T + 1):
        sbs.step(q[t - 1], k[t - 1], v[t - 1], check_scores=(t % 16 == 7))
    sbs.check_scores()
    sbs.check_state()
    assert sbs.evictions == 22
    assert o.seq_len[0] == wl.steady_len
    # meaning check: planted critical tokens that left the local window are retained
    left = [wl.prompt + t - 1 for t in range(1, T - wl.window + 1) if crit[t - 1, 0]]
    kept = set(i32(cache.pos[0, 0, 0, :wl.steady_len]).tolist())
    recall = sum(p in kept for p in left) / max(1, len(left))
    assert recall >= 0.9, recall


def _score_cases(rng, nc):
    """Hand-made score arrays: long equal runs, signed zeros, denormals, infinities, negatives."""
    cases = []
    cases.append(np.full(nc, 0.25, np.float32))
    cases.append(rng.integers(0, 3, nc).astype(np.float32))
    cases.append(rng.choice(np.array([0.0, -0.0, 1e-45, -1e-45, 1e-38], np.float32), nc))
    cases.append(rng.standard_normal(nc).astype(np.float32))
    cases.append(np.arange(nc, dtype=np.float32))
    cases.append(-np.arange(nc, dtype=np.float32))
    a = rng.random(nc).astype(np.float32)
    a[rng.integers(0, nc, 5)] = np.inf
    a[rng.integers(0, nc, 5)] = -np.inf
    cases.append(a)
    a = rng.random(nc).astype(np.float32)
    cut = np.sort(a)[nc // 2]
    a[rng.integers(0, nc, nc // 3)] = cut  # a long run of ties exactly at a plausible cut
    cases.append(a)
    cases.append(np.float32(1.0) + rng.integers(0, 4, nc).astype(np.float32) * np.float32(2 ** -23))
    return cases


@pytest.mark.parametrize("nc,k_keep,window,M", [(300, 100, 16, 10), (2112, 2048, 128, 256), (1040, 1024, 32, 128),
                                                  (4160, 4096, 128, 256), (70, 0, 3, 0), (33, 40, 0, 4), (1, 1, 0, 0),
                                                  (5000, 1500, 2000, 100)])
def test_select_bit_exact_on_given_scores(B, nc, k_keep, window, M):
    """Selection on identical score arrays must equal the oracle's bit for bit, ties included."""
    rng = np.random.default_rng(nc * 7 + k_keep)
    cases = _score_cases(rng, nc + window)
    Nb, Hkv = len(cases), 2
    n = M + nc + window
    cap = n + 8
    cache = B.Cache(1, Nb, 2 * Hkv, Hkv, 64, cap, 1, window, 8, external_scores=True)
    S = np.zeros((Nb, Hkv, cap), np.float32)
    for b, a in enumerate(cases):
        S[b, 0, M:n] = a
        S[b, 1, M:n] = a[::-1]
    S[:, :, :M] = np.inf
    pos = np.broadcast_to(np.arange(cap, dtype=np.int32) * 3, (Nb, Hkv, cap)).copy()
    seq_len = np.full(Nb, n, np.int32)
    n_prompt = np.full(Nb, M, np.int32)
    cache.S[0].copy_(torch.from_numpy(S))
    cache.pos[0].copy_(torch.from_numpy(pos))
    cache.seq_len[0].copy_(torch.from_numpy(seq_len))
    cache.n_prompt.copy_(torch.from_numpy(n_prompt))
    trig = np.ones(Nb, np.uint8)
    trig[1] = 0
    cache.keep_idx.fill_(-1)
    B.dynts_select_evict(cache.ctx, 0, cache.keep_idx, cache.new_len, k_keep, torch.from_numpy(trig).cuda())
    keep_ref, len_ref = orc.select(S.astype(np.float64), pos, seq_len, n_prompt, window, k_keep, trig)
    assert np.array_equal(i32(cache.new_len), len_ref)
    assert np.array_equal(i32(cache.keep_idx), keep_ref)
    assert int(cache.status.item()) == 0


@pytest.mark.parametrize("nc,k_keep,window,M", [(1024, 512, 1, 0), (1025, 1024, 7, 3), (4097, 4096, 0, 0), (16300, 9000, 60, 16),
                                                  (16385, 16384, 5, 2), (33000, 17000, 10, 40)])
def test_select_at_the_edges_of_its_rounds(B, nc, k_keep, window, M):
    """1024 candidates a round, 16 rounds counted together, 16384 slots whose keys are held in LDS."""
    test_select_bit_exact_on_given_scores(B, nc, k_keep, window, M)


@pytest.mark.parametrize("Hq,Hkv,d,cap,k_keep", [(2, 2, 64, 90, 30), (28, 4, 128, 1100, 600), (8, 1, 64, 1030, 1), (7, 1, 128, 4120, 3000),
                                                 (16, 2, 64, 5120, 3000), (16, 2, 64, 5121, 3000), (9, 1, 128, 700, 300),
                                                 (8, 2, 64, 9000, 8000)])
def test_select_makes_the_update_from_kept_logits(B, Hq, Hkv, d, cap, k_keep):
    """A trigger behind an announced step leaves the scores, bit for bit, that the update by a call of its own leaves, of triggered,
    untriggered and idle sequences, and selects from them."""
    rng = np.random.default_rng(cap + Hq)
    Nb, M, window = 4, 11, 17
    lens = np.array([cap - 1, cap // 2, cap - 3, M + 3], np.int32)
    trig = torch.tensor([1, 1, 0, 1], dtype=torch.uint8, device="cuda")
    active = torch.tensor([1, 0, 1, 1], dtype=torch.uint8, device="cuda")
    K, V = _bf16(rng, Nb, Hkv, cap, d).cuda(), _bf16(rng, Nb, Hkv, cap, d).cuda()
    S = torch.from_numpy(rng.random((Nb, Hkv, cap)).astype(np.float32)).cuda()
    q, k, v = _bf16(rng, Nb, Hq, d).cuda(), _bf16(rng, Nb, Hkv, d).cuda(), _bf16(rng, Nb, Hkv, d).cuda()
    out = torch.zeros(Nb, Hq, d, device="cuda")
    got = []
    for by_itself in (True, False):
        c = B.Cache(1, Nb, Hq, Hkv, d, cap, 1, window, 1)
        c.K[0].copy_(K); c.V[0].copy_(V); c.S[0].copy_(S)
        c.seq_len[0].copy_(torch.from_numpy(lens)); c.next_pos[0].copy_(torch.from_numpy(lens)); c.n_prompt.fill_(M)
        B.dynts_hint_trigger(c.ctx, 0)
        B.dynts_decode_step(c.ctx, 0, q, k, v, out, active=active)
        if by_itself:
            B.dynts_update_scores(c.ctx, 0)
        c.keep_idx.fill_(-1)
        B.dynts_select_evict(c.ctx, 0, c.keep_idx, c.new_len, k_keep, trig)
        scores = c.S.clone()
        B.dynts_compact(c.ctx, 0, c.keep_idx, c.new_len, trig)  # (no update is owed any more)
        got.append((scores, c.keep_idx.clone(), c.new_len.clone()))
        assert int(c.status.item()) == 0
    for x, y in zip(*got):
        assert torch.equal(x, y)
    scores, keep, new_len = got[0]
    n = (lens + np.array([1, 0, 1, 1])).astype(np.int32)
    assert not torch.equal(scores[0, 0, :, M:int(n[0])], S[0, :, M:int(n[0])])
    keep_ref, len_ref = orc.select(f64(scores[0]), np.broadcast_to(np.arange(cap, dtype=np.int32), (Nb, Hkv, cap)).copy(), n,
                                   np.full(Nb, M, np.int32), window, k_keep, i32(trig).astype(np.uint8))
    assert np.array_equal(i32(new_len), len_ref) and np.array_equal(i32(keep), keep_ref)


@pytest.mark.parametrize("Nb,nc,k_keep", [(129, 512, 300), (129, 2300, 2200), (257, 2600, 100),             # 512 threads a workgroup
                                          (257, 16500, 9000),                                                # ... keys not held in LDS
                                          (385, 255, 100), (385, 256, 255), (385, 1025, 1024), (400, 1150, 7)])  # 256 threads
def test_select_of_many_units(B, Nb, nc, k_keep):
    """Smaller workgroups: other numbers of rounds, of counts a round, and of threads a bin."""
    rng = np.random.default_rng(nc + Nb)
    Hkv, window, M = 2, 5, 11
    n, cap = M + nc + window, M + nc + window + 3
    cases = _score_cases(rng, nc + window)
    cache = B.Cache(1, Nb, Hkv, Hkv, 64, cap, 1, window, 1, external_scores=True)
    S = np.zeros((Nb, Hkv, cap), np.float32)
    for b in range(Nb):
        for h in range(Hkv):
            S[b, h, M:n] = np.roll(cases[(b + h) % len(cases)], 37 * b)
    S[:, :, :M] = np.inf
    seq_len = np.where(np.arange(Nb) % 5 == 3, n - nc // 2, n).astype(np.int32)
    cache.S[0].copy_(torch.from_numpy(S)); cache.seq_len[0].copy_(torch.from_numpy(seq_len)); cache.n_prompt.fill_(M)
    trig = (np.arange(Nb) % 7 != 1).astype(np.uint8)
    cache.keep_idx.fill_(-1)
    B.dynts_select_evict(cache.ctx, 0, cache.keep_idx, cache.new_len, k_keep, torch.from_numpy(trig).cuda())
    pos = np.broadcast_to(np.arange(cap, dtype=np.int32), (Nb, Hkv, cap)).copy()
    keep_ref, len_ref = orc.select(S.astype(np.float64), pos, seq_len, np.full(Nb, M, np.int32), window, k_keep, trig)
    assert np.array_equal(i32(cache.new_len), len_ref)
    assert np.array_equal(i32(cache.keep_idx), keep_ref)
    assert int(cache.status.item()) == 0


@pytest.mark.parametrize("Nb,Hkv,G,cap", [(129, 2, 4, 700), (260, 2, 1, 2560), (260, 2, 2, 5120), (400, 2, 8, 100), (400, 2, 3, 1100)])
def test_update_from_kept_logits_in_selections_of_many_units(B, Nb, Hkv, G, cap):
    """The scores and lists that the update by a call of its own leads to, bit for bit, with the smaller workgroups."""
    g = torch.Generator(device="cuda").manual_seed(cap)
    bf = lambda *shape: torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(generator=g)
    M, window, d = 7, 9, 64
    K, V, q, k, v = bf(Nb, Hkv, cap, d), bf(Nb, Hkv, cap, d), bf(Nb, Hkv * G, d), bf(Nb, Hkv, d), bf(Nb, Hkv, d)
    S = torch.rand(Nb, Hkv, cap, generator=g, device="cuda")
    lens = torch.tensor([cap - 1 - (b * 13) % (cap // 2) for b in range(Nb)], dtype=torch.int32, device="cuda")
    trig = torch.tensor([b % 4 != 2 for b in range(Nb)], dtype=torch.uint8, device="cuda")
    active = torch.tensor([b % 5 != 1 for b in range(Nb)], dtype=torch.uint8, device="cuda")
    out = torch.zeros(Nb, Hkv * G, d, device="cuda")
    got = []
    for by_itself in (True, False):
        c = B.Cache(1, Nb, Hkv * G, Hkv, d, cap, 1, window, 1)
        c.K[0].copy_(K); c.V[0].copy_(V); c.S[0].copy_(S)
        c.seq_len[0].copy_(lens); c.next_pos[0].copy_(lens); c.n_prompt.fill_(M)
        B.dynts_hint_trigger(c.ctx, 0)
        B.dynts_decode_step(c.ctx, 0, q, k, v, out, active=active)
        if by_itself:
            B.dynts_update_scores(c.ctx, 0)
        c.keep_idx.fill_(-1)
        B.dynts_select_evict(c.ctx, 0, c.keep_idx, c.new_len, cap // 3, trig)
        got.append((c.S.clone(), c.keep_idx.clone(), c.new_len.clone()))
        assert int(c.status.item()) == 0
        c.close()
    for x, y in zip(*got):
        assert torch.equal(x, y)
    assert not torch.equal(got[0][0][0], S)


@pytest.mark.parametrize("paged", [False, True])
@pytest.mark.parametrize("d,Nb,Hkv,G,n,cap", [(128, 3, 2, 7, 2600, 2610), (128, 3, 2, 16, 2400, 2500), (128, 150, 4, 1, 47, 60),
                                              (64, 150, 4, 4, 330, 340), (64, 2, 1, 16, 2700, 2705)])
def test_update_by_itself_from_a_pass_over_k(B, d, Nb, Hkv, G, n, cap, paged):
    """K turned half a tile at a time; caches on either side of 2500 slots, more and fewer units than compute units, ragged lengths."""
    g = torch.Generator(device="cuda").manual_seed(cap + d)
    bf = lambda *shape: torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(generator=g)
    M, Hq = 5, Hkv * G
    c = (B.PagedCache if paged else B.Cache)(1, Nb, Hq, Hkv, d, cap, 1, 1, 1)
    K, q, out = bf(Nb, Hkv, n, d), bf(Nb, Hq, d), torch.zeros(Nb, Hq, d, device="cuda")
    m = torch.tensor([n - (b % 3) * (n // 4) for b in range(Nb)], dtype=torch.int32, device="cuda")
    B.dynts_prefill(c.ctx, 0, K, bf(Nb, Hkv, n, d), m)
    c.n_prompt.fill_(M)
    c.S.fill_(0.0)
    B.dynts_decode_attend_update(c.ctx, 0, q, out)
    B.dynts_update_scores(c.ctx, 0)
    got = c.S[0].double()
    for b in range(Nb):
        nb = int(m[b])
        x = torch.matmul(q[b].double().view(Hkv, G, d), K[b, :, :nb].double().transpose(1, 2)) / np.sqrt(d)
        w = torch.softmax(x, dim=-1).sum(1)
        w[:, :M] = 0.0
        assert_close(got[b, :, :nb].cpu().numpy(), w.cpu().numpy(), "S of sequence %d" % b)
        assert not got[b, :, nb:].any()
    assert int(c.status.item()) == 0


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("d,cap", [(64, 4600), (128, 4096), (64, 100)])
def test_compact_of_lists_beyond_what_is_held(B, d, cap, shift):
    """4096 entries of the keep list are held on chip: one slot evicted in front of, at and behind them, and none."""
    rng = np.random.default_rng(cap + d)
    gone = [0, min(cap, 4096) - 1, cap - 1, cap]
    c = B.Cache(1, len(gone), 1, 1, d, cap, 1, 1, 1)
    K, V = _bf16(rng, len(gone), 1, cap, d).cuda(), _bf16(rng, len(gone), 1, cap, d).cuda()
    c.K[0].copy_(K); c.V[0].copy_(V)
    c.S[0].copy_(torch.arange(cap, device="cuda").float()); c.pos[0].copy_(torch.arange(cap, device="cuda"))
    c.seq_len.fill_(cap)
    for b, slot in enumerate(gone):
        idx = torch.tensor([j for j in range(cap) if j != slot], dtype=torch.int32, device="cuda")[shift:]
        c.keep_idx[b, 0, :len(idx)] = idx
        c.new_len[b] = len(idx)
    idx, m = c.keep_idx.clone(), c.new_len.tolist()
    B.dynts_compact(c.ctx, 0, c.keep_idx, c.new_len)
    assert c.seq_len[0].tolist() == m
    for b in range(len(gone)):
        src = idx[b, 0, :m[b]].long()
        assert torch.equal(c.K[0, b, 0, :m[b]], K[b, 0, src]) and torch.equal(c.V[0, b, 0, :m[b]], V[b, 0, src])
        assert torch.equal(c.pos[0, b, 0, :m[b]].long(), src) and torch.equal(c.S[0, b, 0, :m[b]], src.float())


@pytest.mark.parametrize("paged", [False, True])
@pytest.mark.parametrize("d,Nb,Hkv,cap", [(64, 3, 2, 400), (64, 161, 2, 1000), (128, 107, 2, 1100), (64, 256, 2, 300), (64, 256, 2, 301),
                                          (128, 118, 2, 4200)])
def test_compact_with_either_workgroup(B, d, Nb, Hkv, cap, paged):
    """256 threads where there are more than 1280 workgroups and the cache is small (or beyond 4000 slots), 512 elsewhere; lists up to, at and beyond the 1024 entries
    that the smaller ones hold on chip."""
    g = torch.Generator(device="cuda").manual_seed(cap + d)
    c = (B.PagedCache if paged else B.Cache)(1, Nb, Hkv, Hkv, d, cap, 1, 1, 1)
    bf = lambda: torch.empty(Nb, Hkv, cap, d, dtype=torch.bfloat16, device="cuda").normal_(generator=g)
    K, V = bf(), bf()
    B.dynts_prefill(c.ctx, 0, K, V, torch.full((Nb,), cap, dtype=torch.int32, device="cuda"))
    c.S[0].copy_(torch.arange(cap, device="cuda").float()); c.pos[0].copy_(torch.arange(cap, device="cuda"))
    some = [cap // 3, cap - 1, min(cap, 1024), min(cap, 1025), cap]  # entries of the list
    idx = torch.zeros(Nb, Hkv, cap, dtype=torch.int64, device="cuda")
    m = [some[b % len(some)] for b in range(Nb)]
    for b in range(Nb):
        pick = torch.rand(Hkv, cap, generator=g, device="cuda").argsort(dim=1)[:, :m[b]]
        idx[b, :, :m[b]] = pick.sort(dim=1).values
    c.keep_idx.copy_(idx)
    c.new_len.copy_(torch.tensor(m, dtype=torch.int32))
    B.dynts_compact(c.ctx, 0, c.keep_idx, c.new_len)
    assert c.seq_len[0].tolist() == m
    Kc, Vc = c.K[0], c.V[0]
    for b in range(Nb):
        src = idx[b, :, :m[b]]
        rows = src.unsqueeze(-1).expand(Hkv, m[b], d)
        assert torch.equal(Kc[b, :, :m[b]], torch.gather(K[b], 1, rows)) and torch.equal(Vc[b, :, :m[b]], torch.gather(V[b], 1, rows))
        assert torch.equal(c.pos[0, b, :, :m[b]].long(), src) and torch.equal(c.S[0, b, :, :m[b]], src.float())


@pytest.mark.parametrize("d", [64, 128])
def test_compact_bit_exact(B, d):
    rng = np.random.default_rng(5 + d)
    Nb, Hkv, cap = 4, 3, 777
    cache = B.Cache(1, Nb, Hkv, Hkv, d, cap, 10, 5, 5)
    K = _bf16(rng, Nb, Hkv, cap, d)
    V = _bf16(rng, Nb, Hkv, cap, d)
    S = rng.random((Nb, Hkv, cap)).astype(np.float32)
    pos = np.cumsum(rng.integers(1, 4, (Nb, Hkv, cap)), -1).astype(np.int32)
    seq_len = np.array([777, 500, 64, 300], np.int32)
    cache.K[0].copy_(K); cache.V[0].copy_(V)
    cache.S[0].copy_(torch.from_numpy(S)); cache.pos[0].copy_(torch.from_numpy(pos))
    cache.seq_len[0].copy_(torch.from_numpy(seq_len))
    keep = np.full((Nb, Hkv, cap), -1, np.int32)
    new_len = np.zeros(Nb, np.int32)
    frac = [0.5, 0.97, 0.3, 1.0]
    for b in range(Nb):
        m = int(seq_len[b] * frac[b])
        new_len[b] = m
        for h in range(Hkv):
            sel = np.sort(rng.choice(seq_len[b], m, replace=False))
            if b == 1:  # a long unmoved prefix
                rest = np.sort(rng.choice(np.arange(400, seq_len[b]), m - 400, replace=False))
                sel = np.concatenate([np.arange(400), rest])
            keep[b, h, :m] = sel
    trig = np.array([1, 1, 0, 1], np.uint8)
    cache.keep_idx.copy_(torch.from_numpy(keep)); cache.new_len.copy_(torch.from_numpy(new_len))
    B.dynts_compact(cache.ctx, 0, cache.keep_idx, cache.new_len, torch.from_numpy(trig).cuda())
    Ko, Vo, So, po, sl = f64(K), f64(V), S.astype(np.float64), pos.copy(), seq_len.copy()
    orc.compact(Ko, Vo, So, po, sl, keep, new_len, trig)
    assert np.array_equal(i32(cache.seq_len[0]), sl)
    for b in range(Nb):
        n = sl[b]
        assert np.array_equal(f64(cache.K[0, b, :, :n]), Ko[b, :, :n])
        assert np.array_equal(f64(cache.V[0, b, :, :n]), Vo[b, :, :n])
        assert np.array_equal(f64(cache.S[0, b, :, :n]), So[b, :, :n])
        assert np.array_equal(i32(cache.pos[0, b, :, :n]), po[b, :, :n])
    # the untriggered sequence is untouched, tail included
    assert np.array_equal(f64(cache.K[0, 2]), f64(K[2]))


def test_attention_edge_cases(B):
    """n = 1, one dominant key, uniform attention, large logits: closed forms on the GPU path too."""
    rng = np.random.default_rng(9)
    Nb, Hq, Hkv, d, cap = 4, 8, 2, 128, 600
    cache = B.Cache(1, Nb, Hq, Hkv, d, cap, 500, 10, 10, softmax_scale=1.0)
    o = orc.OracleLayer(Nb, Hq, Hkv, d, cap, 500, 10, 10, softmax_scale=1.0)
    sbs = SideBySide(B, cache, 0, o, "unfused")
    M = [1, 300, 590, 33]
    K0 = _bf16(rng, Nb, Hkv, 590, d, scale=0.1)
    V0 = _bf16(rng, Nb, Hkv, 590, d)
    K0[1, :, 123] = 3.0   # a dominant key for an all-ones query: logit 384 vs ~0
    K0[3] = 0.5           # identical keys: uniform attention
    sbs.prefill(K0, V0, M)
    q = torch.ones(Nb, Hq, d).to(torch.bfloat16)
    # attend over the prompt only (no append): n = M
    B.dynts_decode_attend(cache.ctx, 0, q.cuda(), sbs.out, sbs.lse)
    out_ref, alpha, lse_ref = o.attend(f64(q))
    assert_close(f64(sbs.out), out_ref, "out")
    assert_close(f64(sbs.lse), lse_ref, "lse")
    got = f64(sbs.out)
    assert np.array_equal(got[0, 0], f64(V0[0, 0, 0]))                 # n = 1: the value row itself
    assert np.allclose(got[1, 0], f64(V0[1, 0, 123]), atol=1e-6)      # one-hot
    assert np.allclose(got[3, 5], f64(V0[3, 1, :33]).mean(0), atol=2e-3)


def test_degenerate_batches_and_limits(B):
    """All sequences finished; an empty question window (the first token attends to itself alone); a full cache
    (the append is dropped, the sequence is left alone and the status word says so)."""
    rng = np.random.default_rng(12)
    dev = torch.device("cuda:0")
    Nb, Hq, Hkv, d = 3, 8, 2, 64
    budget, window, E = 6, 2, 2
    cap = 4 + budget + window + E
    cache = B.Cache(1, Nb, Hq, Hkv, d, cap, budget, window, E)
    o = orc.OracleLayer(Nb, Hq, Hkv, d, cap, budget, window, E)
    sbs = SideBySide(B, cache, 0, o, "step")
    sbs.prefill(_bf16(rng, Nb, Hkv, 4, d), _bf16(rng, Nb, Hkv, 4, d), [0, 4, 2])
    # nobody is active: nothing moves
    q, k, v = _bf16(rng, Nb, Hq, d), _bf16(rng, Nb, Hkv, d), _bf16(rng, Nb, Hkv, d)
    before = (cache.K.clone(), cache.S.clone(), cache.seq_len.clone())
    sbs.out.fill_(7.0)
    B.dynts_decode_step(cache.ctx, 0, q.to(dev), k.to(dev), v.to(dev), sbs.out,
                        active=torch.zeros(Nb, dtype=torch.uint8, device=dev))
    B.dynts_update_scores(cache.ctx, 0)
    assert torch.equal(cache.K, before[0]) and torch.equal(cache.S, before[1]) and torch.equal(cache.seq_len, before[2])
    assert bool((sbs.out == 7.0).all())
    # first real step: sequence 0 has no question tokens, its output is the new value row itself
    sbs.step(q, k, v)
    assert np.array_equal(f64(sbs.out)[0], np.repeat(f64(v)[0], Hq // Hkv, axis=0))
    # run without evicting until sequence 1 (4 question tokens) fills the cache
    for _ in range(cap - 4 - 1):
        B.dynts_decode_step(cache.ctx, 0, q.to(dev), k.to(dev), v.to(dev), sbs.out)
    assert int(cache.status.item()) == 0
    assert i32(cache.seq_len[0]).tolist() == [cap - 4, cap, cap - 2]
    B.dynts_update_scores(cache.ctx, 0)
    snap = (cache.K.clone(), cache.seq_len.clone())
    sbs.out.fill_(7.0)
    B.dynts_decode_step(cache.ctx, 0, q.to(dev), k.to(dev), v.to(dev), sbs.out)
    assert int(cache.status.item()) & 1                       # the append of sequence 1 was dropped ...
    assert i32(cache.seq_len[0]).tolist() == [cap - 3, cap, cap - 1]
    assert torch.equal(cache.K[0, 1], snap[0][0, 1])          # ... its rows are untouched ...
    assert bool((sbs.out[1] == 7.0).all()) and not bool((sbs.out[0] == 7.0).any())   # ... and it was not attended
    # the separate append call reports the same condition
    cache.status.zero_()
    B.dynts_update_scores(cache.ctx, 0)
    B.dynts_append(cache.ctx, 0, k.to(dev), v.to(dev))
    assert int(cache.status.item()) & 1 and i32(cache.seq_len[0]).tolist() == [cap - 2, cap, cap]


def test_long_cache_single_unit(B):
    """A cache of 40 000 slots for one (sequence, KV head): many splits, each wave a long range."""
    rng = np.random.default_rng(13)
    dev = torch.device("cuda:0")
    Hq, Hkv, d, M = 4, 1, 128, 100
    n0 = 39_987
    cap = 40_000
    cache = B.Cache(1, 1, Hq, Hkv, d, cap, cap - M - 20, 10, 10)
    o = orc.OracleLayer(1, Hq, Hkv, d, cap, cap - M - 20, 10, 10)
    K = _bf16(rng, 1, Hkv, n0, d)
    V = _bf16(rng, 1, Hkv, n0, d)
    S = torch.from_numpy(rng.random((1, Hkv, n0)).astype(np.float32))
    S[:, :, :M] = float("inf")
    cache.K[0, :, :, :n0] = K.to(dev); cache.V[0, :, :, :n0] = V.to(dev); cache.S[0, :, :, :n0] = S.to(dev)
    cache.pos[0, :, :, :n0] = torch.arange(n0, dtype=torch.int32, device=dev)
    cache.seq_len.fill_(n0); cache.next_pos.fill_(n0); cache.n_prompt.fill_(M)
    o.K[:, :, :n0] = f64(K); o.V[:, :, :n0] = f64(V); o.S[:, :, :n0] = f64(S)
    o.pos[:, :, :n0] = np.arange(n0); o.seq_len[:] = n0; o.next_pos[:] = n0; o.n_prompt[:] = M
    sbs = SideBySide(B, cache, 0, o, "step")
    for t in range(3):
        sbs.step(_bf16(rng, 1, Hq, d, scale=1.5), _bf16(rng, 1, Hkv, d), _bf16(rng, 1, Hkv, d), check_scores=(t == 2))
    assert int(cache.seq_len.item()) == n0 + 3 and int(cache.status.item()) == 0
    # selection and compaction at this length: keep 1000 of the ~39 880 candidates
    cache.keep_idx.fill_(-1)
    B.dynts_select_evict(cache.ctx, 0, cache.keep_idx, cache.new_len, 1000)
    keep_same, len_same = orc.select(f64(cache.S[0]), i32(cache.pos[0]), o.seq_len, o.n_prompt, 10, 1000)
    assert np.array_equal(i32(cache.new_len), len_same) and np.array_equal(i32(cache.keep_idx), keep_same)
    B.dynts_compact(cache.ctx, 0, cache.keep_idx, cache.new_len)
    o.compact(keep_same, len_same)
    n2 = int(len_same[0])
    assert n2 == M + 1000 + 10 and int(cache.seq_len.item()) == n2
    assert np.array_equal(f64(cache.K[0])[:, :, :n2], o.K[:, :, :n2]) and np.array_equal(f64(cache.V[0])[:, :, :n2], o.V[:, :, :n2])
    assert np.array_equal(i32(cache.pos[0])[:, :, :n2], o.pos[:, :, :n2])


@pytest.mark.parametrize("external", [False, True])
def test_native_loop_equals_single_calls(B, external):
    """dynts_decode_loop over several layers (per-step input slabs, ragged activity, trigger steps, one output slab
    per step) does exactly what the same calls issued one by one do (trigger steps announced, as the loop announces
    them): bit-identical caches and outputs."""
    rng = np.random.default_rng(21)
    dev = torch.device("cuda:0")
    L, Nb, Hq, Hkv, d = 3, 4, 8, 2, 64
    M, budget, window, E, T = 6, 20, 5, 9, 70
    cap = M + budget + window + E
    q = _bf16(rng, T, L, Nb, Hq, d).to(dev)
    k = _bf16(rng, T, L, Nb, Hkv, d).to(dev)
    v = _bf16(rng, T, L, Nb, Hkv, d).to(dev)
    s = torch.from_numpy(rng.integers(0, 6, (T, Nb, Hkv)).astype(np.float32)).to(dev) if external else None
    active = (rng.random((T, Nb)) < 0.85).astype(np.uint8)
    active[:, 0] = 1
    act = torch.from_numpy(active).to(dev)
    # trigger steps from the schedule of the always-active sequence
    flags = torch.zeros(T, dtype=torch.uint8)
    for t in range(1, T + 1):
        if t >= budget + window + E and (t - (budget + window + E)) % E == 0:
            flags[t - 1] = 1
    trig = torch.ones((T, Nb), dtype=torch.uint8, device=dev)   # every sequence is trimmed on a trigger step
    K0, V0 = _bf16(rng, Nb, Hkv, M, d).to(dev), _bf16(rng, Nb, Hkv, M, d).to(dev)
    m = torch.tensor([6, 2, 0, 4], dtype=torch.int32, device=dev)

    def fresh():
        c = B.Cache(L, Nb, Hq, Hkv, d, cap, budget, window, E, external_scores=external)
        for l in range(L):
            B.dynts_prefill(c.ctx, l, K0, V0, m)
        return c

    a, b_ = fresh(), fresh()
    outs_a = torch.zeros((T, L, Nb, Hq, d), dtype=torch.float32, device=dev)
    outs_b = torch.zeros_like(outs_a)
    B.dynts_decode_loop(a.ctx, T, q, k, v, outs_a, a.keep_idx, a.new_len, s_new=s, active=act, evict_steps=flags,
                        trigger=trig, out_step_stride=outs_a[0].numel())
    for t in range(T):
        for l in range(L):
            if flags[t]:
                B.dynts_hint_trigger(b_.ctx, l)   # as the loop does on its trigger steps
            B.dynts_decode_step(b_.ctx, l, q[t, l], k[t, l], v[t, l], outs_b[t, l], s_new=s[t] if external else None,
                                active=act[t])
            if flags[t]:
                B.dynts_select_evict(b_.ctx, l, b_.keep_idx, b_.new_len, budget, trig[t])
                B.dynts_compact(b_.ctx, l, b_.keep_idx, b_.new_len, trig[t])
    for l in range(L):
        B.dynts_update_scores(a.ctx, l)
        B.dynts_update_scores(b_.ctx, l)
    torch.cuda.synchronize()
    assert torch.equal(outs_a, outs_b)
    assert torch.equal(a.seq_len, b_.seq_len) and torch.equal(a.next_pos, b_.next_pos)
    for l in range(L):
        for bb in range(Nb):
            n = int(a.seq_len[l, bb])
            assert torch.equal(a.K[l, bb, :, :n], b_.K[l, bb, :, :n]) and torch.equal(a.V[l, bb, :, :n], b_.V[l, bb, :, :n])
            assert torch.equal(a.S[l, bb, :, :n], b_.S[l, bb, :, :n]) and torch.equal(a.pos[l, bb, :, :n], b_.pos[l, bb, :, :n])
    assert int(a.seq_len[0, 0]) < cap and int(flags.sum()) >= 3
    assert int(a.status.item()) == 0 and int(b_.status.item()) == 0


@pytest.mark.parametrize("L,Nb,Hq,Hkv,d,M,budget,window,E,T,external,masked", [
    (1, 1, 8, 2, 64, 64, 128, 32, 16, 200, False, False),      # one tile a wave
    (2, 3, 28, 4, 128, 37, 150, 19, 13, 230, False, True),
    (1, 2, 16, 1, 128, 17, 100, 9, 7, 150, True, True),
    (1, 1, 12, 1, 64, 255, 1, 0, 1, 9, False, False),          # runs of one step and of none
    (1, 3, 16, 1, 64, 1, 255, 0, 1, 260, False, True),         # every slot of the first tiles, one more
    (1, 2, 28, 4, 128, 100, 300, 40, 30, 420, False, True),    # two chunks, the second empty at first: partials
    (2, 2, 8, 2, 64, 50, 350, 61, 51, 600, False, True),
    (1, 2, 16, 2, 128, 250, 250, 8, 4, 280, False, False),     # all 512 slots
    (1, 1, 28, 4, 128, 200, 900, 50, 40, 1100, False, True),   # five chunks, a run longer than there is room for partials
    (2, 2, 8, 2, 64, 100, 1400, 61, 51, 1700, False, True),
    (1, 1, 32, 8, 128, 256, 4096, 128, 64, 4420, False, False),  # 18 chunks: merges of 32 at a time
    (1, 1, 8, 1, 128, 30, 2500, 100, 70, 2800, False, False),  # eight at a time
    (1, 1, 8, 1, 64, 30, 4500, 100, 70, 4800, False, True),
    (1, 1, 16, 1, 128, 30, 1500, 100, 70, 1800, True, False),  # four elements a thread, scores from outside
    (1, 45, 32, 8, 128, 60, 330, 50, 40, 460, False, False),   # two tiles a wave, one chunk
    (1, 90, 4, 2, 64, 60, 330, 50, 40, 460, True, True),
    (1, 3, 8, 2, 64, 20, 30, 10, 200, 250, False, True)])      # two triggers' worth of steps and no more room than that
def test_loop_on_caches_that_stay_on_the_chip_equals_single_calls(B, L, Nb, Hq, Hkv, d, M, budget, window, E, T, external, masked):
    """Runs of steps that the loop makes in one launch, in two calls of it (an update is owed in between): outputs, cache,
    scores before and after the owed update, lengths and status word of the same calls issued one by one, bit for bit."""
    rng = np.random.default_rng(T + d)
    dev = torch.device("cuda:0")
    cap = M + budget + window + E
    q = _bf16(rng, T, L, Nb, Hq, d, scale=1.5).to(dev)
    k, v = _bf16(rng, T, L, Nb, Hkv, d).to(dev), _bf16(rng, T, L, Nb, Hkv, d).to(dev)
    s = torch.from_numpy(rng.integers(0, 6, (T, Nb, Hkv)).astype(np.float32)).to(dev) if external else None
    act = torch.from_numpy((rng.random((T, Nb)) < 0.9).astype(np.uint8)).to(dev) if masked else None
    flags = torch.zeros(T, dtype=torch.uint8)
    flags[budget + window + E - 1::E] = 1
    K0, V0 = _bf16(rng, Nb, Hkv, M, d).to(dev), _bf16(rng, Nb, Hkv, M, d).to(dev)
    m = torch.from_numpy(rng.integers(0 if masked else M, M + 1, Nb).astype(np.int32)).to(dev)
    a, b = (B.Cache(L, Nb, Hq, Hkv, d, cap, budget, window, E, external_scores=external) for _ in range(2))
    for c in (a, b):
        for l in range(L):
            B.dynts_prefill(c.ctx, l, K0, V0, m)
    outs_a = torch.zeros((T, L, Nb, Hq, d), dtype=torch.float32, device=dev)
    outs_b = torch.zeros_like(outs_a)
    cut = T // 3 | 1
    for lo, hi in ((0, cut), (cut, T)):
        B.dynts_decode_loop(a.ctx, hi - lo, q[lo:hi], k[lo:hi], v[lo:hi], outs_a[lo:hi], a.keep_idx, a.new_len, s_new=s[lo:hi] if external else None,
                            active=act[lo:hi] if masked else None, evict_steps=flags[lo:hi].clone(), out_step_stride=outs_a[0].numel())
    for t in range(T):
        for l in range(L):
            if flags[t]:
                B.dynts_hint_trigger(b.ctx, l)
            B.dynts_decode_step(b.ctx, l, q[t, l], k[t, l], v[t, l], outs_b[t, l], s_new=s[t] if external else None, active=act[t] if masked else None)
            if flags[t]:
                B.dynts_select_evict(b.ctx, l, b.keep_idx, b.new_len, budget)
                B.dynts_compact(b.ctx, l, b.keep_idx, b.new_len)

    def same():
        assert torch.equal(outs_a, outs_b)
        assert torch.equal(a.seq_len, b.seq_len) and torch.equal(a.next_pos, b.next_pos) and torch.equal(a.status, b.status)
        for l in range(L):
            for bb in range(Nb):
                n = int(a.seq_len[l, bb])
                for x, y in ((a.K, b.K), (a.V, b.V), (a.S, b.S), (a.pos, b.pos)):
                    assert torch.equal(x[l, bb, :, :n], y[l, bb, :, :n])

    same()
    for l in range(L):
        B.dynts_update_scores(a.ctx, l)
        B.dynts_update_scores(b.ctx, l)
    same()


@pytest.mark.parametrize("d,Hq,Hkv,cap", [(64, 8, 2, 200), (128, 28, 4, 500), (128, 8, 2, 900)])
def test_loop_with_whole_tiles_at_minus_infinity(B, d, Hq, Hkv, cap):
    """Logits that overflow to -inf, over whole tiles of 32 slots (a wave's first among them), weigh nothing, in a run of steps as in
    single calls: every other slot has a logit of zero, so the outputs are the mean of their V rows (sums of fp32: 1e-5)."""
    rng = np.random.default_rng(cap + d)
    dev = torch.device("cuda:0")
    T, n0 = 5, cap - 40
    big = torch.tensor(3e38).bfloat16()
    K0 = torch.zeros((1, Hkv, n0, d), dtype=torch.bfloat16)
    K0[:, :, 32:64] = -big
    K0[:, :, 96:160] = -big
    V0 = _bf16(rng, 1, Hkv, n0, d)
    q = big.expand(T, 1, 1, Hq, d).contiguous().to(dev)
    k = torch.zeros((T, 1, 1, Hkv, d), dtype=torch.bfloat16, device=dev)
    v = _bf16(rng, T, 1, 1, Hkv, d).to(dev)
    a, b = (B.Cache(1, 1, Hq, Hkv, d, cap, cap - 80, 32, 16) for _ in range(2))
    for c in (a, b):
        B.dynts_prefill(c.ctx, 0, K0.to(dev), V0.to(dev), torch.tensor([n0], dtype=torch.int32, device=dev))
    outs_a, outs_b = torch.zeros((T, 1, 1, Hq, d), dtype=torch.float32, device=dev), torch.zeros((T, 1, 1, Hq, d), dtype=torch.float32, device=dev)
    B.dynts_decode_loop(a.ctx, T, q, k, v, outs_a, a.keep_idx, a.new_len, out_step_stride=outs_a[0].numel())
    for t in range(T):
        B.dynts_decode_step(b.ctx, 0, q[t, 0], k[t, 0], v[t, 0], outs_b[t, 0])
    assert torch.equal(outs_a, outs_b)
    alive = torch.cat([V0[0, :, :32], V0[0, :, 64:96], V0[0, :, 160:]], 1).double()
    rows = torch.cat([alive, v[:, 0, 0].cpu().double().transpose(0, 1)], 1)
    for t in range(T):
        want = rows[:, :alive.shape[1] + t + 1].mean(1).repeat_interleave(Hq // Hkv, 0)
        assert float((outs_a[t, 0, 0].cpu().double() - want).abs().max()) <= 1e-5


@pytest.mark.parametrize("L,Nb,Hq,Hkv,d,cap", [(1, 3, 8, 2, 64, 200), (2, 2, 28, 4, 128, 700), (1, 2, 16, 1, 64, 2000), (2, 1, 32, 8, 128, 4544)])
@pytest.mark.parametrize("stride", ["none", "part"])
def test_loop_whose_steps_share_their_outputs(B, L, Nb, Hq, Hkv, d, cap, stride):
    """Without a stride between the steps the outputs that stay are those of the last step that attended the sequence; with less than
    a step's outputs between them later steps overwrite parts of earlier ones: as single calls in order leave them, bit for bit."""
    rng = np.random.default_rng(cap + d)
    dev = torch.device("cuda:0")
    T, M = 40, 30
    q = _bf16(rng, T, L, Nb, Hq, d, scale=1.5).to(dev)
    k, v = _bf16(rng, T, L, Nb, Hkv, d).to(dev), _bf16(rng, T, L, Nb, Hkv, d).to(dev)
    act = torch.from_numpy((rng.random((T, Nb)) < 0.7).astype(np.uint8)).to(dev)
    act[T - 5:, 0] = 0
    n0 = cap - T
    K0, V0 = _bf16(rng, Nb, Hkv, n0, d).to(dev), _bf16(rng, Nb, Hkv, n0, d).to(dev)
    lens = torch.full((Nb,), n0, dtype=torch.int32, device=dev)
    slab = L * Nb * Hq * d
    step = 0 if stride == "none" else Hq * d // 2
    flat = [torch.zeros(slab + T * step, dtype=torch.float32, device=dev) for _ in range(2)]
    a, b = (B.Cache(L, Nb, Hq, Hkv, d, cap, cap - M - 64, 32, 32) for _ in range(2))
    for c in (a, b):
        for l in range(L):
            B.dynts_prefill(c.ctx, l, K0, V0, lens)
    B.dynts_decode_loop(a.ctx, T, q, k, v, flat[0], a.keep_idx, a.new_len, active=act, out_step_stride=step)
    for t in range(T):
        for l in range(L):
            out = flat[1][t * step + l * Nb * Hq * d:][:Nb * Hq * d].view(Nb, Hq, d)
            B.dynts_decode_step(b.ctx, l, q[t, l], k[t, l], v[t, l], out, active=act[t])
    assert torch.equal(flat[0], flat[1]) and bool((flat[0] != 0).any())
    assert torch.equal(a.seq_len, b.seq_len) and torch.equal(a.status, b.status)


@pytest.mark.parametrize("d,Hq,Hkv", [(64, 8, 2), (128, 14, 2), (128, 3, 3)])
def test_attend_then_update_by_any_route(B, d, Hq, Hkv):
    """The unfused attend call keeps its logits for the update behind it.  Two layers share the room for them: whoever
    else uses it in between, and whatever asks for the update (dynts_update_scores, the next fused step, a trigger's
    flush), every attend call's weights reach S once; those of an attend call that another one follows do not."""
    rng = np.random.default_rng(d + Hq)
    Nb, cap, M, G = 2, 203, 17, Hq // Hkv
    lens = np.array([171, 96], np.int32)
    dev = torch.device("cuda:0")
    bf = lambda *s: torch.from_numpy(rng.standard_normal(s).astype(np.float32)).to(torch.bfloat16)
    cache = B.Cache(2, Nb, Hq, Hkv, d, cap, 60, 40, 8)
    K, V = [bf(Nb, Hkv, cap, d) for _ in range(2)], [bf(Nb, Hkv, cap, d) for _ in range(2)]
    for l in range(2):
        B.dynts_prefill(cache.ctx, l, K[l].to(dev), V[l].to(dev), torch.from_numpy(lens).to(dev))
        cache.S[l, :, :, M:] = 0.0
    cache.n_prompt.fill_(M)
    n = [lens.copy(), lens.copy()]
    want = np.zeros((2, Nb, Hkv, cap))
    out = torch.zeros((Nb, Hq, d), dtype=torch.float32, device=dev)

    def attend(l, counts, fused=False):
        q = bf(Nb, Hq, d)
        if fused:
            k1, v1 = bf(Nb, Hkv, d), bf(Nb, Hkv, d)
            B.dynts_decode_step(cache.ctx, l, q.to(dev), k1.to(dev), v1.to(dev), out)
            for b in range(Nb):
                K[l][b, :, n[l][b]], V[l][b, :, n[l][b]] = k1[b], v1[b]
            n[l] += 1
        else:
            B.dynts_decode_attend(cache.ctx, l, q.to(dev), out)
        for b in range(Nb):
            for h in range(Hkv):
                m = n[l][b]
                x = f64(q)[b, h * G:(h + 1) * G] @ f64(K[l])[b, h, :m].T / np.sqrt(d)
                a = np.exp(x - x.max(1, keepdims=True))
                a /= a.sum(1, keepdims=True)
                if counts:
                    want[l, b, h, M:m] += a[:, M:].sum(0)
                assert_close(f64(out)[b, h * G:(h + 1) * G], a @ f64(V[l])[b, h, :m], "out, layer %d" % l)

    def check():
        for l in range(2):
            B.dynts_update_scores(cache.ctx, l)
            for b in range(Nb):
                assert_close(f64(cache.S[l])[b, :, M:n[l][b]], want[l, b, :, M:n[l][b]], "S, layer %d" % l)

    attend(0, True)
    check()
    attend(0, True); attend(1, True)                      # the second layer takes the room
    check()
    attend(0, False); attend(0, True)                     # the first call's weights are dropped, as ever
    check()
    attend(0, True); attend(0, True, fused=True)          # the fused step's pass over K makes the update owed
    check()
    B.dynts_hint_trigger(cache.ctx, 0)
    attend(0, True, fused=True); attend(1, True)          # announced logits stay: the other layer goes without
    check()
    attend(1, True)
    B.dynts_hint_trigger(cache.ctx, 0)
    attend(0, True, fused=True)                           # announced logits take the room from the other layer
    check()
    assert int(cache.status.item()) == 0


@pytest.mark.parametrize("d,Hq,Hkv,cap,nsplit", [(128, 28, 4, 1300, 3), (64, 8, 2, 1500, 6), (128, 4, 1, 5000, 20)])
def test_replayed_steps_leave_no_partial_of_theirs(B, d, Hq, Hkv, cap, nsplit):
    """The replays of a recorded launch share one tag, so the partials of one must not be there for the next, whose merge would
    take them for its own.  Two steps are recorded (the saved query alternates), behind an eager one, whose score update the first
    of them finds owed as it later does the second's; replays against a twin's eager steps."""
    dev = torch.device("cuda:0")
    Nb, n, G, reps = 3, cap - 100, Hq // Hkv, 4
    torch.manual_seed(cap)
    caches = [B.Cache(1, Nb, Hq, Hkv, d, cap, 100, 20, 10, launch_shape=(64, 8)) for _ in range(2)]
    K = torch.randn(Nb, Hkv, cap, d, device=dev).to(torch.bfloat16)
    for c in caches:
        c.K[0].copy_(K)
        c.V[0].copy_(K.flip(2))
        c.seq_len.fill_(n)
        c.n_prompt.fill_(9)
    tokens = [[torch.randn(Nb, h, d, device=dev).to(torch.bfloat16) for h in (Hq, Hkv, Hkv)] for _ in range(2 * reps)]
    now = [[t.clone() for t in tokens[i]] for i in range(2)]
    out = torch.zeros(2, Nb, Hq, d, device=dev)
    for c in caches:
        B.dynts_decode_step(c.ctx, 0, *tokens[0], out[0])
    caches[0].workspace[:Nb * Hkv * nsplit * G * (d + 2) * 8].zero_()
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        for i in range(2):
            B.dynts_decode_step(caches[0].ctx, 0, *now[i], out[i])
    rows = Nb * Hkv * nsplit * G
    partials = caches[0].workspace[:rows * d * 8]  # the head of the workspace, and behind it the statistics
    want = torch.zeros(2, Nb, Hq, d, device=dev)
    for r in range(reps):
        for i in range(2):
            for dst, src in zip(now[i], tokens[2 * r + i]):
                dst.copy_(src)
            B.dynts_decode_step(caches[1].ctx, 0, *tokens[2 * r + i], want[i])
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)
        assert not partials.any() and not caches[0].workspace[(rows * d * 8 + 255) // 256 * 256:][:rows * 16].any()
        assert caches[1].workspace[:rows * d * 8].view(torch.int64).ne(0).sum() > rows * d // 2  # (that is where they lie)
    assert torch.equal(caches[0].S[0], caches[1].S[0]) and torch.equal(caches[0].seq_len, caches[1].seq_len)
    assert int(caches[0].seq_len[0, 0]) == n + 1 + 2 * reps


# a letter per call: A unfused attention, U its update, F a fused attention, of the layer behind it; and the attentions (by
# number) that may still leave their logits in the workspace, the first of a context, which cannot know what follows
@pytest.mark.parametrize("d,Hq,Hkv,calls,keepers", [
    (64, 8, 2, "A0 A0 A0 A0 U0", {0}), (128, 16, 2, "A0 F0 A0 F0 A0 F0 U0", {0}), (128, 14, 2, "A0 A1 A2 U0 U1 U2 A0 A1 A2 U0 U1 U2", {0}),
    (64, 4, 2, "A0 A1 A2 U0 U1 U2 A0 A1 A2 U0 U1 U2 A0 A1 A2 U0 U1 U2", {0, 8}), (128, 8, 2, "A0 U0 A0 F0 A0 U0 A0 F0 A0 U0", {0, 1}),
    (64, 8, 2, "A0 U0 A1 U1 A0 U0 A2 U2", {0, 1, 2, 3}), (64, 16, 2, "A0 U0 A0 U0 A0 U0", set()), (128, 32, 2, "A0 U0 A0 U0", set())])
def test_unfused_attention_keeps_logits_where_its_update_follows(B, d, Hq, Hkv, calls, keepers):
    """The logits an unfused attention keeps for its update cost it a fifth of its time: only callers who ask for the update
    next pay for them, and only where they are fewer bytes than the K rows they spare.  The scores are right in every order."""
    rng = np.random.default_rng(5)
    dev = torch.device("cuda:0")
    L, Nb, cap, n, M, G = 3, 2, 210, 180, 11, Hq // Hkv
    cache = B.Cache(L, Nb, Hq, Hkv, d, cap, 100, 30, 10)
    K = _bf16(rng, L, Nb, Hkv, cap, d)
    cache.K.copy_(K)
    cache.V.copy_(_bf16(rng, L, Nb, Hkv, cap, d))
    cache.seq_len.fill_(n)
    cache.n_prompt.fill_(M)
    kept = cache.workspace[-(Nb * Hq * 224 * 4):]  # the last room in the workspace: [Nb][Hq][cap rounded up to 32] fp32
    want, owed, number = np.zeros((L, Nb, Hkv, cap)), {}, 0
    out = torch.zeros((Nb, Hq, d), device=dev)
    for call in calls.split():
        l = int(call[1])
        if call[0] == "U":
            B.dynts_update_scores(cache.ctx, l)
            want[l] += owed.pop(l, 0.0)
            assert_close(f64(cache.S[l])[..., M:n], want[l][..., M:n], "S, layer %d, %s" % (l, calls))
            continue
        q = _bf16(rng, Nb, Hq, d)
        x = np.matmul(f64(q).reshape(Nb, Hkv, G, d), f64(K[l])[:, :, :n].transpose(0, 1, 3, 2)) / np.sqrt(d)
        a = np.exp(x - x.max(-1, keepdims=True))
        w = np.zeros((Nb, Hkv, cap))
        w[..., M:n] = (a / a.sum(-1, keepdims=True)).sum(2)[..., M:]
        if call[0] == "F":
            B.dynts_decode_attend_update(cache.ctx, l, q.to(dev), out)
            want[l] += owed.pop(l, 0.0)
        else:
            before = kept.clone()
            B.dynts_decode_attend(cache.ctx, l, q.to(dev), out)
            assert torch.equal(kept, before) == (number not in keepers), "attention %d of %s" % (number, calls)
            number += 1
        owed[l] = w
    assert int(cache.status.item()) == 0


@pytest.mark.parametrize("Hq", [4, 32])
def test_kernel_events_of_the_update_behind_an_unfused_attention(B, Hq):
    """dynts_set_kernel_events: the update's launch takes them, whether it adds up kept logits (two heads a group) or reads K."""
    cache = B.Cache(1, 2, Hq, 2, 128, 200, 100, 20, 10)
    cache.seq_len.fill_(150)
    q = torch.randn(2, Hq, 128, device="cuda:0").to(torch.bfloat16)
    out = torch.zeros(2, Hq, 128, device="cuda:0")
    start, stop, between = [torch.cuda.Event(enable_timing=True) for _ in range(3)]
    for e in (start, stop):
        e.record()  # makes the handle
    torch.cuda.synchronize()
    B.dynts_set_kernel_events(cache.ctx, start.cuda_event, stop.cuda_event)
    for _ in range(2):
        B.dynts_decode_attend(cache.ctx, 0, q, out)
        between.record()
        B.dynts_update_scores(cache.ctx, 0)
        torch.cuda.synchronize()
        assert between.elapsed_time(start) > 0 and start.elapsed_time(stop) > 0
    B.dynts_set_kernel_events(cache.ctx, None, None)


@pytest.mark.parametrize("before", ["eager pair", "eager attend", ""])
def test_captured_attend_and_update(B, before):
    """The unfused pair recorded as graphs of their own, per layer: replayed in another order than recorded, with eager calls
    of the same context between, every update adds the weights of its own layer's attention.  One workgroup per unit."""
    dev = torch.device("cuda:0")
    L, Nb, Hq, Hkv, d, M, n = 2, 2, 8, 4, 64, 5, 150
    torch.manual_seed(3)
    cache = B.Cache(L, Nb, Hq, Hkv, d, 200, 100, 20, 10, launch_shape=(1, 8))
    cache.K.normal_()
    cache.V.normal_()
    cache.seq_len.fill_(n)
    cache.n_prompt.fill_(M)
    q = torch.randn(L, Nb, Hq, d, device=dev).to(torch.bfloat16)
    q_other = torch.randn(Nb, Hq, d, device=dev).to(torch.bfloat16)
    out, out_other = torch.zeros(L, Nb, Hq, d, device=dev), torch.zeros(Nb, Hq, d, device=dev)
    if before:
        B.dynts_decode_attend(cache.ctx, 0, q_other, out_other)
    if before == "eager pair":
        B.dynts_update_scores(cache.ctx, 0)
    attend, update = [], []
    torch.cuda.synchronize()
    for l in range(L):
        for what in (attend, update):
            what.append(torch.cuda.CUDAGraph())
            with torch.cuda.graph(what[l]):
                if what is attend:
                    B.dynts_decode_attend(cache.ctx, l, q[l], out[l])
                else:
                    B.dynts_update_scores(cache.ctx, l)
    x = torch.matmul(q.cpu().double().view(L, Nb, Hkv, Hq // Hkv, d), cache.K[:, :, :, :n].cpu().double().transpose(3, 4)) / np.sqrt(d)
    w = torch.softmax(x, dim=-1).sum(3)[..., M:].numpy()
    for replay in range(3):
        cache.S.zero_()
        for g in attend:
            g.replay()
        if replay == 1:  # an attention outside the graphs, which leaves something in the workspace, too
            B.dynts_decode_attend(cache.ctx, 1, q_other, out_other)
            attend[1].replay()
        torch.cuda.synchronize()
        for g in update:
            g.replay()
        torch.cuda.synchronize()
        for l in range(L):
            assert_close(f64(cache.S[l])[..., M:n], w[l], "S, layer %d, replay %d" % (l, replay))
    assert int(cache.status.item()) == 0


def _steps_on_a_large_cache(B, Nb, Hq, Hkv, d, cap, layers, lens, launch_shape=None, masked=False):
    """Every form of the step on the last layer of a dense cache of several hundred MB, against float64.  masked: a quarter of
    the sequences, others each time, sit a step out."""
    G = Hq // Hkv
    dev = torch.device("cuda:0")
    g = torch.Generator(device=dev)
    g.manual_seed(cap)
    normal = lambda *s: torch.randn(s, generator=g, device=dev).to(torch.bfloat16)
    cache = B.Cache(layers, Nb, Hq, Hkv, d, cap, cap - 200, 10, 10, launch_shape=launch_shape)
    layer = layers - 1
    cache.K[layer].copy_(normal(Nb, Hkv, cap, d))
    cache.V[layer].copy_(normal(Nb, Hkv, cap, d))
    M = 7
    cache.S[layer, :, :, :M] = float("inf")
    cache.n_prompt.fill_(M)
    cache.seq_len[layer].copy_(torch.from_numpy(lens).to(dev))
    K, V = cache.K[layer].cpu().double(), cache.V[layer].cpu().double()
    want = torch.zeros((Nb, Hkv, cap), dtype=torch.float64)
    out, lse = torch.zeros((Nb, Hq, d), device=dev), torch.zeros((Nb, Hq), device=dev)
    n = lens.copy()
    on, active = np.ones(Nb, bool), None
    for i, step in enumerate(("first", "step", "hinted", "attend_update", "attend", "step")):
        if masked:
            on = (np.arange(Nb) + i) % 4 != 3
            active = torch.from_numpy(on.astype(np.uint8)).to(dev)
        q, k1, v1 = normal(Nb, Hq, d), normal(Nb, Hkv, d), normal(Nb, Hkv, d)
        if step.startswith("attend"):
            (B.dynts_decode_attend if step == "attend" else B.dynts_decode_attend_update)(cache.ctx, layer, q, out, lse, active)
        else:
            if step == "hinted":
                B.dynts_hint_trigger(cache.ctx, layer)
            B.dynts_decode_step(cache.ctx, layer, q, k1, v1, out, lse=lse, active=active)
            for b in np.flatnonzero(on):
                K[b, :, n[b]], V[b, :, n[b]] = k1[b].cpu().double(), v1[b].cpu().double()
            n[on] += 1
        if step not in ("first", "step"):  # (an unfused call drops what the one before it still owes)
            B.dynts_update_scores(cache.ctx, layer)
        for b in np.flatnonzero(on):
            x = torch.matmul(q[b].cpu().double().view(Hkv, G, d), K[b, :, :n[b]].transpose(1, 2)) / np.sqrt(d)
            if n[b] == 0:
                continue
            a = torch.softmax(x, dim=-1)
            assert_close(f64(out)[b], torch.matmul(a, V[b, :, :n[b]]).reshape(Hq, d).numpy(), "out[%d], %s" % (b, step))
            assert_close(f64(lse)[b], torch.logsumexp(x, dim=-1).reshape(Hq).numpy(), "lse[%d], %s" % (b, step))
            want[b, :, M:n[b]] += a.sum(1)[:, M:]
    B.dynts_update_scores(cache.ctx, layer)
    S = f64(cache.S[layer])
    for b in range(Nb):
        assert_close(S[b, :, M:n[b]], want[b, :, M:n[b]].numpy(), "S[%d]" % b)
        assert np.all(S[b, :, max(M, n[b]):] == 0)
    assert int(cache.status.item()) == 0
    cache.close()


@pytest.mark.parametrize("Nb,Hq,Hkv,d,cap,layers", [(16, 16, 8, 128, 5000, 1), (40, 8, 4, 64, 8100, 1), (16, 16, 8, 128, 1700, 3)])
def test_caches_beyond_the_memory_side_cache(B, Nb, Hq, Hkv, d, cap, layers):
    """Caches of more than 310 MB: tiles at fixed places first, the rest loaded past the memory-side cache.  Ragged lengths
    around the ends of the rounds of fixed tiles, around the length from which the rest goes past the cache, around
    tiles and at both ends, in every form of the step."""
    units = Nb * Hkv
    slot = 4 * layers * units * d
    assert slot * cap > 310e6 and units >= 128 and slot * cap / layers >= 100e6
    fit, per_round = int(310e6 / slot), 8 * 32 * max(1, (256 + units // 2) // units)
    full = int(272e6 / (slot * per_round)) * per_round
    lens = [0, 1, 31, 33, per_round - 1, per_round, per_round + 1, 2 * per_round + 40, full - 1, full, full + 33, fit - 1,
            fit, fit + 1, cap - 35, cap - 4]
    lens = np.array([min(max(x, 0), cap - 4) for x in (lens * 3)[:Nb]], np.int32)
    _steps_on_a_large_cache(B, Nb, Hq, Hkv, d, cap, layers, lens)


@pytest.mark.parametrize("Nb,Hq,Hkv,d,cap,layers,shape,rounds", [
    (16, 16, 8, 128, 1560, 10, None, 0), (32, 28, 4, 128, 1560, 6, None, 1), (32, 8, 4, 128, 1560, 10, (256, 4), 1),
    (32, 8, 4, 64, 3100, 70, (128, 4), 0), (16, 16, 8, 128, 5000, 1, None, 8)])
def test_caches_beyond_the_memory_side_cache_in_deep_stacks(B, Nb, Hq, Hkv, d, cap, layers, shape, rounds):
    """The same with more layers than leave every wave a second fixed tile, or any that go through the cache, with
    four-wave workgroups, and with sequences that sit steps out."""
    units = Nb * Hkv
    slot, waves = 4 * layers * units * d, 8 if shape is None else shape[1]
    per_round = waves * 32 * max(1, ((256 if shape is None else shape[0]) + units // 2) // units)
    assert slot * cap > 310e6 and units >= 128 and slot * cap / layers >= 100e6 and int(272e6 / (slot * per_round)) == rounds
    lens = [0, 1, 31, 32, 33, 65, per_round - 1, per_round, per_round + 1, int(310e6 / slot), int(310e6 / slot) + 1, cap // 2,
            2 * per_round + 40, cap - 35, cap - 7, cap - 6]
    lens = np.array([min(max(x, 0), cap - 6) for x in (lens * 3)[:Nb]], np.int32)
    _steps_on_a_large_cache(B, Nb, Hq, Hkv, d, cap, layers, lens, shape, masked=True)


@pytest.mark.parametrize("Nb,Hq,Hkv,d,cap,layers,shape", [(16, 16, 4, 128, 9700, 1, None), (12, 16, 8, 64, 12800, 1, (96, 4)),
                                                          (25, 28, 4, 128, 3900, 2, None)])
def test_dense_caches_that_write_scores_in_bursts(B, Nb, Hq, Hkv, d, cap, layers, shape):
    """Large caches of fewer units than are loaded past the memory-side cache: a wave's scores leave in runs of up to 16 tiles.
    Ragged lengths around those runs, around tiles and at both ends; a question window that ends inside the first run."""
    assert 4 * Nb * Hkv * cap * d > 192e6 and 4 * layers * Nb * Hkv * cap * d > 310e6 and Nb * Hkv < 128
    first = 32 * (8 if shape is None else shape[1]) * max(1, ((256 if shape is None else shape[0]) + Nb * Hkv // 2) // (Nb * Hkv))
    lens = [0, 1, 31, 33, first - 1, first + 1, first + first * 15, first + first * 16 - 31, first + first * 17 + 5, cap // 3, cap - 35, cap - 4]
    lens = np.array([min(max(x, 0), cap - 4) for x in (lens * 3)[:Nb]], np.int32)
    _steps_on_a_large_cache(B, Nb, Hq, Hkv, d, cap, layers, lens, shape, masked=Nb > 16)


@pytest.mark.parametrize("Hq,Hkv,d,n,shape", [(4, 1, 128, 9001, (256, 8)), (4, 1, 128, 1300, (256, 8)), (8, 1, 128, 4700, (256, 8)),
                                              (16, 1, 128, 2600, (256, 8)), (8, 1, 64, 8448, (256, 8)), (2, 1, 128, 2900, (256, 4)),
                                              (16, 1, 128, 1500, (256, 4)), (5, 1, 64, 1153, (256, 4)), (8, 1, 64, 6000, (256, 8)),
                                              (3, 1, 64, 4205, (256, 8)), (2, 1, 128, 4097, (256, 8)), (5, 1, 128, 1040, (256, 8))])
def test_merge_of_many_chunks(B, Hq, Hkv, d, n, shape):
    """One unit cut into up to 36 chunks: every grouping of the merge (one, two and more output elements per thread), whole and
    partial last groups, chunks that are empty because the sequence is shorter than the capacity."""
    rng = np.random.default_rng(n + Hq)
    dev = torch.device("cuda:0")
    cap = n + 300
    cache = B.Cache(1, 2, Hq, Hkv, d, cap, n, 10, 10, launch_shape=shape)
    lens = [n, max(1, n // 3)]
    cache.K[0].copy_(_bf16(rng, 2, Hkv, cap, d))
    cache.V[0].copy_(_bf16(rng, 2, Hkv, cap, d))
    cache.seq_len[0].copy_(torch.tensor(lens, dtype=torch.int32))
    out, lse = torch.zeros((2, Hq, d), device=dev), torch.zeros((2, Hq), device=dev)
    for _ in range(2):
        q = _bf16(rng, 2, Hq, d, scale=1.5)
        B.dynts_decode_attend_update(cache.ctx, 0, q.to(dev), out, lse)
        for b in range(2):
            x = f64(q)[b] @ f64(cache.K[0, b, 0, :lens[b]]).T / np.sqrt(d)
            a = np.exp(x - x.max(1, keepdims=True))
            assert_close(f64(out)[b], a / a.sum(1, keepdims=True) @ f64(cache.V[0, b, 0, :lens[b]]), "out[%d]" % b)
            assert_close(f64(lse)[b], x.max(1) + np.log(a.sum(1)), "lse[%d]" % b)
    B.dynts_update_scores(cache.ctx, 0)
    assert abs(float(cache.S[0, 0].sum()) - 2 * Hq) < 1e-3 * Hq
