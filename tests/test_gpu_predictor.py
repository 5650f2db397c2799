"""GPU parity of the Importance Predictor head (Sec. 4.1, App. A) against the float64 oracle, synthetic weights."""
import numpy as np
import pytest
import torch

from oracle import dynts_oracle as orc
from tests.helpers import assert_close, f64

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2601_18383_amd import binding
    return binding


def _make(rng, d, m1, m2, bias=True):
    bf = lambda a: torch.from_numpy(a.astype(np.float32)).to(torch.bfloat16)
    W1 = bf(rng.standard_normal((m1, d)) / np.sqrt(d))
    W2 = bf(rng.standard_normal((m2, m1)) / np.sqrt(m1))
    w3 = bf(rng.standard_normal(m2) / np.sqrt(m2))
    b1 = torch.from_numpy(rng.standard_normal(m1).astype(np.float32) * 0.1) if bias else None
    b2 = torch.from_numpy(rng.standard_normal(m2).astype(np.float32) * 0.1) if bias else None
    b3 = torch.from_numpy(rng.standard_normal(1).astype(np.float32)) if bias else None
    return W1, b1, W2, b2, w3, b3


def _run(B, rng, d, m1, m2, batch, act, bias=True, n_rep=1, pack=True):
    dev = torch.device("cuda:0")
    ws = _make(rng, d, m1, m2, bias)
    h = torch.from_numpy(rng.standard_normal((batch, d)).astype(np.float32)).to(torch.bfloat16)
    pred = B.Predictor(*[w.to(dev) if w is not None else None for w in ws], activation=act, pack=pack)
    s = torch.full((batch, n_rep), 7.0, dtype=torch.float32, device=dev)
    B.dynts_predict_scores(pred, h.to(dev), s)
    ref = orc.predictor(f64(h), *[f64(w) if w is not None else None for w in ws], act)
    got = f64(s)
    for r in range(n_rep):
        worst = assert_close(got[:, r], ref, "predictor d=%d batch=%d act=%d" % (d, batch, act), tight=1e-4)
    assert np.all(got == got[:, :1])
    return worst


@pytest.mark.parametrize("act", [0, 1, 2])
@pytest.mark.parametrize("d,m1,m2,batch", [(64, 128, 32, 3), (96, 160, 48, 17), (256, 512, 128, 40),
                                            (512, 1024, 256, 128), (64, 128, 32, 1), (992, 2016, 496, 33)])
def test_small_shapes(B, d, m1, m2, batch, act):
    """Ragged feature groups (m not a multiple of 128), K slices with a partial last chunk, every batch-tile
    variant of the kernel, with and without biases."""
    rng = np.random.default_rng(d + batch + act)
    _run(B, rng, d, m1, m2, batch, act, bias=(batch % 2 == 1), n_rep=1 + batch % 4, pack=(act != 1))


@pytest.mark.parametrize("d,m1,m2,batch", [(256, 512, 592, 24),    # layer 2's workgroups take all of K
                                            (256, 2048, 1040, 24),  # four share it
                                            (12288, 32, 272, 24)])  # the form that cuts K of both layers
def test_replays_take_no_partial_of_another_call(B, d, m1, m2, batch):
    """Every call's words carry the same tag: those that an earlier replay, or a call of another batch on the same scratch, left
    must not be taken for this one's."""
    rng = np.random.default_rng(17)
    dev = torch.device("cuda:0")
    pred = B.Predictor(*[w.to(dev) for w in _make(rng, d, m1, m2)], max_batch=32)
    bf = lambda nb: torch.from_numpy(rng.standard_normal((nb, d)).astype(np.float32)).to(torch.bfloat16).to(dev)
    hs, other = [bf(batch) for _ in range(6)], [bf(nb) for nb in (32, 1, 17)]
    h, s, want = hs[0].clone(), torch.zeros(batch, 1, device=dev), torch.zeros(batch, 1, device=dev)
    aside = torch.zeros(32, 1, device=dev)
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        B.dynts_predict_scores(pred, h, s)
    for i, x in enumerate(hs):
        B.dynts_predict_scores(pred, x, want)
        torch.cuda.synchronize()
        h.copy_(x)
        if i % 2:
            o = other[i // 2]
            B.dynts_predict_scores(pred, o, aside[:o.shape[0]])
        if i == 4:  # words with the tag, counters that have counted
            pred.scratch.view(torch.int32).fill_(1)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(s, want)


@pytest.mark.parametrize("d,batch,hkv", [(3584, 32, 4), (4096, 64, 8), (4096, 128, 8)])
def test_paper_sizes(B, d, batch, hkv):
    """App. C: 3584 -> 7168 -> 1792 -> 1 (R1-Qwen) and 4096 -> 8192 -> 2048 -> 1 (R1-Llama), decode batches of the
    benchmark configs, the score written once per KV head."""
    rng = np.random.default_rng(d + batch)
    _run(B, rng, d, 2 * d, d // 2, batch, orc.ACT_RELU, n_rep=hkv)


def test_pack_is_the_documented_permutation(B):
    """[m][K] -> [m/16][K/32][16][32], bit for bit."""
    dev = torch.device("cuda:0")
    m, K = 48, 96
    W = torch.arange(m * K, dtype=torch.int32).reshape(m, K).to(torch.int16).view(torch.bfloat16).to(dev)
    got = B.dynts_predictor_pack(W).view(torch.int16).cpu().numpy().reshape(m // 16, K // 32, 16, 32)
    want = W.view(torch.int16).cpu().numpy().reshape(m // 16, 16, K // 32, 32).transpose(0, 2, 1, 3)
    assert np.array_equal(got, want)


def test_row_major_weights_at_paper_size(B):
    rng = np.random.default_rng(5)
    _run(B, rng, 3584, 7168, 1792, 32, orc.ACT_SILU, n_rep=4, pack=False)


def test_argument_errors(B):
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(0)
    ws = [w.to(dev) for w in _make(rng, 64, 128, 32)]
    pred = B.Predictor(*ws)
    h = torch.zeros((4, 64), dtype=torch.bfloat16, device=dev)
    s = torch.zeros((4, 300), dtype=torch.float32, device=dev)
    with pytest.raises(B.DyntsError):
        B.dynts_predict_scores(pred, h, s)                       # n_rep too large
    bad = B.dynts_predictor(60, 128, 32, 1, 0, 0, 0, 0, 0, 0, 0)  # d not a multiple of 32
    assert B.dynts_predict_scratch_bytes(bad, 4) == 0
    assert B.dynts_predict_scratch_bytes(pred.w, 129) == 0
    assert B.dynts_predict_scratch_bytes(pred.w, 128) > 0


def test_paper_inference_mode_end_to_end(B):
    """The paper's own inference loop (Sec. 4.1-4.2) in small: every step the predictor head turns the current
    token's hidden state into one score, the token is appended with that score (the same for every KV head),
    attention runs over the retained cache, and when the budget is reached the top-k by predicted score stay.
    HIP path (predictor + fused decode step + selection + compaction) against the oracle chain."""
    from tests.helpers import SideBySide
    rng = np.random.default_rng(77)
    dev = torch.device("cuda:0")
    Nb, Hq, Hkv, d_head, M, budget, window, E = 3, 8, 2, 64, 11, 24, 16, 20
    d_model, m1, m2 = 64, 128, 32
    ws = _make(rng, d_model, m1, m2)
    pred = B.Predictor(*[w.to(dev) for w in ws], activation=B.DYNTS_ACT_SILU)
    cap = M + budget + window + E
    cache = B.Cache(1, Nb, Hq, Hkv, d_head, cap, budget, window, E, external_scores=True)
    o = orc.OracleLayer(Nb, Hq, Hkv, d_head, cap, budget, window, E, external_scores=True)
    sbs = SideBySide(B, cache, 0, o, "step")
    bf = lambda *shape: torch.from_numpy(rng.standard_normal(shape).astype(np.float32)).to(torch.bfloat16)
    sbs.prefill(bf(Nb, Hkv, M, d_head), bf(Nb, Hkv, M, d_head), [M, 5, 8])
    s_dev = torch.zeros((Nb, Hkv), dtype=torch.float32, device=dev)
    T = budget + window + 3 * E + 7
    for t in range(1, T + 1):
        h = bf(Nb, d_model)
        B.dynts_predict_scores(pred, h.to(dev), s_dev)
        s_ref = orc.predictor(f64(h), *[f64(w) for w in ws], orc.ACT_SILU)
        assert_close(f64(s_dev)[:, 0], s_ref, "predicted score, step %d" % t, tight=1e-4)
        # both sides append the HIP path's fp32 score, so that the selection below is decided on identical
        # numbers (the predictor's own parity is asserted just above)
        sbs.step(bf(Nb, Hq, d_head), bf(Nb, Hkv, d_head), bf(Nb, Hkv, d_head), s=s_dev.cpu(), check_scores=(t % 9 == 0))
    assert sbs.evictions == 3
    sbs.check_state()
    # external scores are never changed by attention: every retained thinking slot still holds its predicted score
    S = f64(cache.S[0])
    assert np.all(S[:, 0, :] == S[:, 1, :])
    assert int(cache.status.item()) == 0


@pytest.mark.parametrize("d,m1,m2", [(96, 4128, 1072),   # two tiles a workgroup in both layers, the last of layer 2 alone; an odd number of k-steps
                                     (32, 2080, 1024),   # one k-step in layer 1; four or two workgroups share the K of layer 2
                                     (1056, 96, 16)])    # one group of features, and fewer k-steps than waves
@pytest.mark.parametrize("batch", [1, 16, 17, 33, 49, 64, 65, 96, 97, 128])
def test_tile_edges(B, d, m1, m2, batch):
    """Every number of batch tiles at its edges, with both numbers of feature tiles and shared and unshared K."""
    _run(B, np.random.default_rng(d + batch), d, m1, m2, batch, orc.ACT_RELU, bias=batch % 2 == 1, n_rep=2, pack=batch % 3 != 0)


@pytest.mark.parametrize("d,m1,m2,batch", [
    (12288, 32, 16, 16), (12288, 32, 16, 17), (12288, 160, 48, 64),   # few features and a long K: either side of 1.1 and 1.4 MB a workgroup
    (10912, 64, 16, 48), (10976, 64, 16, 48), (16384, 2048, 16, 33), (16384, 2080, 16, 33),  # ... and of 128 workgroups
    (32, 24576, 16, 5), (32, 24608, 16, 5), (288, 16416, 32, 128),    # many features and a short K
    (512, 16416, 256, 128), (512, 16416, 272, 128),                   # ... with few and with more features in layer 2
    (32, 8192, 16, 32), (32, 8224, 16, 32), (32, 12288, 16, 17), (32, 12320, 16, 17), (32, 8224, 16, 33),  # tiles a workgroup in layer 1
    (32, 8192, 16, 1), (32, 16384, 16, 1), (32, 16384, 16, 128), (64, 16384, 528, 65)])  # workgroups that share K in layer 2
def test_either_side_of_the_plan_rules(B, d, m1, m2, batch):
    _run(B, np.random.default_rng(d + m1 + batch), d, m1, m2, batch, orc.ACT_SILU, bias=batch % 2 == 1, n_rep=2, pack=batch % 3 != 0)


def test_one_scratch_serves_calls_of_any_batch(B):
    """The scratch's layout follows the batch: what a call of one batch leaves is never taken for a word of another's."""
    rng, dev = np.random.default_rng(3), torch.device("cuda:0")
    ws = _make(rng, 128, 2048, 1040)
    pred = B.Predictor(*[w.to(dev) for w in ws], activation=B.DYNTS_ACT_RELU)
    for batch in (128, 3, 70, 128, 33, 17, 3, 48):
        h = torch.from_numpy(rng.standard_normal((batch, 128)).astype(np.float32)).to(torch.bfloat16)
        s = torch.zeros(batch, device=dev)
        B.dynts_predict_scores(pred, h.to(dev), s)
        assert_close(f64(s), orc.predictor(f64(h), *[f64(w) for w in ws], orc.ACT_RELU), "batch %d" % batch, tight=1e-4)


def _chunked_product(x, W, step=1 << 20):
    """x [Nb][K] fp64, W [m][K] bf16 -> x W^T in fp64, some columns at a time."""
    acc = torch.zeros(x.shape[0], W.shape[0], dtype=torch.float64, device=x.device)
    for c in range(0, W.shape[1], step):
        acc += x[:, c:c + step] @ W[:, c:c + step].double().t()
    return acc


@pytest.mark.parametrize("d,m1,m2,batch,pack", [
    (1 << 23, 32, 16, 128, True),      # the hidden states take 2 GiB
    (32, 1 << 22, 32, 17, False),      # so do the second layer's operands for eight batch tiles
    ((1 << 27) - 64, 32, 16, 1, True),  # 16 features' weights take 4 GiB
    ((1 << 26) + 32, 32, 16, 2, False)])
def test_sizes_past_32_bit_offsets(B, d, m1, m2, batch, pack):
    """fp32 sums of K products of two normal values with a variance of 1 / K: errors of some 2^-24 of a result of order 1, times the
    root of the number of terms a sum passes through at most (here some 65536 partial sums), far below the bound of the other sizes."""
    dev = torch.device("cuda:0")
    g = torch.Generator(device=dev).manual_seed(d % 1000 + batch)
    bf = lambda m, k: torch.empty(m, k, dtype=torch.bfloat16, device=dev).normal_(0.0, k ** -0.5, generator=g)
    W1, W2, w3 = bf(m1, d), bf(m2, m1), bf(1, m2)[0].contiguous()
    h = torch.empty(batch, d, dtype=torch.bfloat16, device=dev).normal_(generator=g)
    y = torch.relu(_chunked_product(h.double(), W1))
    y = torch.relu(_chunked_product(y, W2))
    want = (y @ w3.double()).cpu().numpy()
    pred = B.Predictor(W1, None, W2, None, w3, None, activation=B.DYNTS_ACT_RELU, max_batch=batch, pack=pack)
    s = torch.full((batch, 2), 7.0, device=dev)
    B.dynts_predict_scores(pred, h, s)
    got = f64(s)
    assert np.array_equal(got[:, 0], got[:, 1])
    assert_close(got[:, 0], want, "predictor d=%d m1=%d batch=%d" % (d, m1, batch), tight=1e-4)
