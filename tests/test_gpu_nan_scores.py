"""GPU parity with NaN log-probabilities in valid frames: a NaN score counts as
-inf for tokens, repeats and blanks alike, in every decoder; and with scores of
+inf, which order by index.  Against the CPU oracle, N-best: tokens and lengths equal, scores within 1e-4 (the same fp32
operations: 0 expected)."""
import math

import numpy as np
import pytest

import oracle
import paper_2508_07315_amd as P
import workloads as W
from gpu_helpers import compare, device, gpu_boost, gpu_lm, log, oracle_bt, oracle_lm, oracle_threads

pytestmark = pytest.mark.gpu


def _logprobs(B, T, V, seed):
    rng = np.random.default_rng(seed)
    lp = W.random_logprobs(rng, B, T, V)
    lp[0, ::3, V] = np.nan                                  # blanks
    lp[1][rng.random((T, V + 1)) < 0.2] = np.nan            # anything
    for t in range(0, T, 2):                                # runs of labels (whole lane groups)
        a = int(rng.integers(0, V))
        lp[2, t, a:a + 600] = np.nan
    lp[2, 1::4, V] = -np.inf
    lp[3, 5:7] = np.nan                                     # nothing left
    lp[4, ::2, :V] = np.nan                                 # blanks only
    return lp


CASES = [
    # V, K, order, phrases, theta, flags
    (1, 4, 0, 0, math.inf, {}),                             # the small-beam decoder
    (40, 8, 0, 0, math.inf, {}),
    (300, 5, 0, 0, 8.0, {}),
    (1024, 8, 0, 0, math.inf, {}),
    (40, 1, 2, 0, math.inf, {}),                            # one chunk of the general decoder
    (500, 16, 3, 20, math.inf, {}),
    (1024, 8, 3, 0, math.inf, {}),
    (1024, 8, 3, 0, 8.0, {"row_cache": False, "logsumexp": True}),
    (700, 8, 0, 0, math.inf, {"logsumexp": True}),
    (300, 8, 2, 20, math.inf, {"repeat_score": True}),
    (3100, 16, 2, 20, math.inf, {}),                        # several chunks
    (45, 12, 3, 0, math.inf, {}),                           # the class decoder
    (700, 20, 0, 0, 8.0, {"logsumexp": True}),
    (1024, 64, 3, 50, math.inf, {"repeat_score": True}),
    (600, 100, 2, 50, math.inf, {}),
    (2500, 6, 3, 0, math.inf, {}),
]


@pytest.mark.parametrize("V,K,order,phrases,theta,kw", CASES)
def test_nan_scores(V, K, order, phrases, theta, kw):
    import torch
    B, T = 5, 24
    lp = _logprobs(B, T, V, [V, K])
    lens = np.full(B, T, dtype=np.int32)
    counts = (min(6 * V, V * V), 4 * V)[: order - 1] if order else ()
    spec = W.LMSpec(order=order, counts=counts, seed=V + K) if order else None
    bspec = W.BoostSpec(phrases, 2, 4, "zipf", V) if phrases else None
    log("NaN scores", V, K, order, phrases, theta, kw)
    dev = device()
    alpha, w = (0.5 if order else 0.0), (1.25 if phrases else 0.0)
    tok, ln, sc, ws = P.ctcbeam_decode_nbest(
        torch.from_numpy(lp).to(dev), torch.from_numpy(lens).to(dev), K, alpha, 1.0, w,
        gpu_lm(spec, V) if spec else None, gpu_boost(bspec, V) if bspec else None, theta=theta, **kw)
    torch.cuda.synchronize()
    assert P.ctcbeam_query_status(ws) == 0
    okw = {k: v for k, v in kw.items() if k != "row_cache"}
    r = oracle.decode(lp, lens, K, alpha, 1.0, w, theta=theta, lm=oracle_lm(spec, V) if spec else None,
                      bt=oracle_bt(bspec, V) if bspec else None, n_threads=oracle_threads(), want_nbest=True, **okw)
    np.testing.assert_array_equal(ln.cpu().numpy(), r["nbest_lengths"])
    np.testing.assert_array_equal(tok.cpu().numpy(), r["nbest_tokens"])
    np.testing.assert_allclose(sc.cpu().numpy(), r["nbest_scores"], rtol=0, atol=1e-4)


@pytest.mark.parametrize("V,order,phrases", [(40, 2, 0), (256, 0, 20), (1024, 3, 20), (3000, 2, 0)])
def test_nan_scores_greedy(V, order, phrases):
    import torch
    B, T = 5, 60
    lp = _logprobs(B, T, V, V)
    lens = np.full(B, T, dtype=np.int32)
    spec = W.LMSpec(order=order, counts=(6 * V, 4 * V)[: order - 1], seed=V) if order else None
    bspec = W.BoostSpec(phrases, 2, 4, "zipf", V) if phrases else None
    log("NaN scores, greedy", V, order, phrases)
    dev = device()
    alpha, w = (0.5 if order else 0.0), (1.25 if phrases else 0.0)
    tok, ln, sc, _ = P.ctcbeam_greedy_decode(torch.from_numpy(lp).to(dev), torch.from_numpy(lens).to(dev), alpha, 1.0, w,
                                             gpu_lm(spec, V) if spec else None, gpu_boost(bspec, V) if bspec else None)
    torch.cuda.synchronize()
    r = oracle.decode(lp, lens, 1, alpha, 1.0, w, lm=oracle_lm(spec, V) if spec else None,
                      bt=oracle_bt(bspec, V) if bspec else None, n_threads=oracle_threads())
    compare(dict(tokens=tok.cpu().numpy(), lengths=ln.cpu().numpy(), scores=sc.cpu().numpy()), r, what="greedy")


@pytest.mark.parametrize("V,K", [(200, 64), (700, 64), (600, 100), (2500, 64)])
def test_zero_probability_with_negative_alpha(V, K):
    """A negative LM weight makes +inf of an entry of probability 0.  The only
    such context is the state of a poor beam, which comes after more than a
    pass of the class decoder and far below the K-th best of the first pass."""
    import torch
    B, T = 3, 3
    rng = np.random.default_rng([V, K])
    lp = np.full((B, T, V + 1), -200.0, dtype=np.float32)
    toks = np.stack([rng.permutation(V)[:80] for _ in range(B)])
    Z = int(toks[0, 24])
    for b in range(B):
        toks[b] = np.where(toks[b] == Z, toks[b, 24], toks[b])
        toks[b, 24] = Z
        lp[b, 0, toks[b, :64]] = -np.arange(64)
        lp[b, 1:][:, toks[b, 64:]] = -0.1 * np.arange(16)
    lens = np.full(B, T, dtype=np.int32)
    ids = np.stack([np.full(9, Z, dtype=np.int32), np.sort(rng.permutation(V)[:9]).astype(np.int32)], axis=1)
    uni = np.full(V + 2, -2.0, dtype=np.float32)
    # a context of its own for every token
    pairs = np.array([[c, (c + 1) % V] for c in range(V) if c != Z], dtype=np.int32)
    bi = np.concatenate([pairs, ids])
    prob = np.concatenate([np.full(len(pairs), -2.0), np.full(len(ids), -np.inf)]).astype(np.float32)
    at = np.lexsort((bi[:, 1], bi[:, 0]))
    arrays = dict(order=2, V=V, ids=[np.arange(V + 2, dtype=np.int32)[:, None], bi[at]], log10_prob=[uni, prob[at]],
                  log10_bow=[np.zeros(V + 2, dtype=np.float32), None])
    log("zero probability, negative alpha", V, K)
    dev = device()
    tok, ln, sc, ws = P.ctcbeam_decode_nbest(torch.from_numpy(lp).to(dev), torch.from_numpy(lens).to(dev), K, -0.3, 0.0,
                                             0.0, P.ctcbeam_lm_build(arrays))
    torch.cuda.synchronize()
    r = oracle.decode(lp, lens, K, -0.3, 0.0, lm=oracle.LM(arrays), want_nbest=True, n_threads=oracle_threads())
    assert np.isposinf(r["nbest_scores"]).any()
    np.testing.assert_array_equal(ln.cpu().numpy(), r["nbest_lengths"])
    np.testing.assert_array_equal(tok.cpu().numpy(), r["nbest_tokens"])
    np.testing.assert_allclose(sc.cpu().numpy(), r["nbest_scores"], rtol=0, atol=1e-4)
    assert P.ctcbeam_query_status(ws) == 0
