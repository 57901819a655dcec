"""GPU parity of beams over several chunks of the general decoder (fill groups,
the pool carried over the chunks, the extraction after an overflow) at the
edges of the ranges that the class decoder leaves to it: 1801 to 2048 tokens
with phrases and a 3- or 4-gram, above 2048 tokens beams of 3 with a 2- to
4-gram, above 2560 tokens with phrases, above 3072 with an LM.  The class
decoder's side of each edge is run too.  Against the CPU oracle, N-best: tokens
and lengths equal, scores within 1e-4 (the same fp32 operations: 0 expected)."""
import math

import numpy as np
import pytest

import oracle
import paper_2508_07315_amd as P
import workloads as W
from gpu_helpers import device, gpu_boost, gpu_lm, log, oracle_bt, oracle_lm, oracle_threads

pytestmark = pytest.mark.gpu

CASES = [
    # V, K, order, phrases, theta, flags
    (1801, 7, 3, 300, math.inf, {}),
    (2048, 16, 4, 2000, 12.0, {"logsumexp": True}),
    (1900, 16, 3, 300, math.inf, {"repeat_score": True}),
    (2049, 3, 2, 0, math.inf, {}),
    (3072, 3, 4, 0, 12.0, {"repeat_score": True}),
    (2561, 3, 0, 300, math.inf, {}),
    (4096, 4, 0, 3000, 12.0, {"logsumexp": True, "boost_rollback": True}),
    (2561, 16, 3, 2000, math.inf, {}),
    (2700, 13, 5, 500, math.inf, {"repeat_score": True, "boost_rollback": True}),
    (3073, 8, 3, 0, math.inf, {"logsumexp": True}),
    (3073, 16, 1, 0, math.inf, {"row_cache": False}),
    (3500, 9, 2, 300, 12.0, {}),
    (4096, 16, 5, 0, 12.0, {}),
    (4095, 16, 4, 3000, math.inf, {"repeat_score": True, "logsumexp": True}),
    # the class decoder's side
    (1800, 7, 3, 300, math.inf, {}),
    (2048, 6, 4, 300, math.inf, {}),
    (2048, 16, 2, 300, math.inf, {}),
    (2049, 3, 5, 0, math.inf, {}),
    (2560, 3, 0, 300, math.inf, {}),
    (2561, 5, 0, 300, math.inf, {}),
    (4096, 17, 3, 300, math.inf, {}),
    # character sets with phrases change sides at 144 candidates a frame
    (8, 16, 2, 30, math.inf, {}),
    (9, 16, 2, 30, math.inf, {}),
]


def _decode(lp, lens, K, alpha, beta, w, lm, bt, theta, kw):
    import torch
    dev = device()
    tok, ln, sc, ws = P.ctcbeam_decode_nbest(torch.from_numpy(lp).to(dev), torch.from_numpy(lens).to(dev), K, alpha,
                                             beta, w, lm, bt, theta=theta, **kw)
    torch.cuda.synchronize()
    assert P.ctcbeam_query_status(ws) == 0
    return tok.cpu().numpy(), ln.cpu().numpy(), sc.cpu().numpy()


def _compare(g, r):
    np.testing.assert_array_equal(g[1], r["nbest_lengths"])
    np.testing.assert_array_equal(g[0], r["nbest_tokens"])
    np.testing.assert_allclose(g[2], r["nbest_scores"], rtol=0, atol=1e-4)


@pytest.mark.parametrize("V,K,order,phrases,theta,kw", CASES)
def test_multi_chunk(V, K, order, phrases, theta, kw):
    B, T = 4, 40
    rng = np.random.default_rng([V, K, order])
    lp = W.random_logprobs(rng, B, T, V)
    lens = np.array([T, 23, 1, 0], dtype=np.int32)
    counts = (min(6 * V, V * V), 4 * V, 2 * V, 2 * V)[: order - 1] if order else ()
    spec = W.LMSpec(order=order, counts=counts, seed=V + K) if order else None
    bspec = W.BoostSpec(phrases, 2, 4, "zipf", V) if phrases else None
    log("multi-chunk", V, K, order, phrases, theta, kw)
    alpha, w = (0.5 if order else 0.0), (1.25 if phrases else 0.0)
    g = _decode(lp, lens, K, alpha, 1.0, w, gpu_lm(spec, V) if spec else None, gpu_boost(bspec, V) if bspec else None,
                theta, kw)
    okw = {k: v for k, v in kw.items() if k != "row_cache"}
    r = oracle.decode(lp, lens, K, alpha, 1.0, w, theta=theta, lm=oracle_lm(spec, V) if spec else None,
                      bt=oracle_bt(bspec, V) if bspec else None, n_threads=oracle_threads(), want_nbest=True, **okw)
    _compare(g, r)


@pytest.mark.parametrize("V,K,kind,kw", [(3100, 16, "lm", {}), (4096, 9, "lm", {"logsumexp": True}),
                                         (4096, 3, "phrases", {}), (2600, 4, "phrases", {"repeat_score": True})])
def test_multi_chunk_ties(V, K, kind, kw):
    """Rows of equal values under a flat unigram LM (or a phrase that hardly
    any label starts): every label ties, the pool overflows and the index
    order decides."""
    B, T = 2, 7
    lp = np.full((B, T, V + 1), -math.log(V + 1), dtype=np.float32)
    lp[1, 2:, V] = -0.5
    lp[1, 4] = -np.inf
    lp[1, 4, : V // 2] = -2.0
    lens = np.array([T, T], dtype=np.int32)
    log("multi-chunk ties", V, K, kind)
    lm = olm = bt = obt = None
    if kind == "lm":
        ids = [np.arange(V + 2, dtype=np.int32)[:, None]]
        arrays = dict(order=1, V=V, ids=ids, log10_prob=[np.full(V + 2, -2.0, dtype=np.float32)], log10_bow=[None])
        lm, olm = P.ctcbeam_lm_build(arrays), oracle.LM(arrays)
    else:
        off, toks = np.array([0, 2], dtype=np.int32), np.array([V - 2, 5], dtype=np.int32)
        bt, obt = P.ctcbeam_boost_build(V, off, toks), oracle.BT(V, off, toks)
    alpha, w = (0.5 if lm else 0.0), (0.5 if bt else 0.0)
    g = _decode(lp, lens, K, alpha, 0.25, w, lm, bt, math.inf, kw)
    r = oracle.decode(lp, lens, K, alpha, 0.25, w, lm=olm, bt=obt, want_nbest=True, **kw)
    _compare(g, r)
