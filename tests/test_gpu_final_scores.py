"""GPU parity where LM.Final ends hypotheses: </s> has probability 0 (log10
-inf) after some tokens, so a live beam's final score is -inf, or NaN from
0 * -inf with alpha = 0 (a NaN score counts as -inf).  Such a slot is dead:
empty, -inf, ranked last.  Beam, N-best and greedy against the CPU oracle:
tokens and lengths equal, scores within 1e-4."""
import numpy as np
import pytest

import oracle
import paper_2508_07315_amd as P
import workloads as W
from gpu_helpers import compare, device, log, oracle_threads, run_gpu

pytestmark = pytest.mark.gpu


def _lm(V, kind):
    """2-gram over V tokens: no </s> after the even tokens ("some") or at all."""
    uni = np.full(V + 2, -np.log10(V + 2), dtype=np.float32)
    if kind == "all":
        uni[V] = -np.inf
    even = np.arange(0, V, 2, dtype=np.int32)
    bi = np.stack([even, np.full_like(even, V)], axis=1)
    return dict(order=2, V=V, ids=[np.arange(V + 2, dtype=np.int32)[:, None], bi],
                log10_prob=[uni, np.full(len(bi), -np.inf, dtype=np.float32)],
                log10_bow=[np.zeros(V + 2, dtype=np.float32), None])


# one chunk of the general decoder, the class decoder (one and two register
# sets), several chunks of the general decoder
@pytest.mark.parametrize("V,K", [(40, 8), (700, 4), (40, 16), (700, 20), (600, 100), (3100, 16)])
@pytest.mark.parametrize("kind,alpha", [("some", 0.5), ("some", 0.0), ("all", 0.5), ("all", 0.0)])
def test_final_scores(V, K, kind, alpha):
    import torch
    B, T = 4, 30
    rng = np.random.default_rng([V, K])
    lp = W.random_logprobs(rng, B, T, V)
    lens = np.array([T, 13, 2, 0], dtype=np.int32)
    arrays = _lm(V, kind)
    lm, olm = P.ctcbeam_lm_build(arrays), oracle.LM(arrays)
    log("final scores", V, K, kind, alpha)
    r = oracle.decode(lp, lens, K, alpha, 1.0, lm=olm, want_nbest=True, n_threads=oracle_threads())
    if kind == "some":  # the case is what it says
        live = np.isfinite(r["nbest_scores"][:3])
        assert live.any() and not live.all()
    compare(run_gpu(lp, lens, K, alpha, 1.0, lm=lm), r, what="beam")
    dev = device()
    tok, ln, sc, _ = P.ctcbeam_decode_nbest(torch.from_numpy(lp).to(dev), torch.from_numpy(lens).to(dev), K, alpha, 1.0,
                                            0.0, lm)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(ln.cpu().numpy(), r["nbest_lengths"])
    np.testing.assert_array_equal(tok.cpu().numpy(), r["nbest_tokens"])
    np.testing.assert_allclose(sc.cpu().numpy(), r["nbest_scores"], rtol=0, atol=1e-4)


@pytest.mark.parametrize("V", [40, 700, 3100])
@pytest.mark.parametrize("kind,alpha", [("some", 0.5), ("some", 0.0), ("all", 0.5)])
def test_final_scores_greedy(V, kind, alpha):
    import torch
    B, T = 12, 300
    rng = np.random.default_rng(V)
    lp = W.random_logprobs(rng, B, T, V)
    lens = rng.integers(1, T + 1, size=B).astype(np.int32)
    arrays = _lm(V, kind)
    log("final scores, greedy", V, kind, alpha)
    dev = device()
    tok, ln, sc, _ = P.ctcbeam_greedy_decode(torch.from_numpy(lp).to(dev), torch.from_numpy(lens).to(dev), alpha, 1.0,
                                             0.0, P.ctcbeam_lm_build(arrays))
    torch.cuda.synchronize()
    r = oracle.decode(lp, lens, 1, alpha, 1.0, lm=oracle.LM(arrays), n_threads=oracle_threads())
    assert np.isneginf(r["scores"]).any()
    compare(dict(tokens=tok.cpu().numpy(), lengths=ln.cpu().numpy(), scores=sc.cpu().numpy()), r, what="greedy")
