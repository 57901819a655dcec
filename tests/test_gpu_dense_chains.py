"""GPU parity with dense language models over small vocabularies: nearly every
level of every beam's backoff chain holds explicit continuations, so a frame
fills more than 32 runs of arcs at once.  Against the CPU oracle, N-best:
tokens and lengths equal, scores within 1e-4."""
import numpy as np
import pytest

import oracle
import paper_2508_07315_amd as P
import workloads as W
from gpu_helpers import device, gpu_lm, log, oracle_lm, oracle_threads

pytestmark = pytest.mark.gpu

COUNTS = {4: (620, 9000, 40000), 5: (620, 9000, 40000, 60000), 6: (620, 9000, 40000, 60000, 60000)}


@pytest.mark.parametrize("order,K", [(4, 11), (4, 16), (5, 9), (5, 16), (5, 40), (6, 7), (6, 8), (6, 24)])
def test_dense_chains(order, K):
    import torch
    V, B, T = 24, 3, 60
    spec = W.LMSpec(order=order, counts=COUNTS[order], seed=70 + order)
    rng = np.random.default_rng(100 * order + K)
    lp = W.random_logprobs(rng, B, T, V)
    lens = np.array([T, T - 7, T // 2], dtype=np.int32)
    log("dense chains", order, K)
    dev = device()
    tok, ln, sc, ws = P.ctcbeam_decode_nbest(torch.from_numpy(lp).to(dev), torch.from_numpy(lens).to(dev), K,
                                             0.5, 1.0, 0.0, gpu_lm(spec, V))
    torch.cuda.synchronize()
    assert P.ctcbeam_query_status(ws) == 0
    r = oracle.decode(lp, lens, K, 0.5, 1.0, lm=oracle_lm(spec, V), n_threads=oracle_threads(), want_nbest=True)
    np.testing.assert_array_equal(ln.cpu().numpy(), r["nbest_lengths"])
    np.testing.assert_array_equal(tok.cpu().numpy(), r["nbest_tokens"])
    np.testing.assert_allclose(sc.cpu().numpy(), r["nbest_scores"], rtol=0, atol=1e-4)
