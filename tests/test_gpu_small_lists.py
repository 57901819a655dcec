"""GPU parity of the small-beam decoder (K <= 8, no models) where its label
lists can go wrong: vocabularies below, at and above the list length, the lane
count and the labels per lane (64, 256, 1024), lengths at the edges of a batch
of frames (6), and values with many ties (few distinct values, equal rows,
-inf), which the exact keys have to settle.  Against the CPU oracle, N-best:
tokens and lengths equal, scores within 1e-4."""
import math

import numpy as np
import pytest

import oracle
import paper_2508_07315_amd as P
from gpu_helpers import device, log, oracle_threads

pytestmark = pytest.mark.gpu

SIZES = [(1, 1), (1, 8), (2, 3), (8, 8), (9, 8), (10, 8), (11, 7), (29, 5), (63, 8), (64, 4), (65, 8), (255, 2),
         (256, 8), (257, 6), (600, 1), (1000, 8), (1023, 3), (1024, 8)]
LENGTHS = (26, 0, 1, 5, 6, 7, 12, 13)


def _rows(kind, rng, B, T, V):
    W = V + 1
    if kind == "random":
        x = rng.normal(0.0, 3.0, (B, T, W))
    elif kind == "few values":  # ties inside and outside the list
        x = -0.5 * rng.integers(0, 4, (B, T, W))
    elif kind == "equal rows":
        x = np.full((B, T, W), -math.log(W))
        x[:, 3::4, V] = -0.25
    else:  # "floor": most labels at one low value or impossible
        x = np.where(rng.random((B, T, W)) < 0.02, rng.normal(0.0, 2.0, (B, T, W)), -30.0)
        x[:, 2::5, : (V + 1) // 2] = -np.inf
        x[:, 4::9, : V] = -np.inf
    return x.astype(np.float32)


@pytest.mark.parametrize("kind", ["random", "few values", "equal rows", "floor"])
@pytest.mark.parametrize("V,K", SIZES)
def test_small_lists(V, K, kind):
    import torch
    rng = np.random.default_rng([V, K, len(kind)])
    lens = np.array(LENGTHS, dtype=np.int32)
    lp = _rows(kind, rng, len(lens), int(lens.max()), V)
    dev = device()
    for beta, theta in ((1.0, math.inf), (-0.75, 6.0)):
        log("small lists", V, K, kind, beta, theta)
        tok, ln, sc, ws = P.ctcbeam_decode_nbest(torch.from_numpy(lp).to(dev), torch.from_numpy(lens).to(dev), K, 0.0,
                                                 beta, theta=theta)
        torch.cuda.synchronize()
        assert P.ctcbeam_query_status(ws) == 0
        r = oracle.decode(lp, lens, K, 0.0, beta, theta=theta, n_threads=oracle_threads(), want_nbest=True)
        np.testing.assert_array_equal(ln.cpu().numpy(), r["nbest_lengths"])
        np.testing.assert_array_equal(tok.cpu().numpy(), r["nbest_tokens"])
        np.testing.assert_allclose(sc.cpu().numpy(), r["nbest_scores"], rtol=0, atol=1e-4)
