"""The oracle where LM.Final ends hypotheses: -inf or NaN (0 * -inf) final
scores are dead slots, ranked last, empty."""
import numpy as np

import oracle


def test_dead_final_scores():
    V = 3
    uni = np.full(V + 2, -0.7, dtype=np.float32)
    bi = np.array([[0, V]], dtype=np.int32)
    arrays = dict(order=2, V=V, ids=[np.arange(V + 2, dtype=np.int32)[:, None], bi],
                  log10_prob=[uni, np.array([-np.inf], dtype=np.float32)],
                  log10_bow=[np.zeros(V + 2, dtype=np.float32), None])
    lp = np.log(np.array([[[0.6, 0.3, 0.05, 0.05]]], dtype=np.float32))
    for alpha in (0.5, 0.0):
        r = oracle.decode(lp, np.array([1], dtype=np.int32), 3, alpha, 0.0, lm=oracle.LM(arrays), want_nbest=True)
        assert r["tokens"][0, 0] == 1 and np.isfinite(r["scores"][0])
        assert r["nbest_tokens"][0, :, 0].tolist()[0] == 1
        assert r["nbest_lengths"][0, 2] == 0 and r["nbest_tokens"][0, 2, 0] == -1
        assert np.isneginf(r["nbest_scores"][0, 2]) and np.isfinite(r["nbest_scores"][0, :2]).all()


def test_nan_scores_are_dead_candidates():
    """A NaN counts as -inf: the same search as with -inf in its place."""
    rng = np.random.default_rng(3)
    V, T = 6, 12
    lp = np.log(rng.dirichlet(np.ones(V + 1), size=(2, T))).astype(np.float32)
    nan = rng.random(lp.shape) < 0.3
    nan[:, 3, V] = True
    a, b = lp.copy(), lp.copy()
    a[nan], b[nan] = np.nan, -np.inf
    lens = np.array([T, T - 2], dtype=np.int32)
    for kw in ({}, {"logsumexp": True}):
        x, y = (oracle.decode(q, lens, 8, 0.0, 0.5, want_nbest=True, **kw) for q in (a, b))
        for k in ("tokens", "lengths", "scores", "nbest_tokens", "nbest_lengths", "nbest_scores"):
            np.testing.assert_array_equal(x[k], y[k])
