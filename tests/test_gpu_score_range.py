"""GPU parity of scoring at the ends of float32's range: queries so small that
their scale, their scores or their entries are subnormal, and queries so large
that scores overflow, on stores below and above 4,096 rows and for codes that
are scanned as bytes, as float16 values and without their low bits."""
import numpy as np
import pytest

import synth
from oracle import qeps, score
from test_gpu_score import _dev, _store_from_rows

pytestmark = pytest.mark.gpu


def _store(lam, n, d, bits, seed):
    rng = np.random.default_rng(seed)
    x = (synth.unit_rows(rng, n, d) * rng.uniform(0.2, 0.5, (n, 1))).astype(np.float32)
    eps = float(np.abs(x).max()) / (2.0 ** bits - 1.5)
    s = _store_from_rows(lam, x)
    assert s.quantize(eps).bits == bits
    return rng, s, qeps.codes(x, eps).reshape(n, -1), eps


@pytest.mark.parametrize("n", [3000, 5000])
@pytest.mark.parametrize("d,bits", [(32, 8), (768, 8), (32, 10), (768, 11), (32, 15)])
def test_tiny_queries(lam, n, d, bits):
    """One-hot, sparse and Gaussian queries times 2^-e: from e = 100 on the
    float32 score scale leaves the normal range, from 114 on the power of two
    that scales the query up does, and from 126 on the entries are subnormal.
    Scores are multiples of 2^-149, so they are compared, and may be ordered,
    to within one."""
    rng, s, c, eps = _store(lam, n, d, bits, 7 * d + bits)
    base = np.zeros((4, d))
    base[0, 0] = 1.0
    base[1, 1], base[1, 5] = -1.0, 0.75
    base[2:] = synth.unit_rows(rng, 2, d)
    expo = [90, 100, 106, 110, 113, 114, 120, 127, 140]
    q = np.concatenate([base * 2.0 ** -e for e in expo]).astype(np.float32)
    gs, gi, gb = (t.cpu().numpy() for t in s.score_topk(_dev(q), 10))
    for i, e in enumerate(expo):
        r, f = slice(4 * i, 4 * i + 4), 2.0 ** e
        tol = max(1e-5, f * 2.0 ** -149)
        S = score.scores(q[r].astype(np.float64) * f, c, eps)
        kth = np.sort(S, axis=1)[:, -10]
        for j in range(4):
            row = gi[r][j]
            assert np.unique(row).size == 10 and row.min() >= 0, (e, j)
            assert np.all(np.abs(gs[r][j].astype(np.float64) * f - S[j, row]) <= tol), (e, j)
            assert np.all(S[j, row] >= kth[j] - 2 * tol) and np.all(np.diff(S[j, row]) <= 2 * tol), (e, j)
    beta = score.bound(q, eps)
    assert np.all(gb >= beta) and np.all(gb.astype(np.float64) - beta <= 2.0 ** -149 + beta * 2.0 ** -22)


@pytest.mark.parametrize("n", [3000, 6000])
@pytest.mark.parametrize("eps", [1.0, 0.05])
def test_overflowing_scores(lam, n, eps):
    """Rows of entries up to 200 against queries near float32's largest value:
    every score -inf, every score +inf, both, and one finite query among them.
    The k best are those of the scores rounded to float32, equal ones by id."""
    rng = np.random.default_rng(int(100 * eps) + n)
    d, k = 32, 10
    x = rng.uniform(1.0, 200.0, (n, d)).astype(np.float32)
    x[:, 0] = rng.uniform(-200.0, 200.0, n).astype(np.float32)
    s = _store_from_rows(lam, x)
    s.quantize(eps)
    q = np.zeros((7, d), np.float32)
    q[0, 1:] = -3e38
    q[1, 1:] = 3e38
    q[2, 0] = 3e38
    q[3, 0] = -3e38
    q[4] = rng.standard_normal(d)
    q[5, 1:] = -1.1e35                     # the best scores finite, about half of all -inf
    q[6, 1:] = 1.1e35                      # about half of all +inf
    gs, gi, _ = (t.cpu().numpy() for t in s.score_topk(_dev(q), k))
    with np.errstate(over="ignore"):
        want = score.scores(q, qeps.codes(x, eps).reshape(n, -1), eps).astype(np.float32)
    ts, ti = score.topk(want, np.arange(n), k)
    for j in (0, 1, 2, 3, 6):
        assert np.array_equal(gs[j], ts[j]) and np.array_equal(gi[j], ti[j]), j
    for j in (4, 5):
        assert np.allclose(gs[j], ts[j], rtol=1e-5) and np.all(gi[j] >= 0), j
