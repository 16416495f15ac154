"""GPU parity of the scoring passes at the edges of their tiles: dimensions
that fill no whole slab of 64 (and none at all), odd and even code widths, row
and query counts one past a tile, every range of k, and more near-equal rows
than the rescoring takes or the candidate buffer holds."""
import numpy as np
import pytest

import synth
from oracle import qeps
from test_gpu_score import _compare, _dev, _flip_store, _store_from_rows

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,n,nq,k,eps", [
    (32, 4225, 1, 64, 1e-3),       # half a slab, one row past a tile, one query
    (96, 5001, 129, 17, 4e-3),     # a slab and a half, one query past a tile
    (160, 12289, 33, 1, 2e-2),     # 5-bit codes
    (384, 9001, 300, 50, 1e-3),    # 9-bit codes, six slabs
    (416, 4500, 64, 5, 3e-4),      # seven slabs, the last one half full
    (1536, 4353, 130, 16, 1e-3),   # 24 slabs
])
def test_dimensions_and_edges(lam, d, n, nq, k, eps):
    rng = np.random.default_rng(d + n)
    x = synth.unit_rows(rng, n, d).astype(np.float32)
    s = _store_from_rows(lam, x)
    s.quantize(eps)
    q = synth.unit_rows(rng, nq, d)
    h = nq // 2
    q[:h] = synth.members(rng, x[rng.choice(n, h)].astype(np.float64), rng.uniform(0.6, 0.99, h)) if h else q[:h]
    q = q.astype(np.float32)
    gs, gi, _ = s.score_topk(_dev(q), k)
    c = qeps.codes(x, eps).reshape(n, -1)
    _compare(gs.cpu().numpy(), gi.cpu().numpy(), c, np.arange(n), q, eps, k)


@pytest.mark.parametrize("group,n", [(1500, 6000), (4500, 9000)])
@pytest.mark.parametrize("k", [1, 10, 64])
def test_many_equal_rows(lam, group, n, k):
    """`group` rows tied with row 200 (identical codes): more than the 1,024
    rows that are rescored, and more than the 4,096 candidates that are kept;
    the k best are the tied rows in id order."""
    x, q = _flip_store(n=n, group=group)
    s = _store_from_rows(lam, x)
    eps = 2.0 ** -11
    s.quantize(eps)
    c = qeps.codes(x, eps).reshape(n, -1)
    gs, gi, _ = s.score_topk(_dev(q), k)
    gi = gi.cpu().numpy()
    assert np.array_equal(gi[2], np.concatenate([[200], np.arange(300, 300 + k - 1)]))
    _compare(gs.cpu().numpy(), gi, c, np.arange(n), q, eps, k)
