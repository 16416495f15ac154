"""GPU parity of the scoring passes at the edges of their tiles: dimensions
that fill no whole slab of 64 (and none at all), odd and even code widths, row
and query counts one past a tile, every range of k, and more near-equal rows
than the rescoring takes or the candidate buffer holds."""
import numpy as np
import pytest

import synth
from oracle import qeps, score
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


@pytest.mark.parametrize("d,n,bits,absmax", [
    (96, 4225, 13, None),       # one low bit left out of the scan, one row past a tile
    (160, 5000, 15, None),
    (384, 4500, 22, None),      # ten bits left out
    (64, 4300, 16, 50.0),       # a declared absmax far above the rows: 16-bit codes of 10-bit values
])
def test_wide_codes_scan(lam, d, n, bits, absmax):
    """Codes of more than 12 bits are scanned without their low bits; the
    scores and the order are those of the whole codes.  A query entry that
    overflows float32 when scaled by 2^11 makes its row invalid."""
    rng = np.random.default_rng(bits)
    x = synth.unit_rows(rng, n, d).astype(np.float32)
    s = _store_from_rows(lam, x)
    eps = (absmax or float(np.abs(x).max())) / 2.0 ** bits * 1.01
    p = s.quantize(eps, absmax=absmax)
    assert p.bits == bits
    q = np.concatenate([synth.unit_rows(rng, 20, d),
                        synth.members(rng, x[rng.choice(n, 20)].astype(np.float64), rng.uniform(0.6, 0.99, 20))])
    q = q.astype(np.float32)
    q[5, 3] = 1e36
    gs, gi, gb = (t.cpu().numpy() for t in s.score_topk(_dev(q), 20))
    assert np.all(gi[5] == -1) and np.all(np.isnan(gs[5])) and np.isnan(gb[5])
    keep = [j for j in range(q.shape[0]) if j != 5]
    c = qeps.codes(x, eps).reshape(n, -1)
    _compare(gs[keep], gi[keep], c, np.arange(n), q[keep], eps, 20)


def _rows_above(q, c, eps, k):
    """Per query, the rows that the sample tells of above the byte scan's
    threshold, by the rule that chooses between the scans (past a limit that
    grows with the launch's tiles the query's group of 256 takes the fp16 scan),
    from binary64 scores."""
    q = q.astype(np.float64)
    n, d = c.shape
    R = np.sqrt(((c * (2 * eps)) ** 2).sum(1).max()) + eps * np.sqrt(d)
    mx = np.abs(q).max(1, keepdims=True)
    e = 14 - np.floor(np.log2(mx))
    h = (q * 2.0 ** e).astype(np.float16) * 2.0 ** -e
    v = np.rint(q / (mx / 127)) * (mx / 127)
    qn, dh, db = (np.linalg.norm(a, axis=1) for a in (q, q - h, q - v))
    err = (dh + (2 * (d + 64) * 2.0 ** -24 + 2.0 ** -21) * (qn + dh) + db + 2.0 ** -21 * (qn + db)) * R
    tiles = min(n // 128, -(-max(4096, -(-k * n // 256)) // 128))
    best = score.scores(q, c[:tiles * 128], eps).reshape(len(q), tiles * 2, 8, 2, 4).max(axis=(2, 4))
    best = best.reshape(len(q), -1)                       # each entry the best of 32 rows
    kth = np.sort(best, axis=1)[:, -k]
    f = (best >= (kth - err)[:, None]).mean(1)
    return -np.log(np.maximum(1 - f, 1e-6)) * n / 32


@pytest.mark.parametrize("kind", ["gaussian", "spiky", "concentrated"])
@pytest.mark.parametrize("d,n,nq,bits,absmax", [
    (96, 4225, 130, 3, None),      # a partly empty slab of bytes
    (160, 9000, 257, 7, None),     # two groups of queries
    (768, 33001, 2100, 8, None),   # the large tile
    (128, 6000, 40, 10, 1.9),      # 10-bit storage of 8-bit codes
])
def test_byte_scan(lam, kind, d, n, nq, bits, absmax):
    """Codes that fit 8 bits are scanned as bytes: Gaussian queries; queries
    whose largest entry dominates (a wide error bound, in one group of 256
    queries only); rows so close together that the bound covers many of them."""
    rng = np.random.default_rng(bits)
    if kind == "concentrated":
        x = synth.members(rng, np.repeat(synth.unit_rows(rng, 1, d), n, axis=0), rng.uniform(0.97, 0.99, n))
    else:
        x = synth.unit_rows(rng, n, d)
    x = x.astype(np.float32)
    top = float(np.abs(x).max())
    s = _store_from_rows(lam, x)
    eps = absmax / 2.0 ** bits * 1.01 if absmax else top / (2 ** bits - 1.5) if bits < 8 else top / 250.0
    p = s.quantize(eps, absmax=absmax)
    assert p.bits == bits and top / (2 * eps) < 127
    q = synth.members(rng, x[rng.choice(n, nq)].astype(np.float64), rng.uniform(0.5, 0.99, nq))
    if kind == "spiky":
        q[: nq // 2, rng.integers(0, d)] = 3.0
    q = q.astype(np.float32)
    gs, gi, _ = s.score_topk(_dev(q), 10)
    c = qeps.codes(x, eps).reshape(n, -1)
    # the scan that each group of 256 queries takes, from inputs clear of the limit
    above = _rows_above(q, c, eps, 10)
    limit = 2048 if -(-nq // 128) * -(-n // 128) >= 2048 else 256
    above = np.array([above[g:g + 256].max() for g in range(0, nq, 256)])
    fp16 = {("spiky", 768): [True] * 5 + [False] * 4, ("concentrated", 768): [True] * 9,
            ("concentrated", 160): [True, False], ("concentrated", 128): [True]}.get((kind, d), [False] * len(above))
    assert np.all(above[fp16] > 1.4 * limit) and np.all(above[np.logical_not(fp16)] < limit / 1.4)
    pick = np.unique(np.concatenate([rng.choice(nq, min(nq, 60), replace=False), [0, nq - 1]]))
    _compare(gs.cpu().numpy()[pick], gi.cpu().numpy()[pick], c, np.arange(n), q[pick], eps, 10, tol=3e-5)


@pytest.mark.parametrize("d,n,nq,flagged,k,bits", [
    (96, 9000, 40, 7, 10, 15),        # few flagged queries: one per work item
    (64, 6000, 150, 131, 64, 10),     # groups of four, the last one of three
    (768, 20000, 300, 257, 1, 9),     # the last one of one
    (4096, 5000, 140, 130, 10, 8),    # the widest rows, the last one of two
])
def test_many_flagged_queries(lam, d, n, nq, flagged, k, bits):
    """4,400 rows of the same codes lead for `flagged` of the queries, which
    overflow and are scored exactly, several to a work item; the others, and
    all-zero ones among them, are not disturbed."""
    rng = np.random.default_rng(d + n)
    v = synth.unit_rows(rng, 1, d)
    x = synth.unit_rows(rng, n, d)
    eps = float(max(np.abs(x).max(), np.abs(v).max())) / (2.0 ** bits - 2.5)
    g = np.sort(rng.permutation(n)[:4400])
    x[g] = np.round(v / (2 * eps)) * (2 * eps) + rng.uniform(-0.4, 0.4, (4400, d)) * eps
    x = x.astype(np.float32)
    s = _store_from_rows(lam, x)
    assert s.quantize(eps).bits == bits
    c = qeps.codes(x, eps).reshape(n, -1)
    assert np.all(c[g] == c[g[0]]) and s.info().size == n
    q = synth.unit_rows(rng, nq, d)
    f = np.sort(rng.permutation(nq)[:flagged])
    q[f] = v + 0.3 / np.sqrt(d) * rng.standard_normal((flagged, d))
    q = q.astype(np.float32)
    rest = np.setdiff1d(np.arange(nq), f)
    q[rest[:3]] = 0.0
    gs, gi, _ = (t.cpu().numpy() for t in s.score_topk(_dev(q), k))
    assert np.array_equal(gi[f], np.broadcast_to(g[:k], (flagged, k)))
    assert np.array_equal(gi[rest[:3]], np.broadcast_to(np.arange(k), (3, k))) and np.all(gs[rest[:3]] == 0.0)
    pick = np.concatenate([rest[3:23], f[:20], f[-3:]])
    _compare(gs[pick], gi[pick], c, np.arange(n), q[pick], eps, k, tol=2e-5)


@pytest.mark.parametrize("n", [300, 4500])
def test_more_queries_than_one_pass(lam, n):
    """65,536 queries share one pass's scratch; a call of more gives each query
    what a smaller call gives it."""
    import torch
    rng = np.random.default_rng(n)
    x = synth.unit_rows(rng, n, 32).astype(np.float32)
    s = _store_from_rows(lam, x)
    s.quantize(2e-3)
    q = torch.randn((65536 + 777, 32), generator=torch.Generator(device="cuda").manual_seed(n), device="cuda")
    got = s.score_topk(q, 7)
    for a, b in [(0, 130), (65400, 65536), (65536, 66313)]:
        assert all(torch.equal(g[a:b], w) for g, w in zip(got, s.score_topk(q[a:b].contiguous(), 7)))
