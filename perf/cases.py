"""The calls whose speed matters to a user of this framework, with their inputs.

Each case is one pass of a public operation over seeded synthetic inputs with
the distributions of ``synth`` (unit-norm embeddings in clusters of about 47
to 60 records whose members lie at cosine U(0.80, 0.999) from their centre,
queries near random centres at cosine U(0.5, 0.9), raw values half N(0, 0.04^2)
and half U(-1, 1)), drawn on the GPU.  The operations:

  qeps    Q_eps encode and decode of a float32 array (``quantize``/``dequantize``)
  ingest  the greedy near-duplicate test over a stream of records, call by call,
          into an emptied store (``Store.ingest``; with ``band_width`` the
          candidates come from the band index)
  score   top-k retrieval of a batch of queries against a quantized store
          (``Store.score_topk``)
  codec   the store's codecs: Q_eps codes of the retained rows, their per-block
          encoding exported and decoded, and retrieval from the blocks

``exact`` gives the floating outputs in binary64 from plain torch.
"""
from __future__ import annotations

import math

import torch

import paper_2609_32256_amd as lam

TAU = 0.95
CORPUS_ROWS, CORPUS_QUERIES = 361802, 4096
BULK_ROWS, BULK_DIM = 131072, 1024
KEEP = 0.85          # share of a clustered stream retained at TAU


def listed():
    return [
        # one small array quantized and read back: the latency of a call
        dict(name="qeps_call", op="qeps", n=10007, eps=1e-3, mode="bits", declared=False),
        # the quantizer microbenchmark: 2^26 values, 10-bit codes
        dict(name="qeps_bulk", op="qeps", n=1 << 26, eps=1e-3, mode="bits", declared=True),
        # an agent admits the chunks of its trajectories as they finish: eight
        # calls of 47 records, each waiting for its decisions
        dict(name="ingest_calls", op="ingest", n=376, dim=768, batch=47, wait=True, shuffled=False, band_width=0, rel=0.0),
        # the 600-trajectory stream in batches of 1,024, calls that do not wait
        dict(name="ingest_stream", op="ingest", n=27986, dim=768, batch=1024, wait=False, shuffled=False, band_width=0,
             rel=0.0),
        # a small encoder's embeddings in ragged batches
        dict(name="ingest_384", op="ingest", n=20011, dim=384, batch=1999, wait=False, shuffled=True, band_width=0,
             rel=0.0),
        # building a large store: 4,096-row calls of 1,024-dimensional records
        dict(name="ingest_bulk", op="ingest", n=BULK_ROWS, dim=BULK_DIM, batch=4096, wait=False, shuffled=True,
             band_width=0, rel=0.0),
        # the stream with candidates from the band index (bands of 8 at 0.3 sigma)
        dict(name="ingest_banded", op="ingest", n=27986, dim=768, batch=1024, wait=False, shuffled=False, band_width=8,
             rel=0.3),
        # one query of a serving loop against the whole corpus
        dict(name="score_one", op="score", nq=1, n=CORPUS_ROWS, dim=768, k=10, eps=1e-3),
        # a batch of queries against the retained rows of the stream
        dict(name="score_store", op="score", nq=1024, n=23969, dim=768, k=10, eps=1e-3),
        # a small encoder's store, ragged sizes, long result lists
        dict(name="score_384", op="score", nq=300, n=120001, dim=384, k=50, eps=1e-3),
        # the retrieval benchmark: 4,096 queries against the whole corpus
        dict(name="score_corpus", op="score", nq=CORPUS_QUERIES, n=CORPUS_ROWS, dim=768, k=10, eps=1e-3),
        # the codecs of the stream's store, and retrieval from its blocks
        dict(name="codec_store", op="codec", nq=64, n=23969, dim=768, k=10, eps=1e-3),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["qeps", "ingest", "ingest", "banded", "score", "score", "score", "codec"])
    if op == "qeps":
        return dict(op="qeps", n=_log_int(rng, 1000, 1 << 26), eps=10.0 ** rng.uniform(-5, -2),
                    mode=rng.choice(["bits", "bits", "bytes"]), declared=rng.random() < 0.5)
    dim = rng.choice([128, 256, 384, 512, 768, 768, 1024, 1024, 1536])
    if op == "ingest":
        n = min(_log_int(rng, 64, BULK_ROWS), int(math.sqrt(float(BULK_ROWS) ** 2 * BULK_DIM / dim)))
        batch = min(n, max(_log_int(rng, 16, 4096), -(-n // 128)))
        return dict(op="ingest", n=n, dim=dim, batch=batch, wait=rng.random() < 0.4, shuffled=rng.random() < 0.5,
                    band_width=0, rel=0.0)
    if op == "banded":
        n = _log_int(rng, 1000, 28000)
        return dict(op="ingest", n=n, dim=dim, batch=min(n, max(_log_int(rng, 64, 4096), -(-n // 64))),
                    wait=rng.random() < 0.4, shuffled=rng.random() < 0.5, band_width=rng.choice([8, 8, 16]),
                    rel=rng.choice([0.1, 0.2, 0.3]))
    # eps from 1e-2 (codes of about 5 bits) to 1e-5 (about 15 bits, the split form)
    eps = 10.0 ** rng.uniform(-5, -2)
    k = rng.choice([1, 5, 10, 10, 20, 50, 64])
    if op == "score":
        n = _log_int(rng, 1000, CORPUS_ROWS)
        most = CORPUS_QUERIES * CORPUS_ROWS * 768 // (n * dim * (4 if eps < 1e-4 else 1))
        return dict(op="score", nq=min(_log_int(rng, 1, CORPUS_QUERIES), max(1, most)), n=n, dim=dim, k=k, eps=eps)
    return dict(op="codec", nq=_log_int(rng, 1, 1024), n=_log_int(rng, 1000, 60000), dim=dim, k=k, eps=eps)


# ------------------------------------------------------------------ inputs
def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _unit(v):
    return v / torch.linalg.vector_norm(v, dim=1, keepdim=True)


def _near(g, mu, lo, hi):
    """One unit row per row of mu, at cosine U(lo, hi) to it."""
    c = lo + (hi - lo) * torch.rand((mu.shape[0], 1), generator=g, device="cuda")
    u = torch.randn(mu.shape, generator=g, device="cuda")
    u -= (u * mu).sum(dim=1, keepdim=True) * mu
    return _unit(c * mu + torch.sqrt(1.0 - c * c) * _unit(u))


def _records(g, n, dim, per_cluster, shuffled):
    """n clustered unit rows (the clusters contiguous, or in random order) and
    the cluster centres."""
    clusters = max(1, n // per_cluster)
    centres = _unit(torch.randn((clusters, dim), generator=g, device="cuda"))
    label = torch.arange(n, device="cuda") * clusters // n
    if shuffled:
        label = label[torch.randperm(n, generator=g, device="cuda")]
    x = torch.empty((n, dim), device="cuda")
    for s in range(0, n, 1 << 16):
        x[s:s + (1 << 16)] = _near(g, centres[label[s:s + (1 << 16)]], 0.80, 0.999)
    return x, centres


def _queries(g, centres, nq):
    return _near(g, centres[torch.randint(0, centres.shape[0], (nq,), generator=g, device="cuda")], 0.5, 0.9)


def _raw(seed, n):
    g = _generator(seed)
    x = torch.empty(n, device="cuda")
    h = n // 2
    x[:h] = 0.04 * torch.randn(h, generator=g, device="cuda")
    x[h:] = 2.0 * torch.rand(n - h, generator=g, device="cuda") - 1.0
    return x


def _retrieval(case, seed):
    g = _generator(seed)
    x, centres = _records(g, case["n"], case["dim"], 60, True)
    return x, _queries(g, centres, case["nq"])


# ------------------------------------------------------------------ the cases
def prepare(case, seed):
    if case["op"] == "qeps":
        x = _raw(seed, case["n"])
        return dict(case=case, x=x, absmax=float(x.abs().max()) if case["declared"] else None)
    if case["op"] == "ingest":
        x, _ = _records(_generator(seed), case["n"], case["dim"], 47, case["shuffled"])
        band = {}
        if case["band_width"]:
            band = dict(eps_band=case["rel"] / math.sqrt(case["dim"]), band_width=case["band_width"])
        return dict(case=case, batches=x.split(case["batch"]), store=lam.Store(case["dim"], TAU, case["n"], **band))
    # a store that keeps every record (tau = 1 merges exact copies only)
    x, q = _retrieval(case, seed)
    store = lam.Store(case["dim"], 1.0, case["n"])
    for rows in x.split(4096):
        store.ingest(rows, sync=False)
    store.quantize(case["eps"])
    return dict(case=case, store=store, q=q)


def run(state):
    case = state["case"]
    if case["op"] == "qeps":
        codes, p = lam.quantize(state["x"], case["eps"], absmax=state["absmax"], mode=case["mode"])
        return dict(codes=codes, xhat=lam.dequantize(codes, p))
    store = state["store"]
    if case["op"] == "ingest":
        store.clear()
        rep = [store.ingest(rows, sync=case["wait"])[0] for rows in state["batches"]]
        # the retained ids, padded to the arrivals: their number depends on the data
        return dict(rep=rep if len(rep) <= 8 else torch.cat(rep), ids=_padded(store.ids(), case["n"]),
                    delta_hat=store.info().delta_hat_run)
    if case["op"] == "score":
        scores, ids, bound = store.score_topk(state["q"], case["k"])
        return dict(scores=scores, ids=ids, bound=bound)
    store.quantize(case["eps"])
    store.block_encode()
    widths, row_off, data = store.block_export()
    xhat = store.block_decode()
    scores, ids, bound = store.score_topk_blocks(state["q"], case["k"])
    data = _padded(data, case["n"] * case["dim"] * (_bits(case) + 1) // 32)
    return dict(widths=widths, row_off=row_off, data=data, xhat=xhat, scores=scores, ids=ids, bound=bound)


def _padded(v, n):
    return torch.nn.functional.pad(v, (0, max(0, n - v.shape[0])), value=-1)


def _bits(case):
    """About the code width of unit rows (largest coordinate near 5 sigma) or raw values."""
    top = 1.0 if case["op"] == "qeps" else 5.0 / math.sqrt(case["dim"])
    return max(1, math.ceil(math.log2(top / case["eps"] + 1)))


def work(case):
    n = case["n"]
    if case["op"] == "qeps":
        b = _bits(case)
        if case["mode"] == "bytes":
            b = 8 if b <= 8 else 16 if b <= 16 else 32
        return dict(bytes=n * (8 + 2 * b / 8), flops=0)
    dim = case["dim"]
    if case["op"] == "ingest":
        # each record read once; a retained one stored in float32
        pairs = 0 if case["band_width"] else KEEP * n * (n - 1) / 2
        return dict(bytes=n * dim * 4 * (1 + KEEP), flops=2.0 * dim * pairs)
    codes, q = n * dim * _bits(case) / 8, case["nq"] * (dim * 4 + case["k"] * 12)
    if case["op"] == "score":
        return dict(bytes=codes + q, flops=2.0 * dim * n * case["nq"])
    # rows to codes, codes to blocks, blocks out, blocks to rows, blocks to scores
    return dict(bytes=n * dim * 8 + 7 * codes + q, flops=2.0 * dim * n * case["nq"])


def tolerance(case):
    if case["op"] == "qeps":
        return "exact"
    if case["op"] == "ingest":
        return dict(rel=2.5e-7)   # the decisions are exact; delta_hat is compared in float32
    # float32 scores; two records whose scores agree to rounding may change places
    # (fp32 accumulation over a small store is within 4e-7 of the binary64 scores)
    return dict(rel=1.6e-6, max=1.6e-5, differ=1e-3)


# ------------------------------------------------------------------ binary64 values
def _codes64(x, eps):
    return torch.round(x.double() / (2.0 * eps))   # half to even


def _scores64(x, q, eps, k):
    """The k best q . x_hat of every query, descending, padded with -inf."""
    best = torch.full((q.shape[0], k), -math.inf, dtype=torch.float64, device="cuda")
    for rows in x.split(1 << 15):
        s = q.double() @ (_codes64(rows, eps) * (2.0 * eps)).T.contiguous()
        best = torch.cat([best, s], dim=1).topk(k, dim=1).values
    return best


def _delta64(x):
    """The largest distance from a dropped row to its representative under the
    greedy test over all earlier retained rows."""
    n = x.shape[0]
    x = x.double()
    half = 0.5 * (x * x).sum(dim=1)
    near = {}
    for s in range(0, n, 2048):
        e = min(n, s + 2048)
        d2 = 2.0 * (half[s:e, None] + half[None, :e] - x[s:e] @ x[:e].T)
        ok = (d2 <= 2.0 - 2.0 * TAU) & (torch.arange(e, device="cuda")[None, :] < torch.arange(s, e, device="cuda")[:, None])
        for i, j in ok.nonzero().tolist():   # ascending j within each row
            near.setdefault(s + i, []).append(j)
    kept, pairs = [True] * n, []
    for i in range(n):
        for j in near.get(i, ()):
            if kept[j]:
                kept[i] = False
                pairs.append((i, j))
                break
    if not pairs:
        return 0.0
    p = torch.tensor(pairs, device="cuda")
    return float(torch.linalg.vector_norm(x[p[:, 0]] - x[p[:, 1]], dim=1).max())


def exact(case, seed):
    if case["op"] == "qeps":
        return dict(codes=None, xhat=_codes64(_raw(seed, case["n"]), case["eps"]) * (2.0 * case["eps"]))
    if case["op"] == "ingest":
        if case["band_width"]:
            return None   # the candidates are those of the band index
        x, _ = _records(_generator(seed), case["n"], case["dim"], 47, case["shuffled"])
        return dict(rep=None, ids=None, delta_hat=_delta64(x))
    x, q = _retrieval(case, seed)
    out = dict(scores=_scores64(x, q, case["eps"], case["k"]), ids=None,
               bound=case["eps"] * q.double().abs().sum(dim=1))
    if case["op"] == "codec":
        out.update(widths=None, row_off=None, data=None, xhat=_codes64(x, case["eps"]) * (2.0 * case["eps"]))
    return out
