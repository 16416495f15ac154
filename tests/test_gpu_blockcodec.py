"""GPU parity of the per-block codec of the store's codes against the oracle
(oracle/blockcodec.py): widths, row offsets and bit-plane words bit for bit,
decode equal to the store's Q_eps decode, scores equal to the fixed-width
scorer's, sizes and ratios as defined."""
import numpy as np
import pytest
import torch

import synth
from test_gpu_score import _compare
from oracle import blockcodec, dedup, qeps

pytestmark = pytest.mark.gpu


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _store(lam, x, tau, eps, batch=1024, spare=0):
    s = lam.Store(x.shape[1], tau, x.shape[0] + spare)
    xd = _dev(x)
    for b0 in range(0, x.shape[0], batch):
        s.ingest(xd[b0:b0 + batch])
    p = s.quantize(eps)
    return s, p


@pytest.fixture(scope="module")
def subset():
    cfg = synth.subset_ingest()
    return cfg, dedup.greedy(cfg["x"], 0.95)


@pytest.mark.parametrize("eps", [1e-2, 1e-3, 1e-4])
def test_subset_store_blocks_bit_exact(lam, subset, eps):
    """The whole 27,986-row subset stream at tau = 0.95, its store coded at
    each eps: the fixed-width codes and the block encoding equal the oracle's
    bit for bit, and top-10 scores of the stream's 1,024 queries match the
    oracle's."""
    cfg, ref = subset
    x = cfg["x"]
    s, p = _store(lam, x, 0.95, eps)
    kept = s.ids().cpu().numpy()
    assert np.array_equal(kept, ref["kept"])
    codes = qeps.codes(x[kept], eps).reshape(kept.size, -1)
    assert p.bits == qeps.plan(eps, float(np.abs(x[kept]).max()))["bits"]
    assert np.array_equal(s.codes().cpu().numpy().view(np.uint32), qeps.pack(codes, p.bits))
    ref = blockcodec.encode(codes)
    st = s.block_encode()
    w, ro, d = s.block_export()
    assert np.array_equal(w.cpu().numpy(), ref["widths"])
    assert np.array_equal(ro.cpu().numpy().astype(np.uint64), ref["row_off"])
    assert np.array_equal(d.cpu().numpy().view(np.uint32), ref["data"])
    sz = blockcodec.sizes(ref, codes.size)
    assert st["data_bytes"] == sz["data_bytes"] and st["meta_bytes"] == sz["meta_bytes"]
    assert st["bits_per_code"] == pytest.approx(sz["bits_per_code"], rel=1e-12)
    assert st["plain_bits"] == p.bits
    assert st["composite_ratio"] == pytest.approx(x.shape[0] * x.shape[1] * 4 / sz["total_bytes"], rel=1e-12)
    # lossless: the decode is the store's Q_eps decode, bit for bit
    assert torch.equal(s.block_decode(), s.dequantize())
    q = cfg["q"]
    gs, gi, _ = s.score_topk(torch.from_numpy(q).cuda(), 10)
    worst = _compare(gs.cpu().numpy(), gi.cpu().numpy(), codes, kept, q, eps, 10)
    assert worst <= 1e-5
    print(f"eps={eps}: b={p.bits}, {st['bits_per_code']:.3f} bits/code, codec x{st['codec_ratio']:.2f}, "
          f"composite x{st['composite_ratio']:.2f}")


def test_scores_from_blocks_equal_fixed_width(lam):
    t = synth.tiny_ingest()
    s, p = _store(lam, t["x"], t["tau"], t["eps"])
    s.block_encode()
    q = _dev(t["q"])
    for k in (1, 10, 64):
        a = s.score_topk(q, k)
        b = s.score_topk_blocks(q, k)
        assert all(torch.equal(u, v) for u, v in zip(a, b))


def test_zero_blocks_and_state(lam):
    """All-zero rows cost no data words; a stale encoding is refused."""
    rng = np.random.default_rng(3)
    x = synth.unit_rows(rng, 40, 96).astype(np.float32)
    x[5] = 0.0
    s, p = _store(lam, x, 1.0, 1e-3, spare=4)
    st = s.block_encode()
    w, ro, d = s.block_export()
    ro = ro.cpu().numpy()
    kept = s.ids().cpu().numpy().tolist()
    r5 = kept.index(5)
    assert ro[r5 + 1] == ro[r5] and w.cpu().numpy()[r5].tolist() == [0, 0, 0]
    s.ingest(_dev(synth.unit_rows(rng, 1, 96).astype(np.float32)))
    s.quantize(1e-3)
    with pytest.raises(lam.LamError) as e:
        s.block_decode()
    assert e.value.name == "LAM_ESTATE"
    s.block_encode()
    assert torch.equal(s.block_decode(), s.dequantize())


@pytest.mark.parametrize("bits,n,dim", [
    (1, 5, 32), (2, 257, 32), (7, 300, 96), (8, 33, 768), (9, 11, 4096), (15, 19, 160), (16, 130, 64),
    (17, 21, 384), (24, 9, 1024), (31, 13, 96), (32, 40, 224)])
def test_every_field_width_bit_exact(lam, bits, n, dim):
    """Code widths on both sides of the 8-, 16- and 32-bit fields a lane holds a
    block in, with row lengths and counts that leave a workgroup's threads, and
    the last workgroup's rows, over; blocks of every width from 0 to `bits`."""
    rng = np.random.default_rng(bits)
    x = rng.uniform(-1, 1, (n, dim // 32, 32)) * 2.0 ** -rng.integers(0, bits + 3, (n, dim // 32, 1))
    x = x.reshape(n, dim).astype(np.float32)
    x[0, 0], x[1, 1] = 1.0, -1.0
    x[3, :32] = 0.0
    eps = 1.0 if bits == 1 else 0.5 / ((1 << (bits - 1)) - 1.5 if bits > 2 else 1.0)
    s, p = _store(lam, x, 1.0, eps)
    assert p.bits == bits
    kept = s.ids().cpu().numpy()
    codes = qeps.codes(x[kept], eps).reshape(kept.size, -1)
    ref = blockcodec.encode(codes)
    s.block_encode()
    w, ro, d = s.block_export()
    assert np.array_equal(w.cpu().numpy(), ref["widths"])
    assert np.array_equal(ro.cpu().numpy().astype(np.uint64), ref["row_off"])
    assert np.array_equal(d.cpu().numpy().view(np.uint32), ref["data"])
    want = s.dequantize()
    assert torch.equal(s.block_decode(), want)
    # an output that is only word aligned
    buf = torch.empty(kept.size * dim + 1, device="cuda")
    assert torch.equal(s.block_decode(out=buf[1:].view(kept.size, dim)), want)
    if bits <= 22:   # the widest codes that scoring takes
        q = _dev(synth.unit_rows(rng, 3, dim).astype(np.float32))
        assert all(torch.equal(u, v) for u, v in zip(s.score_topk(q, 5), s.score_topk_blocks(q, 5)))


def test_encoding_memory_and_regrowth(lam):
    """The device holds the encoding in about its own size, not the codes' (one
    wide block in 32 per row here), and a store encoded again at a finer, then a
    coarser step gives the oracle's encoding each time (a buffer that has to
    grow, and one that is larger than needed)."""
    rng = np.random.default_rng(91)
    n, dim = 20000, 1024
    x = np.zeros((n, dim), np.float32)
    x[:, 64:96] = rng.uniform(-1, 1, (n, 32)).astype(np.float32)
    x[0, 64] = 1.0
    s, p = _store(lam, x, 1.0, 2.0 ** -12)
    s.info()
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    st = s.block_encode()
    torch.cuda.synchronize()
    used = before - torch.cuda.mem_get_info()[0]
    assert st["data_bytes"] * 16 < p.code_bytes
    assert used <= st["total_bytes"] + 4 * n + (8 << 20), (used, st["total_bytes"], p.code_bytes)
    for eps in (2.0 ** -15, 2.0 ** -9, 2.0 ** -17):
        s.quantize(eps)
        s.block_encode()
        ref = blockcodec.encode(qeps.codes(x[:300], eps).reshape(300, dim))
        w, ro, d = s.block_export()
        assert np.array_equal(w.cpu().numpy().reshape(n, -1)[:300], ref["widths"].reshape(300, -1))
        assert np.array_equal(ro.cpu().numpy().astype(np.uint64)[:301], ref["row_off"])
        words = int(ref["row_off"][-1])
        assert np.array_equal(d.cpu().numpy().view(np.uint32)[:words], ref["data"][:words])
        assert torch.equal(s.block_decode(), s.dequantize())


def test_empty_store(lam):
    """The encoding of an empty store has one row offset, 0, in memory that held
    other rows before."""
    n, dim = 4096, 64
    a = lam.Store(dim, 1.0, n)
    a.ingest(_dev(np.random.default_rng(5).uniform(-1, 1, (n, dim)).astype(np.float32)))
    a.info()
    del a
    stores = [lam.Store(dim, 1.0, c) for c in (n * dim // 2 - 1, n * dim // 4 - 1, n * dim // 8 - 1)]
    for s in stores:
        s.quantize(1e-3)
        assert s.block_encode()["rows"] == 0
        w, ro, d = s.block_export()
        assert w.numel() == 0 and d.numel() == 0 and ro.cpu().tolist() == [0]
