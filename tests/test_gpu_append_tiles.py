"""Appends of several scan tiles (512 positions each) at once (GPU): the running query sums and the partial
representative scores against float64 sums on the host, where tiles are full, ragged, of one position, the
chunk is short, and where the tokens that leave the window precede the chunk or lie inside it."""
import numpy as np
import pytest
import torch

from paper_2402_04617_amd import infllm as F
from tests.gpu_util import Layer, dev, host, log
from tests.test_gpu_kernels import rand_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,G,D,lL,chunks", [
    ("bf16", 4, 128, 1100, (700, 1536, 512)),  # tiles of all kinds: before the chunk, inside it
    ("bf16", 3, 64, 2000, (1300, 1025)),       # run-time group size, a last tile of one position
    ("f32", 2, 64, 40, (1100, 9, 600)),        # a window shorter than a tile
    ("bf16", 8, 128, 513, (513, 1024, 1)),
    # short chunks: one thread per dim, 8 or 16 positions at a time; the window inside the chunk
    ("bf16", 4, 128, 60, (100, 9, 16, 17, 32, 33, 8, 24)),
    ("bf16", 3, 64, 12, (32, 31, 25)),
    ("f32", 1, 128, 200, (230, 32, 1, 20)),
])
def test_append_tiles(dtype, G, D, lL, chunks):
    rng = np.random.default_rng(lL)
    Hkv, B, lI, S = 2, 1, 5, sum(chunks)
    ring = lL + max(chunks) + 7
    p = F.params(G * Hkv, Hkv, D, lI, lL, 64, 2, 2, dtype)
    q, k, v = rand_inputs(rng, G * Hkv, Hkv, S, D, dtype, B=B)
    L = Layer(p, B, S, chunk=max(chunks), ring=ring)
    qd, kd, vd = dev(q, dtype), dev(k, dtype), dev(v, dtype)
    pref = np.cumsum(q.astype(np.float64).reshape(B, Hkv, G, S, D).sum(axis=2), axis=2)
    past = 0
    for n in chunks:
        log(f"[append tiles] {dtype} G={G} D={D} l_L={lL} past={past} n={n}")
        off = past * D * L.esize
        F.infllm_append(p, L.mem.struct, qd.data_ptr() + off, S * D, kd.data_ptr() + off, vd.data_ptr() + off, S * D,
                        n, past)
        torch.cuda.synchronize()
        got, part = host(L.mem.qprefix), host(L.mem.rpart)
        for t in range(past, past + n):
            assert np.allclose(got[:, :, t % ring], pref[:, :, t], rtol=1e-12, atol=1e-12), t
        for pos in range(max(past, lI + lL), past + n):
            t = pos - lL
            w = k[:, :, t].astype(np.float64) * (pref[:, :, pos] - pref[:, :, t])
            exp = w.reshape(B, Hkv, D // 8, 8).sum(-1)
            assert np.allclose(part[:, :, :, t % ring], exp, rtol=1e-10, atol=1e-10), t
        past += n


@pytest.mark.parametrize("dtype,G,D,lL,chunks", [
    ("bf16", 4, 128, 4096, (32, 32, 9)),        # a slice per wave
    ("bf16", 3, 64, 700, (100, 513, 8)),        # whole blocks, a second tile
    ("f32", 2, 128, 300, (100, 60, 3, 130)),    # a window shorter than a tile
])
def test_append_ring_shorter_than_window(dtype, G, D, lL, chunks):
    """Short chunks at the start of a stream need no ring slot of a token that leaves the window: a ring that
    holds one chunk is accepted, and only the running sums are written."""
    rng = np.random.default_rng(lL + 1)
    Hkv, lI, S, ring = 2, 5, sum(chunks), max(chunks) + 1
    assert ring <= lL and S <= lI + lL
    p = F.params(G * Hkv, Hkv, D, lI, lL, 64, 2, 2, dtype)
    q, k, v = rand_inputs(rng, G * Hkv, Hkv, S, D, dtype)
    L = Layer(p, 1, S, chunk=max(chunks), ring=ring)
    L.mem.rpart.fill_(3.0)
    qd, kd, vd = dev(q, dtype), dev(k, dtype), dev(v, dtype)
    pref = np.cumsum(q.astype(np.float64).reshape(1, Hkv, G, S, D).sum(axis=2), axis=2)
    past = 0
    for n in chunks:
        log(f"[append short ring] {dtype} G={G} D={D} l_L={lL} ring={ring} past={past} n={n}")
        off = past * D * L.esize
        F.infllm_append(p, L.mem.struct, qd.data_ptr() + off, S * D, kd.data_ptr() + off, vd.data_ptr() + off, S * D,
                        n, past)
        torch.cuda.synchronize()
        got = host(L.mem.qprefix)
        for t in range(past, past + n):
            assert np.allclose(got[:, :, t % ring], pref[:, :, t], rtol=1e-12, atol=1e-12), t
        past += n
    assert (L.mem.rpart == 3.0).all()
    assert np.array_equal(host(L.mem.k)[:, :, :S], k) and np.array_equal(host(L.mem.v)[:, :, :S], v)


@pytest.mark.parametrize("dtype,lI,lL,chunks", [
    ("bf16", 5, 300, (100, 90, 110)),   # the first chunk lies within the window
    ("f32", 200, 8, (20, 90, 60)),      # ... within the initial tokens
    ("bf16", 0, 513, (513, 12)),
])
def test_append_of_stored_keys(dtype, lI, lL, chunks):
    """k and v absent: the caller has stored them, and no token of a chunk leaves the window inside it."""
    rng = np.random.default_rng(lL + 2)
    Hkv, G, D, S = 2, 4, 64, sum(chunks)
    ring = lL + max(chunks) + 1
    p = F.params(G * Hkv, Hkv, D, lI, lL, 64, 2, 2, dtype)
    q, k, v = rand_inputs(rng, G * Hkv, Hkv, S, D, dtype)
    L = Layer(p, 1, S, chunk=max(chunks), ring=ring)
    qd = dev(q, dtype)
    L.mem.k.copy_(dev(k, dtype))
    L.mem.v.copy_(dev(v, dtype))
    pref = np.cumsum(q.astype(np.float64).reshape(1, Hkv, G, S, D).sum(axis=2), axis=2)
    past = 0
    for n in chunks:
        log(f"[append stored] {dtype} l_I={lI} l_L={lL} past={past} n={n}")
        F.infllm_append(p, L.mem.struct, qd.data_ptr() + past * D * L.esize, S * D, None, None, 0, n, past)
        torch.cuda.synchronize()
        got, part = host(L.mem.qprefix), host(L.mem.rpart)
        for t in range(past, past + n):
            assert np.allclose(got[:, :, t % ring], pref[:, :, t], rtol=1e-12, atol=1e-12), t
        for pos in range(max(past, lI + lL), past + n):
            t = pos - lL
            w = k[:, :, t].astype(np.float64) * (pref[:, :, pos] - pref[:, :, t])
            assert np.allclose(part[:, :, :, t % ring], w.reshape(1, Hkv, D // 8, 8).sum(-1), rtol=1e-10, atol=1e-10), t
        past += n
