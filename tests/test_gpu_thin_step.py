"""Steps of a few tokens whose append and scoring share a launch and whose attention selects the units
(GPU): scores against infllm_score_units, the lookup against the oracle's selection from those scores (at
the row lengths and unit counts where the select changes, and with massive ties), the appended rows and
rings against infllm_append, the attention against infllm_chunk_attend on the same lookup."""
import numpy as np
import pytest
import torch

from oracle import infllm_oracle as O
from paper_2402_04617_amd import infllm as F
from tests.gpu_util import Layer, host, log, oparams

pytestmark = pytest.mark.gpu

LI, LL, LBS = 3, 40, 4
#        dtype, G, Hkv, D, n_q, units, k, mode, batch
CASES = [
    ("bf16", 4, 2, 128, 1, 233, 16, "tokens", 2),
    ("bf16", 1, 3, 64, 1, 1023, 48, "tokens", 1),    # most units of the candidate ranking
    ("bf16", 2, 1, 128, 1, 1024, 49, "mean", 1),     # longest row one wave selects from; one unit more
    ("bf16", 8, 1, 64, 1, 1025, 32, "tokens", 1),    # a row longer: separate selection
    ("bf16", 4, 1, 128, 1, 700, 300, "remap", 2),
    ("bf16", 4, 2, 64, 1, 64, 63, "remap", 1),
    ("bf16", 4, 2, 64, 1, 65, 65, "tokens", 1),      # every unit
    ("bf16", 4, 2, 128, 8, 130, 7, "remap", 1),      # longest thin chunk, matrix-core attention
    ("bf16", 3, 2, 64, 3, 500, 33, "mean", 2),
    ("f32", 2, 2, 64, 5, 300, 20, "tokens", 2),
    ("f32", 3, 1, 128, 1, 129, 12, "remap", 1),
]


def _layer(case, ties):
    dtype, G, Hkv, D, n_q, units, k, mode, B = case
    past = LI + LL + units * LBS + 1
    p = F.params(G * Hkv, Hkv, D, LI, LL, LBS, 2, k, dtype, sm_scale=D ** -0.5,
                 rope_inv_freq=F.rope_frequencies(D) if mode == "remap" else None,
                 repr_mode="mean" if mode == "mean" else "tokens")
    assert O.partition(past, oparams(p)).n_units == units
    L = Layer(p, B, past + n_q, chunk=max(n_q, 8))
    g = torch.Generator(device="cuda").manual_seed(units * 31 + k)
    for t in (L.mem.k, L.mem.v, L.mem.k_rot, L.mem.unit_ksum, L.mem.qprefix):
        if t is not None:
            t.copy_(torch.randn(t.shape, generator=g, device="cuda"))
    if ties:
        L.mem.unit_ksum.zero_()  # every score 0 but a few: the k-th place falls among the ties
        L.mem.unit_ksum[:, :, 0, 5:9] = 1.0
    q = torch.randn((B, G * Hkv, n_q, D), generator=g, device="cuda").to(L.dt)
    kv = [torch.randn((B, Hkv, n_q, D), generator=g, device="cuda").to(L.dt) for _ in range(2)]
    return p, L, past, q, kv


@pytest.mark.parametrize("ties", [False, True], ids=["random", "ties"])
@pytest.mark.parametrize("case", CASES, ids=[str(c) for c in CASES])
def test_thin_step(case, ties):
    dtype, G, Hkv, D, n_q, units, k, mode, B = case
    p, L, past, q, (kk, vv) = _layer(case, ties)
    _, L2, _, _, _ = _layer(case, ties)
    log(f"[thin] {case} ties={ties}")
    out = torch.zeros_like(q)
    lse = torch.zeros((B, G * Hkv, n_q), device="cuda")
    scores = torch.zeros((B, Hkv, units), device="cuda")
    idx = torch.full((B, Hkv, k), 7, dtype=torch.int32, device="cuda")
    F.infllm_step(p, L.mem.struct, q, n_q * D, kk, vv, n_q * D, n_q, past, units, scores, idx, out, n_q * D, lse, L.ws)
    # the general entry points, one after the other, on a copy of the memory
    F.infllm_append(p, L2.mem.struct, q, n_q * D, kk, vv, n_q * D, n_q, past)
    want = torch.zeros_like(scores)
    F.infllm_score_units(p, L2.mem.struct, q, n_q * D, n_q, units, want, L2.ws)
    torch.cuda.synchronize()
    scale = float(want.abs().max())
    # float32 sums of D products in another order: a few ulp of the largest partial sum
    assert float((scores - want).abs().max()) <= 2e-6 * max(scale, 1e-3) * D ** 0.5
    for a, b in zip((L.mem.k, L.mem.v, L.mem.k_rot, L.mem.qprefix, L.mem.rpart),
                    (L2.mem.k, L2.mem.v, L2.mem.k_rot, L2.mem.qprefix, L2.mem.rpart)):
        assert a is None or torch.equal(a, b)
    sc, got = host(scores).astype(np.float64), host(idx)
    for b in range(B):
        for g in range(Hkv):
            assert np.array_equal(got[b, g], O.select_units(sc[b, g], oparams(p))), (b, g)
    out2, lse2 = torch.zeros_like(out), torch.zeros_like(lse)
    F.infllm_chunk_attend(p, L2.mem.struct, q, n_q * D, n_q, past, idx, k, out2, n_q * D, lse2, L2.ws)
    torch.cuda.synchronize()
    if dtype == "f32" or (n_q == 1 and G in (1, 2, 4, 8)):
        # the same kernel, lookup and parts
        assert torch.equal(out, out2) and torch.equal(lse, lse2)
    else:
        # the matrix-core kernel splits the keys elsewhere when it selects: bf16 probabilities against another
        # maximum (2^-9 each), fp16 partials, a bf16 result
        assert float((out.float() - out2.float()).abs().max()) <= 1e-2 * float(out2.float().abs().max())
        assert float((lse - lse2).abs().max()) <= 1e-3


@pytest.mark.parametrize("n_q", [1, 4])
def test_thin_step_varlen(n_q):
    """Sequences with no units, some and many: each as its own step."""
    G, Hkv, D, k = 4, 2, 64, 9
    units = [0, 3, 9, 400]
    pasts = [20] + [LI + LL + u * LBS + 2 for u in units[1:]]
    p = F.params(G * Hkv, Hkv, D, LI, LL, LBS, 2, k, "bf16", sm_scale=D ** -0.5)
    gen = torch.Generator(device="cuda").manual_seed(5)
    L = Layer(p, 4, max(pasts) + n_q, chunk=8)
    for t in (L.mem.k, L.mem.v, L.mem.unit_ksum, L.mem.qprefix):
        t.copy_(torch.randn(t.shape, generator=gen, device="cuda"))
    q = torch.randn((4, G * Hkv, n_q, D), generator=gen, device="cuda").to(L.dt)
    kk, vv = (torch.randn((4, Hkv, n_q, D), generator=gen, device="cuda").to(L.dt) for _ in range(2))
    mu = L.max_units
    log(f"[thin varlen] n_q={n_q}")
    out, lse = torch.zeros_like(q), torch.zeros((4, G * Hkv, n_q), device="cuda")
    scores = torch.zeros((4, Hkv, mu), device="cuda")
    idx = torch.full((4, Hkv, k), 7, dtype=torch.int32, device="cuda")
    F.infllm_step_varlen(p, L.mem.struct, q, n_q * D, kk, vv, n_q * D, n_q, pasts, units, scores, idx, out, n_q * D,
                         lse, L.ws)
    for b in range(4):
        s = L.mem.struct
        one = F.Memory(1, s.capacity, L.mem.k[b].data_ptr(), L.mem.v[b].data_ptr(), s.max_units,
                       L.mem.repr_idx[b].data_ptr(), L.mem.unit_ksum[b].data_ptr(), L.mem.qprefix[b].data_ptr(),
                       L.mem.rpart[b].data_ptr(), s.ring, None)
        o1, l1 = torch.zeros_like(q[:1]), torch.zeros((1, G * Hkv, n_q), device="cuda")
        s1 = torch.zeros((Hkv, max(1, units[b])), device="cuda")
        i1 = torch.zeros((1, Hkv, k), dtype=torch.int32, device="cuda")
        F.infllm_step(p, one, q[b], n_q * D, kk[b], vv[b], n_q * D, n_q, pasts[b], units[b], s1, i1, o1, n_q * D, l1,
                      L.ws)
        torch.cuda.synchronize()
        assert torch.equal(i1[0], idx[b])
        if units[b]:
            assert torch.equal(s1, scores[b, :, :units[b]])
        # another part count than the batch's: partial rows of 11 bits, results of 8 (and as above)
        assert float((o1[0].float() - out[b].float()).abs().max()) <= 1e-2 * float(o1.float().abs().max())
        assert float((l1[0] - lse[b]).abs().max()) <= 1e-3


@pytest.mark.parametrize("B,Hkv,G,D,keys", [(5, 8, 8, 128, 4201), (3, 4, 8, 128, 8400), (9, 8, 4, 64, 1101),
                                            (5, 8, 1, 64, 3001), (1, 8, 4, 128, 6400), (22, 8, 1, 64, 1400)])
def test_decode_parts_fit_the_chip(B, Hkv, G, D, keys):
    """No part count whose last few workgroups begin a round of their own (two to a compute unit, 512 in all)
    while a context is short enough for their rounds to show; the rows of the parts merged are those of one part."""
    p = F.params(G * Hkv, Hkv, D, 4, 16384, 32, 2, 4, "bf16", sm_scale=D ** -0.5)
    gen = torch.Generator(device="cuda").manual_seed(keys)
    L = Layer(p, B, keys, chunk=1)
    for t in (L.mem.k, L.mem.v):
        t.copy_(torch.randn(t.shape, generator=gen, device="cuda"))
    q = torch.randn((B, G * Hkv, 1, D), generator=gen, device="cuda").to(L.dt)
    idx = torch.full((B, Hkv, 4), -1, dtype=torch.int32, device="cuda")
    out, lse = torch.zeros_like(q), torch.zeros((B, G * Hkv, 1), device="cuda")
    one, lse1 = torch.zeros_like(q), torch.zeros_like(lse)
    log(f"[decode parts] B={B} Hkv={Hkv} G={G} D={D} keys={keys}")
    parts = F.infllm_attend_partial(p, L.mem.struct, q, D, 1, keys - 1, idx, 4, out, D, lse, L.ws)
    assert parts > 1 and parts * B * Hkv <= 512
    F.infllm_lse_merge(p, B, 1, parts, L.ws, out, D, lse)
    F.infllm_chunk_attend(p, L.mem.struct, q, D, 1, keys - 1, idx, 4, one, D, lse1, None)
    torch.cuda.synchronize()
    # partial rows are rounded to 11 bits, outputs to 8
    assert float((out.float() - one.float()).abs().max()) <= 2.0 ** -7 * float(one.float().abs().max())
    assert float((lse - lse1).abs().max()) <= 1e-5 * max(1.0, float(lse1.abs().max()))


#        G, D, most keys that one workgroup takes whole
@pytest.mark.parametrize("G,D,whole", [(1, 64, 1000), (2, 64, 750), (1, 128, 500), (4, 128, 250), (8, 128, 150)])
def test_short_context_decode_parts(G, D, whole):
    """Decoding over a short context: one part, which needs no merge, up to where a split pays; the same rows on
    both sides of the line as in one part."""
    Hkv, B = 2, 2
    p = F.params(G * Hkv, Hkv, D, 4, 4096, 32, 2, 4, "bf16", sm_scale=D ** -0.5)
    gen = torch.Generator(device="cuda").manual_seed(whole)
    L = Layer(p, B, whole + 300, chunk=1)
    for t in (L.mem.k, L.mem.v):
        t.copy_(torch.randn(t.shape, generator=gen, device="cuda"))
    q = torch.randn((B, G * Hkv, 1, D), generator=gen, device="cuda").to(L.dt)
    idx = torch.full((B, Hkv, 4), -1, dtype=torch.int32, device="cuda")
    for keys in (1, 337, whole, whole + 1, whole + 257):
        log(f"[short decode] G={G} D={D} keys={keys}")
        out, lse = torch.zeros_like(q), torch.zeros((B, G * Hkv, 1), device="cuda")
        one, lse1 = torch.zeros_like(q), torch.zeros_like(lse)
        parts = F.infllm_attend_partial(p, L.mem.struct, q, D, 1, keys - 1, idx, 4, out, D, lse, L.ws)
        assert keys == whole + 1 or (parts == 1) == (keys <= whole), keys
        if parts > 1:
            F.infllm_lse_merge(p, B, 1, parts, L.ws, out, D, lse)
        F.infllm_chunk_attend(p, L.mem.struct, q, D, 1, keys - 1, idx, 4, one, D, lse1, None)
        torch.cuda.synchronize()
        # partial rows are rounded to 11 bits, outputs to 8
        assert float((out.float() - one.float()).abs().max()) <= 2.0 ** -7 * float(one.float().abs().max())
        assert float((lse - lse1).abs().max()) <= 1e-5 * max(1.0, float(lse1.abs().max()))
