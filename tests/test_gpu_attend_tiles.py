"""The matrix-core attention where its tile loop can go wrong (GPU): key groups of one key (l_I or l_bs
not a multiple of 8) over more tiles than the position table holds, odd and even tile counts down to one,
row tiles whose last waves have no rows, and lookup entries to skip in each.  Expected values: the oracle,
at the bars of the other attention cases."""
import pytest
import torch

from paper_2402_04617_amd import infllm as F
from tests.gpu_util import Layer, log
from tests.test_gpu_kernels import _attend_case

pytestmark = pytest.mark.gpu

#         dtype, G, Hkv, D, lI, lL, lbs, k_m, past, n_q, B
CASES = [
    # single-key groups, 84 and more tiles in one part: the position table moves along
    ("bf16", 3, 1, 128, 5, 300, 20, 250, 7000, 11, 1),    # 33 rows: one whole wave and one row
    ("bf16", 4, 1, 64, 8, 300, 36, 160, 9000, 65, 1),     # 260 rows: a row tile of four rows
    # 8-key groups, l_I and l_bs multiples of 8 but not of a tile
    ("bf16", 2, 2, 128, 24, 500, 40, 30, 6000, 47, 1),
    # one, two and three tiles in all
    ("bf16", 4, 2, 128, 0, 16, 16, 2, 9, 40, 1),
    ("bf16", 1, 2, 64, 4, 64, 16, 2, 70, 40, 2),
    ("bf16", 4, 2, 128, 16, 64, 16, 4, 110, 77, 1),
]


@pytest.mark.parametrize("case", CASES, ids=[str(c) for c in CASES])
@pytest.mark.parametrize("mode", ["parts", "one-part", "skipped-entry", "skipped-entry-one-part"])
def test_chunk_attend_tiles(case, mode):
    _attend_case(case, workspace="one-part" not in mode, invalid_entry=mode.startswith("skipped"))


# The float32 kernel at the edges of its tiles (32 keys, 32 rows a wave, 1, 2 or 4 waves): one row to several
# row tiles, part and tile remainders, a lookup longer than the entries it keeps in LDS.
F32_CASES = [
    ("f32", 1, 2, 128, 5, 40, 12, 6, 300, 1, 1),       # one row
    ("f32", 3, 1, 64, 16, 100, 20, 5, 700, 11, 2),     # 33 rows: two waves
    ("f32", 1, 1, 128, 8, 64, 32, 9, 900, 65, 1),      # 65 rows: four waves
    ("f32", 4, 2, 64, 0, 33, 7, 40, 500, 33, 1),       # 132 rows: a second row tile of four rows
    ("f32", 2, 1, 128, 16, 64, 16, 4, 20, 31, 1),      # no units yet
    ("f32", 1, 1, 64, 4, 40, 2, 2100, 5000, 9, 1),     # 2,100 entries
]


@pytest.mark.parametrize("case", F32_CASES, ids=[str(c) for c in F32_CASES])
@pytest.mark.parametrize("mode", ["parts", "one-part", "skipped-entry"])
def test_chunk_attend_f32_tiles(case, mode):
    _attend_case(case, workspace=mode != "one-part", invalid_entry=mode == "skipped-entry")


@pytest.mark.parametrize("D,G,n_q,remap", [(64, 4, 45, False), (128, 1, 70, False), (64, 2, 19, True)])
def test_f32_hidden_values_stay_hidden(D, G, n_q, remap):
    """Values that are not finite reach the rows that see their key and no others: a token inside the chunk,
    and position 0, which stands in for the keys of a skipped lookup entry."""
    lL, lbs, past, hot = 40, 20, 300, 7
    p = F.params(G, 1, D, 0, lL, lbs, 2, 4, "f32", rope_inv_freq=F.rope_frequencies(D) if remap else None)
    S = past + n_q
    L = Layer(p, 1, S, chunk=n_q, ring=n_q + lL + 1)
    g = torch.Generator(device="cuda").manual_seed(D + n_q)
    for t in (L.mem.k, L.mem.v, L.mem.k_rot):
        if t is not None:
            t.copy_(torch.randn(t.shape, generator=g, device="cuda"))
    q = torch.randn((1, G, n_q, D), generator=g, device="cuda")
    idx = torch.tensor([[[3, 5, 8, 10 ** 6]]], dtype=torch.int32, device="cuda")  # unit 0 is not looked up

    def attend():
        out, lse = torch.zeros_like(q), torch.zeros((1, G, n_q), device="cuda")
        log(f"[attend] hidden values D={D} G={G} n_q={n_q} remap={remap}")
        F.infllm_chunk_attend(p, L.mem.struct, q, n_q * D, n_q, past, idx, 4, out, n_q * D, lse, L.ws)
        torch.cuda.synchronize()
        return out, lse

    clean, lse = attend()
    L.mem.v[:, :, 0] = float("nan")
    L.mem.v[:, :, past + hot] = float("inf")
    out, lse2 = attend()
    assert torch.equal(lse, lse2)
    # the same products in the same order, but for the sums of the keys taken apart
    assert (out[:, :, :hot] - clean[:, :, :hot]).abs().max().item() <= 1e-5
    assert not torch.isfinite(out[:, :, hot:]).any()


@pytest.mark.parametrize("D,Hkv,n_q", [(128, 8, 512), (64, 8, 512), (128, 2, 512)])
def test_parts_without_tiles(D, Hkv, n_q):
    """The first chunk of a document, split over the keys: parts that lie past the last key of a row tile's
    queries hold no tile.  Their rows are zeros with an lse of -inf, whatever the queries are, and queries that
    are not finite leave the other rows as they were (8 and 4 waves of rows)."""
    G, rows = 4, 4 * Hkv * n_q
    p = F.params(G * Hkv, Hkv, D, 128, 4096, 128, 4, 32, "bf16", sm_scale=D ** -0.5)
    L = Layer(p, 1, n_q, chunk=n_q, ring=n_q + 1)
    g = torch.Generator(device="cuda").manual_seed(n_q + D)
    for t in (L.mem.k, L.mem.v):
        t.copy_(torch.randn(t.shape, generator=g, device="cuda"))
    q = torch.randn((1, G * Hkv, n_q, D), generator=g, device="cuda").to(L.dt)
    idx = torch.full((1, Hkv, 32), -1, dtype=torch.int32, device="cuda")
    # the first rows of every 256-row tile: what a late query load would leave in the staged output rows
    hot = torch.arange(n_q, device="cuda") % 64 < 4

    def partial(qq):
        out, lse = torch.zeros_like(q), torch.zeros((1, G * Hkv, n_q), device="cuda")
        L.ws.fill_(0xA5)
        log(f"[partial] parts without tiles D={D} Hkv={Hkv} n_q={n_q}")
        parts = F.infllm_attend_partial(p, L.mem.struct, qq, n_q * D, n_q, 0, idx, 32, out, n_q * D, lse, L.ws)
        assert parts > 1
        o = L.ws[:parts * rows * D * 2].view(torch.float16).view(parts, G * Hkv, n_q, D).clone()
        part_lse = L.ws[parts * rows * D * 2:][:parts * rows * 4].view(torch.float32).view(parts, G * Hkv, n_q).clone()
        F.infllm_lse_merge(p, 1, n_q, parts, L.ws, out, n_q * D, lse)
        torch.cuda.synchronize()
        return o, part_lse, out, lse

    o, part_lse, out, lse = partial(q)
    empty = part_lse == float("-inf")
    assert empty.any(0)[:, :64].all() and not empty.all(0).any()
    assert (o[empty] == 0).all()
    bad = q.clone()
    bad[:, :, hot] = float("nan")
    o2, part_lse2, out2, lse2 = partial(bad)
    assert (o2[empty & ~hot] == 0).all()
    assert torch.equal(o2[:, :, ~hot], o[:, :, ~hot]) and torch.equal(part_lse2[:, :, ~hot], part_lse[:, :, ~hot])
    assert torch.equal(out2[:, :, ~hot], out[:, :, ~hot]) and torch.equal(lse2[:, :, ~hot], lse[:, :, ~hot])


@pytest.mark.parametrize("Hkv,G,n_q,B,past", [(8, 8, 1500, 1, 0), (8, 4, 3000, 3, 0), (8, 8, 1500, 1, 300)])
def test_long_prompt_is_not_split(Hkv, G, n_q, B, past):
    """A prompt with more row tiles than compute units: the short row tiles follow the long ones, and a split of
    the keys (which starts more workgroups than it shortens) and its merge are not worth it."""
    D = 128
    p = F.params(G * Hkv, Hkv, D, 128, 4096, 128, 4, 32, "bf16", sm_scale=D ** -0.5)
    L = Layer(p, B, past + n_q, chunk=n_q, ring=n_q + 1)
    g = torch.Generator(device="cuda").manual_seed(n_q)
    for t in (L.mem.k, L.mem.v):
        t.copy_(torch.randn(t.shape, generator=g, device="cuda"))
    q = torch.randn((B, G * Hkv, n_q, D), generator=g, device="cuda").to(L.dt)
    idx = torch.full((B, Hkv, 32), -1, dtype=torch.int32, device="cuda")
    out, lse = torch.zeros_like(q), torch.zeros((B, G * Hkv, n_q), device="cuda")
    log(f"[prompt] Hkv={Hkv} G={G} n_q={n_q} B={B} past={past}")
    assert F.infllm_attend_partial(p, L.mem.struct, q, n_q * D, n_q, past, idx, 32, out, n_q * D, lse, L.ws) == 1
    torch.cuda.synchronize()
    b, h = B - 1, G + 1  # one head against float32
    x, k, v = (t.float() for t in (q[b, h], L.mem.k[b, h // G, :past + n_q], L.mem.v[b, h // G, :past + n_q]))
    z = (x @ k.T * D ** -0.5).masked_fill(torch.arange(past + n_q, device="cuda")[None] >
                                          past + torch.arange(n_q, device="cuda")[:, None], float("-inf"))
    assert float((z.softmax(-1) @ v - out[b, h].float()).abs().max()) <= 2e-2
    assert float((z.logsumexp(-1) - lse[b, h]).abs().max()) <= 1e-3
