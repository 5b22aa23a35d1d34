"""The unit lookup by every route it takes (GPU): the selection entry point, the decode kernel's prologue and the
matrix-core attention's (short and long rows), at the row lengths and unit counts where the select changes, for
scores that crowd: equal, equal but for their low bits, large in a few lanes only, not numbers.  Expected values:
the oracle's selection, exactly."""
import numpy as np
import pytest
import torch

from oracle import infllm_oracle as O
from paper_2402_04617_amd import infllm as F
from tests.gpu_util import Layer, host, log, oparams

pytestmark = pytest.mark.gpu

PATTERNS = ["random", "close", "few values", "equal", "few lanes", "few lanes long", "nan", "ascending"]


def _pattern(name, n, rng):
    if name == "random":
        return rng.standard_normal(n)
    if name == "close":       # the upper sixteen bits agree
        return 100.0 + rng.permutation(n) * 2.0 ** -14
    if name == "few values":
        return rng.integers(0, 3, n).astype(np.float64)
    if name == "equal":
        return np.full(n, -2.5)
    if name == "few lanes":   # sixteen of the 64 residues hold all large scores
        return rng.standard_normal(n) + np.where(np.arange(n) % 64 < 16, 50.0, 0.0)
    if name == "few lanes long":  # the same within every wave's 1,024 elements, and crowded
        return np.where(np.arange(n) % 64 < 40, 100.0 + rng.permutation(n) * 2.0 ** -14, -1.0)
    if name == "nan":
        return np.where(rng.random(n) < 0.5, np.nan, rng.standard_normal(n))
    return np.arange(n) * 0.125


def _expected(s, k):
    op = O.Params(1, 1, 64, 0, 1, 1, 1, k)
    return O.select_units(np.where(np.isnan(s), -1e30, s).astype(np.float32).astype(np.float64), op)


@pytest.mark.parametrize("n", [49, 65, 130, 512, 513, 987, 1024, 1025, 2000, 4096, 5100, 8155])
def test_select_topk_routes(n):
    rng = np.random.default_rng(n)
    s = np.stack([_pattern(name, n, rng) for name in PATTERNS]).astype(np.float32)
    sd = torch.from_numpy(s).cuda()
    for k in (1, 32, 36, 37, 47, 48, 49, 64, 128):
        if k >= n:
            continue
        log(f"[topk] n={n} k={k}")
        idx = torch.full((len(PATTERNS), k), 7, dtype=torch.int32, device="cuda")
        F.infllm_select_topk(len(PATTERNS), sd, n, k, idx)
        got = host(idx)
        for r, name in enumerate(PATTERNS):
            assert np.array_equal(got[r], _expected(s[r], k)), (name, k)


@pytest.mark.parametrize("n_q,D", [(1, 64), (4, 128)], ids=["decode", "chunk"])
@pytest.mark.parametrize("units,k", [(49, 48), (130, 48), (300, 49), (987, 47), (987, 64), (1024, 48), (1024, 49),
                                     (300, 300), (1025, 48), (2000, 48), (5500, 48), (8155, 37), (8155, 48)])
def test_step_lookup_routes(n_q, D, units, k):
    G, LI, LL, LBS = 4, 3, 40, 4
    Hkv = len(PATTERNS)
    past = LI + LL + units * LBS + 1
    p = F.params(G * Hkv, Hkv, D, LI, LL, LBS, 2, k, "bf16", sm_scale=D ** -0.5)
    assert O.partition(past, oparams(p)).n_units == units
    rng = np.random.default_rng(units + k)
    s = np.stack([_pattern(name, units, rng) for name in PATTERNS]).astype(np.float32)
    L = Layer(p, 1, past + n_q, chunk=8)
    # one dimension carries the scores: a query sum of 4 or 16 there, exact products
    L.mem.unit_ksum[0, :, 0, :units, 0] = torch.from_numpy(s).cuda()
    q = torch.zeros((1, G * Hkv, n_q, D), dtype=torch.bfloat16, device="cuda")
    q[..., 0] = 1.0
    kv = torch.zeros((1, Hkv, n_q, D), dtype=torch.bfloat16, device="cuda")
    out, lse = torch.zeros_like(q), torch.zeros((1, G * Hkv, n_q), device="cuda")
    scores = torch.zeros((1, Hkv, units), device="cuda")
    idx = torch.full((1, Hkv, k), 7, dtype=torch.int32, device="cuda")
    log(f"[step lookup] n_q={n_q} units={units} k={k}")
    F.infllm_step(p, L.mem.struct, q, n_q * D, kv, kv, n_q * D, n_q, past, units, scores, idx, out, n_q * D, lse, L.ws)
    torch.cuda.synchronize()
    assert np.array_equal(host(scores)[0], s * np.float32(G * n_q), equal_nan=True)
    got = host(idx)[0]
    for g, name in enumerate(PATTERNS):
        assert np.array_equal(got[g], _expected(s[g], k)), name
