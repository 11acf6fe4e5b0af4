"""Selection over long rows of keys, where one pass over K gives the row sums
and a bound on every chunk's score, and only the chunks that the bound leaves
are scored exactly: against the oracle's chunk scores, on scores that the
bound settles and on scores that it cannot settle (the head is then scored in
full)."""
import math

import numpy as np
import pytest
import torch

import oracle as O
import paper_2608_30295_amd as ck
from gpu_util import DEV, check_topk

pytestmark = pytest.mark.gpu

# heads * padded rows * keys must reach 2^27 and the budget stay below a 48th of the chunks for the one-pass route
CASES = [
    # kind, hq, hkv, l_obs, keys, cs, chunks kept
    ("heavy", 8, 8, 64, 262144, 8, 256),            # 64 rows per head: two row tiles
    ("heavy", 4, 4, 16, 524288 + 5, 8, 1),          # 16 rows padded to 64, one chunk kept, ragged last chunk
    ("heavy", 8, 4, 37, 262144 + 37, 12, 440),      # 74 rows padded to 128; a chunk size that does not divide 64
    ("heavy", 16, 4, 64, 131072 + 29, 64, 32),      # 256 rows; chunks of a whole tile
    ("heavy", 16, 2, 64, 131072 + 64, 4, 680),      # 512 rows; 1764 candidates
    ("heavy", 8, 8, 64, 299008 + 1, 32, 190),       # chunk of one key at the end
    ("flat", 8, 8, 64, 262144, 8, 64),              # near-equal scores: nothing is settled
    ("one tied", 8, 8, 64, 262144, 8, 64),          # equal keys in one head: lower indices win there
    ("spikes", 8, 8, 64, 262144, 8, 64),            # terms 600 nats above the sampled ones: sums overflow
]


@pytest.mark.parametrize("kind,hq,hkv,l_obs,keys,cs,b", CASES)
def test_one_pass_selection(kind, hq, hkv, l_obs, keys, cs, b):
    n, G, d = keys + l_obs, hq // hkv, 128
    g = torch.Generator(device=DEV).manual_seed(keys + b)
    q = torch.randn((hq, l_obs, d), generator=g, device=DEV).bfloat16()
    k = torch.empty((hkv, n, d), dtype=torch.bfloat16, device=DEV)
    for h in range(hkv):
        x = torch.randn((n, d), generator=g, device=DEV)
        if kind == "flat":
            x *= 1e-3
        else:
            x[torch.rand(n, generator=g, device=DEV) < 0.01] *= 3
        k[h] = x
    if kind == "one tied":
        k[1] = k[1, :1]
    if kind == "spikes":
        u = q[G:2 * G].float().reshape(-1, d).mean(dim=0)
        k[1, [9001, 200003]] = (600.0 * math.sqrt(d) * u / u.norm() ** 2).bfloat16()
    heads = list(range(hkv))[::-1]
    print(f"one pass {kind} hq={hq} hkv={hkv} l_obs={l_obs} keys={keys} cs={cs} b={b}", flush=True)
    idx = ck.select_critical(q, k, heads, cs, b).cpu().numpy()
    again = ck.select_critical(q, k, heads, cs, b).cpu().numpy()
    assert np.array_equal(idx, again)
    qf = q.float().cpu().numpy().astype(np.float64)
    for h in (0, 1):
        kf = k[h:h + 1].float().cpu().numpy().astype(np.float64)
        sc = O.chunk_scores(qf[h * G:(h + 1) * G], kf, 0, G, l_obs, cs, 1 / math.sqrt(d))
        if kind == "one tied" and h == 1:
            sc = np.full_like(sc, sc[0])
            assert np.array_equal(idx[heads.index(h)], np.arange(b))
        check_topk(idx[heads.index(h)], sc, b)


# Scores at the ends of fp32's exponent range.  Keys lie on a few axes: with
# queries 32 e_a + 0.25 e_b a key x e_a + y e_b scores 32 x + 0.25 y exactly,
# x and y on bf16's grid.
C = math.log2(math.e) / math.sqrt(128)      # log2 units per unit of q . k
SAMPLES = 32                                 # 32-key tiles that the row sums are estimated from


def _axes(log2, sx):
    """x, y with 32 x + 0.25 y as close to log2 / C as y's grid allows; x of log2's sign, on a grid of sx."""
    s = log2 / C
    x = math.trunc(s / 32 / sx) * sx
    y = torch.tensor((s - 32 * x) / 0.25).bfloat16().item()
    return x, y


def _random_heads(hkv, rows, n, head):
    g = torch.Generator(device=DEV).manual_seed(n + head)
    q = torch.randn((hkv, rows, 128), generator=g, device=DEV).bfloat16()
    k = torch.empty((hkv, n, 128), dtype=torch.bfloat16, device=DEV)
    for h in range(hkv):
        x = torch.randn((n, 128), generator=g, device=DEV)
        x[torch.rand(n, generator=g, device=DEV) < 0.01] *= 3
        k[h] = x
    q[head], k[head] = 0, 0
    return q, k


def _select_head(q, k, head, cs, b):
    hkv = k.shape[0]
    idx = ck.select_critical(q, k, list(range(hkv)), cs, b).cpu().numpy()
    qf, kf = (t[head:head + 1].float().cpu().numpy().astype(np.float64) for t in (q, k))
    sc = O.chunk_scores(qf, kf, 0, 1, q.shape[1], cs, 1 / math.sqrt(128))
    return idx[head], sc


def test_estimates_far_below_the_sums():
    """Every row's sum lies 2^126 to 2^128 above its estimate, the spikes all
    outside the sampled tiles: the rows' estimate-to-sum ratios are below
    fp32's normal numbers, and the bound on the other chunks with them.  The
    best chunk is one of row 0's; 70 chunks of row 1, whose ratio is three
    times smaller, rank above it by their weighted mass."""
    n_keys, head = 262144, 3
    q, k = _random_heads(8, 2, n_keys + 2, head)
    q[head, 0, 0], q[head, 0, 1], q[head, 1, 2], q[head, 1, 3] = 32, 0.25, 32, 0.25
    base = math.log2(n_keys)                 # every other key scores 0
    first = torch.arange(SAMPLES) * (n_keys - 32) // (SAMPLES - 1)
    free = [c for c in range(100, n_keys // 8 - 8, 211) if ((first + 32 <= 8 * c) | (first >= 8 * c + 8)).all()]
    best, a, b = free[75], free[:69], free[76:146]

    def put(chunks, dim, log2):
        x, y = _axes(log2, 0.25)
        for c in chunks:
            k[head, 8 * c + 5, dim], k[head, 8 * c + 5, dim + 1] = x, y
    put([best], 0, base + 126.4 + math.log2(0.0165))
    put(a, 0, base + 126.4 + math.log2((1 - 0.0165) / 69))
    put(b, 2, base + 127.8 - math.log2(70))
    idx, sc = _select_head(q, k, head, 8, 1)
    assert np.argmax(sc) == best
    check_topk(idx, sc, 1)


def test_estimates_far_above_the_sums():
    """Six keys carry the row's whole sum, one in each of six sampled groups:
    the estimate is 341 times the sum, and against it every other key's
    weight is below fp32's normal numbers, though its share of the exact mass
    is not."""
    n_keys, head = 262144, 3
    q, k = _random_heads(8, 1, n_keys + 1, head)
    q[head, 0, 0], q[head, 0, 1] = 32, 0.25
    low, mid = _axes(-118.0, 0.25), _axes(-116.5, 0.25)
    k[head, :n_keys, 0], k[head, :n_keys, 1] = low
    upper = [20000 + 7 * i for i in range(200)]          # chunks with one key of 2^1.5 times the mass of the others
    for c in upper:
        k[head, 8 * c + 2, 0], k[head, 8 * c + 2, 1] = mid
    for t in range(6):
        k[head, (n_keys - 32) * t // (SAMPLES - 1) + 5, :2] = 0
    idx, sc = _select_head(q, k, head, 8, 64)
    check_topk(idx, sc, 64)


def test_sampled_keys_all_masked():
    """Keys hidden by a component of -inf: all the sampled ones, so there is
    nothing to estimate the rows' sums from; the visible ones score -200 in
    log2 units."""
    n_keys, head = 262144, 3
    q, k = _random_heads(8, 16, n_keys + 16, head)
    g = torch.Generator(device=DEV).manual_seed(9)
    q[head] = torch.randn((16, 128), generator=g, device=DEV).bfloat16()
    q[head, :, 0], q[head, :, 1] = 1, 16
    k[head, :, 0] = -math.inf
    lo = 135400                                          # 4096 visible keys between two sampled tiles
    k[head, lo:lo + 4096] = torch.randn((4096, 128), generator=g, device=DEV).bfloat16()
    k[head, lo:lo + 4096, 0], k[head, lo:lo + 4096, 1] = 0, -98
    first = torch.arange(SAMPLES) * (n_keys - 32) // (SAMPLES - 1)
    assert ((first + 32 <= lo) | (first >= lo + 4096)).all()
    idx = ck.select_critical(q, k, list(range(8)), 8, 64).cpu().numpy()[head]
    vis = k[head:head + 1, lo:lo + 4096].float().cpu().numpy().astype(np.float64)
    qf = q[head:head + 1].float().cpu().numpy().astype(np.float64)
    sc = np.zeros(n_keys // 8)
    pad = np.concatenate([vis, np.zeros((1, 16, 128))], axis=1)
    sc[lo // 8:(lo + 4096) // 8] = O.chunk_scores(qf, pad, 0, 1, 16, 8, 1 / math.sqrt(128))
    check_topk(idx, sc, 64)
