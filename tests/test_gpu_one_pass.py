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
from gpu_util import DEV, ONE_PASS, TILE, check_topk, select_redone, select_route

pytestmark = pytest.mark.gpu

CASES = [
    # kind, hq, hkv, l_obs, keys, cs, chunks kept: candidates are 4 of them, up to 64 more below 1024
    ("heavy", 8, 8, 64, 262144, 8, 256),            # 64 rows per head: two row tiles
    ("heavy", 4, 4, 16, 524288 + 5, 8, 1),          # 16 rows padded to 64, one chunk kept, ragged last chunk
    ("heavy", 8, 4, 37, 262144 + 37, 12, 440),      # 74 rows padded to 128; a chunk size that does not divide 64
    ("heavy", 16, 4, 64, 131072 + 29, 64, 32),      # 256 rows; chunks of a whole tile
    ("heavy", 16, 2, 64, 131072 + 64, 4, 680),      # 512 rows: two passes
    ("heavy", 8, 8, 64, 299008 + 1, 32, 190),       # chunk of one key at the end
    ("heavy", 16, 4, 32, 262144, 8, 600),           # 2400 candidates, four per lane; 32768 chunks
    ("heavy", 8, 4, 64, 262144, 4, 1200),           # 4800 candidates, eight per lane; four slices of chunks
    ("heavy", 8, 8, 64, 262144 + 3, 1, 64),         # every key a chunk
    ("heavy", 4, 4, 16, 524288 + 7, 2, 600),        # chunks of two keys, 16 slices, candidates capped at 2048
    ("flat", 8, 8, 64, 262144, 8, 64),              # near-equal scores: nothing is settled
    ("gauss", 16, 4, 64, 131072, 8, 256),           # no heavy keys; 256 rows
    ("gauss", 4, 4, 64, 600001, 12, 300),           # and 64
    ("one tied", 8, 8, 64, 262144, 8, 64),          # equal keys in one head: lower indices win there
    ("spikes", 8, 8, 64, 262144, 8, 64),            # terms 600 nats above the sampled ones: sums overflow
    ("sink", 8, 4, 64, 262144, 8, 256),             # the first keys have most of the mass
]


def _sampled(n_keys):
    """The keys that the row sums are estimated from: the first 32, and steps of the golden ratio."""
    u = np.arange(8192, dtype=np.uint64)
    step = np.uint64(32) + ((u * np.uint64(2654435769) & np.uint64(0xFFFFFFFF)) * np.uint64(n_keys - 32) >> np.uint64(32))
    return np.where(u < 32, u, step).astype(np.int64)


def _free_chunks(n_keys, cs):
    """Whole chunks without a sampled key."""
    return np.setdiff1d(np.arange(n_keys // cs), _sampled(n_keys) // cs)


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
        elif kind != "gauss":
            x[torch.rand(n, generator=g, device=DEV) < 0.01] *= 3
        k[h] = x
    if kind == "one tied":
        k[1] = k[1, :1]
    for h in range(hkv if kind == "sink" else 0):
        u = q[h * G:(h + 1) * G].float().reshape(-1, d).mean(dim=0)
        k[h, :4] = (k[h, :4].float() + 45.0 * u / u.norm()).bfloat16()
    if kind == "spikes":
        u = q[G:2 * G].float().reshape(-1, d).mean(dim=0)
        k[1, [9001, 200003]] = (600.0 * math.sqrt(d) * u / u.norm() ** 2).bfloat16()
    heads = list(range(hkv))[::-1]
    one_pass = G * l_obs <= 256
    assert select_route(hq, hkv, l_obs, n, cs, hkv, b) == (ONE_PASS if one_pass else TILE)
    print(f"one pass {kind} hq={hq} hkv={hkv} l_obs={l_obs} keys={keys} cs={cs} b={b}", flush=True)
    ws = ck.workspace(ck.select_workspace(hq, hkv, l_obs, n, cs, hkv), DEV)
    idx = ck.select_critical(q, k, heads, cs, b, ws=ws).cpu().numpy()
    if one_pass:
        full = select_redone(ws, hq, hkv, l_obs, n, cs, hkv, b)[::-1]
        print("scored in full:", np.nonzero(full)[0], flush=True)
        want = {"flat": range(hkv), "one tied": [1], "spikes": [1]}.get(kind, [])
        assert np.array_equal(np.nonzero(full)[0], want)
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
    """Every row's sum lies 2^126 to 2^128 above its estimate, no spike being
    among the sampled keys: the rows' estimate-to-sum ratios are below fp32's
    normal numbers, and the bound on the other chunks with them.  The best
    chunk is one of row 0's; 70 chunks of row 1 (there are 68 candidates),
    whose ratio is three times smaller, rank above it by their weighted mass."""
    n_keys, head = 262144, 3
    assert select_route(8, 8, 2, n_keys + 2, 8, 8, 1) == ONE_PASS
    q, k = _random_heads(8, 2, n_keys + 2, head)
    q[head, 0, 0], q[head, 0, 1], q[head, 1, 2], q[head, 1, 3] = 32, 0.25, 32, 0.25
    base = math.log2(n_keys)                 # every other key scores 0
    free = _free_chunks(n_keys, 8)[100::150]
    best, a, b = free[75], free[:69], free[76:146]
    assert len(a) == 69 and len(b) == 70

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
    """Eight keys carry the row's whole sum, one in each of the eight groups of
    samples: the estimate is 32 times the sum, and against it every other
    key's weight is below fp32's normal numbers, though its share of the
    exact mass is not."""
    n_keys, head = 262144, 3
    assert select_route(8, 8, 1, n_keys + 1, 8, 8, 64) == ONE_PASS
    q, k = _random_heads(8, 1, n_keys + 1, head)
    q[head, 0, 0], q[head, 0, 1] = 32, 0.25
    low, mid = _axes(-121.0, 0.25), _axes(-119.5, 0.25)
    k[head, :n_keys, 0], k[head, :n_keys, 1] = low
    upper = [20000 + 7 * i for i in range(200)]          # chunks with one key of 2^1.5 times the mass of the others
    for c in upper:
        k[head, 8 * c + 2, 0], k[head, 8 * c + 2, 1] = mid
    for key in _sampled(n_keys)[40::1024]:
        k[head, key, :2] = 0
    idx, sc = _select_head(q, k, head, 8, 64)
    check_topk(idx, sc, 64)


def test_sampled_keys_all_masked():
    """Keys hidden by a component of -inf: all the sampled ones, so there is
    nothing to estimate the rows' sums from; the visible ones score -200 in
    log2 units."""
    n_keys, head = 262144, 3
    assert select_route(8, 8, 16, n_keys + 16, 8, 8, 64) == ONE_PASS
    q, k = _random_heads(8, 16, n_keys + 16, head)
    g = torch.Generator(device=DEV).manual_seed(9)
    q[head] = torch.randn((16, 128), generator=g, device=DEV).bfloat16()
    q[head, :, 0], q[head, :, 1] = 1, 16
    k[head, :, 0] = -math.inf
    chunks = _free_chunks(n_keys, 8)[12000:12512]
    keys = torch.from_numpy((chunks[:, None] * 8 + np.arange(8)).reshape(-1)).to(DEV)
    x = torch.randn((4096, 128), generator=g, device=DEV)
    x[:, 0], x[:, 1] = 0, -98
    k[head, keys] = x.bfloat16()
    idx = ck.select_critical(q, k, list(range(8)), 8, 64).cpu().numpy()[head]
    vis = k[head:head + 1, keys].float().cpu().numpy().astype(np.float64)
    qf = q[head:head + 1].float().cpu().numpy().astype(np.float64)
    sc = np.zeros(n_keys // 8)
    pad = np.concatenate([vis, np.zeros((1, 16, 128))], axis=1)
    sc[chunks] = O.chunk_scores(qf, pad, 0, 1, 16, 8, 1 / math.sqrt(128))
    check_topk(idx, sc, 64)
