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
