"""The bf16 score passes on both sides of the lengths where a call goes over
from the tiles of score.h to the waves of score_wave.h and back: which side a
call takes (on the host, for 256 compute units), and selections and CV scores
of either side against the oracle."""
import math
import os

import numpy as np
import pytest
import torch

import oracle as O
import paper_2608_30295_amd as ck
from gpu_util import DEV, TILE, WAVE, check_topk, score_route, select_route

built = pytest.mark.skipif(not os.path.exists(ck.LIB_PATH), reason="libcatekv.so not built")


@built
@pytest.mark.parametrize("l_obs,G,n_sel,last_tile,first_wave", [
    # keys per head: blocks of 640 keys still run on score.h up to 128 rows, of 256 keys at 256 rows
    (16, 1, 1, 256 * 640, 256 * 640 + 1), (64, 1, 3, 85 * 640, 85 * 640 + 1), (64, 2, 8, 32 * 640, 32 * 640 + 1),
    (48, 4, 1, 256 * 256, 256 * 256 + 1), (64, 4, 3, 85 * 256, 85 * 256 + 1),
])
def test_route_by_length(l_obs, G, n_sel, last_tile, first_wave):
    for keys, want in ((64, TILE), (last_tile, TILE), (first_wave, WAVE)):
        b = -(-keys // 8) // 40 + 1                                   # too many chunks kept for one pass
        assert select_route(8 * G, 8, l_obs, keys + l_obs, 8, n_sel, b) == want, keys
        assert score_route(n_sel * G, n_sel, l_obs, keys + 40, 32, 8) == want, keys
        assert select_route(8 * G, 8, l_obs, keys + l_obs, 8, n_sel, b, bf16=False) == TILE


@built
def test_route_of_long_rows_and_of_512():
    two = lambda l_obs, G, n_sel, keys: select_route(8 * G, 8, l_obs, keys + l_obs, 8, n_sel, keys // 320)
    assert two(64, 1, 5, 1 << 18) == WAVE and two(64, 1, 5, (1 << 18) + 64) == TILE     # 64 rows: K beyond the cache
    assert two(64, 2, 5, (1 << 18) + 64) == WAVE
    assert score_route(5, 5, 64, (1 << 18) + 104, 32, 8) == WAVE
    assert two(64, 8, 5, 1 << 18) == TILE and score_route(40, 5, 64, (1 << 18) + 40, 32, 8) == TILE


def _keys(hkv, n, g):
    k = torch.empty((hkv, n, 128), dtype=torch.bfloat16, device=DEV)
    for h in range(hkv):
        x = torch.randn((n, 128), generator=g, device=DEV)
        x[torch.rand(n, generator=g, device=DEV) < 0.01] *= 3
        k[h] = x
    return k


@pytest.mark.gpu
@pytest.mark.parametrize("hq,hkv,l_obs,keys,cs,b,want", [
    (2, 2, 16, 81921, 8, 700, WAVE),          # one key in the last block of 672
    (2, 2, 16, 81920, 8, 700, TILE),
    (2, 2, 64, 90007, 12, 300, WAVE),         # chunks across blocks: column mass in memory
    (4, 2, 37, 100003, 64, 40, WAVE),         # 74 rows padded to 128, a chunk per 64 keys
    (4, 2, 64, 81920, 16, 300, TILE),
    (8, 2, 64, 32769, 8, 300, WAVE),
    (8, 2, 64, 32768, 1, 900, TILE),
    (16, 2, 30, 50001, 32, 60, WAVE),         # 240 rows of 8 query heads
    (2, 2, 64, 700001, 8, 2200, TILE),        # K beyond the last-level cache
])
def test_selection_either_side(hq, hkv, l_obs, keys, cs, b, want):
    n, G = keys + l_obs, hq // hkv
    assert select_route(hq, hkv, l_obs, n, cs, hkv, b) == want
    g = torch.Generator(device=DEV).manual_seed(keys + cs)
    q, k = torch.randn((hq, l_obs, 128), generator=g, device=DEV).bfloat16(), _keys(hkv, n, g)
    print(f"selection hq={hq} hkv={hkv} l_obs={l_obs} keys={keys} cs={cs} b={b}", flush=True)
    idx = ck.select_critical(q, k, [1, 0], cs, b).cpu().numpy()
    h = 1
    qf = q[h * G:(h + 1) * G].float().cpu().numpy().astype(np.float64)
    sc = O.chunk_scores(qf, k[h:h + 1].float().cpu().numpy().astype(np.float64), 0, G, l_obs, cs, 1 / math.sqrt(128))
    check_topk(idx[0], sc, b)


@pytest.mark.gpu
@pytest.mark.parametrize("hq,hkv,lq,keys,calib,want", [
    (2, 2, 16, 81921, False, WAVE),
    (2, 2, 64, 81920, True, TILE),
    (4, 2, 37, 90011, False, WAVE),
    (8, 2, 64, 32769, True, WAVE),
    (8, 2, 64, 32768, False, TILE),
    (16, 2, 30, 40001, False, WAVE),
])
def test_cv_either_side(hq, hkv, lq, keys, calib, want):
    n, G = keys + 40, hq // hkv
    assert score_route(hq, hkv, lq, n, 32, 8) == want
    g = torch.Generator(device=DEV).manual_seed(keys + lq)
    q, k = torch.randn((hq, lq, 128), generator=g, device=DEV).bfloat16(), _keys(hkv, n, g)
    pos = n if calib else n - lq
    print(f"cv hq={hq} hkv={hkv} lq={lq} keys={keys} calib={calib}", flush=True)
    cv = ck.score_heads(q, k, q_pos0=pos, l_init=32, l_rec=8, k_pct=0.996, alpha=1.0).cpu().numpy()
    h = 1
    qf = q[h * G:(h + 1) * G].float().cpu().numpy().astype(np.float64)
    ref = O.score_heads(qf, pos, k[h:h + 1].float().cpu().numpy().astype(np.float64), 32, 8, 0.996, 1.0)
    np.testing.assert_allclose(cv[h], ref[0], rtol=1e-4, atol=1e-6)
