"""CV scoring where column blocks are longer than the columns that are counted
at a time (many KV heads share the compute units), with odd key counts, and
with observation values so close together that the bracket spans few keys of
the float order: two heads against the oracle."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2608_30295_amd as ck
from gpu_util import DEV

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hkv,G,lq,n,scale,dtype", [
    (64, 1, 16, 135000 + 37, 1.0, torch.bfloat16),     # blocks of 16896 columns on 256 compute units: two counting windows
    (64, 1, 16, 190000 + 37, 1.0, torch.bfloat16),     # 23808: well beyond the first window's 16384
    (32, 2, 33, 70001, 1.0, torch.bfloat16),
    (8, 4, 16, 30011, 0.02, torch.bfloat16),           # near-uniform rows
    (64, 1, 8, 20005, 1.0, torch.float32),
])
def test_cv_long_blocks(hkv, G, lq, n, scale, dtype):
    g = torch.Generator(device=DEV).manual_seed(n)
    q = torch.randn((hkv * G, lq, 128), generator=g, device=DEV).to(dtype)
    k = torch.empty((hkv, n, 128), dtype=dtype, device=DEV)
    for h in range(hkv):
        x = torch.randn((n, 128), generator=g, device=DEV) * scale
        x[torch.rand(n, generator=g, device=DEV) < 0.01] *= 3
        k[h] = x
    l_init, l_rec = 32, 8
    print(f"cv blocks hkv={hkv} G={G} lq={lq} n={n} scale={scale} {dtype}", flush=True)
    cv = ck.score_heads(q, k, q_pos0=n - lq, l_init=l_init, l_rec=l_rec, k_pct=0.996, alpha=1.0).cpu().numpy()
    for h in (0, hkv - 1):
        qf = q[h * G:(h + 1) * G].float().cpu().numpy().astype(np.float64)
        kf = k[h:h + 1].float().cpu().numpy().astype(np.float64)
        ref = O.score_heads(qf, n - lq, kf, l_init, l_rec, 0.996, 1.0)
        np.testing.assert_allclose(cv[h], ref[0], rtol=1e-4, atol=1e-6)


UNTOUCHED = 0x7FBADBAD


@pytest.mark.parametrize("hkv,lq,n_keys,repeat", [
    (8, 64, 131072, 1),      # rows of a power of two: an even step over the entries meets the same keys in every row
    (16, 32, 65536, 1),
    (16, 32, 65536, 8),      # keys in runs of eight alike
    (16, 32, 65531, 8),
])
def test_cv_sample_brackets_the_quantile(hkv, lq, n_keys, repeat):
    """No head's sample misses the quantile: the observation matrix, which is
    written out for such a head alone, stays untouched in the workspace."""
    G, n = 4, n_keys + 40
    g = torch.Generator(device=DEV).manual_seed(n_keys + repeat)
    q = torch.randn((hkv * G, lq, 128), generator=g, device=DEV).bfloat16()
    k = torch.empty((hkv, n, 128), dtype=torch.bfloat16, device=DEV)
    for h in range(hkv):
        x = torch.randn((-(-n // repeat), 128), generator=g, device=DEV)
        x[torch.rand(x.shape[0], generator=g, device=DEV) < 0.01] *= 3
        k[h] = x.repeat_interleave(repeat, dim=0)[:n]
    print(f"cv sample hkv={hkv} lq={lq} n_keys={n_keys} repeat={repeat}", flush=True)
    ws = ck.workspace(ck.score_heads_workspace(hkv * G, hkv, lq, n, 32, 8), DEV)
    words = ws[:ws.numel() // 4 * 4].view(torch.int32)
    words.fill_(UNTOUCHED)
    cv = ck.score_heads(q, k, q_pos0=n - lq, l_init=32, l_rec=8, k_pct=0.996, alpha=1.0, ws=ws).cpu().numpy()
    edges = torch.nonzero(words != UNTOUCHED).flatten()
    assert int((edges[1:] - edges[:-1]).max()) > hkv * lq * n_keys
    for h in (0, hkv - 1):
        qf = q[h * G:(h + 1) * G].float().cpu().numpy().astype(np.float64)
        kf = k[h:h + 1].float().cpu().numpy().astype(np.float64)
        ref = O.score_heads(qf, n - lq, kf, 32, 8, 0.996, 1.0)
        np.testing.assert_allclose(cv[h], ref[0], rtol=1e-4, atol=1e-6)


def test_cv_radix_route_of_clustered_scores():
    """64 keys alike in a row at the 0.984 percentile: the entries at and above
    the quantile lie in few columns, whose buffers overflow, and heads take
    the radix route over the stored matrix."""
    hkv, G, lq, n = 16, 4, 32, 65536 + 40
    g = torch.Generator(device=DEV).manual_seed(5)
    q = torch.randn((hkv * G, lq, 128), generator=g, device=DEV).bfloat16()
    x = torch.randn((hkv, 1025, 128), generator=g, device=DEV)
    x[torch.rand((hkv, 1025), generator=g, device=DEV) < 0.01] *= 3
    k = x.repeat_interleave(64, dim=1)[:, :n].bfloat16().contiguous()
    ws = ck.workspace(ck.score_heads_workspace(hkv * G, hkv, lq, n, 32, 8), DEV)
    words = ws[:ws.numel() // 4 * 4].view(torch.int32)
    words.fill_(UNTOUCHED)
    cv = ck.score_heads(q, k, q_pos0=n - lq, l_init=32, l_rec=8, k_pct=0.984, alpha=1.0, ws=ws).cpu().numpy()
    edges = torch.nonzero(words != UNTOUCHED).flatten()
    assert int((edges[1:] - edges[:-1]).max()) < hkv * lq * 65536       # some head's matrix was stored
    for h in (0, 5, hkv - 1):
        qf = q[h * G:(h + 1) * G].float().cpu().numpy().astype(np.float64)
        ref = O.score_heads(qf, n - lq, k[h:h + 1].float().cpu().numpy().astype(np.float64), 32, 8, 0.984, 1.0)
        np.testing.assert_allclose(cv[h], ref[0], rtol=1e-4, atol=1e-6)
