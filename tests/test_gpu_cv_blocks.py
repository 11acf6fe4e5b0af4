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
    (64, 1, 16, 135000 + 37, 1.0, torch.bfloat16),     # blocks of 16887 columns: two counting windows
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
