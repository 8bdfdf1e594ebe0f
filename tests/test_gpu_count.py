"""The attention statistic's counts over walks that are cut into parts.

Uneven lists (empty, short and full rows), an odd number of blocks, a short
tail block and text tokens, at sizes where a walk has one, two and four parts.
A block's count may differ from the fp64 count only by entries whose
log-probability lies within 2e-4 of the threshold (the decision is taken in
fp32 on fp32 row sums); unlisted blocks keep the zeros they start with.
"""
import math

import numpy as np
import pytest

import workloads as W
from parity import bf16_tensor

import paper_2601_11641_amd as M
from test_gpu_parity import _uneven_lists

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


@pytest.mark.parametrize("d,bs,n,text", [(128, 128, 15, 0), (128, 128, 31, 0), (64, 64, 33, 0), (128, 64, 67, 0),
                                         (64, 128, 71, 300), (128, 128, 65, 100)])
def test_counts_of_cut_walks(d, bs, n, text):
    H, eta = 2, 3e-3
    T = (n * bs - text - 23) // 2
    Lv = 2 * T
    L = Lv + text
    nv = -(-Lv // bs)
    assert -(-L // bs) == n
    rng = np.random.default_rng(n)
    q, k, v = (bf16_tensor(W.to_bf16_bits(rng.standard_normal((1, H, L, d)).astype(np.float32) * 1.3))
               for _ in range(3))
    rows, idx, cnt = _uneven_lists(1, H, n, n + d)
    shape = M.make_shape(1, H, L, d, bs, T, text)
    o, lse = torch.empty_like(q), torch.empty((1, H, L), dtype=torch.float32, device="cuda")
    M.mod_block_sparse_attn_fwd(shape, q, k, v, idx, cnt, 0.0, o, lse)
    with M.Stats(shape, M.make_params(warmup_m=1, statistic="attention", eta=eta)) as st:
        M.mod_update_stats(st.handle, q, k, lse, idx, cnt, 1)
        G = M.mod_stats_get_block_mass(st.handle, 1, H, nv)[0]
    sizes = np.array([min(bs, L - i * bs) for i in range(n)], dtype=np.float64)
    pad = n * bs - L
    for h in range(H):
        p = (q[0, h].double() @ k[0, h].double().t()) / math.sqrt(d) - lse[0, h].double()[:, None] - math.log(eta)
        p = torch.nn.functional.pad(p, (0, pad, 0, pad), value=-math.inf).view(n, bs, n, bs)
        p = torch.nan_to_num(p, nan=-math.inf, posinf=math.inf, neginf=-math.inf)
        want = (p >= 0).sum((1, 3)).cpu().numpy()
        band = (p.abs() < 2e-4).sum((1, 3)).cpu().numpy()
        got = G[h] * sizes[:nv, None] * sizes[None, :nv]
        for i in range(nv):
            kept = np.zeros(nv, dtype=bool)
            kept[[j for j in rows[0][h][i] if j < nv]] = True
            assert (G[h, i, ~kept] == 0).all(), (h, i)
            assert (np.abs(got[i] - want[i, :nv])[kept] <= band[i, :nv][kept] + 1e-6).all(), (h, i)
        assert want.sum() > 0
