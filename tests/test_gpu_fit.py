"""GPU parity of the fit (block logits, map, sums, solve) where its launches
change with the shape, against the oracle in fp64.

A head's whole fit runs in one launch up to 64 and up to 128 blocks (and as
many frames), beyond that in row chunks of 4, 8 or 16 rows; the logits use 32-
or 64-row tiles.  Sizes on both sides of each line, short last chunks and
tiles, frames that straddle blocks, more frames than blocks.  The statistic
and the coefficients must agree to rounding level: 1e-10 and 1e-9 relative, as
in the other parity tests.
"""
import numpy as np
import pytest

import oracle as O
from parity import bf16_to_f64

import paper_2601_11641_amd as M

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

# heads, frames, tokens per frame, block, d
SHAPES = {
    "n5": (1, 2, 150, 64, 64),
    "n63": (3, 7, 573, 64, 64),
    "n64": (2, 4, 1024, 64, 128),
    "n65": (2, 5, 831, 64, 64),
    "n62f70": (2, 70, 56, 64, 64),       # more frames than a 64-block fit holds
    "n123f140": (2, 140, 56, 64, 64),    # and than a 128-block fit
    "n127": (2, 3, 5414, 128, 128),
    "n128": (5, 8, 1024, 64, 128),
    "n129": (2, 4, 2050, 64, 64),        # chunks of 4 rows, the last of one
    "n229h36": (36, 4, 3660, 64, 64),    # 8 rows, the last chunk of five; 64-row logit tiles
    "n330h60": (60, 3, 7030, 64, 64),    # 16 rows, the last chunk of ten
}


def _setup(name):
    H, F, T, bs, d = SHAPES[name]
    L = F * T
    gen = torch.Generator(device="cuda").manual_seed(len(name) + H * L)
    base = torch.randn((1, H, F, 1, d), device="cuda", generator=gen)
    q, k = ((base + torch.randn((1, H, F, T, d), device="cuda", generator=gen)).reshape(1, H, L, d).bfloat16()
            .contiguous() for _ in range(2))
    return H, L, d, bs, T, q, k, M.make_shape(1, H, L, d, bs, T), O.frame_regions(L, bs, T)


def _check_fit(st, H, G, regions, heads):
    X, _ = M.mod_stats_get_anchor(st.handle, 0, 1, H, st.p)
    for h in heads:
        ref = O.fit(G[h], regions)
        assert np.abs(X[0, h] - ref).max() <= 1e-9 * max(1.0, np.abs(ref).max()), h


@pytest.mark.parametrize("name", sorted(SHAPES))
def test_pooled_fit(name):
    H, L, d, bs, T, q, k, shape, regions = _setup(name)
    heads = range(H) if H < 6 else (0, H // 2, H - 1)
    with M.Stats(shape, M.make_params(warmup_m=1)) as st:
        M.mod_collect_stats(st.handle, q, k, 1)
        G = M.mod_stats_get_block_mass(st.handle, 1, H, st.n)[0]
        for h in heads:
            qb, kb = (O.pool(bf16_to_f64(x[0, h]), bs) for x in (q, k))
            ref = O.block_mass(qb, kb, O.block_sizes(L, bs), 1.0 / np.sqrt(d))
            np.testing.assert_allclose(G[h], ref, rtol=1e-10, atol=1e-15)
        _check_fit(st, H, G, regions, heads)


@pytest.mark.parametrize("name", ["n62f70", "n64", "n65", "n129", "n229h36"])
def test_attention_statistic_fit(name):
    """The same launches over a stored map, which they must leave as it is."""
    H, L, d, bs, T, q, k, shape, regions = _setup(name)
    heads = range(H) if H < 6 else (0, H // 2, H - 1)
    n = M.mod_num_blocks(shape)
    idx = torch.arange(n, dtype=torch.int32, device="cuda").expand(1, H, n, n).contiguous()
    cnt = torch.full((1, H, n), n, dtype=torch.int32, device="cuda")
    o, lse = torch.empty_like(q), torch.empty((1, H, L), dtype=torch.float32, device="cuda")
    M.mod_block_sparse_attn_fwd(shape, q, k, q, idx, cnt, 0.0, o, lse)
    with M.Stats(shape, M.make_params(warmup_m=1, statistic="attention", eta=1e-3)) as st:
        M.mod_update_stats(st.handle, q, k, lse, idx, cnt, 1)
        G = M.mod_stats_get_block_mass(st.handle, 1, H, n)[0]
        sizes = O.block_sizes(L, bs)
        counts = G * sizes[:, None] * sizes[None, :]
        assert np.abs(counts - np.round(counts)).max() <= 1e-9 * bs * bs and G.max() > 0
        _check_fit(st, H, G, regions, heads)


@pytest.mark.parametrize("F,T", [(3, 65550), (2, 131060)])
def test_fit_of_wide_maps(F, T):
    """3073 and 4096 blocks (the largest): the block mass on sampled rows, and X
    as the minimum-norm solution of the normal equations -- the residual G - M X
    sums to zero over every diagonal, column and frame square, and X has no
    component along the null vector.  An error of 1e-9 of the largest
    coefficient (as above) in each of a cell's three terms, over n cells."""
    L, d, bs = F * T, 64, 64
    n, regions = O.num_blocks(L, bs), O.frame_regions(L, bs, T)
    gen = torch.Generator(device="cuda").manual_seed(n)
    base = torch.randn((1, 1, F, 1, d), device="cuda", generator=gen)
    q, k = ((base + torch.randn((1, 1, F, T, d), device="cuda", generator=gen)).reshape(1, 1, L, d).bfloat16()
            .contiguous() for _ in range(2))
    with M.Stats(M.make_shape(1, 1, L, d, bs, T), M.make_params(warmup_m=1)) as st:
        M.mod_collect_stats(st.handle, q, k, 1)
        G = M.mod_stats_get_block_mass(st.handle, 1, 1, n)[0, 0]
        X = M.mod_stats_get_anchor(st.handle, 0, 1, 1, st.p)[0][0, 0]
    qb, kb = (O.pool(bf16_to_f64(x[0, 0]), bs) for x in (q, k))
    sample = sorted({0, 1, 15, 16, n // 2, n - 2, n - 1, *np.random.default_rng(n).integers(0, n, 24).tolist()})
    np.testing.assert_allclose(G[sample], O.block_mass(qb[sample], kb, O.block_sizes(L, bs), 1.0 / np.sqrt(d)),
                               rtol=1e-10, atol=1e-15)
    bound = 3 * n * 1e-9 * np.abs(X).max()
    assert np.abs(O.rhs(G - O.reconstruct(X, n, regions), regions)).max() <= bound
    assert abs(X @ O.null_vector(n, F)) <= bound


def test_handle_memory_of_short_maps():
    """A handle of short maps owns what the header states, and none of the long
    maps' row-chunk sums (284 MB here)."""
    H, n, d = 16384, 128, 64
    T = n * 64 // 2
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    with M.Stats(M.make_shape(1, H, 2 * T, d, 64, T), M.make_params(warmup_m=1)):
        used = free - torch.cuda.mem_get_info()[0]
    stated = H * (2 * n * d + n * n + 29 * n) * 8
    assert abs(used - stated) < 128 << 20, (used, stated)
