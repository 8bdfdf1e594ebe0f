"""The extrapolation and selection launch against the oracle's selection of
the same prediction.

The lists of every row must equal what the oracle selects from the prediction
and the gate read back from the handle (fp64, so both sides rank the same
float32 keys): at the row widths where the keys per lane change and where a
row is shared by a work-group's waves (above 2304 blocks, up to the limit of
4096), with one and with two rows per wave, boundaries found bit by bit and by
galloping, aligned and straddling chunks of rows, tied keys
(constant Q and K: the order by block or pattern index decides), forced frame
blocks, and a text segment.  MASS sums its fp64 masses in another order than
the oracle: a row whose target lies within 1e-12 of a prefix is left out.
"""
import numpy as np
import pytest

import oracle as O
import workloads as W
from parity import bf16_tensor

import paper_2601_11641_amd as M

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

# heads, frames, tokens per frame, text tokens, block (n blocks)
LAYERS = {
    "n5": (1, 2, 160, 0, 64),
    "n64": (3, 4, 1024, 0, 64),
    "n65": (2, 5, 819, 0, 64),
    "n257": (2, 3, 5483, 0, 64),
    "n640": (1, 2, 20480, 0, 64),
    "n1024": (1, 4, 16384, 0, 64),
    "n1025": (1, 4, 16385, 0, 64),
    "n229h36": (36, 4, 3660, 0, 64),        # two rows per wave, the last chunk short
    "n229h36text": (36, 4, 3660, 77, 64),   # and a block of video and text
    "n65text": (2, 5, 832, 130, 64),        # the text starts on a block
    "n129": (2, 3, 2740, 0, 64),
    "n192": (2, 4, 3072, 0, 64),
    "n193": (1, 2, 6160, 0, 64),
    "n448": (1, 4, 7168, 0, 64),
    "n2063": (1, 3, 44000, 0, 64),
    "n2304": (1, 2, 73728, 0, 64),
    "n2305": (1, 5, 29501, 0, 64),          # a row per work-group from here on
    "n2561h2": (2, 4, 40963, 0, 64),
    "n3073text": (1, 3, 65550, 130, 64),
    "n3585": (1, 4, 57345, 0, 64),
    "n4096": (1, 2, 131060, 0, 64),
}


def _rows(kv_idx, kv_cnt):
    idx, cnt = kv_idx.cpu().numpy(), kv_cnt.cpu().numpy()
    return [[[idx[b, h, i, :cnt[b, h, i]].tolist() for i in range(cnt.shape[2])] for h in range(cnt.shape[1])]
            for b in range(cnt.shape[0])][0]


@pytest.mark.parametrize("name", sorted(LAYERS))
@pytest.mark.parametrize("tied", [False, True])
def test_selection_of_the_predicted_scores(name, tied):
    H, F, T, text, bs = LAYERS[name]
    d, L = 64, F * T + text
    n, nv = -(-L // bs), -(-F * T // bs)
    gen = torch.Generator(device="cuda").manual_seed(n + H)
    q, k, q1, k1 = (torch.randn((1, H, 1 if tied else L, d), device="cuda", generator=gen).bfloat16()
                    .expand(1, H, L, d).contiguous() for _ in range(4))
    shape = M.make_shape(1, H, L, d, bs, T, text)
    regions = O.frame_regions(F * T, bs, T)
    heads = range(H) if H < 5 else (0, 17, H - 1)
    # frame blocks forced in every head, in none (a very wide handle takes seconds to create: one of both)
    for tau_e in (-1e9, 1e9) if n < 3000 else (-1e9 if tied else 1e9,):
        with M.Stats(shape, M.make_params(warmup_m=2, delta_t=0, tau_e=tau_e)) as st:
            M.mod_collect_stats(st.handle, q, k, 1)
            M.mod_collect_stats(st.handle, q1, k1, 2)
            for step, (mode, kw) in enumerate([("topk", dict(density=0.2)), ("topk", dict(density=1.0)),
                                               ("mass", dict(mass=0.7)), ("mass", dict(mass=1.0)),
                                               ("pattern", dict(patterns=1)),
                                               ("pattern", dict(patterns=max(1, nv // 2)))], start=3):
                idx = torch.full((1, H, n, n), -1, dtype=torch.int32, device="cuda")
                cnt = torch.zeros((1, H, n), dtype=torch.int32, device="cuda")
                M.mod_predict_block_mask(st.handle, None, None, step, M.make_budget(mode, **kw), idx, cnt)
                rows = [_rows(idx[:, h:h + 1], cnt[:, h:h + 1])[0] for h in heads]
                pred = M.mod_stats_get_prediction(st.handle, 1, H, nv)[0]
                gate = M.mod_stats_get_gate(st.handle, 1, H)[0]
                X2, X1 = (M.mod_stats_get_anchor(st.handle, s, 1, H, st.p)[0][0] for s in (0, 1))
                assert (gate == (tau_e < 0)).all()
                for h in heads:
                    ref = X2[h, :3 * nv - 1] + (X2[h, :3 * nv - 1] - X1[h, :3 * nv - 1]) * (step - 2)
                    np.testing.assert_allclose(pred[h], ref, rtol=0, atol=1e-14 * max(1.0, np.abs(X2[h]).max()) * step)
                    c, dd = pred[h, :2 * nv - 1], pred[h, 2 * nv - 1:]
                    sig = O.scores(c, dd, nv)
                    # every row of a narrow layer; of a wide one the first and the
                    # last, those around a change of work-group, and random ones
                    some = range(n) if n <= 1300 else sorted(
                        {*range(6), nv // 2, *range(nv - 5, n), *np.random.default_rng(n + step).integers(0, n, 24)})
                    forced = O.forced_mask(nv, regions, bool(gate[h]))
                    if text and (F * T) % bs:
                        forced[:, nv - 1] = True
                    if mode == "pattern":
                        want = [r.kept for r in O.select_patterns(c, dd, nv, kw["patterns"], forced)]
                        sure = [True] * nv
                    else:
                        sel = {i: O.select_row_topk(sig[i], forced[i], O.topk_count(kw["density"], nv)) if mode == "topk"
                               else O.select_row_mass(sig[i], forced[i], kw["mass"]) for i in some if i < nv}
                        want = {i: r.kept for i, r in sel.items()}
                        sure = {i: mode == "topk" or r.mass_margin > 1e-12 for i, r in sel.items()}
                    for i in some:
                        if text and i >= F * T // bs:
                            assert rows[heads.index(h)][i] == list(range(n)), (h, i)
                        elif sure[i]:
                            assert rows[heads.index(h)][i] == want[i].tolist() + list(range(nv, n)), (
                                name, tau_e, mode, kw, h, i)
