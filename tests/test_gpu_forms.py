"""GPU parity of the attention's (head width, block size) forms where the
launch differs between them, against the oracle.

Each form keeps a different number of work-groups on a compute unit and
fetches further items once its first is done: layers with more (head, pair)
items than groups resident at once, uneven random lists (empty, full, short
and long rows), a short tail block, sampled query blocks.
"""
import math

import numpy as np
import pytest

import oracle as O
import workloads as W
from parity import LSE_ABS, MAX_ABS, MEAN_ABS, attention_errors, bf16_tensor, bf16_to_f64

import paper_2601_11641_amd as M
from test_gpu_parity import PLAN_MISC_INT, _uneven_lists

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


def _layer(B, H, L, d, seed, spread=1.5):
    """N(0, 1) values, Q and K scaled by spread, as bf16 bits and tensors."""
    rng = np.random.default_rng(seed)
    host = [W.to_bf16_bits(rng.standard_normal((B, H, L, d)).astype(np.float32) * (spread if t < 2 else 1.0))
            for t in range(3)]
    return host, tuple(bf16_tensor(x) for x in host)


def _check_rows(host, rows, o, lse, d, bs, L, heads, sample):
    scale = 1.0 / math.sqrt(d)
    og, lg = bf16_to_f64(o), lse.cpu().numpy().astype(np.float64)
    for b, h in heads:
        qf, kf, vf = (W.bf16_bits_to_f64(x[b, h]) for x in host)
        Oo, Lo = O.attention(qf, kf, vf, rows[b][h], bs, scale, rows=sample)
        for i in sample:
            sl = slice(i * bs, min(L, (i + 1) * bs))
            mx, mean = attention_errors(og[b, h, sl], Oo[sl])
            assert mx <= MAX_ABS and mean <= MEAN_ABS, (b, h, i, mx, mean)
            fin = np.isfinite(Lo[sl])
            assert (np.isneginf(lg[b, h, sl]) == ~fin).all(), (b, h, i)
            if fin.any():
                assert np.abs(lg[b, h, sl][fin] - Lo[sl][fin]).max() <= LSE_ABS, (b, h, i)


@pytest.mark.parametrize("d,bs,tail", [(128, 128, 1), (128, 64, 63), (64, 128, 37), (64, 64, 16)])
def test_attention_more_items_than_resident_groups(d, bs, tail):
    # 18 heads x 51 pairs, the last of one block (22 heads where 1024 groups are resident)
    B, H, n = 2, 11 if d == bs == 64 else 9, 101
    L = (n - 1) * bs + tail
    host, (q, k, v) = _layer(B, H, L, d, 100 + d + bs)
    rows, idx, cnt = _uneven_lists(B, H, n, 7)
    shape = M.make_shape(B, H, L, d, bs)
    for ws_bytes in (M.mod_attn_workspace_bytes(shape), M.mod_attn_plan_bytes(shape)):
        ws = torch.zeros(ws_bytes, dtype=torch.uint8, device="cuda")
        o = torch.full_like(q, float("nan"))
        lse = torch.full((B, H, L), float("nan"), dtype=torch.float32, device="cuda")
        M.mod_block_sparse_attn_fwd(shape, q, k, v, idx, cnt, 0.0, o, lse, ws, ws_bytes)
        assert not torch.isnan(o.float()).any() and not torch.isnan(lse).any()
        _check_rows(host, rows, o, lse, d, bs, L, [(0, 0), (0, 8), (1, 4)], [0, 1, 2, 49, 50, 98, 99, 100])


@pytest.mark.parametrize("d,bs,H,n", [(64, 128, 2, 150), (128, 64, 3, 99), (64, 64, 2, 230)])
def test_attention_fewer_items_than_resident_groups(d, bs, H, n):
    """Planned launches whose items, split or not, leave resident groups
    without one: those leave at once (the plan counts the items), the others
    do all of them."""
    L = (n - 1) * bs + 9
    host, (q, k, v) = _layer(1, H, L, d, n + bs)
    rng = np.random.default_rng(n)
    shape = M.make_shape(1, H, L, d, bs)
    pairs = H * ((n + 1) // 2)
    size = M.mod_attn_workspace_bytes(shape)
    for keep in (n // 4, n):
        rows = [[np.sort(rng.choice(n, size=keep, replace=False)).tolist() for _ in range(n)] for _ in range(H)]
        idx = torch.zeros((1, H, n, n), dtype=torch.int32)
        idx[0, :, :, :keep] = torch.tensor(rows, dtype=torch.int32)
        cnt = torch.full((1, H, n), keep, dtype=torch.int32, device="cuda")
        ws = torch.full((size,), 0x5A, dtype=torch.uint8, device="cuda")
        o = torch.full_like(q, float("nan"))
        lse = torch.full((1, H, L), float("nan"), dtype=torch.float32, device="cuda")
        M.mod_block_sparse_attn_fwd(shape, q, k, v, idx.cuda(), cnt, 0.0, o, lse, ws, size)
        head = ws[:4 * (PLAN_MISC_INT + 3)].view(torch.int32).cpu().tolist()
        lens, (splits, steps, items) = head[PLAN_MISC_INT - 16:PLAN_MISC_INT - 8], head[PLAN_MISC_INT:]
        assert items == sum(lens) and (splits > 0) == (keep == n), (lens, splits, steps, items)
        assert (items == pairs) if splits == 0 else (pairs < items), (items, pairs)
        assert not torch.isnan(o.float()).any() and not torch.isnan(lse).any()
        _check_rows(host, [rows], o, lse, d, bs, L, [(0, 0), (0, H - 1)], [0, 1, n // 2, n - 2, n - 1])


@pytest.mark.parametrize("d,bs,tail", [(128, 64, 1), (64, 128, 65), (64, 128, 64), (64, 64, 33)])
def test_attention_narrow_tiles_edges(d, bs, tail):
    """Walks of zero, one and two tiles in either part, and a short tail block
    in any position of them: its valid rows end inside the first or the
    second half tile, or exactly between them."""
    n, H = 9, 3
    L = (n - 1) * bs + tail
    host, (q, k, v) = _layer(1, H, L, d, 40 + d + bs + tail, spread=2.5)
    t = n - 1
    pick = [[[], [t], [0], [0, t], [t], [t], [1, 2], [1, 2, t], [0, 1, 2, t]],
            [[0, 1], [2, t], [3], [], [0, 3, t], [0, 3, t], [t], [5], [t]],
            [[2, 4, t], [2, 4, 6, t], [2], [3], [], [], list(range(n)), [t], [1]]]
    idx = torch.full((1, H, n, n), -1, dtype=torch.int32)
    cnt = torch.zeros((1, H, n), dtype=torch.int32)
    for h in range(H):
        for i, js in enumerate(pick[h]):
            cnt[0, h, i] = len(js)
            idx[0, h, i, :len(js)] = torch.tensor(js, dtype=torch.int32)
    o = torch.full_like(q, float("nan"))
    lse = torch.full((1, H, L), float("nan"), dtype=torch.float32, device="cuda")
    M.mod_block_sparse_attn_fwd(M.make_shape(1, H, L, d, bs), q, k, v, idx.cuda(), cnt.cuda(), 0.0, o, lse)
    _check_rows(host, [pick], o, lse, d, bs, L, [(0, h) for h in range(H)], list(range(n)))


@pytest.mark.parametrize("d,bs", [(128, 128), (128, 64), (64, 128), (64, 64)])
def test_attention_row_does_not_depend_on_the_other_row_of_its_pair(d, bs):
    """A query block's output is the same, bit for bit, whether the other block
    of its pair keeps the same list (every tile in the shared part of the
    walk) or none (every tile in its own part): the softmax steps cover the
    same kv rows in both.  Scores wide enough that the running max moves in the
    middle of a tile, a short tail block."""
    n, H = 13, 2
    L = (n - 1) * bs + bs // 2 + 3
    _, (q, k, v) = _layer(1, H, L, d, 300 + d + bs, spread=2.5)
    rng = np.random.default_rng(d + bs)
    shape = M.make_shape(1, H, L, d, bs)
    lists = [[np.sort(rng.choice(n, size=int(rng.integers(1, n + 1)), replace=False)) for _ in range((n + 1) // 2)]
             for _ in range(H)]

    def run(keeps):
        idx = torch.zeros((1, H, n, n), dtype=torch.int32)
        cnt = torch.zeros((1, H, n), dtype=torch.int32)
        for h in range(H):
            for i in range(n):
                if keeps(i):
                    js = lists[h][i // 2]
                    cnt[0, h, i] = len(js)
                    idx[0, h, i, :len(js)] = torch.from_numpy(js)
        o = torch.empty_like(q)
        lse = torch.empty((1, H, L), dtype=torch.float32, device="cuda")
        M.mod_block_sparse_attn_fwd(shape, q, k, v, idx.cuda(), cnt.cuda(), 0.0, o, lse)
        return o.view(torch.int16), lse

    o_both, lse_both = run(lambda i: True)
    for side in (0, 1):
        o, lse = run(lambda i: i % 2 == side)
        for i in range(side, n, 2):
            rows = slice(i * bs, min(L, (i + 1) * bs))
            assert torch.equal(lse[:, :, rows], lse_both[:, :, rows]), (side, i)
            assert torch.equal(o[:, :, rows], o_both[:, :, rows]), (side, i)


@pytest.mark.parametrize("d,bs,n", [(128, 128, 101), (64, 64, 64), (128, 64, 33)])
def test_attention_plan_without_counts(d, bs, n):
    """Fewer items than resident groups and no slots (short sequences, or a
    plan-only workspace): one item per group without a plan, uneven and empty
    rows, on a workspace of exactly the plan's size with stale contents."""
    H, L = 2, (n - 1) * bs + 17
    host, (q, k, v) = _layer(1, H, L, d, n)
    rows, idx, cnt = _uneven_lists(1, H, n, n)
    shape = M.make_shape(1, H, L, d, bs)
    size = M.mod_attn_plan_bytes(shape)
    ws = torch.full((size + 64,), 0x5A, dtype=torch.uint8, device="cuda")
    for _ in range(2):
        o = torch.full_like(q, float("nan"))
        lse = torch.full((1, H, L), float("nan"), dtype=torch.float32, device="cuda")
        M.mod_block_sparse_attn_fwd(shape, q, k, v, idx, cnt, 0.0, o, lse, ws, size)
        _check_rows(host, rows, o, lse, d, bs, L, [(0, 0), (0, 1)], sorted({0, 1, 2, n // 2, n - 2, n - 1}))
    assert (ws[size:] == 0x5A).all()


def test_attention_plan_of_sums_beyond_32_bits():
    """512 heads of 2048 blocks, every count 2048: the plan's sums over all
    pairs need 64 bits.  Every row lists its own block, the next one and a few
    rows all; the other slots hold -1, which the attention skips."""
    H, n, d, bs = 512, 2048, 64, 64
    L = n * bs
    cost = H * (n // 2) * (4 + 2 * n)
    assert cost >= 2**31
    host, small = _layer(1, 1, L, d, 3)
    q, k, v = (x.expand(1, H, L, d).contiguous() for x in small)
    own = torch.arange(n, dtype=torch.int32)
    row = torch.stack([own, (own + 1) % n], 1).sort(1).values.cuda()
    idx = torch.full((1, H, n, n), -1, dtype=torch.int32, device="cuda")
    idx[..., :2] = row
    cnt = torch.full((1, H, n), n, dtype=torch.int32, device="cuda")
    full = [0, 777, n - 1]
    for i in full:
        idx[:, :, i] = own.cuda()
    o = torch.empty_like(q)
    lse = torch.empty((1, H, L), dtype=torch.float32, device="cuda")
    shape = M.make_shape(1, H, L, d, bs)
    ws = torch.zeros(M.mod_attn_plan_bytes(shape), dtype=torch.uint8, device="cuda")
    M.mod_block_sparse_attn_fwd(shape, q, k, v, idx, cnt, 0.0, o, lse, ws, ws.numel())
    # the cost before each head and in all, and every pair in exactly one list
    at = 4 * (PLAN_MISC_INT + 16)
    before = ws[at:at + 8 * (H + 1)].view(torch.int64).cpu()
    assert torch.equal(before, torch.arange(H + 1) * (cost // H)) and int(before[-1]) == cost
    at += 8 * 8 * (H + 1)
    items = ws[at:at + 4 * H * (n // 2)].view(torch.int32)
    assert torch.equal(items.sort().values, torch.arange(H * (n // 2), dtype=torch.int32, device="cuda"))
    rows = [[list(range(n)) if i in full else sorted({i, (i + 1) % n}) for i in range(n)]]
    for h in (0, 200, H - 1):
        _check_rows(host, [rows], o[:, h:h + 1], lse[:, h:h + 1], d, bs, L, [(0, 0)], [0, 1, 776, 777, 1500, n - 1])
    assert torch.equal(o[0, 1].view(torch.int16), o[0, H - 1].view(torch.int16))


@pytest.mark.parametrize("H,n,keep", [(1, 195, 176), (2, 131, 131)])
def test_attention_split_in_equal_parts(H, n, keep):
    """Few equal long walks: split into the number of parts whose rounds of
    items end first, and merged."""
    d = bs = 128
    L = (n - 1) * bs + 5
    host, (q, k, v) = _layer(1, H, L, d, n)
    rng = np.random.default_rng(n)
    rows = [[np.sort(rng.choice(n, size=keep, replace=False)).tolist() for _ in range(n)] for _ in range(H)]
    idx = torch.zeros((1, H, n, n), dtype=torch.int32)
    idx[0, :, :, :keep] = torch.tensor(rows, dtype=torch.int32)
    cnt = torch.full((1, H, n), keep, dtype=torch.int32, device="cuda")
    shape = M.make_shape(1, H, L, d, bs)
    size = M.mod_attn_workspace_bytes(shape)
    ws = torch.zeros(size, dtype=torch.uint8, device="cuda")
    o = torch.full_like(q, float("nan"))
    lse = torch.full((1, H, L), float("nan"), dtype=torch.float32, device="cuda")
    M.mod_block_sparse_attn_fwd(shape, q, k, v, idx.cuda(), cnt, 0.0, o, lse, ws, size)
    split, steps = ws.view(torch.int32)[PLAN_MISC_INT:PLAN_MISC_INT + 2].cpu().tolist()
    assert split > 0 and steps >= 64, (split, steps)
    _check_rows(host, [rows], o, lse, d, bs, L, [(0, h) for h in range(H)], [0, 1, n // 2, n - 2, n - 1])
