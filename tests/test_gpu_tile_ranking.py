"""Token tiles beyond 128 tokens, which every wave of the tiled projections ranks from counts and mask (moe_rank_tiles):
hand-made tables with experts on both sides of lane 63 / 64, rows at the edges of 16, 96, 112 and 128, empty and masked experts
first, last and in runs, and a single working expert, every row against the oracle (these tables are small, and the down
projection takes tiles of 128 rows for all but one); then tables for which it takes every tile height and number of K
splits, with the tiles read off the block timeline."""
import numpy as np
import pytest

import oracle
from paper_2602_03495_amd import workloads as wl
from helpers import OUT_TOL, SENTINEL, rel_err

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

EDGES = [1, 15, 16, 17, 95, 96, 97, 111, 112, 113, 127, 128, 129, 191, 192, 193, 224, 225, 255, 256, 257, 384]


def _rows(N, at):
    rows = np.zeros(N, np.int32)
    for e, n in at.items():
        rows[e % N] = n
    return rows


# rows per expert, experts masked off (None: no mask)
CASES = {
    "1": (_rows(1, {0: 129}), None),
    "63-edges": (_rows(63, {2 * i: n for i, n in enumerate(EDGES)} | {-1: 3}), [0, 4]),
    "64-last": (_rows(64, {0: 5, 63: 260}), None),
    "65-last": (_rows(65, {63: 130, 64: 97}), [63]),
    "128-spread": (_rows(128, {(17 * i + 5) % 128: n for i, n in enumerate(EDGES)} | {127: 33}), [5, 22, 126]),
    "128-one": (_rows(128, {64: 600, 3: 9}), [3]),
    "128-all": (np.full(128, 9, np.int32), list(range(0, 128, 3))),
}


@pytest.mark.parametrize("name", CASES)
@pytest.mark.parametrize("d", [256, 1024])           # column tiles of 128 and, with many token tiles, more
def test_every_row_of_hand_made_tables(name, d):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_03495_amd import binding as B, layer as Lm
    B.load_library()
    rows, off = CASES[name]
    N, T, I = len(rows), int(rows.sum()), 128
    assert T > 128, "the case must take the ranked tiles"
    cfg = wl.scaled(wl.CONFIGS["tiny"], d=d, I=I, N=N, k=1)
    h, (w1, w3, w2) = wl.hidden_states(cfg, T), wl.expert_weights(cfg)
    perm = np.random.default_rng(N).permutation(T).astype(np.int32)
    topk_idx = np.empty((T, 1), np.int32)
    topk_idx[perm, 0] = np.repeat(np.arange(N), rows)
    mask = np.ones(N, np.uint8)
    if off is not None:
        mask[off] = 0
    offsets = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)

    s = B.shape(T, d, N, 1, I)
    y = torch.empty((T, d), dtype=torch.bfloat16, device="cuda")
    y.view(torch.int16).fill_(SENTINEL)
    dev = lambda a: torch.from_numpy(a).cuda()
    packed = [B.moe_pack_weights(Lm.to_device_bf16(w)) for w in (w1, w3, w2)]
    print(f"tile ranking {name} d={d} T={T}", flush=True)
    B.moe_expert_ffn(s, Lm.to_device_bf16(h), dev(perm), dev(offsets), dev(rows), *packed, None if off is None else dev(mask), y,
                     B.alloc_workspace(s))
    torch.cuda.synchronize()
    bits = Lm.from_device_bf16(y)
    on = np.repeat(mask.astype(bool), rows)
    assert np.all(bits[~on] == SENTINEL), "a row of a masked-off expert was written"
    ref = oracle.expert_rows(h, topk_idx, w1, w3, w2, mask, tokens=perm[on])[:, 0]
    got = wl.bf16_bits_to_f32(bits[on])
    worst = max(rel_err(got[i], ref[i]) for i in range(len(got)))
    assert worst <= OUT_TOL, worst


def _down_launch(rows, T, d, I):
    """What the tiled down projection does with these rows (k = 1, all experts on), as the kernels decide it: token-tile
    height and K splits."""
    N, tiles = len(rows), lambda h: int(sum(-(-int(r) // h) for r in rows))
    est = max(-(-T // 128), min(N, T))
    nf = 4 if est * -(-d // 512) >= 256 else 2 if est * -(-d // 256) >= 256 else 1
    n_ntc = -(-d // (128 * nf))
    nsp_max = 1
    while nsp_max < 8 and (I // 32) % (16 * nsp_max) == 0 and I // 32 // (2 * nsp_max) >= 32 and 2 * nsp_max * T * d * 4 <= 64 << 20:
        nsp_max *= 2
    height = 128
    if tiles(128) * n_ntc >= 256:
        def cost(h):
            items = tiles(h) * n_ntc
            return (2 * -(-items // 256) if items <= 512 else (2 * items + 255) // 256 + 1) * (h + 64)
        height = min((128, 112, 96), key=cost)                      # of equals the tallest
    items = tiles(height) * n_ntc
    nsp, best, finer = 1, -(-items // 256) * 64, 2
    while finer <= nsp_max:
        c = -(-items * finer // 256) * (64 // finer)
        if c * 100 <= best * 85:
            nsp, best = finer, c
        finer *= 2
    return height, nsp


# rows per expert, d, I, height and K splits of the down projection
LAUNCHES = {
    "128 rows": ([128 * (1 + e % 2) for e in range(128)], 256, 128, 128, 1),
    "112 rows": ([193 + e % 32 for e in range(128)], 256, 128, 112, 1),
    "96 rows": ([96 * (1 + e % 2) - e % 5 for e in range(128)], 256, 128, 96, 1),
    "2 splits": ([129, 0, 31, 100, 1], 384, 2048, 128, 2),
    "4 splits": ([1, 0, 257, 16, 112], 256, 4096, 128, 4),
    "8 splits": ([33, 128, 0, 96, 17], 640, 8192, 128, 8),
    "4 of 8 splits": ([128] * 14 + [1, 100], 512, 8192, 128, 4),
}


@pytest.mark.parametrize("name", LAUNCHES)
def test_every_tile_height_and_split_of_the_down_projection(name):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_03495_amd import binding as B, layer as Lm
    B.load_library()
    rows, d, I, height, nsp = LAUNCHES[name]
    N, T = len(rows), sum(rows)
    assert _down_launch(rows, T, d, I) == (height, nsp), _down_launch(rows, T, d, I)
    cfg = wl.scaled(wl.CONFIGS["tiny"], d=d, I=I, N=N, k=1)
    h, (w1, w3, w2) = wl.hidden_states(cfg, T), wl.expert_weights(cfg)
    perm = np.random.default_rng(N).permutation(T).astype(np.int32)
    topk_idx = np.empty((T, 1), np.int32)
    topk_idx[perm, 0] = np.repeat(np.arange(N), rows)
    offsets = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    s = B.shape(T, d, N, 1, I)
    y = torch.empty((T, d), dtype=torch.bfloat16, device="cuda")
    y.view(torch.int16).fill_(SENTINEL)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    packed = [B.moe_pack_weights(Lm.to_device_bf16(w)) for w in (w1, w3, w2)]
    records = torch.zeros(2 * B.TRACE_MAX_BLOCKS * 8, dtype=torch.int64, device="cuda")
    print(f"down projection launch {name} d={d} I={I} T={T}", flush=True)
    B.moe_debug_set_trace(records)
    B.moe_expert_ffn(s, Lm.to_device_bf16(h), dev(perm), dev(offsets), dev(np.array(rows, np.int32)), *packed, None, y, B.alloc_workspace(s))
    torch.cuda.synchronize()
    B.moe_debug_set_trace(None)
    t = records.cpu().numpy().reshape(2, B.TRACE_MAX_BLOCKS, 8)[1]
    t = t[t[:, 7] == 1]
    tiles = sorted((e, min(height, n - m)) for e, n in enumerate(rows) for m in range(0, n, height))
    col = sorted(map(tuple, t[t[:, 6] == 0][:, 4:6].tolist()))
    assert col == sorted(tiles * nsp), "the launch's tiles of the first columns"
    # the first and last rows of every expert, and of its tiles
    edge = {o + j for o, n in zip(offsets, rows) for m in range(0, n, height) for j in (m, min(n, m + height) - 1)}
    pick = np.array(sorted(edge))[:: max(1, len(edge) // 400)]
    ref = oracle.expert_rows(h, topk_idx, w1, w3, w2, np.ones(N, np.uint8), tokens=perm[pick].astype(np.int32))[:, 0]
    bits = Lm.from_device_bf16(y)
    assert not np.any(np.all(bits == SENTINEL, axis=1)), "a row was not written"
    got = wl.bf16_bits_to_f32(bits[pick])
    worst = max(rel_err(got[i], ref[i]) for i in range(len(pick)))
    assert worst <= OUT_TOL, worst


# rows per expert, inner size, blocks of the up projection that have an item.  384 items, a round and a half: with a mean of 86 and 65 rows
# to a tile the last 128 run as two blocks each (those of a ragged column tile, 4 of the 16 of every XCD, as one), with one row
# all of them, three rounds; one tile more: none
UP_ITEMS = {"a round and 256 half-width items": ([257] * 128, 256, 512), "one tile more": ([257] * 127 + [385], 256, 385),
            "768 half-width items, one tile per expert": ([1] * 128, 768, 768),
            "a round and 224 half-width items": ([130] * 32 + [0] * 8, 1408, 480)}


@pytest.mark.parametrize("name", UP_ITEMS)
def test_every_item_of_the_up_projection_has_a_block(name):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_03495_amd import binding as B, layer as Lm
    B.load_library()
    rows, I, items = UP_ITEMS[name]
    N, T, d = len(rows), sum(rows), 128
    cfg = wl.scaled(wl.CONFIGS["tiny"], d=d, I=I, N=N, k=1)
    h, (w1, w3, w2) = wl.hidden_states(cfg, T), wl.expert_weights(cfg)
    perm = np.random.default_rng(N).permutation(T).astype(np.int32)
    topk_idx = np.empty((T, 1), np.int32)
    topk_idx[perm, 0] = np.repeat(np.arange(N), rows)
    offsets = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    s = B.shape(T, d, N, 1, I)
    y = torch.empty((T, d), dtype=torch.bfloat16, device="cuda")
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    packed = [B.moe_pack_weights(Lm.to_device_bf16(w)) for w in (w1, w3, w2)]
    records = torch.zeros(2 * B.TRACE_MAX_BLOCKS * 8, dtype=torch.int64, device="cuda")
    print(f"up projection items {name} I={I} T={T}", flush=True)
    B.moe_debug_set_trace(records)
    B.moe_expert_ffn(s, Lm.to_device_bf16(h), dev(perm), dev(offsets), dev(np.array(rows, np.int32)), *packed, None, y, B.alloc_workspace(s))
    torch.cuda.synchronize()
    B.moe_debug_set_trace(None)
    t = records.cpu().numpy().reshape(2, B.TRACE_MAX_BLOCKS, 8)[0]
    assert int((t[:, 7] == 1).sum()) == items
    last = [o + n - 1 for o, n in zip(offsets, rows) if n]                 # the last row of every expert, and some others
    pick = np.array(sorted(set(last) | set(range(0, T, max(1, T // 200)))))
    ref = oracle.expert_rows(h, topk_idx, w1, w3, w2, np.ones(N, np.uint8), tokens=perm[pick].astype(np.int32))[:, 0]
    got = wl.bf16_bits_to_f32(Lm.from_device_bf16(y)[pick])
    worst = max(rel_err(got[i], ref[i]) for i in range(len(pick)))
    assert worst <= OUT_TOL, worst
