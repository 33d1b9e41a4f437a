"""Tiled expert FFN: the items of a last round that would fill half of the compute units or less run as two of half the width, and
those of an up projection of 257 to 384 all of them, where that is two rounds or their token tiles are short.

Row tables whose launches end in such a round, just beside it and in an exact half of one, on both sides of the rule of the up
projection: the blocks that had an item, and the results against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2602_03495_amd import workloads as wl
from helpers import OUT_TOL, SENTINEL, rel_err

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# rows per expert, d, I, blocks with an item of the up and of the down projection
LAUNCHES = {
    "24 of 280 cut": ([130] * 70 + [0] * 58, 1024, 512, 304, 304),
    # short tiles: all 270 of the up projection as halves
    "at most one tile per expert": ([1] * 90 + [0] * 38, 1024, 768, 540, 464),
    "32 rows to a tile": ([32] * 90, 128, 768, 540, 90),
    "33 rows to a tile": ([33] * 90, 128, 768, 284, 90),
    # 258 items with a ragged last column tile are 473 halves: two rounds of them
    "two rounds of halves": ([2] * 43 + [0] * 20, 256, 1408, 473, 86),
    "two rounds of halves, full tiles": ([128] * 43, 256, 1408, 473, 86),
    "a half less than a third round": ([64] * 46 + [0], 256, 1408, 506, 92),
    "halves would need a third round": ([64] * 47, 256, 1408, 303, 94),
    "three column tiles": ([9] * 90, 128, 640, 450, 90),
    "a whole round of items": ([3] * 64, 256, 1024, 256, 128),
    "384, long tiles": ([40] * 128, 128, 768, 512, 128),
    "384, short tiles": ([32] * 128, 128, 768, 768, 128),
    "384, ragged and short": ([3] * 64, 256, 1408, 704, 128),
    "384 of the down projection": ([20] * 96, 2048, 128, 96, 512),
    "half a round beyond two": ([3] * 128, 128, 1280, 768, 128),
    # half of the last column tile of 512 and of 256 columns: 8 of the 44 items that are cut have no second half
    "ragged down projection": ([20] * 60, 2304, 128, 60, 336),
    "ragged down projection, narrow tiles": ([20] * 60, 1152, 128, 60, 336),
    "beyond 384": ([3] * 97, 128, 1024, 388, 97),
    "half a round": ([5] * 64 + [0] * 64, 1024, 512, 256, 256),
    "more than half a round": ([4] * 43, 2048, 768, 129, 432),
    "full tiles, deep prefetch": ([1030] * 8, 1024, 2048, 640, 448),
    # a ragged column tile (128 of 256) has no second half: 8 of the 16 items that are cut; the narrowest down tiles stay whole
    "ragged columns": ([130] * 44, 640, 1408, 536, 440),
}


@pytest.mark.parametrize("name", LAUNCHES)
def test_items_of_a_short_last_round_run_as_halves(name):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_03495_amd import binding as B, layer as Lm
    B.load_library()
    rows, d, I, up, down = LAUNCHES[name]
    N, T = len(rows), sum(rows)
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
    print(f"short last round {name} d={d} I={I} T={T}", flush=True)
    B.moe_debug_set_trace(records)
    B.moe_expert_ffn(s, Lm.to_device_bf16(h), dev(perm), dev(offsets), dev(np.array(rows, np.int32)), *packed, None, y, B.alloc_workspace(s))
    torch.cuda.synchronize()
    B.moe_debug_set_trace(None)
    t = records.cpu().numpy().reshape(2, B.TRACE_MAX_BLOCKS, 8)
    assert [int((t[i, :, 7] == 1).sum()) for i in (0, 1)] == [up, down]
    bits = Lm.from_device_bf16(y)
    assert not np.any(bits == SENTINEL), "an element was not written"
    last = [o + n - 1 for o, n in zip(offsets, rows) if n]
    pick = np.array(sorted(set(last) | set(range(0, T, max(1, T // 100)))))
    ref = oracle.expert_rows(h, topk_idx, w1, w3, w2, np.ones(N, np.uint8), tokens=perm[pick].astype(np.int32))[:, 0]
    got = wl.bf16_bits_to_f32(bits[pick])
    worst = max(rel_err(got[i], ref[i]) for i in range(len(pick)))
    assert worst <= OUT_TOL, worst
