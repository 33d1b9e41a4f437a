"""Token tiles beyond 128 tokens, which every wave of the tiled projections ranks from counts and mask (moe_rank_tiles):
hand-made tables with experts on both sides of lane 63 / 64, rows at every edge of the three tile heights (96, 112, 128),
empty and masked experts first, last and in runs, and a single working expert.  Every row against the oracle."""
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
