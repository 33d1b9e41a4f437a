"""Whole FFN over a long inner size (8192 or more, 48 MB of activations or more) with few output columns, where the tiled down
projection works alone, against the oracle, with routing tables made by hand so that every row tile edge occurs: experts
with 1 row, one below, at and above 32, 64, 128, 192 and 256 rows, several tiles, and none.  The kernel for long inner sizes
(ffn_wide.h) is tested in test_gpu_long_k_down.py."""
import numpy as np
import pytest

import oracle
from paper_2602_03495_amd import workloads as wl
from helpers import OUT_TOL, SENTINEL, rel_err

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# rows per expert; I / 32 an odd multiple of 4 in the second case
CASES = [(128, 8192, [1, 31, 32, 33, 63, 64, 65, 127, 128, 129, 191, 192, 193, 255, 256, 257, 0, 1100], []),
         (384, 8320, [640, 1, 250, 513, 300, 1200, 0, 131], [0, 4])]


@pytest.mark.parametrize("d,I,rows,off", CASES)
def test_long_inner_size_down_projection_matches_the_oracle(d, I, rows, off):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_03495_amd import binding as B, layer as Lm
    B.load_library()
    N, T = len(rows), sum(rows)
    assert T * I * 2 >= 48 << 20, "a long inner size with many activations"
    cfg = wl.scaled(wl.CONFIGS["tiny"], d=d, I=I, N=N, k=1)
    h, (w1, w3, w2) = wl.hidden_states(cfg, T), wl.expert_weights(cfg)
    rng = np.random.default_rng(d)
    perm = rng.permutation(T).astype(np.int32)                  # expert-grouped rows -> tokens, as any routing could give
    topk_idx = np.empty((T, 1), np.int32)
    topk_idx[perm, 0] = np.repeat(np.arange(N), rows)
    mask = np.ones(N, np.uint8)
    mask[off] = 0
    counts, offsets = np.array(rows, np.int32), np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)

    s = B.shape(T, d, N, 1, I)
    ws = B.alloc_workspace(s)
    y = torch.empty((T, d), dtype=torch.bfloat16, device="cuda")
    y.view(torch.int16).fill_(SENTINEL)
    dev = lambda a: torch.from_numpy(a).cuda()
    packed = [B.moe_pack_weights(Lm.to_device_bf16(w)) for w in (w1, w3, w2)]
    print(f"long inner size d={d} I={I} rows={rows} off={off}", flush=True)
    B.moe_expert_ffn(s, Lm.to_device_bf16(h), dev(perm), dev(offsets), dev(counts), *packed, dev(mask), y, ws)
    torch.cuda.synchronize()
    bits = Lm.from_device_bf16(y)
    on = np.repeat(mask.astype(bool), rows)
    assert np.all(bits[~on] == SENTINEL), "a row of a masked-off expert was written"
    assert not np.any(np.all(bits[on] == SENTINEL, axis=1)), "a row of a masked-on expert was not written"

    # all rows of the short experts, the last 40 and some other rows of the long ones
    pick = [offsets[e] + j for e in range(N) if mask[e] for j in range(rows[e]) if rows[e] <= 65 or j >= rows[e] - 40 or j % 37 == 0]
    ref = oracle.expert_rows(h, topk_idx, w1, w3, w2, mask, tokens=perm[pick].astype(np.int32))[:, 0]
    got = wl.bf16_bits_to_f32(bits[pick])
    errs = [rel_err(got[i], ref[i]) for i in range(len(pick))]
    print(f"  {len(pick)} rows, worst {max(errs):.2e}", flush=True)
    assert max(errs) <= OUT_TOL, (pick[int(np.argmax(errs))], max(errs))
