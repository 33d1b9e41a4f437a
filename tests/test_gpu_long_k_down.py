"""Which kernel takes the down projection over a long inner size, and what it computes there.  Both kernels are launched and
the rows of the experts at work decide on the device (wide_faster): tables by hand on either side, with the kernel read off
the block timeline (its items hold up to 256 rows, those of the tiled kernel at most 128), every row against a float64
product of the same activations."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

SENTINEL = 0x5A5A


@pytest.fixture(scope="module")
def binding():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_03495_amd import binding as B
    B.load_library()
    return B


def down(B, d, I, k, rows, off=(), seed=0):
    """The down stage alone on activations and weights N(0, 1) and N(0, 1/I).  Returns the timeline's records (expert, rows,
    column tile) and asserts that every row of the experts at work is right and no other is written."""
    N, R = len(rows), sum(rows)
    assert R % k == 0
    T = R // k
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    s = B.shape(T, d, N, k, I)
    ws = B.alloc_workspace(s)
    first = (-ws.data_ptr()) % 256
    act = ws[first:first + 2 * R * I].view(torch.bfloat16).view(R, I)      # the activations open the workspace
    act.normal_(0.0, 1.0, generator=gen)
    w2 = torch.empty((N, d, I), dtype=torch.bfloat16, device="cuda")
    for e in range(N):
        w2[e].normal_(0.0, I ** -0.5, generator=gen)
    packed = B.moe_pack_weights(w2)
    mask = np.ones(N, np.uint8)
    mask[list(off)] = 0
    offsets = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    y = torch.empty((R, d), dtype=torch.bfloat16, device="cuda")
    y.view(torch.int16).fill_(SENTINEL)
    h = torch.zeros((T, d), dtype=torch.bfloat16, device="cuda")
    records = torch.zeros(2 * B.TRACE_MAX_BLOCKS * 8, dtype=torch.int64, device="cuda")
    args = (s, h, dev(np.arange(R, dtype=np.int32)), dev(offsets), dev(np.array(rows, np.int32)), packed, packed, packed, dev(mask), y, ws,
            B.STAGE_DOWN)
    print(f"long inner size d={d} I={I} k={k} rows={list(rows)} off={list(off)}", flush=True)
    B.moe_debug_set_trace(records)
    B.moe_expert_ffn_stage(*args)
    torch.cuda.synchronize()
    B.moe_debug_set_trace(None)
    first_y = y.clone()
    B.moe_expert_ffn_stage(*args)
    torch.cuda.synchronize()
    assert torch.equal(y.view(torch.int16), first_y.view(torch.int16)), "two runs differ"
    for e in range(N):
        a, b = int(offsets[e]), int(offsets[e + 1])
        if not mask[e]:
            assert bool((y.view(torch.int16)[a:b] == SENTINEL).all()), "a row of a masked-off expert was written"
            continue
        # the result rounded to bf16 (2^-9, taken twice), and fp32 sums of I / 32 steps, 32 products each, up to 16 pieces
        for c in range(a, b, 512):
            x, w = act[c:min(b, c + 512)].double(), w2[e].double()
            ref, size = x @ w.T, x.abs() @ w.abs().T
            bound = ref.abs() * 2.0 ** -8 + size * ((I // 32 + 32 + 16) * 2.0 ** -24)
            assert bool(((y[c:min(b, c + 512)].double() - ref).abs() <= bound).all()), (e, c)
    t = records.cpu().numpy().reshape(2, B.TRACE_MAX_BLOCKS, 8)[1]
    return t[t[:, 7] == 1][:, 4:7]


# d, I, k, rows, experts off, whether the long-K kernel works; beside each the down projection on the tiled and on that kernel
CHOICE = [
    (4096, 14336, 2, [1441, 190, 398, 889, 618, 286, 140, 134], [6, 7], True),                   # 617 and 423 us
    (4096, 14336, 2, [1540, 379, 283, 550, 165, 954, 126, 99], [5, 7], True),                    # 375 and 331
    (4096, 14336, 2, [436, 451, 436, 436, 436, 445, 436, 436], [0, 2, 3, 4, 6, 7], True),        # 196 and 114
    (1024, 11008, 1, [5193, 2428], [], True),                                                    # 227 and 156
    (4096, 14336, 2, [280, 249, 274, 266, 248, 262, 255, 254], [1, 4], False),                   # 230 and 354
    (4096, 14336, 2, [200, 842, 484, 120, 303, 225, 80, 40], [0, 3, 6, 7], False),               # 223 and 277
    (4096, 14336, 2, [600, 665, 656, 619, 612, 611, 596, 583], [0, 7], False),                   # 374 and 442
    (4096, 8192, 4, [320] * 32, [], False),                                                      # 686 and 815
    (2048, 8192, 4, [1331, 1033, 792, 598, 437, 375, 271, 250, 197, 194, 143, 133, 120, 101, 94, 75], list(range(4, 16)), False),   # 117 and 167
]


@pytest.mark.parametrize("d,I,k,rows,off,wide", CHOICE)
def test_the_faster_kernel_takes_the_down_projection(binding, d, I, k, rows, off, wide):
    rec = down(binding, d, I, k, rows, off)
    assert bool((rec[:, 1] > 128).any()) == wide
    assert set(rec[:, 0].tolist()) == {e for e in range(len(rows)) if e not in off}


# d (odd multiples of 128: the last column tile is half a tile), I (8320 / 128 = 65: pieces of uneven length), rows, experts
# off, items that run whole, items that are cut, their pieces.  Rows at the edges of every body (32, 64, 128, 192, 256 rows).
PLANS = [
    (3968, 8192, [1, 32, 33, 1086, 63, 64, 65, 127, 128, 129, 191, 192, 193, 255, 256, 257], [3], 256, 0, 1),    # one exact round
    (3968, 8320, [1, 33, 64, 942, 65, 127, 129, 191, 193, 255, 256, 257, 512], [3], 224, 0, 1),                  # too many to be cut
    (3968, 8192, [1, 33, 64, 65, 127, 129, 191, 193, 255, 256, 257, 512, 700, 513], [], 256, 64, 4),
    (4224, 8320, [1, 33, 700, 642, 64, 65, 127, 129, 191, 193, 255, 256, 257, 512, 600], [3], 256, 84, 3),
    (1920, 8320, [1, 256, 33, 3629, 257, 129, 65], [3], 0, 56, 4),
    (1920, 14336, [1, 255, 513, 3568, 33], [3], 0, 48, 5),
]


@pytest.mark.parametrize("d,I,rows,off,whole,cut,pieces", PLANS)
def test_row_edges_in_whole_and_in_cut_items(binding, d, I, rows, off, whole, cut, pieces):
    rec = down(binding, d, I, 1, rows, off)
    assert bool((rec[:, 1] > 128).any()), "the case must take the long-K kernel"
    assert len(rec) == whole + cut * pieces
    # every block took an item of its own or, of a cut one, a piece
    want = [(e, min(256, n - m), c) for e, n in enumerate(rows) if e not in off for c in range((d + 255) // 256) for m in range(0, n, 256)]
    got = sorted(map(tuple, rec.tolist()))
    assert got == sorted(want[:whole] + want[whole:] * pieces)


def test_a_replayed_graph_takes_the_kernel_that_its_mask_asks_for(binding):
    # one captured down stage, replayed with a mask that leaves six experts (the tiled kernel) and one that leaves two (the long-K
    # kernel): nothing of the choice stays from one replay to the next
    B = binding
    d, I, k, rows = 4096, 14336, 2, [280, 249, 274, 266, 248, 262, 255, 254]
    N, R = len(rows), sum(rows)
    gen = torch.Generator(device="cuda").manual_seed(7)
    s = B.shape(R // k, d, N, k, I)
    ws = B.alloc_workspace(s)
    first = (-ws.data_ptr()) % 256
    ws[first:first + 2 * R * I].view(torch.bfloat16).normal_(0.0, 1.0, generator=gen)
    w2 = torch.empty((N, d, I), dtype=torch.bfloat16, device="cuda")
    for e in range(N):
        w2[e].normal_(0.0, I ** -0.5, generator=gen)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    offsets = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    mask = torch.zeros(N, dtype=torch.uint8, device="cuda")
    y = torch.empty((R, d), dtype=torch.bfloat16, device="cuda")
    args = (s, torch.zeros((R // k, d), dtype=torch.bfloat16, device="cuda"), dev(np.arange(R, dtype=np.int32)), dev(offsets),
            dev(np.array(rows, np.int32)), w2, w2, w2, mask, y, ws, B.STAGE_DOWN)
    masks = {off: dev(np.array([e not in off for e in range(N)], np.uint8)) for off in ((1, 4), (1, 3, 4, 5, 6, 7), tuple(range(N)))}
    records = torch.zeros(2 * B.TRACE_MAX_BLOCKS * 8, dtype=torch.int64, device="cuda")
    want, most_rows = {}, {}
    for off, m in masks.items():
        mask.copy_(m)
        y.view(torch.int16).fill_(SENTINEL)
        records.zero_()
        B.moe_debug_set_trace(records)
        B.moe_expert_ffn_stage(*args)
        torch.cuda.synchronize()
        B.moe_debug_set_trace(None)
        want[off] = y.clone()
        t = records.view(2, B.TRACE_MAX_BLOCKS, 8)[1]
        most_rows[off] = int(t[:, 5].max())
    assert [most_rows[off] > 128 for off in masks] == [False, True, False] and most_rows[tuple(range(N))] == 0
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        B.moe_expert_ffn_stage(*args)
    torch.cuda.current_stream().wait_stream(side)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        B.moe_expert_ffn_stage(*args)
    for off in list(masks) * 3 + [(1, 4), (1, 4)]:
        mask.copy_(masks[off])
        y.view(torch.int16).fill_(SENTINEL)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y.view(torch.int16), want[off].view(torch.int16)), off
