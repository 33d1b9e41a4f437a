"""Decode-sized down projection with an inner size of at most 2048 on either side of the line between the weight-streaming
kernel and the tiled one (256 items of 128 columns, 160 at I = 128): whole layers against the oracle, every row compared, with shares of K
per wave that are short, uneven (I = 1408: 11 steps, I = 128: 1) and long."""
import pytest

from helpers import run_layer
from paper_2602_03495_amd import workloads as wl

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("I", [128, 384, 1408, 2048, 2176])
@pytest.mark.parametrize("d,k,T", [(2048, 8, 1), (2048, 8, 2), (2048, 5, 3), (2176, 5, 3), (256, 8, 15), (256, 8, 16), (384, 1, 1)])
def test_down_projection_on_both_sides_of_the_line(I, d, k, T):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_03495_amd import binding as B, layer as Lm
    B.load_library()
    cfg = wl.scaled(wl.CONFIGS["tiny"], d=d, I=I, N=16, k=k)
    print(f"short down projection d={d} I={I} k={k} T={T}", flush=True)
    run_layer(B, Lm, cfg, T, [None, wl.mask_random(cfg, 9)], B.FFN_SKINNY, draw=T)


@pytest.mark.parametrize("I,d,tiled", [(128, 2432, False), (128, 2560, True), (256, 2560, False), (256, 3968, False), (256, 4096, True)])
def test_line_by_inner_size(I, d, tiled):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_03495_amd import binding as B, layer as Lm
    B.load_library()
    cfg = wl.scaled(wl.CONFIGS["tiny"], d=d, I=I, N=8, k=8)
    print(f"line of the short down projection I={I} d={d}", flush=True)
    run_layer(B, Lm, cfg, 1, [None, wl.mask_random(cfg, 3)], B.FFN_SKINNY)
    s = B.shape(1, d, 8, 8, I)
    dev = lambda *v: torch.tensor(v, dtype=torch.int32, device="cuda")
    w = torch.zeros(8 * I * d, dtype=torch.bfloat16, device="cuda")
    h, y = torch.zeros(1, d, dtype=torch.bfloat16, device="cuda"), torch.empty(8, d, dtype=torch.bfloat16, device="cuda")
    records = torch.zeros(2 * B.TRACE_MAX_BLOCKS * 8, dtype=torch.int64, device="cuda")
    B.moe_debug_set_trace(records)
    B.moe_expert_ffn(s, h, dev(*range(8)), dev(*range(9)), dev(*[1] * 8), w, w, w, None, y, B.alloc_workspace(s))
    torch.cuda.synchronize()
    B.moe_debug_set_trace(None)
    ran = int((records.reshape(2, B.TRACE_MAX_BLOCKS, 8)[1, :, 7] == 1).sum())
    assert ran == (8 * d // 128 if tiled else 0)
