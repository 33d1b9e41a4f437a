"""Decode-sized down projection with an inner size of at most 2048 on either side of the line between the weight-streaming
kernel and the tiled one (256 items of 128 columns): whole layers against the oracle, every row compared, with shares of K
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
