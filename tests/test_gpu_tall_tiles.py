"""The up projection's tiles of up to 256 rows at half width (taken where every expert has at most 256 rows, one more than 128, such
items number 192 to 256, the whole items more than 128 and the hidden size is 2048 or more), and the launches just beside those lines,
against a float32 product."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

# rows, d, I, masked-off experts, blocks of the up launch (128 columns of every expert each where the tall tiles are taken)
CASES = {
    "every height": ([129, 1, 16, 17, 33, 64, 65, 96, 97, 128, 144, 145, 160, 161, 192, 193, 208, 256, 255, 2], 2176, 1280, (), 200),
    "all but two experts off": ([140, 30, 256, 256], 2048, 12288, (2, 3), 192),
    "exactly one round": ([200, 7], 2048, 16384, (), 256),
    "ragged inner columns": ([130] * 20, 2048, 1408, (), 220),
    "a whole item beyond half a round": ([129] + [40] * 63, 2048, 512, (), 256),
    "half a round of whole items": ([129, 40, 40], 2048, 8192, (), None),
    "a narrow layer": ([200, 7], 1920, 16384, (), None),
    "a tile short of the line": ([200, 5], 2048, 12160, (), None),
    "more than one round": ([200, 5, 9], 2048, 12288, (), None),
    "no expert beyond 128 rows": ([128, 100], 2048, 16384, (), None),
    "an expert beyond 256 rows": ([257, 3], 2048, 16384, (), None),
}


@pytest.mark.parametrize("name", CASES)
def test_tall_tiles_of_the_up_projection(name):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_03495_amd import binding as B
    B.load_library()
    rows, d, I, off, blocks = CASES[name]
    N, T = len(rows), sum(rows)
    gen = torch.Generator(device="cuda").manual_seed(T)
    w1, w3 = ((torch.randn(N, I, d, generator=gen, device="cuda") * d ** -0.5).bfloat16() for _ in range(2))
    h = torch.randn(T, d, generator=gen, device="cuda").bfloat16()
    perm = torch.randperm(T, generator=gen, device="cuda").int()
    offsets = torch.from_numpy(np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)).cuda()
    counts = torch.tensor(rows, dtype=torch.int32, device="cuda")
    mask = torch.ones(N, dtype=torch.uint8, device="cuda")
    mask[list(off)] = 0
    s = B.shape(T, d, N, 1, I)
    ws = B.alloc_workspace(s)
    act = ws[: T * I * 2].view(torch.bfloat16).view(T, I)          # the workspace begins with the activations
    act.view(torch.int16).fill_(0x7B7B)
    records = torch.zeros(2 * B.TRACE_MAX_BLOCKS * 8, dtype=torch.int64, device="cuda")
    y = torch.empty(T, d, dtype=torch.bfloat16, device="cuda")
    print(f"up projection {name} d={d} I={I} T={T}", flush=True)
    p1, p3 = B.moe_pack_weights(w1), B.moe_pack_weights(w3)
    B.moe_debug_set_trace(records)
    B.moe_expert_ffn_stage(s, h, perm, offsets, counts, p1, p3, p1, mask, y, ws, B.STAGE_UP)
    torch.cuda.synchronize()
    B.moe_debug_set_trace(None)
    ran = records.cpu().numpy().reshape(2, B.TRACE_MAX_BLOCKS, 8)[0]
    ran = ran[ran[:, 7] == 1]
    assert len(ran) > 0
    if blocks is None:
        assert ran[:, 5].max() <= 128
    else:
        assert len(ran) == blocks and ran[:, 5].max() == max(r for e, r in enumerate(rows) if e not in off)
    at = 0
    for e, r in enumerate(rows):
        got = act[at:at + r]
        if e in off:
            assert (got.view(torch.int16) == 0x7B7B).all()
        else:
            x = h[perm[at:at + r].long()].float()
            ref = torch.nn.functional.silu(x @ w1[e].float().T) * (x @ w3[e].float().T)
            # one rounding to bf16 (2^-9) and fp32 sums of d products in another order
            assert (got.float() - ref).abs().max() <= 2 ** -8 * ref.abs().max(), (name, e)
        at += r
