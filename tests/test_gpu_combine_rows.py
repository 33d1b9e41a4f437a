"""combine_kernel with every number of working slots (1 to 8 selections, 0 to 3 shared experts, masks that leave any subset
of the slots) at widths below, at and beyond a wave's 512 and a block's 2048 columns.  Rows of masked-off experts hold NaN
and must not be read into a sum."""
import numpy as np
import pytest

from paper_2602_03495_amd import workloads as wl

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("S", [0, 1, 2, 3])
@pytest.mark.parametrize("d", [128, 512, 640, 2048, 2176, 4096, 8192])
def test_any_number_of_working_slots(d, S):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_03495_amd import binding as B
    B.load_library()
    print(f"combine d={d} S={S}", flush=True)
    N, T = 16, 33
    for k in range(1, 9):
        rng = np.random.default_rng(1000 * d + 10 * S + k)
        idx = np.stack([rng.permutation(N)[:k] for _ in range(T)]).astype(np.int32)
        inv = rng.permutation(T * k).astype(np.int32).reshape(T, k)
        w, scale = rng.random((T, k), dtype=np.float32), rng.random(T, dtype=np.float32)
        mask = (rng.random(N) < 0.6).astype(np.uint8)
        y = torch.from_numpy(rng.standard_normal((T * k, d), dtype=np.float32)).bfloat16()
        on = mask[idx] != 0
        y[inv[~on]] = float("nan")
        sy = torch.from_numpy(rng.standard_normal((max(S, 1), T, d), dtype=np.float32)).bfloat16()
        out = torch.empty((T, d), dtype=torch.bfloat16, device="cuda")
        dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
        s = B.shape(T, d, N, k, 128)
        B.moe_combine(s, y.cuda(), dev(idx), dev(w), dev(inv), dev(mask), sy.cuda() if S else None, S, dev(scale) if S else None, out)
        torch.cuda.synchronize()
        terms = np.where(on[:, :, None], w[:, :, None] * np.nan_to_num(y.double().numpy()[inv]), 0.0)
        if S:
            terms = np.concatenate([terms, (scale[:, None] * sy.double().numpy()).transpose(1, 0, 2)], axis=1)
        ref = terms.sum(axis=1)
        # one rounding to bf16 (2^-9 of the value), up to 11 fp32 sums (2^-24 each of the absolute sum)
        bound = 2.0 ** -8 * np.abs(ref) + 16 * 2.0 ** -24 * np.abs(terms).sum(axis=1)
        assert np.all(np.abs(out.double().cpu().numpy() - ref) <= bound), k


@pytest.mark.parametrize("d", [1024, 1152, 2048, 2176, 8192])
@pytest.mark.parametrize("k", [1, 2, 3, 4])
@pytest.mark.parametrize("mask_of", ["none", "half", "all off"])
@pytest.mark.parametrize("n_shared", [0, 1, 3])
def test_many_tokens_give_the_bits_of_few(d, k, mask_of, n_shared):
    # more than 1024 tokens with up to 3 slots run on a kernel of their own; the sums are the same, in the same order
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_03495_amd import binding as B
    T, N = 1025, 8
    gen = torch.Generator(device="cuda").manual_seed(d + k)
    idx = torch.rand(T, N, generator=gen, device="cuda").topk(k, dim=1).indices.int().contiguous()
    w = torch.rand(T, k, generator=gen, device="cuda")
    inv = torch.randperm(T * k, generator=gen, device="cuda").int()
    y = torch.randn(T * k, d, generator=gen, device="cuda").bfloat16()
    shared = torch.randn(max(1, n_shared), T, d, generator=gen, device="cuda").bfloat16() if n_shared else None
    scale = torch.rand(T, generator=gen, device="cuda") if n_shared == 1 else None
    mask = {"none": None, "half": torch.arange(N, device="cuda", dtype=torch.uint8) % 2, "all off": torch.zeros(N, device="cuda", dtype=torch.uint8)}[mask_of]

    def combine(a, b):
        out = torch.full((b - a, d), float("nan"), dtype=torch.bfloat16, device="cuda")
        sy = None if shared is None else shared[:, a:b].contiguous()
        return B.moe_combine(B.shape(b - a, d, N, k, 128), y, idx[a:b].contiguous(), w[a:b].contiguous(), inv[a * k:b * k].contiguous(), mask,
                             sy, n_shared, None if scale is None else scale[a:b].contiguous(), out)

    whole, parts = combine(0, T), torch.cat([combine(0, 512), combine(512, 1024), combine(1024, T)])
    torch.cuda.synchronize()
    assert torch.equal(whole.view(torch.int16), parts.view(torch.int16))
    # fp32 sums of at most 7 rows, rounded to bf16 once
    on = torch.ones(T, k, dtype=torch.bool, device="cuda") if mask is None else mask[idx.long()].bool()
    ref = (y[inv.long()].view(T, k, d).double() * (w * on).double()[:, :, None]).sum(1)
    if shared is not None:
        ref += (shared.double() * (1.0 if scale is None else scale.double()[None, :, None])).sum(0)
    assert bool(((whole.double() - ref).abs() <= ref.abs() * 2.0 ** -8 + 1e-5).all())
