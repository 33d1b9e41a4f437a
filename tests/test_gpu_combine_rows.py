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
