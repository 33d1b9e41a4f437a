"""Counts, offsets and the stable permutation of moe_route at the edges of the permutation kernel's register loads (1, 4 and
16 selections per thread of 1024, and a second load), and the p largest predicted workloads with ties; all of it whole
numbers, compared exactly with numpy on the GPU's own selections."""
import numpy as np
import pytest

import oracle
from paper_2602_03495_amd import workloads as wl

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_03495_amd import binding, layer
    binding.load_library()
    return binding, layer


@pytest.mark.parametrize("N,k,T", [(128, 1, 17), (128, 1, 1023), (128, 1, 1024), (1, 1, 1025), (37, 3, 1365), (128, 8, 512),
                                   (64, 1, 4097), (8, 2, 8192), (60, 1, 16385), (128, 8, 4097)])
def test_tables_are_the_stable_grouping_of_the_selections(gpu, N, k, T):
    B, Lm = gpu
    print(f"tables N={N} k={k} T={T} rows={T * k}", flush=True)
    cfg = wl.scaled(wl.CONFIGS["qwen3"], d=128, I=128)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(N * 100003 + T)
    h = torch.randn(T, cfg.d, generator=gen, device="cuda").bfloat16()
    W = (torch.randn(N, cfg.d, generator=gen, device="cuda") * cfg.d ** -0.5).bfloat16()
    b = -torch.arange(N, device="cuda").float().add(1).log()          # skewed: the last experts get few rows or none
    s = B.shape(T, cfg.d, N, k, cfg.I)
    ws = B.alloc_workspace(s)
    r = B.alloc_routing(s)
    B.moe_route(s, h, W, b, cfg.norm_mode, r, ws)
    p = min(N, 9)
    pc, top = torch.empty(N, dtype=torch.int32, device="cuda"), torch.empty(p, dtype=torch.int32, device="cuda")
    B.moe_predict_workload(s, h, torch.zeros(cfg.d, device="cuda"), W, b, p, pc, top, ws)
    torch.cuda.synchronize()
    idx = r.topk_idx.cpu().numpy().reshape(-1)
    counts = np.bincount(idx, minlength=N)
    perm = np.argsort(idx, kind="stable")
    assert np.array_equal(r.counts.cpu().numpy(), counts)
    assert np.array_equal(r.offsets.cpu().numpy(), np.concatenate([[0], np.cumsum(counts)]))
    assert np.array_equal(r.perm.cpu().numpy(), perm)
    assert np.array_equal(r.inv_perm.cpu().numpy()[perm], np.arange(T * k))
    assert np.array_equal(pc.cpu().numpy(), counts)
    assert np.array_equal(top.cpu().numpy(), oracle.top_p(counts, p))


@pytest.mark.parametrize("N,T", [(128, 3), (128, 200), (70, 16)])
def test_largest_workloads_with_ties_and_every_expert_asked_for(gpu, N, T):
    # a zero gate: the first k experts get every token, the others none; p = N orders all of them
    B, Lm = gpu
    d, k = 128, 2
    s = B.shape(T, d, N, k, 128)
    z = lambda *n: torch.zeros(*n, device="cuda")
    pc, top = (torch.full((N,), -1, dtype=torch.int32, device="cuda") for _ in range(2))
    B.moe_predict_workload(s, z(T, d).bfloat16(), z(d), z(N, d).bfloat16(), None, N, pc, top, B.alloc_workspace(s))
    torch.cuda.synchronize()
    assert pc.tolist() == [T] * k + [0] * (N - k)
    assert top.tolist() == list(range(N))
