"""The gate product at the edges of its tiles: blocks that walk several token tiles (with a residual vector 13 tokens each), runs of
K shorter than, equal to and longer than the steps a wave keeps in registers, expert slices that are not full.  Routing is compared
with the oracle under the rules of helpers.py and the prediction through its counts; a logit is a function of its token and
expert alone, so a token routed by itself gets the same bits as inside the batch."""
import ctypes

import numpy as np
import pytest

import oracle
from helpers import check_routing, exempt_tokens
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


@pytest.mark.parametrize("d,N,k,T", [(128, 128, 8, 1000), (640, 60, 4, 417), (2048, 49, 4, 833), (2176, 64, 6, 53), (4096, 8, 2, 300),
                                     (4096, 70, 8, 27), (512, 33, 3, 530), (1024, 65, 5, 16), (1152, 64, 6, 29), (8192, 128, 8, 40), (8192, 17, 2, 14), (2048, 128, 8, 16), (4096, 8, 2, 13)])
def test_route_and_predict_at_the_edges_of_the_gate_tiles(gpu, d, N, k, T):
    B, Lm = gpu
    print(f"gate tiles d={d} N={N} k={k} T={T}", flush=True)
    cfg = wl.scaled(wl.CONFIGS["qwen3"], d=d, N=N, k=k, I=128)
    h = wl.hidden_states(cfg, T)
    W0, b0, W1, b1 = wl.gate_weights(cfg, 0), wl.gate_bias(cfg, 0), wl.gate_weights(cfg, 1), wl.gate_bias(cfg, 1)
    rv = wl.layer_drift(cfg)
    assert np.any(rv.view(np.uint32) & 0xFFFF)           # not bf16 numbers: all three parts of the split count
    up = lambda a: Lm.to_device_bf16(a)
    hd, W0d, W1d, b0d, b1d, rvd = up(h), up(W0), up(W1), *(torch.from_numpy(a).cuda() for a in (b0, b1, rv))
    s, p = B.shape(T, d, N, k, cfg.I), min(N, 5)
    ws, r = B.alloc_workspace(s), B.alloc_routing(s)
    pc, top = torch.empty(N, dtype=torch.int32, device="cuda"), torch.empty(p, dtype=torch.int32, device="cuda")
    B.moe_route_predict(s, hd, W0d, b0d, cfg.norm_mode, r, rvd, W1d, b1d, p, pc, top, ws)
    torch.cuda.synchronize()
    host = lambda t: t.cpu().numpy()
    lg, o_idx, o_w, o_counts = oracle.route(h, W0, b0, k, cfg.norm_mode)
    idx, w = host(r.topk_idx), host(r.topk_w)
    check_routing(lg, o_idx, o_w, o_counts, idx, w, host(r.counts), host(r.offsets), host(r.perm), host(r.inv_perm), N, k)
    plg, _, p_counts, _ = oracle.predict_workload(h, rv, W1, b1, k, p)
    got = host(pc)
    assert got.sum() == T * k
    assert int(np.abs(got.astype(np.int64) - p_counts).sum()) <= 2 * int(exempt_tokens(plg, k).sum())
    assert np.array_equal(host(top), oracle.top_p(got, p))

    s1 = B.shape(1, d, N, k, cfg.I)
    for workspace in (B.alloc_workspace(s1), None):      # the product spread over blocks, and one block for all of it
        r1 = B.alloc_routing(s1)
        for t in sorted({0, 12, 13, T // 2, T - 1} & set(range(T))):
            B.moe_route(s1, hd[t:t + 1], W0d, b0d, cfg.norm_mode, r1, workspace)
            torch.cuda.synchronize()
            assert np.array_equal(host(r1.topk_idx)[0], idx[t]) and np.array_equal(host(r1.topk_w)[0], w[t]), t


def test_an_infinite_residual_element_makes_infinite_logits_not_nan(gpu):
    # its lower parts are zero: an infinity less itself would make every logit NaN
    B, _ = gpu
    d, N, k, T = 256, 8, 2, 21
    W = torch.zeros(N, d, device="cuda")
    W[0::2, 7], W[1::2, 7] = 1.0, -1.0
    rv = torch.zeros(d, device="cuda")
    rv[7], rv[8] = float("inf"), 3.4e38                 # rv[8]: beyond the largest bf16 number, times zero
    s = B.shape(T, d, N, k, 128)
    pc, top = torch.empty(N, dtype=torch.int32, device="cuda"), torch.empty(2, dtype=torch.int32, device="cuda")
    B.moe_predict_workload(s, torch.ones(T, d, device="cuda").bfloat16(), rv, W.bfloat16(), None, 2, pc, top, B.alloc_workspace(s))
    torch.cuda.synchronize()
    assert pc.tolist() == [T, 0, T, 0, 0, 0, 0, 0] and top.tolist() == [0, 2]


@pytest.mark.parametrize("T,N", [(1, 8), (13, 16), (16, 8), (16, 40), (21, 8), (21, 64)])
def test_an_infinite_gate_weight_makes_an_infinite_logit_not_nan(gpu, T, N):
    # the residual's lower parts are zero where it is a bf16 number: times an infinity they are NaN, and such a logit comes last
    B, _ = gpu
    d, k = 256, 2
    W = torch.zeros(N, d, device="cuda")
    W[3, 7], W[5, 7] = float("inf"), float("-inf")
    rv = torch.zeros(d, device="cuda")
    rv[7] = 1.0
    s = B.shape(T, d, N, k, 128)
    pc, top = torch.empty(N, dtype=torch.int32, device="cuda"), torch.empty(2, dtype=torch.int32, device="cuda")
    h = torch.zeros(T, d, device="cuda")
    h[:, 7] = 1.0                                        # zero times infinity in the token's own product is NaN in any order
    B.moe_predict_workload(s, h.bfloat16(), rv, W.bfloat16(), None, 2, pc, top, B.alloc_workspace(s))
    torch.cuda.synchronize()
    assert pc.tolist() == [T, 0, 0, T] + [0] * (N - 4) and top.tolist() == [0, 3]


def _kernels(call):
    """Kernel launches of a call: the nodes of a graph it is captured into."""
    call()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        call()
    with open("/proc/self/maps") as maps:
        hip = ctypes.CDLL(next(line.split()[-1] for line in maps if "libamdhip64" in line))
    n = ctypes.c_size_t(0)
    assert hip.hipGraphGetNodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(n)) == 0
    return n.value


@pytest.mark.parametrize("d,N,k", [(128, 8, 2), (4096, 8, 2), (8192, 16, 8), (2176, 3, 3)])
def test_decode_prediction_of_few_experts(gpu, d, N, k):
    """Up to 16 experts and 16 tokens: one launch, also where tokens and the residual's rows are more than the 16 of a tile, and with
    every token's prediction as it is alone and in a batch of several tiles."""
    B, Lm = gpu
    cfg = wl.scaled(wl.CONFIGS["qwen3"], d=d, N=N, k=k, I=128)
    dev = lambda a: torch.from_numpy(a).cuda()
    h, W0, W1 = (Lm.to_device_bf16(a) for a in (wl.hidden_states(cfg, 45), wl.gate_weights(cfg, 0), wl.gate_weights(cfg, 1)))
    b0, b1, rv = dev(wl.gate_bias(cfg, 0)), dev(wl.gate_bias(cfg, 1)), dev(wl.layer_drift(cfg))

    def predict(T, first, fused):
        s, x = B.shape(T, d, N, k, 128), h[first:first + T].contiguous()
        ws, r, pc, top = B.alloc_workspace(s), B.alloc_routing(s), torch.full((N,), -1, dtype=torch.int32, device="cuda"), \
            torch.full((N,), -1, dtype=torch.int32, device="cuda")
        call = (lambda: B.moe_route_predict(s, x, W0, b0, 1, r, rv, W1, b1, N, pc, top, ws)) if fused else \
            (lambda: B.moe_predict_workload(s, x, rv, W1, b1, N, pc, top, ws))
        n = _kernels(call)
        counts = pc.cpu().numpy()
        assert np.array_equal(top.cpu().numpy(), oracle.top_p(counts, N))
        return counts, n

    alone = [predict(1, t, t % 2 == 0)[0] for t in range(45)]
    for T in (1, 12, 13, 14, 16):
        for fused in (False, True):
            print(f"few experts d={d} N={N} T={T} fused={fused}", flush=True)
            counts, n = predict(T, 0, fused)
            assert n == 1, n
            assert np.array_equal(counts, sum(alone[:T]))
    assert np.array_equal(predict(45, 0, False)[0], sum(alone))


@pytest.mark.parametrize("d,N,k,T", [(128, 16, 8, 53), (4096, 8, 2, 4100), (128, 17, 8, 53), (8192, 33, 4, 300), (1024, 20, 2, 8300),
                                     (2048, 48, 4, 4200), (4224, 48, 4, 4200)])
def test_a_large_batch_is_predicted_as_its_decode_batches(gpu, d, N, k, T):
    """Few experts beyond decode sizes: blocks that hold tokens and residual side by side, and (17 to 48 experts, many blocks) the
    stored logits; alone and with the routing, which has to be what it is alone."""
    B, Lm = gpu
    print(f"large prediction d={d} N={N} k={k} T={T}", flush=True)
    cfg = wl.scaled(wl.CONFIGS["qwen3"], d=d, N=N, k=k, I=128)
    dev = lambda a: torch.from_numpy(a).cuda()
    h, W0, W1 = (Lm.to_device_bf16(a) for a in (wl.hidden_states(cfg, T), wl.gate_weights(cfg, 0), wl.gate_weights(cfg, 1)))
    b0, b1, rv = dev(wl.gate_bias(cfg, 0)), dev(wl.gate_bias(cfg, 1)), dev(wl.layer_drift(cfg))
    i32 = dict(dtype=torch.int32, device="cuda")
    top, expect = torch.empty(N, **i32), torch.zeros(N, dtype=torch.int64, device="cuda")
    ws16 = B.alloc_workspace(B.shape(16, d, N, k, 128))
    for t in range(0, T, 16):
        pc = torch.empty(N, **i32)
        B.moe_predict_workload(B.shape(min(16, T - t), d, N, k, 128), h[t:t + 16], rv, W1, b1, N, pc, top, ws16)
        expect += pc
    s = B.shape(T, d, N, k, 128)
    ws, alone, both = B.alloc_workspace(s), B.alloc_routing(s), B.alloc_routing(s)
    B.moe_route(s, h, W0, b0, 1, alone, ws)
    counts = [torch.empty(N, **i32) for _ in range(2)]
    B.moe_predict_workload(s, h, rv, W1, b1, N, counts[0], top, ws)
    B.moe_route_predict(s, h, W0, b0, 1, both, rv, W1, b1, N, counts[1], top, ws)
    torch.cuda.synchronize()
    for c in counts:
        assert torch.equal(c.long(), expect)
    assert np.array_equal(top.cpu().numpy(), oracle.top_p(counts[1].cpu().numpy(), N))
    for name in ("topk_idx", "topk_w", "counts", "offsets", "perm", "inv_perm"):
        assert torch.equal(getattr(alone, name), getattr(both, name)), name
