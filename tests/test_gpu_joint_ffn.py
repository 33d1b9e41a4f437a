"""Both projections of the routed and the shared experts as one launch (called directly, whatever the rule of moe_layer_ffn says of the
sizes; the rule: test_joint_rule.py), against moe_expert_ffn on either set of experts.
A projection whose K is not split adds its products in the same order in both, so the rows are the same bits; where the separate
down projection splits K (fp32 sums of 2 or more parts) the rows differ by one bf16 rounding of y at most, 2^-8 of the value, and
of sums of that size where terms cancel (2^-8 of the largest value)."""
import numpy as np
import pytest
import torch

from paper_2602_03495_amd import workloads as wl

pytestmark = pytest.mark.gpu

SENTINEL = 0x7B7B

# rows of the experts, k, d, I, masked-off experts, shared experts, their inner size
CASES = {
    "three tiles to an expert": ([3072 // 8] * 8, 1, 256, 128, (), 0, 0),
    "one expert with a row less": ([3072 // 8] * 7 + [383], 1, 256, 128, (), 0, 0),
    "ragged tiles of every height": ([1, 16, 17, 32, 33, 64, 65, 96, 97, 127, 128, 129, 0, 255, 257, 5000], 1, 640, 384, (), 0, 0),
    "wide, ragged inner columns": ([700, 1, 2500, 0, 130, 3000], 1, 2048, 1408, (4,), 0, 0),
    "every expert masked off": ([3100, 3100], 1, 256, 256, (0, 1), 0, 0),
    "one expert on": ([3100, 3100], 1, 1152, 640, (0,), 0, 0),
    "128 experts": ([60] * 64 + [1] * 63 + [2500], 1, 384, 256, tuple(range(0, 128, 3)), 0, 0),
    "8 slots, wide tiles": ([100] * 70 + [0, 1, 999], 8, 2048, 128, (3, 72), 0, 0),
    "6 slots, long inner size": ([200, 129, 200, 5, 200, 66, 0, 200, 200], 6, 1152, 8064, (1,), 0, 0),
    "6 slots, shared": ([100, 17, 1, 100, 0, 82, 100, 100, 100], 6, 640, 384, (0,), 2, 384),
    "shared, few tokens": ([3, 0, 14], 1, 256, 256, (), 2, 256),
    "shared, long inner size": ([300, 2, 40], 1, 1152, 384, (1,), 1, 1408),
    "shared, long inner size, wide tiles": ([90] * 60, 1, 2176, 128, (5,), 1, 640),
    "shared, all routed experts masked off": ([200, 200], 1, 512, 256, (0, 1), 2, 256),
    "shared, separate projection splits K": ([140, 30], 1, 512, 1408, (), 1, 4096),
}


class Layer:
    """Tables, weights and buffers of one call: rows of the experts (k slots per token), shared experts S of inner size Is."""

    def __init__(self, B, rows, k, d, I, off=(), S=0, Is=0):
        self.B, self.rows, self.off, self.d, self.S = B, rows, off, d, S
        N, R = len(rows), sum(rows)
        self.T = T = R // k
        assert T * k == R and max(rows) <= T
        self.gen = gen = torch.Generator(device="cuda").manual_seed(N + R)

        def weights(n, r, K):
            return B.moe_pack_weights((torch.randn(n, r, K, generator=gen, device="cuda") * K ** -0.5).bfloat16())

        self.h = torch.randn(T, d, generator=gen, device="cuda").bfloat16()
        self.mask = torch.ones(N, dtype=torch.uint8, device="cuda")
        self.mask[list(off)] = 0
        self.s = B.shape(T, d, N, k, I)
        self.tables = (torch.randperm(R, generator=gen, device="cuda").int(),
                       torch.from_numpy(np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)).cuda(),
                       torch.tensor(rows, dtype=torch.int32, device="cuda"))
        self.w = weights(N, I, d), weights(N, I, d), weights(N, d, I)
        self.ws = B.alloc_workspace(self.s)
        if S:
            i32 = dict(dtype=torch.int32, device="cuda")
            self.ss = B.shape(T, d, S, S, Is)
            counts, offsets, perm = torch.empty(S, **i32), torch.empty(S + 1, **i32), torch.empty(T * S, **i32)
            B.moe_dense_route(self.ss, counts, offsets, perm)
            self.stables, self.sw = (perm, offsets, counts), (weights(S, Is, d), weights(S, Is, d), weights(S, d, Is))
            self.sws = B.alloc_workspace(self.ss)
        self.row_on = torch.from_numpy(~np.repeat(np.isin(np.arange(N), list(off)), rows)).cuda()

    def fresh(self):
        """Results of the routed and of the shared experts, filled with the sentinel."""
        y = [torch.empty((n, self.d), dtype=torch.bfloat16, device="cuda") for n in (sum(self.rows), self.T * self.S) if n]
        for a in y:
            a.view(torch.int16).fill_(SENTINEL)
        return y

    def call(self, y, masked=True):
        shared = (self.ss, *self.stables, *self.sw, y[1], self.sws) if self.S else None
        self.B.moe_layer_ffn(self.s, self.h, *self.tables, *self.w, self.mask if masked else None, y[0], self.ws, shared)

    def joint(self, y, polls=1 << 21):
        """The joint launch itself.  polls = 0: as if every wait had run out."""
        import ctypes as C
        p = self.B._ptr
        tail = (C.c_void_p(0),) * 9
        if self.S:
            tail = (C.byref(self.ss), *map(p, self.stables), *map(p, self.sw), p(y[1]), self.B._ws_ptr(self.sws))
        rc = self.B.load_library().moe_ffn_joint_impl(C.byref(self.s), p(self.h), *map(p, self.tables), *map(p, self.w), p(self.mask),
                                                      p(y[0]), self.B._ws_ptr(self.ws), *tail, C.c_int(polls), self.B._stream())
        assert rc == 0

    def separate(self, y):
        self.B.moe_expert_ffn(self.s, self.h, *self.tables, *self.w, self.mask, y[0], self.B.alloc_workspace(self.s))
        if self.S:
            self.B.moe_expert_ffn(self.ss, self.h, *self.stables, *self.sw, None, y[1], self.B.alloc_workspace(self.ss))


def bits(y):
    return y.view(torch.int16)


@pytest.mark.parametrize("name", CASES)
def test_joint_launch_writes_what_the_separate_launches_write(name):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_03495_amd import binding as B
    B.load_library()
    print(f"joint launch: {name} {CASES[name][1:]}", flush=True)
    L = Layer(B, *CASES[name])
    exact = name != "shared, separate projection splits K"
    got, graph = L.fresh(), None
    for turn in range(4):
        # other hidden states every time over the workspace of the time before: activations of an earlier pass must not be read
        L.h.normal_(generator=L.gen)
        ref = L.fresh()
        L.separate(ref)
        if turn == 0:
            for ws in [L.ws] + ([L.sws] if L.S else []):
                ws.fill_(0xFF)                    # arbitrary contents: counters and activations alike
        if graph is not None:
            graph.replay()
        else:
            L.joint(got)
        for i, (a, b) in enumerate(zip(got, ref)):
            if exact or i == 0:
                assert torch.equal(bits(a), bits(b)), (name, turn)
            else:
                x, r = a.float(), b.float()
                assert (x - r).abs().max() <= 2 ** -8 * r.abs().max(), (name, turn)
        if turn == 1:
            side = torch.cuda.Stream()
            side.wait_stream(torch.cuda.current_stream())
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=side):
                L.joint(got)
    assert (bits(got[0])[~L.row_on] == SENTINEL).all()


def test_two_joint_launches_beside_each_other():
    """On two streams, each with blocks for the whole chip: whichever of them get a place, no block waits for one that has none."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_03495_amd import binding as B
    B.load_library()
    print("two joint launches on two streams", flush=True)
    layers = [Layer(B, [150] * 40, 3, 2048, 384, (1,), 2, 768), Layer(B, [90] * 64 + [240], 2, 1024, 640, (2, 9))]
    got, ref = [L.fresh() for L in layers], [L.fresh() for L in layers]
    for L, r in zip(layers, ref):
        L.separate(r)
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    for _ in range(8):
        for L, g, st in zip(layers, got, streams):
            with torch.cuda.stream(st):
                L.joint(g)
    torch.cuda.synchronize()
    for r, g in zip(ref, got):
        assert all(torch.equal(bits(a), bits(b)) for a, b in zip(g, r))


# rows, k, d, I, masked-off experts, shared experts, their inner size; the down items are 128, 256 and 512 columns wide
VOIDED = {
    "128 columns": ([400] * 8, 2, 256, 128, (2,), 0, 0),
    "256 columns, ragged": ([60] * 90, 1, 640, 128, (0, 89), 0, 0),
    "512 columns, ragged, shared": ([60] * 100, 1, 1152, 128, (7,), 1, 640),
}


@pytest.mark.parametrize("name", VOIDED)
def test_rows_whose_activations_were_not_waited_for_are_nan(name):
    """A wait that runs out leaves NaN in the whole rows of its item and nothing elsewhere; the launch after it is whole again."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_03495_amd import binding as B
    B.load_library()
    print(f"waits that ran out: {name}", flush=True)
    L = Layer(B, *VOIDED[name])
    y = L.fresh()
    L.joint(y, polls=0)
    assert (bits(y[0])[L.row_on] == 0x7FC0).all() and (bits(y[0])[~L.row_on] == SENTINEL).all()
    assert all((bits(a) == 0x7FC0).all() for a in y[1:])
    ref = L.fresh()
    L.separate(ref)
    L.joint(y)
    assert (bits(y[0])[L.row_on] == bits(ref[0])[L.row_on]).all()
    assert all((bits(a) == bits(b)).all() for a, b in zip(y[1:], ref[1:]))


def launched_jointly(B, call):
    """Whether call, of more than 16 tokens, ran as a joint launch: the blocks of separate launches leave records."""
    records = torch.zeros(2 * B.TRACE_MAX_BLOCKS * 8, dtype=torch.int64, device="cuda")
    B.moe_debug_set_trace(records)
    call()
    torch.cuda.synchronize()
    B.moe_debug_set_trace(None)
    return not bool((records.view(-1, 8)[:, 7] == 1).any())


def test_calls_take_the_launch_that_the_rule_names():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_03495_amd import binding as B
    import test_joint_rule as rule
    for rows, shape, shared in (([165] * 55 + [141], (2048, 56, 1, 1152), ()), ([165] * 55 + [140], (2048, 56, 1, 1152), ()),
                                ([65, 64], (256, 2, 1, 256), (1, 640)), ([64, 64], (256, 2, 1, 256), (1, 640))):
        d, N, k, I = shape
        L = Layer(B, rows, k, d, I, (), *shared)
        for masked in (False, True):
            y, ref = L.fresh(), L.fresh()
            want = rule.joint(masked, L.T, d, N, k, I, shared)
            print(f"route: {L.T} tokens {shape} {shared} masked {masked}: joint {want}", flush=True)
            assert launched_jointly(B, lambda: L.call(y, masked)) == want
            L.separate(ref)
            assert all(torch.equal(bits(a), bits(b)) for a, b in zip(y, ref))


def test_ffn_and_gates_use_parts_of_the_workspace_of_their_own():
    """What lets a prediction on another stream run beside the FFN: neither writes where the other does."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_03495_amd import binding as B, layer as Lm
    cfg = wl.LayerConfig(71, "parts", d=256, N=32, k=3, I=128, norm_mode=wl.NORM_RENORM, bias_law="normal", n_shared=2, I_shared=256,
                         shared_gate="one")
    T, fill = 1024, 0x5C
    w = Lm.LayerWeights.upload(wl.gate_weights(cfg), wl.gate_bias(cfg), *wl.expert_weights(cfg), wl.shared_expert_weights(cfg))
    L = Lm.MoeLayer(cfg, T)
    h = Lm.to_device_bf16(wl.hidden_states(cfg, T))
    top = torch.empty(2, dtype=torch.int32, device="cuda")
    res_vec = torch.zeros(cfg.d, device="cuda")

    def routing_bytes(s):                 # the tail of the workspace
        up = lambda n: (n + 255) // 256 * 256
        return up(128 * 4) + 2 * up(s.T * s.k * 4) + 2 * up(max(s.T, 16) * s.N * 4)

    def parts(ws, s):
        n = B.workspace_bytes(s)
        ws = ws[B._ws_ptr(ws).value - ws.data_ptr():][:n]
        return ws[:n - routing_bytes(s)], ws[n - routing_bytes(s):]

    for gates in (lambda: L.route(h, w), lambda: L.predict(h, res_vec, w, 2, top), lambda: L.route_predict(h, w, res_vec, w, 2, top)):
        L.ws.fill_(fill)
        gates()
        ffn, gate = parts(L.ws, L.shape)
        assert (ffn == fill).all()
    assert (gate != fill).any()
    L.ws.fill_(fill)
    L.sws.fill_(fill)
    assert launched_jointly(B, lambda: L.all_ffn(h, w, None))
    for ws, s in ((L.ws, L.shape), (L.sws, L.sshape)):
        ffn, gate = parts(ws, s)
        assert (gate == fill).all() and (ffn != fill).any()


def test_two_workspaces_and_one_batch_are_required():
    import ctypes as C
    from paper_2602_03495_amd import binding as B
    lib = B.load_library()
    p, q, z = C.c_void_p(0x1000), C.c_void_p(0x2000), C.c_void_p(0)
    s, ss = B.shape(16, 256, 8, 2, 512), B.shape(16, 256, 1, 1, 512)
    call = lambda ss, a=p, w=q: lib.moe_layer_ffn(C.byref(s), p, p, p, p, p, p, p, z, p, p, C.byref(ss), p, p, p, p, p, a, p, w, z)
    assert call(ss, w=p) == -1                              # the same workspace twice
    assert call(ss, a=z) == -1                              # no w2 of the shared experts
    assert call(B.shape(17, 256, 1, 1, 512)) == -1          # another batch
    assert call(B.shape(16, 128, 1, 1, 512)) == -1          # another hidden size
    assert call(ss, w=C.c_void_p(0x1010)) == -4             # misaligned workspace
    ss.weight_layout = 0
    assert call(ss) == -2                                   # row-major weights
