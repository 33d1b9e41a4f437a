"""The passes whose speed this repository cares about: one MoE layer, called as a program that serves a model calls it.

A case is a layer shape of ``workloads.CONFIGS``, a batch size and how the layer is called.  ``listed()`` is a fixed
selection, ``draw(rng)`` gives further cases of the same ranges.  All inputs are made on the GPU from a seed with the laws
of ``workloads.py`` (hidden states N(0,1), weights N(0, 1/fan_in), Zipf-skewed gate bias, expert masks from a previous
step's workloads)."""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2602_03495_amd import binding as B
from paper_2602_03495_amd import layer as Lm
from paper_2602_03495_amd import workloads as wl

MERGED_MAX_T = 64      # up to here a layer with shared experts runs them inside the grouped launches


def _case(name, config, tokens, on, predict=False, graph=False):
    """on: experts placed on this GPU (0 = no mask, all of them); predict: the next layer's workload is predicted with the
    routing; graph: the pass is captured once and replayed, as a decode loop does."""
    c = {"config": config, "tokens": tokens, "on": on, "predict": predict, "graph": graph}
    if name is not None:
        c = {"name": name, **c}
    return c


def listed():
    return [
        # decode of a single sequence, shared expert inside the grouped launches: all latency and launches
        _case("qwen15_decode_1", "qwen15", 1, 0, graph=True),
        # a decode batch issued call by call, half of the experts on this GPU
        _case("deepseek_decode_16", "deepseek", 16, 32),
        # one layer of the 48-layer decode stack, with the prediction that drives its prefetching
        _case("qwen3_decode_16", "qwen3", 16, 64, predict=True, graph=True),
        # decode with large experts: weight streaming
        _case("mixtral_decode_1", "mixtral", 1, 0, graph=True),
        _case("mixtral_decode_13", "mixtral", 13, 6),
        # a batch between decode and prefill (many sequences, or a short prompt), ragged
        _case("qwen3_mid_77", "qwen3", 77, 64),
        # most experts live on the host: two of eight here
        _case("mixtral_mid_200_few", "mixtral", 200, 2),
        # prompts: many small experts, with and without shared ones, with the prediction, ragged
        _case("deepseek_prefill_2048", "deepseek", 2048, 32),
        _case("qwen3_prefill_1531", "qwen3", 1531, 64, predict=True),
        _case("qwen15_prefill_4096", "qwen15", 4096, 0),
        # prompts through large experts; the first is the workload of bench.py
        _case("mixtral_prefill_2048", "mixtral", 2048, 6),
        _case("mixtral_prefill_8192", "mixtral", 8192, 0),
    ]


def draw(rng):
    config = rng.choice(["mixtral", "deepseek", "qwen15", "qwen3"])
    tokens = int(round(math.exp(rng.uniform(0.0, math.log(8192.0)))))
    N = wl.CONFIGS[config].N
    on = rng.choice([0, 0, N // 2, (3 * N) // 4, N // 4])
    return _case(None, config, max(1, min(8192, tokens)), on, predict=rng.random() < 0.3,
                 graph=tokens <= 16 and rng.random() < 0.5)


# ---------------------------------------------------------------------------------------------------------------------

def _merged(cfg, case):
    return cfg.n_shared > 0 and case["tokens"] <= MERGED_MAX_T and not case["predict"]


def _zipf(cfg, gen):
    """[N] fp32 gate bias: -s ln(rank), ranks a random permutation, shifted to zero mean (on gen's device)."""
    rank = torch.randperm(cfg.N, generator=gen, device=gen.device).double() + 1.0
    b = -cfg.zipf_s * rank.log()
    return (b - b.mean()).float()


def _mask(cfg, case, bias, gen):
    """uint8 [N], the `on` experts with the largest workloads of a previous step of the same size, or None."""
    if case["on"] == 0:
        return None
    logits = torch.randn(case["tokens"], cfg.N, generator=gen, device=gen.device) + bias
    prev = torch.bincount(logits.topk(cfg.k, dim=1).indices.reshape(-1), minlength=cfg.N)
    mask = torch.zeros(cfg.N, dtype=torch.uint8, device=gen.device)
    mask[torch.sort(prev, descending=True, stable=True).indices[: case["on"]]] = 1
    return mask


def _weights(n, rows, K, gen, chunk=8):
    """Row-major [n, rows, K] bf16, N(0, 1/K)."""
    w = torch.empty((n, rows, K), dtype=torch.bfloat16, device=gen.device)
    for i in range(0, n, chunk):
        w[i:i + chunk].normal_(0.0, K ** -0.5, generator=gen)
    return w


def prepare(case, seed):
    cfg, T = wl.CONFIGS[case["config"]], case["tokens"]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    h = torch.randn(T, cfg.d, generator=gen, device="cuda").bfloat16()
    gate_w = _weights(1, cfg.N, cfg.d, gen)[0]
    bias = _zipf(cfg, gen)
    mask = _mask(cfg, case, bias, gen)
    w1, w3, w2 = (_weights(cfg.N, cfg.I, cfg.d, gen), _weights(cfg.N, cfg.I, cfg.d, gen), _weights(cfg.N, cfg.d, cfg.I, gen))
    layer = Lm.MoeLayer(cfg, T)
    w = Lm.LayerWeights(gate_w, bias, None, None, None)
    if cfg.n_shared:
        S, Is = cfg.n_shared, cfg.I_shared
        s1, s3, s2 = _weights(S, Is, cfg.d, gen), _weights(S, Is, cfg.d, gen), _weights(S, cfg.d, Is, gen)
        if cfg.shared_gate == "sigmoid":
            w.w_sg = torch.randn(cfg.d, generator=gen, device="cuda").mul_(cfg.d ** -0.5).bfloat16()
        if _merged(cfg, case):
            # a shared expert of inner size m I as m experts of inner size I behind the routed ones
            m = Is // cfg.I
            s2 = s2.view(S, cfg.d, m, cfg.I).transpose(1, 2).reshape(S * m, cfg.d, cfg.I)
            w.xw1 = B.moe_pack_weights(torch.cat([w1, s1.view(S * m, cfg.I, cfg.d)]))
            w.xw3 = B.moe_pack_weights(torch.cat([w3, s3.view(S * m, cfg.I, cfg.d)]))
            w.xw2 = B.moe_pack_weights(torch.cat([w2, s2]))
        else:
            w.sw1, w.sw3, w.sw2 = B.moe_pack_weights(s1), B.moe_pack_weights(s3), B.moe_pack_weights(s2)
    if w.xw1 is None:
        w.w1, w.w3, w.w2 = B.moe_pack_weights(w1), B.moe_pack_weights(w3), B.moe_pack_weights(w2)
    state = {"case": case, "layer": layer, "h": h, "w": w, "mask": mask, "graph": None,
             "merged": _merged(cfg, case), "xmask": None}
    if state["merged"] and mask is not None:
        state["xmask"] = layer.merged_mask(mask)
    if case["predict"]:
        # the next layer's gate; the drift between the layers is N(0, 0.1) per dimension
        state["next_w"] = Lm.LayerWeights(_weights(1, cfg.N, cfg.d, gen)[0], _zipf(cfg, gen), None, None, None)
        state["res_vec"] = torch.randn(cfg.d, generator=gen, device="cuda") * 0.1 ** 0.5
        state["p"] = max(1, cfg.N // 16)
        state["top"] = torch.empty(state["p"], dtype=torch.int32, device="cuda")
    if case["graph"]:
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            _pass(state)
        torch.cuda.current_stream().wait_stream(side)
        state["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(state["graph"]):
            _pass(state)
    return state


def _pass(s):
    layer, h, w, mask = s["layer"], s["h"], s["w"], s["mask"]
    if s["merged"]:
        layer.forward_merged(h, w, s["xmask"])
    elif s["case"]["predict"]:
        layer.route_predict(h, w, s["res_vec"], s["next_w"], s["p"], s["top"])
        layer.expert_ffn(h, w, mask)
        if layer.n_shared:
            layer.shared_ffn(h, w)
        layer.combine(mask)
    else:
        layer.forward(h, w, mask)


def run(state):
    if state["graph"] is not None:
        state["graph"].replay()
    else:
        _pass(state)
    layer = state["layer"]
    r = layer.routing
    outputs = {"out": layer.out, "topk_idx": r.topk_idx, "topk_w": r.topk_w, "counts": r.counts}
    if state["case"]["predict"]:
        outputs["pred_counts"] = layer.pred_counts
        outputs["top_experts"] = state["top"]
    return outputs


def work(case):
    """The weights of the experts that have rows and are on this GPU, the hidden states and the gate once in, the layer's
    output and tables once out; 6 d I flops per routed row on this GPU.  How many experts and rows that is follows from
    the routing law; it is taken from one simulated batch."""
    cfg, T = wl.CONFIGS[case["config"]], case["tokens"]
    gen = torch.Generator()
    gen.manual_seed(1)
    bias = _zipf(cfg, gen)
    mask = _mask(cfg, case, bias, gen)
    logits = torch.randn(T, cfg.N, generator=gen) + bias
    counts = torch.bincount(logits.topk(cfg.k, dim=1).indices.reshape(-1), minlength=cfg.N).numpy()
    if mask is not None:
        counts = counts * mask.numpy()
    active, rows = int(np.count_nonzero(counts)), int(counts.sum())
    expert, gates = 3 * cfg.d * cfg.I, 2 if case["predict"] else 1
    byts = 2.0 * expert * active + 2.0 * gates * cfg.N * cfg.d + 2.0 * 2.0 * T * cfg.d + 8.0 * T * cfg.k
    flops = 2.0 * expert * rows + 2.0 * gates * T * cfg.N * cfg.d
    if cfg.n_shared:
        shared = 3 * cfg.d * cfg.I_shared * cfg.n_shared
        byts += 2.0 * shared
        flops += 2.0 * shared * T
    return {"bytes": byts, "flops": flops}


def tolerance(case):
    """bf16 results of fp32 sums: the inner activations, the expert rows and the output are each rounded to bf16 once.
    Against the same pass in float64 the output of every listed case differs by 2.9e-3 (2-norm), the weights by 1.5e-7."""
    # differ: a token whose k-th and (k+1)-th logits agree to fp32 rounding may take either expert
    return {"rel": 1e-2, "differ": 0.02}
