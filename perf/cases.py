"""Performance cases of the MoE layer path.

A case is one pass of N tokens through a few consecutive MoE layers, called the
way a serving program calls them: `layer_forward` per layer for a stack whose
experts are resident on the device (routing, cross-layer prediction,
permutation and the quantised expert FFN), or `OffloadedStack.layer` for a stack
whose routed experts live in pinned host memory behind the expert cache.  Every
layer has weights and inputs of its own, so weights come from HBM (or over the
link), not out of a cache that the previous call warmed.
"""
import copy
import dataclasses
import math
import weakref

import numpy as np
import torch

import paper_2502_12224_amd.binding as B
from paper_2502_12224_amd.stack import LayerBuffers, OffloadedStack, layer_forward
from workloads import SHAPES, default_m, gen_expert, gen_gate, gen_hidden, gen_shared_gate, unit_rmsnorm_bf16

_DIMS = ("H", "E", "k", "I", "bits", "n_shared", "I_shared", "shared_bits")
_OUTPUTS = ("ids", "w", "pred_ids", "pred_w", "pred_pop", "counts", "offsets", "perm", "inv_perm", "order", "y")


def _case(name, shape, tokens, layers, **options):
    """shape: the entry of workloads.SHAPES that gives the dimensions (options override them) and the
    distributions of gate and bias; steps: passes with inputs of their own inside one run."""
    case = {"name": name, "shape": shape, "tokens": tokens, "layers": layers, "steps": 1, "zero_points": False,
            "low_percent": 0, "y_bf16": False, "graph": False, "offload": False}
    case.update({d: getattr(SHAPES[shape], d) for d in _DIMS})
    case.update(options)
    return case


def listed():
    return [
        # two small int8 layers with groups of 64, 16 requests: launches and host calls are all there is
        _case("tiny_16", "tiny", 16, 2),
        # one user generating: a token through all 24 layers, replayed from a graph as a serving loop does
        _case("qwen_decode_1", "qwen", 1, 24, graph=True),
        # the same without a graph, 8-bit shared experts: every layer is a call from Python
        _case("deepseek_decode_1", "deepseek", 1, 12),
        # a small decode batch: most of the experts of a layer are read for one or two tokens each
        _case("deepseek_decode_8", "deepseek", 8, 8),
        # one user on a model with few large experts: nothing but weight bytes
        _case("mixtral_decode_1", "mixtral", 1, 4),
        # an odd decode batch beyond the one-call layer
        _case("qwen_decode_13", "qwen", 13, 6),
        # a large decode batch, or a very short prompt: nearly every expert is read for a few rows
        _case("deepseek_batch_48", "deepseek", 48, 4),
        # a short prompt on experts of the asymmetric quantiser, the least popular quarter moved at 2 bits, bf16 out
        _case("qwen_prefill_131_hybrid", "qwen_prefill", 131, 4, zero_points=True, low_percent=25, y_bf16=True),
        # prompts with skewed routing: the usual length, and a long one
        _case("qwen_prefill_512", "qwen_prefill", 512, 4),
        _case("qwen_prefill_2048", "qwen_prefill", 2048, 4),
        # a long prompt on large experts: matrix-core work
        _case("mixtral_prefill_2048", "mixtral", 2048, 2),
        # decoding with the routed experts in host memory: four steps of 8 requests, about a fifth of every deep
        # layer's experts cached, the cache step and its transfers in between
        _case("deepseek_offload_8", "deepseek", 8, 5, offload=True, steps=4),
    ]


def _log_int(rng, lo, hi):
    return min(hi, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))


def draw(rng):
    kind = rng.random()
    if kind < 0.12:
        tokens = _log_int(rng, 1, 128)
        return _pure(_case("", rng.choice(["qwen", "deepseek"]), tokens, rng.randint(3, 5), offload=True,
                           steps=2))
    if kind < 0.40:
        tokens = _log_int(rng, 1, 8)
    elif kind < 0.58:
        tokens = rng.randint(9, 63)
    else:
        tokens = _log_int(rng, 64, 2048)
    shape = rng.choice(["qwen", "qwen_prefill", "deepseek", "mixtral", "generic", "generic", "generic"])
    options = {}
    if shape == "generic":
        shape = rng.choice(["qwen", "qwen_prefill", "deepseek", "mixtral"])
        E = rng.randint(8, 128)
        n_shared = rng.randint(0, 2)
        options = {"H": 1024 * rng.randint(1, 4), "E": E, "k": rng.randint(1, 8), "I": 128 * rng.randint(4, 22),
                   "bits": rng.choice([4, 4, 8]), "n_shared": n_shared,
                   "I_shared": 128 * rng.randint(4, 22) if n_shared else 0, "shared_bits": rng.choice([4, 8])}
    case = _case("", shape, tokens, 1, **options)
    case["zero_points"] = case["bits"] == 4 and rng.random() < 0.2
    case["low_percent"] = 25 if tokens > 16 and case["bits"] == 4 and rng.random() < 0.3 else 0
    case["y_bf16"] = rng.random() < 0.3
    case["graph"] = rng.random() < 0.3
    # as many layers as stay within a few GB of weights and the work of the largest listed case
    stored = case["E"] * _expert_bytes(case["H"], case["I"], case["bits"]) + \
        case["n_shared"] * _expert_bytes(case["H"], case["I_shared"], case["shared_bits"])
    flops = work(case)["flops"]
    case["layers"] = max(1, min(rng.randint(2, 8), int(2.5e9 / stored), int(2.5e12 / flops)))
    return _pure(case)


def _pure(case):
    del case["name"]
    return case


def _config(case, seed):
    return dataclasses.replace(SHAPES[case["shape"]], seed=seed, layers=case["layers"], **{d: case[d] for d in _DIMS})


class _Layer:
    """Weights of one resident layer, with the attributes layer_forward reads."""

    def __init__(self, cfg, case, layer):
        dev = "cuda"
        self.Wg, self.bias = gen_gate(cfg, layer, dev)
        self.shared_gate = gen_shared_gate(cfg, layer, dev)
        # the least popular experts of a prefill travel as 2-bit copies
        order = range(cfg.E) if self.bias is None else torch.argsort(self.bias, descending=True).tolist()
        low = set(list(order)[cfg.E - cfg.E * case["low_percent"] // 100:])
        self.packed = [B.PackedExpert(gen_expert(cfg, layer, e, device=dev, bits=2 if e in low else None,
                                                 zero_points=case["zero_points"]), dev) for e in range(cfg.E)]
        self.shared = [B.PackedExpert(gen_expert(cfg, layer, s, shared=True, device=dev), dev)
                       for s in range(cfg.n_shared)]
        self.table = B.expert_table([p.struct() for p in self.packed], dev)
        self.shared_table = B.expert_table([p.struct() for p in self.shared], dev) if cfg.n_shared else None


def _buffers(cfg, N, count, y_bf16):
    """Output buffers of `count` layer calls in common arenas; one workspace, since the calls are ordered."""
    first = LayerBuffers(cfg, N, "cuda")
    if y_bf16:
        first.desc.y_is_fp32 = 0
        first.y = first.y.to(torch.bfloat16)
    bufs, outputs = [copy.copy(first) for _ in range(count)], {}
    for name in _OUTPUTS:
        t = getattr(first, name)
        n = t.numel()
        # one row per call, padded (with zeros) so that every row starts on a 16-byte boundary
        outputs[name] = torch.zeros(count, (n + 7) // 8 * 8, dtype=t.dtype, device=t.device)
        for i, b in enumerate(bufs):
            setattr(b, name, outputs[name][i, :n].view(t.shape))
    return bufs, outputs


def _release(lib, cache, engine):
    torch.cuda.synchronize()
    lib.fate_cache_destroy(cache)
    lib.fate_hip_engine_destroy(engine)


def prepare(case, seed):
    cfg = _config(case, seed)
    N, L, steps = case["tokens"], case["layers"], case["steps"]
    xs = [unit_rmsnorm_bf16(gen_hidden(cfg, N, step=i, device="cuda")) for i in range(L * steps)]
    bufs, outputs = _buffers(cfg, N, L * steps, case["y_bf16"])
    state = {"cfg": cfg, "case": case, "xs": xs, "bufs": bufs, "outputs": outputs, "graph": None}
    if case["offload"]:
        # one shallow layer cached in full, then a fifth of the experts per layer; at most one expert prefetched
        # per layer, as the ratio of compute to transfer time allows
        stack = OffloadedStack(cfg, cfg.E + (L - 1) * (cfg.E // 5), 1, staging_slots=3 * cfg.E, L_shallow=1)
        weakref.finalize(stack, _release, stack.lib, stack.cache, stack.engine)
        state["stack"] = stack
        return state
    state["layers"] = [_Layer(cfg, case, l) for l in range(L)]
    if case["graph"]:
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            _enqueue(state)
            side.synchronize()
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=side):
                _enqueue(state)
        torch.cuda.current_stream().wait_stream(side)
        state["graph"] = graph
    return state


def _enqueue(state):
    layers, xs, bufs = state["layers"], state["xs"], state["bufs"]
    # (zero-points and 2-bit copies are formats of the separate calls, not of the one-call decode layer)
    one_launch = None if not (state["case"]["zero_points"] or state["case"]["low_percent"]) else False
    for l, layer in enumerate(layers):
        layer_forward(state["cfg"], layer, layers[l + 1] if l + 1 < len(layers) else None, xs[l], bufs[l],
                      one_launch=one_launch)


def run(state):
    case = state["case"]
    if case["offload"]:
        L = case["layers"]
        for i in range(L * case["steps"]):
            state["stack"].layer(i % L, state["xs"][i], state["bufs"][i])
    elif state["graph"] is not None:
        state["graph"].replay()
    else:
        _enqueue(state)
    return state["outputs"]


def _expert_bytes(H, I, bits, group=128):
    return 3 * (H * I * bits // 8 + H * I // group * 2)


def _active_experts(case):
    """Expected number of experts that N tokens select: gate logits are N(0, 1) plus the bias."""
    shape, E, N = SHAPES[case["shape"]], case["E"], case["tokens"]
    rng = np.random.default_rng(7)
    bias = np.zeros(E)
    if shape.zipf_s > 0:
        bias = -shape.zipf_s * np.log(np.arange(1, E + 1))
    elif shape.bias_std > 0:
        bias = rng.normal(0.0, shape.bias_std, E)
    trials = 1 if N >= 256 else 8
    seen = 0
    for _ in range(trials):
        top = np.argsort(-(rng.normal(size=(N, E)) + bias), axis=1)[:, :case["k"]]
        seen += len(np.unique(top))
    return seen / trials


def work(case):
    """Every activated expert (codes and scales) read once per layer call, gates, inputs, outputs; the
    products of every (token, expert) pair and of both gates.  An offloaded stack counts the same: which
    of these bytes also cross the host link depends on the cache."""
    H, E, N, k = case["H"], case["E"], case["tokens"], case["k"]
    m = default_m(E, k)
    group = SHAPES[case["shape"]].group
    wide = _expert_bytes(H, case["I"], case["bits"], group)
    low = case["low_percent"] / 100
    active = _active_experts(case)
    extra = 3 * H * case["I"] // group * 2 if case["zero_points"] else 0
    weights = active * ((1 - low) * wide + low * _expert_bytes(H, case["I"], 2, group) + extra)
    weights += case["n_shared"] * _expert_bytes(H, case["I_shared"], case["shared_bits"], group)
    acts = N * H * (2 + (2 if case["y_bf16"] else 4)) + N * (k * 8 + m * 8 + k * 8)
    flops = 6.0 * H * N * (k * case["I"] + case["n_shared"] * case["I_shared"]) + 4.0 * N * H * E
    calls = case["layers"] * case["steps"]
    return {"bytes": calls * (weights + 2 * E * H * 2 + acts), "flops": calls * flops}


def tolerance(case):
    """fp16 products of fp16-rounded activations and weights, fp32 sums: three roundings of 2^-11 in a chain
    of two products; bf16 outputs add a rounding of 2^-9.  Identifiers and counts are whole numbers: exact."""
    return {"rel": 4e-3, "max": 4e-2} if case["y_bf16"] else {"rel": 1e-3, "max": 1e-2}
