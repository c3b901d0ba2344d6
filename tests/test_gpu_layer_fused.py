"""One-launch decode layer against the separate calls and the oracle."""
import numpy as np
import pytest
import torch

from oracle import moe as O
import paper_2502_12224_amd.binding as B
from paper_2502_12224_amd.stack import LayerBuffers, LayerWeights, layer_forward
from workloads import SHAPES, gen_hidden
from helpers import DEV, bias_np, f32, ffn_rel_err, oracle_expert

pytestmark = pytest.mark.gpu

ROUTE_FIELDS = ("ids", "w", "counts", "offsets", "perm", "inv_perm", "order")
PRED_FIELDS = ("pred_ids", "pred_w", "pred_pop")


def _snapshot(buf, fields):
    return {f: getattr(buf, f).clone() for f in fields}


@pytest.mark.parametrize("name,N,last", [("tiny", 1, False), ("tiny", 8, False), ("tiny", 5, True),
                                         ("qwen", 1, False), ("qwen", 1, True), ("qwen", 6, False),
                                         ("deepseek", 8, False), ("deepseek", 1, False), ("mixtral", 1, False),
                                         ("mixtral", 4, False)])
def test_one_launch_layer_equals_separate_calls_and_oracle(name, N, last):
    _one_launch_case(SHAPES[name], name, N, last)


# the other kernel instantiations of the one-token form, and a layer without shared experts: the Qwen shape with
# 8-bit routed experts, with an 8-bit shared expert, with both, and with no shared expert at all
import dataclasses
_QWEN = SHAPES["qwen"]
VARIANTS = {
    "qwen-routed8": dataclasses.replace(_QWEN, name="qwen-routed8", bits=8),
    "qwen-shared8": dataclasses.replace(_QWEN, name="qwen-shared8", shared_bits=8),
    "qwen-both8": dataclasses.replace(_QWEN, name="qwen-both8", bits=8, shared_bits=8),
    "qwen-noshared": dataclasses.replace(_QWEN, name="qwen-noshared", n_shared=0, I_shared=0, shared_gate=False),
}


@pytest.mark.parametrize("name,N", [("qwen-routed8", 1), ("qwen-shared8", 1), ("qwen-both8", 1), ("qwen-noshared", 1),
                                    ("qwen-noshared", 3)])
def test_one_launch_layer_on_other_formats_and_without_shared_experts(name, N):
    _one_launch_case(VARIANTS[name], name, N, False)


def _one_token_workgroups(cfg):
    """Workgroups of a one-token layer with both gates: the gates' rows, 32 neurons of every expert, 32 outputs of every
    part of the down projection (pieces of at most 768 columns of int4 or 384 of int8, four a workgroup).  The kernel of
    three waves per SIMD takes launches of more than 512."""
    pieces = lambda I, bits: -(-I // (768 if bits == 4 else 384))
    parts = -(-max(cfg.n_shared * pieces(cfg.I_shared, cfg.shared_bits), cfg.k * pieces(cfg.I, cfg.bits)) // 4)
    return 2 * cfg.E // 4 + cfg.n_shared * cfg.I_shared // 32 + cfg.k * cfg.I // 32 + parts * cfg.H // 32


# one-token layers of more workgroups than two per compute unit hold (618 and 662 with five and six of the
# Qwen-shaped experts, 726 to 854 with 8-bit ones) run the kernel of three waves per SIMD; one instantiation per pair of formats
@pytest.mark.parametrize("bits,shared_bits,k", [(4, 4, 5), (4, 4, 6), (4, 8, 6), (8, 4, 6), (8, 8, 6)])
def test_one_token_layer_of_more_workgroups_than_two_per_compute_unit(bits, shared_bits, k):
    cfg = dataclasses.replace(_QWEN, name=f"qwen-k{k}-{bits}-{shared_bits}", k=k, bits=bits, shared_bits=shared_bits)
    assert _one_token_workgroups(cfg) > 512
    _one_token_case_with_hints(cfg)


# the kernel of two waves per SIMD, of every pair of formats; with three, the largest tables and selections
@pytest.mark.parametrize("bits,shared_bits,k,I_shared,E,workgroups", [
    (4, 4, 4, 5632, 60, 510), (4, 8, 2, 1408, 60, 226), (8, 4, 2, 1408, 60, 290), (8, 8, 4, 1408, 60, 506),
    (4, 4, 8, 1408, 256, 780),
])
def test_one_token_layer_on_both_sides_of_two_workgroups_per_compute_unit(bits, shared_bits, k, I_shared, E, workgroups):
    cfg = dataclasses.replace(_QWEN, name=f"qwen-{bits}-{shared_bits}-k{k}-{I_shared}-{E}", k=k, bits=bits, shared_bits=shared_bits,
                              I_shared=I_shared, E=E)
    assert _one_token_workgroups(cfg) == workgroups
    _one_token_case_with_hints(cfg)


def _one_token_case_with_hints(cfg):
    k = cfg.k
    one, (x, lw, ln) = _one_launch_case(cfg, cfg.name, 1, False)
    # hints: all right, one wrong, all wrong; y differs at most in the order of its fp32 sums
    true = one.ids.cpu().numpy()[0].tolist()
    others = [e for e in range(cfg.E) if e not in true]
    y_ref = f32(one.y).astype(np.float64)
    for h in (true, true[:1] + [others[0]] + true[2:], others[:k]):
        print(f"  hint {h}", flush=True)
        one.y.fill_(float("nan"))
        layer_forward(cfg, lw, ln, x, one, one_launch=True, hint_ids=torch.tensor(h, dtype=torch.int32, device=DEV))
        torch.cuda.synchronize()
        assert one.status() == 0
        assert ffn_rel_err(f32(one.y), y_ref).max() <= 1e-5, h


def _one_launch_case(cfg, name, N, last):
    print(f"case {name} N={N} last={last}", flush=True)
    x = gen_hidden(cfg, N, device=DEV)
    lw = LayerWeights(cfg, 0, DEV)
    ln = None
    if not last:
        ln = LayerWeights(cfg, 1, DEV, experts=[])
    sep = LayerBuffers(cfg, N, DEV)
    one = LayerBuffers(cfg, N, DEV)
    assert one.one_launch_ok
    layer_forward(cfg, lw, ln, x, sep, one_launch=False)
    torch.cuda.synchronize()
    y_sep = sep.y.clone()
    fields = ROUTE_FIELDS + (() if last else PRED_FIELDS)
    want = _snapshot(sep, fields)
    P = N * cfg.k
    # three calls in a row on the same workspace: the counters must come back to zero each time
    for rep in range(3):
        one.y.fill_(float("nan"))
        layer_forward(cfg, lw, ln, x, one, one_launch=True)
        torch.cuda.synchronize()
        assert one.status() == 0, f"status {one.status()} on call {rep}"
        for f in fields:
            a, b = getattr(one, f), want[f]
            if f in ("perm", "inv_perm"):
                a, b = a[:P], b[:P]
            assert torch.equal(a, b), (f, rep)
        y_one = f32(one.y)
        assert np.isfinite(y_one).all()
        # same weights and activations; the two paths differ in the order of the fp32 sums and in how
        # the codes' offset is removed (per code, or per group after the matrix cores), which can
        # move an fp16 rounding of h
        assert ffn_rel_err(y_one, f32(y_sep).astype(np.float64)).max() <= 5e-4, rep
    sync_words = one.layer_ws[:8].view(torch.int32).cpu().numpy()
    assert sync_words[0] == 3 and sync_words[1] == 0       # epoch = number of calls, exit counter back at zero
    # against the oracle
    rid, rw, _, rz = O.gate_route(f32(x), f32(lw.Wg), bias_np(lw.bias), cfg.k, cfg.renorm)
    if len(O.near_tie_rows(rz, cfg.k)) == 0:
        assert np.array_equal(one.ids.cpu().numpy(), rid)
    ids_h = one.ids.cpu().numpy()
    from workloads import gen_expert
    experts = {int(e): oracle_expert(gen_expert(cfg, 0, int(e), device=DEV)) for e in set(ids_h.ravel().tolist())}
    shared = [oracle_expert(gen_expert(cfg, 0, s, shared=True, device=DEV)) for s in range(cfg.n_shared)]
    sg = None if lw.shared_gate is None else f32(lw.shared_gate)
    y_ref = O.moe_ffn(f32(x), ids_h, one.w.cpu().numpy().astype(np.float64), experts, shared, sg)
    err = ffn_rel_err(f32(one.y), y_ref).max()
    print(f"  max row error vs oracle {err:.2e}")
    assert err <= 2e-3
    return one, (x, lw, ln)


def test_one_launch_layer_rejects_large_batches():
    cfg = SHAPES["tiny"]
    d = B.make_ffn_desc(9, cfg.H, cfg.E, cfg.k, cfg.I, cfg.bits, cfg.group, 0, 0, cfg.bits, cfg.group, True, 0)
    nbytes, _ = B.fate_moe_layer_decode_workspace(d)
    ws = torch.zeros(nbytes, dtype=torch.uint8, device=DEV)
    buf = LayerBuffers(cfg, 9, DEV)
    lw = LayerWeights(cfg, 0, DEV)
    x = gen_hidden(cfg, 9, device=DEV)
    with pytest.raises(B.FateError):
        B.fate_moe_layer_decode(d, x, lw.Wg, lw.bias, None, None, cfg.m, cfg.renorm, buf.ids, buf.w, None, None, None,
                                buf.counts, buf.offsets, buf.perm, buf.inv_perm, buf.order, lw.table, None, None,
                                buf.y, ws)

@pytest.mark.parametrize("name,N", [("qwen", 1), ("qwen", 4), ("mixtral", 2)])
def test_one_launch_layer_with_outlier_activations(name, N):
    """Activations with a large common component and a few outlier channels: the one-launch body feeds
    the matrix cores with codes + constant and removes the constant's share afterwards from the sum of
    the activations of a group, which is where such inputs would cost accuracy."""
    cfg = SHAPES[name]
    print(f"case {name} N={N} outliers", flush=True)
    g = torch.Generator(device="cpu").manual_seed(1234 + N)
    xf = torch.randn(N, cfg.H, generator=g) + 3.0                       # common offset: every group sum is large
    cols = torch.randperm(cfg.H, generator=g)[:8]
    xf[:, cols] *= 40.0                                                  # outlier channels
    x = xf.to(torch.bfloat16).to(DEV)
    lw = LayerWeights(cfg, 0, DEV)
    one = LayerBuffers(cfg, N, DEV)
    layer_forward(cfg, lw, None, x, one, one_launch=True)
    torch.cuda.synchronize()
    assert one.status() == 0
    ids_h = one.ids.cpu().numpy()
    from workloads import gen_expert
    experts = {int(e): oracle_expert(gen_expert(cfg, 0, int(e), device=DEV)) for e in set(ids_h.ravel().tolist())}
    shared = [oracle_expert(gen_expert(cfg, 0, s, shared=True, device=DEV)) for s in range(cfg.n_shared)]
    sg = None if lw.shared_gate is None else f32(lw.shared_gate)
    y_ref = O.moe_ffn(f32(x), ids_h, one.w.cpu().numpy().astype(np.float64), experts, shared, sg)
    err = ffn_rel_err(f32(one.y), y_ref).max()
    print(f"  max row error vs oracle {err:.2e}")
    assert err <= 2e-3

@pytest.mark.parametrize("name,N,how", [("qwen", 1, "null"), ("qwen", 6, "null"), ("mixtral", 1, "null"),
                                        ("qwen", 1, "zero_points"), ("qwen", 6, "zero_points"),
                                        ("deepseek", 1, "null"), ("deepseek", 1, "zero_points")])
def test_one_launch_layer_with_an_expert_that_is_not_resident(name, N, how):
    """An activated expert whose table entry holds NULL pointers, or is stored in a format the one-launch
    layer does not read (here: with zero-points): status bit 0 is raised, its pairs contribute nothing,
    everything else is as usual (one-token kernels of two and three waves per SIMD, GEMMs)."""
    cfg = SHAPES[name]
    assert N > 1 or name == "mixtral" or (_one_token_workgroups(cfg) > 512) == (name == "deepseek")
    print(f"case {name} N={N} one expert absent ({how})", flush=True)
    x = gen_hidden(cfg, N, device=DEV)
    lw = LayerWeights(cfg, 0, DEV)
    one = LayerBuffers(cfg, N, DEV)
    layer_forward(cfg, lw, None, x, one, one_launch=True)
    torch.cuda.synchronize()
    ids_h = one.ids.cpu().numpy()
    gone = int(ids_h[0, 0])                                  # the first token's first expert
    saved = lw.table.clone()
    sz = __import__('ctypes').sizeof(B.fate_qexpert)
    if how == "null":
        lw.table[gone * sz:(gone + 1) * sz].zero_()
    else:                      # a non-NULL zero-point pointer (the scales' address: never read)
        o = B.fate_qexpert
        lw.table[gone * sz + o.z1.offset:gone * sz + o.z1.offset + 8] = \
            lw.table[gone * sz + o.s1.offset:gone * sz + o.s1.offset + 8].clone()
    one.y.fill_(float("nan"))
    layer_forward(cfg, lw, None, x, one, one_launch=True)
    torch.cuda.synchronize()
    lw.table.copy_(saved)
    assert one.status() == 1
    assert np.array_equal(one.ids.cpu().numpy(), ids_h)
    from workloads import gen_expert
    experts = {int(e): oracle_expert(gen_expert(cfg, 0, int(e), device=DEV)) for e in set(ids_h.ravel().tolist())}
    shared = [oracle_expert(gen_expert(cfg, 0, s, shared=True, device=DEV)) for s in range(cfg.n_shared)]
    sg = None if lw.shared_gate is None else f32(lw.shared_gate)
    w_ref = one.w.cpu().numpy().astype(np.float64)
    w_ref[ids_h == gone] = 0.0
    y_ref = O.moe_ffn(f32(x), ids_h, w_ref, experts, shared, sg)
    err = ffn_rel_err(f32(one.y), y_ref).max()
    print(f"  max row error vs oracle {err:.2e}")
    assert err <= 2e-3


@pytest.mark.parametrize("name,N", [("qwen", 1), ("deepseek", 8)])
def test_one_launch_layer_replayed_from_a_graph(name, N):
    """The layer call captured once and replayed with new inputs, with eager calls and synchronisations
    between the replays: every replay gives what the eager call gives on the same input, bit for bit
    (one-token kernel and GEMM form; the call's epoch lives on the device, so a replay advances it)."""
    cfg = SHAPES[name]
    print(f"case {name} N={N} graph replays", flush=True)
    lw = LayerWeights(cfg, 0, DEV)
    ln = LayerWeights(cfg, 1, DEV, experts=[])
    xs = [gen_hidden(cfg, N, step=s, device=DEV) for s in range(4)]
    eager = LayerBuffers(cfg, N, DEV)
    fields = ROUTE_FIELDS + PRED_FIELDS
    want = []
    for x in xs:
        layer_forward(cfg, lw, ln, x, eager, one_launch=True)
        torch.cuda.synchronize()
        assert eager.status() == 0
        want.append((_snapshot(eager, fields), eager.y.clone()))
    cap = LayerBuffers(cfg, N, DEV)
    x_in = torch.zeros_like(xs[0])
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        x_in.copy_(xs[0])
        layer_forward(cfg, lw, ln, x_in, cap, one_launch=True)     # warm before capture
        side.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            layer_forward(cfg, lw, ln, x_in, cap, one_launch=True)
    torch.cuda.synchronize()
    for s in (1, 3, 0, 2, 2):
        x_in.copy_(xs[s])
        cap.y.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert cap.status() == 0
        for f in fields:
            assert torch.equal(getattr(cap, f), want[s][0][f]), f"{f} of a replay (input {s}) differs from the eager call"
        assert torch.equal(cap.y, want[s][1]), f"y of a replay (input {s}) differs from the eager call"
        # eager work of the program between the replays
        layer_forward(cfg, lw, ln, xs[(s + 1) % 4], eager, one_launch=True)
        torch.cuda.synchronize()


@pytest.mark.parametrize("name", ["qwen", "deepseek"])
def test_one_token_layer_with_prefetch_hints(name):
    """The previous layer's prediction handed in as a hint (section 4.3): the routed work groups start on
    the hinted experts before the gate is known.  Whatever the hint - exact, permuted, partly or wholly
    wrong, repeated, out of range, pointing at an expert that is not resident - the routing outputs are
    those of the call without a hint, bit for bit, and y differs at most in the order of its fp32 sums."""
    cfg = SHAPES[name]
    E, k = cfg.E, cfg.k
    x = gen_hidden(cfg, 1, step=11, device=DEV)
    lw = LayerWeights(cfg, 0, DEV)
    ln = LayerWeights(cfg, 1, DEV, experts=[])
    ref = LayerBuffers(cfg, 1, DEV)
    layer_forward(cfg, lw, ln, x, ref, one_launch=True)
    torch.cuda.synchronize()
    assert ref.status() == 0
    true = ref.ids.cpu().numpy()[0].tolist()
    others = [e for e in range(E) if e not in true]
    # an expert that is not selected and not resident: a hint may name it without consequences
    gone = others[0]
    sz = __import__('ctypes').sizeof(B.fate_qexpert)
    lw.table[gone * sz:(gone + 1) * sz].zero_()
    hints = {
        "exact": true,
        "reversed": true[::-1],
        "one wrong": true[:1] + [others[1]] + true[2:],
        "all wrong": others[1:1 + k],
        "repeated": [true[0]] * k,
        "out of range": [-1, E + 5] + true[:k - 2],
        "not resident": [gone] + true[1:],
    }
    y_ref = f32(ref.y).astype(np.float64)
    fields = ROUTE_FIELDS + PRED_FIELDS
    got = LayerBuffers(cfg, 1, DEV)
    for what, h in hints.items():
        print(f"case {name} hint {what}: {h}", flush=True)
        hint = torch.tensor(h, dtype=torch.int32, device=DEV)
        got.y.fill_(float("nan"))
        layer_forward(cfg, lw, ln, x, got, one_launch=True, hint_ids=hint)
        torch.cuda.synchronize()
        assert got.status() == 0, what
        for f in fields:
            assert torch.equal(getattr(got, f), getattr(ref, f)), (what, f)
        assert ffn_rel_err(f32(got.y), y_ref).max() <= 1e-5, what
    # against the oracle once more, with the exact hint
    hint = torch.tensor(true, dtype=torch.int32, device=DEV)
    layer_forward(cfg, lw, ln, x, got, one_launch=True, hint_ids=hint)
    torch.cuda.synchronize()
    from workloads import gen_expert
    experts = {int(e): oracle_expert(gen_expert(cfg, 0, int(e), device=DEV)) for e in true}
    shared = [oracle_expert(gen_expert(cfg, 0, s, shared=True, device=DEV)) for s in range(cfg.n_shared)]
    sg = None if lw.shared_gate is None else f32(lw.shared_gate)
    y_orc = O.moe_ffn(f32(x), ref.ids.cpu().numpy(), ref.w.cpu().numpy().astype(np.float64), experts, shared, sg)
    assert ffn_rel_err(f32(got.y), y_orc).max() <= 2e-3


def test_layers_of_two_shapes_share_a_workspace():
    """One workspace for calls of two shapes: a call of eight tokens leaves its activations as plain fp16, all of them pairs
    (1, 0) here, and the one-token call behind it runs at the epoch with those bits (0x3c00).  Its words with an epoch tag
    lie where no other shape keeps data, so it must not take them for its own: same bits as on a workspace of its own."""
    tiny = SHAPES["tiny"]
    a = dataclasses.replace(tiny, layers=1, H=2048, E=8, k=1, I=2048, bits=4, group=128, gate_var=1.0 / 2048)
    b = dataclasses.replace(tiny, layers=1, H=1024, E=8, k=1, I=384, bits=8, group=128, gate_var=1.0 / 1024)
    la, lb = LayerWeights(a, 0, DEV), LayerWeights(b, 0, DEV)
    xa = torch.zeros(8, a.H, dtype=torch.bfloat16, device=DEV)
    xa[:, 0::2] = 1.0
    xb = gen_hidden(b, 1, device=DEV)
    ba, alone, after = LayerBuffers(a, 8, DEV), LayerBuffers(b, 1, DEV), LayerBuffers(b, 1, DEV)
    layer_forward(b, lb, None, xb, alone, one_launch=True)
    shared = torch.zeros(max(ba.layer_ws.numel(), after.layer_ws.numel()), dtype=torch.uint8, device=DEV)
    shared[:4].view(torch.int32).fill_(0x3c00 - 2)
    ba.layer_ws = after.layer_ws = shared
    layer_forward(a, la, None, xa, ba, one_launch=True)
    layer_forward(b, lb, None, xb, after, one_launch=True)
    torch.cuda.synchronize()
    assert int(shared[:4].view(torch.int32)[0]) == 0x3c00
    assert after.status() == 0 and ba.status() == 0
    for f in ROUTE_FIELDS + ("y",):
        assert torch.equal(getattr(after, f), getattr(alone, f)), f


@pytest.mark.parametrize("H,E,k,I,bits,group,n_shared,I_shared,N", [
    (2048, 16, 4, 1408, 4, 128, 2, 512, 5),        # two waves per column range, two quarters each
    (768, 16, 2, 2048, 4, 128, 0, 0, 8),           # six groups: quarters of one and two
    (512, 16, 4, 2048, 4, 256, 0, 0, 3),           # two groups: quarters without any
    (1280, 16, 4, 1280, 4, 256, 0, 0, 6),          # five groups: one wave
    (1024, 16, 4, 1152, 8, 64, 1, 384, 7),
    (1280, 16, 4, 1152, 4, 64, 1, 384, 8),         # two groups per stage, five stages per wave
    (1152, 16, 4, 1280, 4, 64, 0, 0, 4),           # the same, nine stages: one wave
])
def test_layer_by_gemms_gives_the_bits_of_the_separate_calls(H, E, k, I, bits, group, n_shared, I_shared, N):
    """The two forms of the decode-sized GEMM differ in how many waves share the columns of the up projection, not in the
    order of any sum (without a shared gate, whose dot product is taken by one wave in one form and by four in the other)."""
    cfg = dataclasses.replace(SHAPES["tiny"], name="edge", layers=1, H=H, E=E, k=k, I=I, bits=bits, group=group,
                              gate_var=1.0 / H, n_shared=n_shared, I_shared=I_shared, shared_bits=bits)
    print(f"case {H} {E} {k} {I} int{bits} g{group} N={N}", flush=True)
    x = gen_hidden(cfg, N, device=DEV)
    lw = LayerWeights(cfg, 0, DEV)
    one, sep = LayerBuffers(cfg, N, DEV), LayerBuffers(cfg, N, DEV)
    layer_forward(cfg, lw, None, x, one, one_launch=True)
    layer_forward(cfg, lw, None, x, sep, one_launch=False)
    torch.cuda.synchronize()
    assert one.status() == 0
    for f in ROUTE_FIELDS + ("y",):
        assert torch.equal(getattr(one, f), getattr(sep, f)), f


@pytest.mark.parametrize("bits,shared_bits,group", [(4, 8, 128), (8, 4, 128), (8, 8, 128), (4, 4, 128), (4, 4, 64)])
def test_layer_and_separate_calls_round_h_alike(bits, shared_bits, group):
    """Both forms round h to fp16 once, in every copy of the code.  A row whose copy rounds to fp32 in between differs in
    about one value of 2^15: eight tokens, 13312 values of h each, eight inputs."""
    cfg = dataclasses.replace(SHAPES["tiny"], name="rounding", layers=1, H=512, E=16, k=2, I=1024, bits=bits, group=group,
                              gate_var=1.0 / 512, n_shared=2, I_shared=5632, shared_bits=shared_bits)
    lw = LayerWeights(cfg, 0, DEV)
    one, sep = LayerBuffers(cfg, 8, DEV), LayerBuffers(cfg, 8, DEV)
    for step in range(8):
        print(f"int{bits} int{shared_bits} g{group} input {step}", flush=True)
        x = gen_hidden(cfg, 8, step=step, device=DEV)
        layer_forward(cfg, lw, None, x, one, one_launch=True)
        layer_forward(cfg, lw, None, x, sep, one_launch=False)
        torch.cuda.synchronize()
        assert one.status() == 0
        assert torch.equal(one.y, sep.y), (one.y != sep.y).any(1).nonzero().flatten().tolist()


@pytest.mark.parametrize("H,E,k,I,bits,shared_bits,group,n_shared,I_shared,N,distinct,zipf,whole", [
    (512, 64, 6, 1408, 4, 8, 128, 2, 384, 8, 8, 0.0, True),        # about 35 experts of 11 tiles
    (512, 64, 6, 1408, 4, 8, 128, 2, 384, 8, 2, 0.0, False),       # the same call, tokens equal but for two: about 11
    (1024, 48, 8, 1152, 4, 4, 64, 0, 0, 7, 7, 0.0, True),          # groups of 64
    (512, 64, 6, 1536, 4, 4, 256, 1, 2048, 8, 8, 0.0, True),       # of 256: a group per range of columns
    (512, 60, 4, 1408, 4, 4, 128, 1, 5632, 8, 8, 0.0, True),       # 88 shared tiles, a uniform gate ...
    (512, 60, 4, 1408, 4, 4, 128, 1, 5632, 8, 8, 1.5, False),      # ... and a Zipf gate
    (512, 64, 8, 2816, 4, 4, 128, 0, 0, 8, 8, 0.0, True),          # whole tiles beyond a round too
    (4096, 64, 6, 1408, 4, 8, 128, 2, 384, 8, 8, 0.0, True),       # long rows: two rounds of split tiles, one of whole ones
    (4096, 64, 6, 1408, 4, 8, 128, 2, 384, 8, 4, 0.0, False),
])
def test_layer_of_chosen_tiles_gives_the_bits_of_the_separate_calls(H, E, k, I, bits, shared_bits, group, n_shared, I_shared, N,
                                                                    distinct, zipf, whole):
    """Whole or split routed tiles by the number of experts that the tokens name: the same bits, and both are met."""
    cfg = dataclasses.replace(SHAPES["tiny"], name="tiles", layers=1, H=H, E=E, k=k, I=I, bits=bits, group=group,
                              gate_var=1.0 / H, n_shared=n_shared, I_shared=I_shared, shared_bits=shared_bits, zipf_s=zipf)
    print(f"case {H} {E} {k} {I} g{group} N={N} distinct {distinct} zipf {zipf}", flush=True)
    x = gen_hidden(cfg, N, device=DEV)
    x = x[:distinct].repeat(N // distinct + 1, 1)[:N].contiguous()
    lw = LayerWeights(cfg, 0, DEV)
    one, sep = LayerBuffers(cfg, N, DEV), LayerBuffers(cfg, N, DEV)
    layer_forward(cfg, lw, None, x, one, one_launch=True)
    layer_forward(cfg, lw, None, x, sep, one_launch=False)
    torch.cuda.synchronize()
    assert one.status() == 0
    # the side of the line that this case is meant for
    named = int((one.counts > 0).sum())
    tiles, shared = (I + 127) // 128, 2 * n_shared * ((I_shared + 127) // 128)
    split, whole_tiles = 2 * named * tiles + shared, named * tiles + shared
    assert (split > 512 if H <= 3072 else split > 768 and whole_tiles <= 512) == whole, (named, split, whole_tiles)
    for f in ROUTE_FIELDS + ("y",):
        assert torch.equal(getattr(one, f), getattr(sep, f)), f


@pytest.mark.parametrize("H,E,k,I,group,n_shared,I_shared,N", [
    (512, 64, 6, 1408, 128, 2, 384, 8),            # about 35 experts: 814 tiles of 64 neurons, whole routed ones instead
    (1024, 48, 8, 1152, 64, 0, 0, 7),              # the same in groups of 64
    (512, 64, 6, 1536, 256, 1, 2048, 8),           # of 256: a group per range of columns
    (512, 64, 6, 1408, 128, 2, 384, 4),            # fewer tokens: split tiles for both
])
def test_layer_of_whole_routed_and_split_shared_tiles_gives_the_bits_of_the_separate_calls(H, E, k, I, group, n_shared, I_shared, N):
    test_layer_by_gemms_gives_the_bits_of_the_separate_calls(H, E, k, I, 4, group, n_shared, I_shared, N)


@pytest.mark.parametrize("H,E,k,I,group,n_shared,I_shared,N", [
    (512, 64, 6, 1408, 128, 2, 384, 8),            # about 35 experts: 782 tiles of 64 neurons, whole routed ones instead
    (1024, 48, 8, 1152, 64, 0, 0, 7),              # the same in groups of 64
    (512, 64, 6, 1536, 256, 1, 2048, 8),           # of 256: a group per range of columns
    (512, 64, 6, 1408, 128, 2, 384, 4),            # fewer tokens: split tiles for both
])
def test_layer_of_whole_routed_and_split_shared_tiles_gives_the_bits_of_the_separate_calls(H, E, k, I, group, n_shared, I_shared, N):
    test_layer_by_gemms_gives_the_bits_of_the_separate_calls(H, E, k, I, 4, group, n_shared, I_shared, N)
