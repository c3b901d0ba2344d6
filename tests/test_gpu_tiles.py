"""The GEMM kernels at the edges of their tiles and the routing kernels at the edges of their row loads.
Same bars as the other tests: FFN per token row max_i |y - y_ref| / max_i |y_ref| <= 2e-3 (h is rounded to fp16 once,
weights in tiles of more than 32 rows, too, 2^-11 relative each), ids and permutations equal."""
import dataclasses

import numpy as np
import pytest
import torch

from oracle import moe as O
import paper_2502_12224_amd.binding as B
from paper_2502_12224_amd.stack import LayerBuffers, layer_forward
from workloads import SHAPES, gen_expert, gen_gate, gen_hidden
from helpers import DEV, GpuLayer, f32, ffn_rel_err, gpu_permute, gpu_route, oracle_expert
from test_gpu_layer_fused import _one_launch_case

pytestmark = pytest.mark.gpu

ROWS = (1, 31, 32, 33, 64, 65, 96, 97, 128, 129)        # rows per expert: both sides of every tile size


@pytest.mark.parametrize("H,I,bits,n_shared,I_shared", [
    (256, 384, 4, 0, 0),                    # whole sums, fp16 outputs
    (384, 2048, 4, 0, 0),                   # parts of the reduction dimension, fp32 outputs
    (256, 2048, 8, 1, 384),                 # parts of the routed experts' only, tiles of 64 rows
    (256, 384, 4, 1, 2048),                 # parts of the shared expert's only
    (256, 1536, 4, 2, 1152),                # parts of both
])
def test_prefill_gemm_at_its_tile_edges(H, I, bits, n_shared, I_shared):
    cfg = dataclasses.replace(SHAPES["tiny"], name="edge", layers=1, H=H, E=len(ROWS), k=1, I=I, bits=bits, group=128,
                              gate_var=1.0 / H, n_shared=n_shared, I_shared=I_shared)
    ids = np.repeat(np.arange(cfg.E), ROWS)
    ids = np.random.default_rng(7).permutation(ids).astype(np.int32)[:, None]
    N = len(ids)
    x = gen_hidden(cfg, N, device=DEV)
    w = torch.rand(N, 1, generator=torch.Generator().manual_seed(3)).to(DEV) + 0.1
    L = GpuLayer(cfg, 0)
    y, ws = L.ffn(x, *gpu_permute(torch.from_numpy(ids).to(DEV), cfg.E), w, mode=2, ws_fill=0xff)
    assert int(ws[:4].view(torch.int32)[0]) == 0
    sg = None if L.shared_gate is None else f32(L.shared_gate)
    y_ref = O.moe_ffn_grouped(f32(x), ids, w.cpu().numpy().astype(np.float64),
                              {e: oracle_expert(L.host[e]) for e in range(cfg.E)},
                              [oracle_expert(s) for s in L.shared_host], sg)
    assert ffn_rel_err(f32(y), y_ref).max() <= 2e-3


@pytest.mark.parametrize("bits,widths,zp", [(4, (2, 8), False), (4, (2, 4), True), (8, (4, 8, 2), False)])
def test_prefill_gemm_on_entries_of_other_widths(bits, widths, zp):
    """Entries of another width than the layer's nominal one: 2- and 8-bit rows in passes of 64 within tiles of 128 rows
    (4-bit layer), 4-bit rows in tiles of 64 (8-bit layer)."""
    cfg = dataclasses.replace(SHAPES["tiny"], name="edge", layers=1, H=256, E=len(ROWS), k=1, I=384, bits=bits, group=128,
                              gate_var=1.0 / 256)
    ids = np.repeat(np.arange(cfg.E), ROWS)
    for turn in range(len(widths)):         # every number of rows at every width
        print(f"case nominal {bits} widths {widths} turn {turn} zp={zp}", flush=True)
        order = np.random.default_rng(turn).permutation(len(ids))
        ids_t = ids[order].astype(np.int32)[:, None]
        x = gen_hidden(cfg, len(ids), device=DEV)
        w = torch.rand(len(ids), 1, generator=torch.Generator().manual_seed(3)).to(DEV) + 0.1
        L = GpuLayer(cfg, 0, experts=[])
        for e in range(cfg.E):
            L.host[e] = gen_expert(cfg, 0, e, device=DEV, bits=widths[(e + turn) % len(widths)], zero_points=zp)
            L.packed[e] = B.PackedExpert(L.host[e], DEV)
        L.table = B.expert_table([L.packed[e].struct() for e in range(cfg.E)], DEV)
        y, ws = L.ffn(x, *gpu_permute(torch.from_numpy(ids_t).to(DEV), cfg.E), w, mode=2, ws_fill=0xff)
        assert int(ws[:4].view(torch.int32)[0]) == 0
        y_ref = O.moe_ffn_grouped(f32(x), ids_t, w.cpu().numpy().astype(np.float64),
                                  {e: oracle_expert(L.host[e]) for e in range(cfg.E)}, [], None)
        assert ffn_rel_err(f32(y), y_ref).max() <= 2e-3


_QWEN = SHAPES["qwen"]
LAYERS = {
    "64pairs": (dataclasses.replace(_QWEN, H=1152, E=200, k=8, gate_var=1 / 1152), 8),       # one range of columns, E > 64
    "int8g64": (dataclasses.replace(_QWEN, H=1024, E=96, I=896, bits=8, group=64, n_shared=2, I_shared=384,
                                    shared_bits=4, gate_var=1 / 1024), 3),
    "odd-blocks": (dataclasses.replace(_QWEN, H=768, E=17, k=5, I=1152, n_shared=0, I_shared=0, gate_var=1 / 768), 7),
    "one-token": (dataclasses.replace(_QWEN, H=1280, E=10, k=4, I=4096, n_shared=0, I_shared=0, gate_var=1 / 1280), 1),
}


@pytest.mark.parametrize("name", list(LAYERS))
def test_decode_layer_by_gemms_at_its_edges(name):
    cfg, N = LAYERS[name]
    _one_launch_case(cfg, name, N, False)


@pytest.mark.parametrize("H", [64, 256, 1024])
def test_infinite_gate_weight_stays_in_its_column(H):
    """An infinite gate weight makes its expert's logit infinite (never NaN: lanes past the end of a row must not
    multiply it by zero), so the expert leads every token's selection."""
    cfg = dataclasses.replace(SHAPES["tiny"], H=H, E=12, k=2, gate_var=1.0 / H)
    x = gen_hidden(cfg, 5, device=DEV)
    x[:, 0] = 1.0
    Wg, b = gen_gate(cfg, 0, device=DEV)
    Wg[7, 0] = float("inf")
    ids, _, _ = gpu_route(x, Wg, b, cfg.k, False, want_probs=False)
    assert ids[:, 0].tolist() == [7] * 5


FEW_ROWS = (1, 15, 16, 17, 31, 32, 33)   # both sides of the few-row forms' blocks of 16 and of their end


@pytest.mark.parametrize("bits,group,zp,scale", [        # scale 0: a common component and outlier channels
    (4, 64, False, 1.0),                    # stages of 64 columns
    (4, 64, True, 1.0),
    (4, 192, False, 1.0),                   # the same, groups of three stages
    (4, 128, False, 1.0),                   # stages of 128 columns
    (4, 256, True, 1.0),                    # groups of two stages
    (8, 64, False, 1.0),
    (2, 128, False, 1.0),
    (2, 256, True, 1.0),
    (4, 128, False, 2.0 ** -3),             # small and large activations
    (4, 128, False, 2.0 ** 5),
    (4, 128, False, 0), (4, 64, True, 0), (8, 64, False, 0), (2, 128, False, 0), (2, 128, True, 0),
])
def test_tiles_of_few_rows_in_every_format(bits, group, zp, scale):
    """The forms for tiles of at most 32 rows (and the next larger one) in every format they read.  (With x scaled by
    2^-3 h is about 2^-9, far above the 2^-14 below which fp16 loses bits; by 2^5 about 2^8.)  Activations with a common
    component and a few channels 40 times as large make every group's sum large: with zero-points their share of the
    products comes from that sum."""
    cfg = dataclasses.replace(SHAPES["tiny"], name="few", layers=1, H=768, E=len(FEW_ROWS), k=1, I=768, bits=bits,
                              group=group, gate_var=1.0 / 768)
    print(f"case bits={bits} group={group} zp={zp} scale={scale}", flush=True)
    ids = np.random.default_rng(5).permutation(np.repeat(np.arange(cfg.E), FEW_ROWS)).astype(np.int32)[:, None]
    x = gen_hidden(cfg, len(ids), device=DEV).float() * (scale or 1.0)
    if not scale:
        x += 3.0
        x[:, 5::97] *= 40.0
    x = x.to(torch.bfloat16)
    w = torch.rand(len(ids), 1, generator=torch.Generator().manual_seed(3)).to(DEV) + 0.1
    L = GpuLayer(cfg, 0, experts=[])
    for e in range(cfg.E):
        L.host[e] = gen_expert(cfg, 0, e, device=DEV, zero_points=zp)
        L.packed[e] = B.PackedExpert(L.host[e], DEV)
    L.table = B.expert_table([L.packed[e].struct() for e in range(cfg.E)], DEV)
    y, ws = L.ffn(x, *gpu_permute(torch.from_numpy(ids).to(DEV), cfg.E), w, mode=2, ws_fill=0xff)
    assert int(ws[:4].view(torch.int32)[0]) == 0
    y_ref = O.moe_ffn_grouped(f32(x), ids, w.cpu().numpy().astype(np.float64),
                              {e: oracle_expert(L.host[e]) for e in range(cfg.E)}, [], None)
    assert ffn_rel_err(f32(y), y_ref).max() <= 2e-3


def _overflowing(ex, how):
    """h: intermediate neuron 5 leaves the range of fp16 for about every second token.  x: every W1 and W3 weight positive, a
    row of W2 of one sign, so that an infinite activation makes h infinite and y infinite of the row's sign."""
    if how == "h":
        ex.s1[5], ex.s3[5] = 64.0, 64.0
    else:
        for w in (ex.w1, ex.w3, ex.w2):
            w.fill_(0x7f if ex.bits == 8 else 0xff)
        ex.w2[1::2] = {8: 0x81, 4: 0x11, 2: 0x00}[ex.bits]
    return ex


# (the decode layer reads symmetric entries of 4 and 8 bits, and an infinite x makes its gate's logits NaN)
_INFINITE = [(form, how, *fmt) for form in ("prefill", "decode", "layer") for how in ("h", "x")
             for fmt in ((4, 128, False), (4, 64, False), (8, 64, False), (4, 128, True), (4, 64, True), (2, 128, False), (2, 128, True))
             if form != "layer" or (how == "h" and fmt[0] != 2 and not fmt[2])]


@pytest.mark.parametrize("form,how,bits,group,zp", _INFINITE)
def test_infinite_activations_are_infinite_in_every_form(form, how, bits, group, zp):
    """A token whose x is infinite, or whose h leaves the range of fp16: every column of y is what IEEE arithmetic on the
    stored weights gives, +-inf or NaN (a weight of zero), however many rows its expert has; the other tokens of its tile
    are as precise as ever.  Tiles of 1 to 33 rows, the decode-sized call, the decode layer."""
    rows = FEW_ROWS if form == "prefill" else (1, 8, 5, 2) if form == "decode" else (2, 2, 2, 2)
    H, I = (256, 256) if form == "prefill" else (256, 4096)
    cfg = dataclasses.replace(SHAPES["tiny"], name="inf", layers=1, H=H, E=len(rows), k=1, I=I, bits=bits, group=group,
                              gate_var=1.0 / H)
    print(f"case {form} infinite {how} bits={bits} group={group} zp={zp}", flush=True)
    ids = np.random.default_rng(5).permutation(np.repeat(np.arange(cfg.E), rows)).astype(np.int32)[:, None]
    x = gen_hidden(cfg, len(ids), device=DEV)
    if how == "x":
        x.abs_()                            # (all neurons have nearly the same h: a negative sum would make them vanish in fp16)
        x[::3, 77] = float("inf")
    w = torch.rand(len(ids), 1, generator=torch.Generator().manual_seed(3)).to(DEV) + 0.1
    L = GpuLayer(cfg, 0, experts=[])
    for e in range(cfg.E):
        L.host[e] = _overflowing(gen_expert(cfg, 0, e, device=DEV, zero_points=zp), how)
        L.packed[e] = B.PackedExpert(L.host[e], DEV)
    L.table = B.expert_table([L.packed[e].struct() for e in range(cfg.E)], DEV)
    if form == "layer":
        # a gate that gives every token its expert of ids
        L.Wg, L.bias = torch.zeros(cfg.E, H, dtype=torch.bfloat16, device=DEV), None
        L.Wg[:, :4] = torch.eye(4, device=DEV)
        x[:, :4] = 0.0
        x[torch.arange(len(ids)), torch.from_numpy(ids[:, 0].astype(np.int64))] = 8.0
        buf = LayerBuffers(cfg, len(ids), DEV)
        layer_forward(cfg, L, None, x, buf, one_launch=True)
        torch.cuda.synchronize()
        assert buf.status() == 0 and torch.equal(buf.ids.cpu(), torch.from_numpy(ids))
        y, w = f32(buf.y), buf.w
    else:
        y, ws = L.ffn(x, *gpu_permute(torch.from_numpy(ids).to(DEV), cfg.E), w, mode=2 if form == "prefill" else 1, ws_fill=0xff)
        assert int(ws[:4].view(torch.int32)[0]) == 0
        y = f32(y)
    x, w = f32(x).astype(np.float64), w.cpu().numpy().astype(np.float64)
    experts = [oracle_expert(L.host[e]) for e in range(cfg.E)]
    infinite = 0
    for t in range(len(ids)):
        ex = experts[ids[t, 0]]
        with np.errstate(all="ignore"):
            g, u = (ex.W1 * x[t]).sum(axis=1), (ex.W3 * x[t]).sum(axis=1)
            h = g / (1.0 + np.exp(-g)) * u
            h[np.abs(h) >= 65520.0] = np.copysign(np.inf, h[np.abs(h) >= 65520.0])
            ref = w[t, 0] * (ex.W2 * h).sum(axis=1)
        if np.isinf(h).any():
            infinite += 1
            assert not np.isfinite(ref).any() and (ref > 0).any() and (ref < 0).any()
            assert np.array_equal(np.isnan(y[t]), np.isnan(ref)) and np.array_equal(y[t] > 0, ref > 0), (t, rows[ids[t, 0]])
        else:
            assert np.abs(y[t] - ref).max() <= 2e-3 * np.abs(ref).max(), t
    assert 0 < infinite < len(ids)
