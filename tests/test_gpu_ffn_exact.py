"""The GEMM's decode-sized form (up to 16 tokens, exact weights) and the decode kernels that remain for small or
unaligned layers, at the edges of their ranges: groups that end inside a part of the reduction dimension, 16 rows
in one expert, experts smaller than I_max, sizes that are no multiple of 128.  Same bar as the other FFN tests:
per token row max_i |y - y_ref| / max_i |y_ref| <= 2e-3 (one fp16 rounding of h, 2^-11 relative)."""
import dataclasses

import numpy as np
import pytest
import torch

from oracle import moe as O
import paper_2502_12224_amd.binding as B
from paper_2502_12224_amd.stack import LayerBuffers, layer_forward
from workloads import SHAPES, gen_expert, gen_gate, gen_hidden
from helpers import DEV, GpuLayer, f32, ffn_rel_err, gpu_permute, gpu_route, oracle_expert

pytestmark = pytest.mark.gpu

SHAPE = dict(layers=1, E=4, k=4, renorm=True)       # every token selects every expert: N rows per expert


@pytest.mark.parametrize("H,I,bits,group,n_shared,I_shared,N", [
    (256, 5120, 4, 256, 0, 0, 16),          # groups of 256, parts of 640 columns in the down projection
    (1024, 4096, 4, 64, 0, 0, 16),          # two groups per stage
    (1024, 4096, 8, 128, 0, 0, 15),         # a group of two stages, a row short of the tile
    (512, 4096, 4, 128, 1, 1024, 1),        # one row; a shared expert of another size
    (192, 576, 4, 64, 0, 0, 16),            # no multiple of 128: decode kernels
    (256, 512, 4, 128, 0, 0, 9),            # small layer: decode kernels, two passes of 8 rows
])
def test_decode_sized_ffn_matches_oracle(H, I, bits, group, n_shared, I_shared, N):
    cfg = dataclasses.replace(SHAPES["tiny"], name="edge", H=H, I=I, bits=bits, group=group, gate_var=1.0 / H,
                              n_shared=n_shared, I_shared=I_shared, **SHAPE)
    x = gen_hidden(cfg, N, device=DEV)
    Wg, b = gen_gate(cfg, 0, device=DEV)
    ids, w, _ = gpu_route(x, Wg, b, cfg.k, cfg.renorm, want_probs=False)
    counts, offsets, perm, inv, order = gpu_permute(ids, cfg.E)
    L = GpuLayer(cfg, 0)
    y, ws = L.ffn(x, counts, offsets, perm, inv, order, w, mode=0, ws_fill=0)
    torch.cuda.synchronize()
    assert int(ws[:4].view(torch.int32)[0]) == 0
    y_ref = O.moe_ffn(f32(x), ids.cpu().numpy(), w.cpu().numpy().astype(np.float64),
                      {e: oracle_expert(L.host[e]) for e in range(cfg.E)}, [oracle_expert(s) for s in L.shared_host], None)
    assert ffn_rel_err(f32(y), y_ref).max() <= 2e-3


def _layer_of_unequal_experts(cfg, sizes, zero_points=False, groups=(None,)):
    """A layer whose expert e has sizes[e % len(sizes)] intermediate neurons (at most cfg.I) and the group
    groups[e % len(groups)] (None: the layer's); shared experts likewise, cfg.I_shared - 64 the first one."""
    L = GpuLayer(cfg, 0, experts=[])
    for e in range(cfg.E):
        c = dataclasses.replace(cfg, I=sizes[e % len(sizes)])
        L.host[e] = gen_expert(c, 0, e, device=DEV, group=groups[e % len(groups)], zero_points=zero_points)
        L.packed[e] = B.PackedExpert(L.host[e], DEV)
    L.table = B.expert_table([L.packed[e].struct() for e in range(cfg.E)], DEV)
    for s in range(cfg.n_shared):
        c = dataclasses.replace(cfg, I_shared=cfg.I_shared - (64 if s == 0 else 0))
        L.shared_host[s] = gen_expert(c, 0, s, shared=True, device=DEV)
        L.shared_packed[s] = B.PackedExpert(L.shared_host[s], DEV)
    if cfg.n_shared:
        L.shared_table = B.expert_table([p.struct() for p in L.shared_packed], DEV)
    return L


def _oracle_ffn(L, cfg, x, ids, w):
    return O.moe_ffn_grouped(f32(x), ids.cpu().numpy(), w.cpu().numpy().astype(np.float64),
                             {e: oracle_expert(L.host[e]) for e in range(cfg.E)}, [oracle_expert(s) for s in L.shared_host], None)


def _edge(H, E, k, I, bits, group, n_shared=0, I_shared=0, shared_bits=4):
    return dataclasses.replace(SHAPES["tiny"], name="edge", layers=1, H=H, E=E, k=k, I=I, bits=bits, group=group,
                               gate_var=1.0 / H, n_shared=n_shared, I_shared=I_shared, shared_bits=shared_bits)


@pytest.mark.parametrize("bits,group,groups,zp,N,mode", [
    (4, 64, (None,), False, 8, 0),
    (4, 64, (None,), True, 16, 0),
    (8, 64, (None,), False, 16, 1),
    (4, 128, (64,), False, 13, 0),          # the layer's group is 128, its experts' 64
    (4, 64, (None,), False, 40, 2),         # prefill form
    (4, 64, (None,), True, 40, 2),
    (8, 64, (None,), False, 40, 2),
])
@pytest.mark.parametrize("E,k,I,sizes", [
    (64, 8, 256, (192, 256, 64)),                       # whole sums
    (16, 4, 2048, (1984, 2048, 64, 1088)),              # parts of the reduction dimension
])
def test_experts_smaller_than_i_max(E, k, I, sizes, bits, group, groups, zp, N, mode):
    """Entries whose intermediate size is any multiple of 64 up to I_max, routed and shared: the down projection
    takes all of their columns."""
    cfg = _edge(512, E, k, I, bits, group, n_shared=2, I_shared=384, shared_bits=bits)
    print(f"case E={E} I={I} bits={bits} group={group}{groups} zp={zp} N={N} mode={mode}", flush=True)
    if groups != (None,):
        cfg = dataclasses.replace(cfg, n_shared=0, I_shared=0)      # (a shared entry of 320 neurons has no groups of 128)
    x = gen_hidden(cfg, N, device=DEV)
    Wg, b = gen_gate(cfg, 0, device=DEV)
    ids, w, _ = gpu_route(x, Wg, b, cfg.k, cfg.renorm, want_probs=False)
    L = _layer_of_unequal_experts(cfg, sizes, zp, groups)
    y, ws = L.ffn(x, *gpu_permute(ids, cfg.E), w, mode=mode, ws_fill=0xff)
    assert int(ws[:4].view(torch.int32)[0]) == 0
    assert ffn_rel_err(f32(y), _oracle_ffn(L, cfg, x, ids, w)).max() <= 2e-3


@pytest.mark.parametrize("bits,E,k,I,sizes,N", [
    (4, 64, 8, 256, (192, 256, 64), 8),
    (8, 64, 8, 256, (192, 256, 64), 8),
    (4, 16, 4, 2048, (1984, 2048, 64, 1088), 5),
])
def test_decode_layer_of_experts_smaller_than_i_max(bits, E, k, I, sizes, N):
    cfg = _edge(512, E, k, I, bits, 64, n_shared=2, I_shared=384, shared_bits=bits)
    print(f"case decode layer E={E} I={I} bits={bits} N={N}", flush=True)
    x = gen_hidden(cfg, N, device=DEV)
    L = _layer_of_unequal_experts(cfg, sizes)
    L.Wg, L.bias = gen_gate(cfg, 0, device=DEV)
    buf = LayerBuffers(cfg, N, DEV)
    layer_forward(cfg, L, None, x, buf, one_launch=True)
    torch.cuda.synchronize()
    assert buf.status() == 0
    assert ffn_rel_err(f32(buf.y), _oracle_ffn(L, cfg, x, buf.ids, buf.w)).max() <= 2e-3


@pytest.mark.parametrize("bits,group,zp,N,k", [(4, 128, False, 16, 4), (4, 64, True, 13, 4), (8, 64, False, 16, 8), (4, 128, False, 9, 3)])
def test_tokens_that_name_an_expert_more_than_once(bits, group, zp, N, k):
    """Ids need not be distinct within a token (padding rows name one expert k times): an expert then has up to N * k
    rows, in calls of up to 16 tokens more than one tile of the decode-sized form."""
    cfg = _edge(512, 16, k, 2048, bits, group)
    print(f"case repeated ids bits={bits} group={group} zp={zp} N={N} k={k}", flush=True)
    ids = torch.randint(0, cfg.E, (N, k), dtype=torch.int32, generator=torch.Generator().manual_seed(N))
    ids[: N - N // 4] = 5                   # (the rest of the tokens adds the rows that end inside a tile)
    ids[-1, :] = 9
    ids = ids.to(DEV)
    w = (torch.rand(N, k, generator=torch.Generator().manual_seed(3)) + 0.1).to(DEV)
    x = gen_hidden(cfg, N, device=DEV)
    L = _layer_of_unequal_experts(cfg, (2048, 1024 + 128), zp)
    y, ws = L.ffn(x, *gpu_permute(ids, cfg.E), w, ws_fill=0xff)
    assert int(ws[:4].view(torch.int32)[0]) == 0
    assert ffn_rel_err(f32(y), _oracle_ffn(L, cfg, x, ids, w)).max() <= 2e-3
