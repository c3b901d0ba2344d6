"""The GEMM's decode-sized form (up to 16 tokens, exact weights) and the decode kernels that remain for small or
unaligned layers, at the edges of their ranges: groups that end inside a part of the reduction dimension, 16 rows
in one expert, experts smaller than I_max, sizes that are no multiple of 128.  Same bar as the other FFN tests:
per token row max_i |y - y_ref| / max_i |y_ref| <= 2e-3 (one fp16 rounding of h, 2^-11 relative)."""
import dataclasses

import numpy as np
import pytest
import torch

from oracle import moe as O
from workloads import SHAPES, gen_gate, gen_hidden
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
