"""GPU parity of routing, prediction and permutation against the oracle
(through the C ABI).  Integer outputs must match bit for bit; rows whose
oracle logits have a top-k gap below 1e-5 are counted apart."""
import dataclasses

import numpy as np
import pytest
import torch

from oracle import moe as O
import paper_2502_12224_amd.binding as B
from workloads import SHAPES, gen_gate, gen_hidden
from helpers import DEV, bias_np, check_routing, f32, gpu_permute, gpu_predict, gpu_route

pytestmark = pytest.mark.gpu

CASES = [("tiny", 16), ("qwen", 1), ("qwen", 5), ("qwen", 77), ("qwen_prefill", 512), ("qwen_prefill", 2048),
         ("deepseek", 8), ("deepseek", 1024), ("mixtral", 1), ("mixtral", 3), ("mixtral", 300), ("mixtral", 2048)]


@pytest.mark.parametrize("name,N", CASES)
def test_gate_route_matches_oracle(name, N):
    cfg = SHAPES[name]
    x = gen_hidden(cfg, N, device=DEV)
    Wg, b = gen_gate(cfg, 0, device=DEV)
    ids, w, probs = gpu_route(x, Wg, b, cfg.k, cfg.renorm)
    torch.cuda.synchronize()
    rid, rw, rp, rz = O.gate_route(f32(x), f32(Wg), bias_np(b), cfg.k, cfg.renorm)
    nt = check_routing(ids, w, rid, rw, rz, cfg.k, f"{name} N={N}")
    assert nt <= max(1, N // 200)
    p = probs.cpu().numpy().astype(np.float64)
    assert np.abs(p - rp).max() <= 1e-6 and np.allclose(p.sum(1), 1, atol=1e-5)


@pytest.mark.parametrize("name,N", CASES)
def test_cross_layer_predict_matches_oracle(name, N):
    cfg = SHAPES[name]
    x = gen_hidden(cfg, N, device=DEV)
    Wg1, b1 = gen_gate(cfg, 1, device=DEV)
    m = cfg.m
    ids, w, pop = gpu_predict(x, Wg1, b1, cfg.k, m)
    torch.cuda.synchronize()
    rid, rw, rpop, rz = O.cross_layer_predict(f32(x), f32(Wg1), bias_np(b1), m)
    nt = check_routing(ids, w, rid, rw, rz, m, f"{name} N={N}")
    if nt == 0:
        assert np.array_equal(pop.cpu().numpy(), rpop)
    assert int(pop.sum()) == N * m
    # identity: the same gate on the same input is that layer's true routing
    tid, tw, _ = gpu_route(x, Wg1, b1, cfg.k, False, want_probs=False)
    assert torch.equal(tid, ids[:, :cfg.k]) and torch.equal(tw, w[:, :cfg.k])


@pytest.mark.parametrize("N,k,E", [(0, 2, 8), (1, 4, 60), (16, 2, 8), (5, 6, 64), (512, 4, 60), (2048, 6, 64),
                                   (4096, 8, 256), (1000, 1, 3),
                                   # both sides of the popularity order's two forms, and of the ids kept in registers
                                   (65, 1, 64), (64, 8, 60), (513, 1, 64), (65, 1, 65), (300, 1, 200), (8193, 1, 64)])
def test_permute_matches_oracle(N, k, E):
    rng = np.random.default_rng(N * 7 + k)
    # skewed draws without repeats inside a row
    pw = 1.0 / np.arange(1, E + 1) ** 1.1
    ids = np.stack([rng.choice(E, size=k, replace=False, p=pw / pw.sum()) for _ in range(N)]).astype(np.int32) \
        if N else np.zeros((0, k), np.int32)
    g = gpu_permute(torch.from_numpy(ids).to(DEV), E)
    torch.cuda.synchronize()
    ref = O.permute(ids, E)
    for a, r, nm in zip(g, ref, ("counts", "offsets", "perm", "inv_perm", "expert_order")):
        assert np.array_equal(a.cpu().numpy(), r), nm


def test_permute_drops_out_of_range_ids():
    ids = torch.tensor([[0, 9], [3, -1], [3, 0]], dtype=torch.int32, device=DEV)
    counts, offsets, perm, inv, order = gpu_permute(ids, 4)
    assert counts.tolist() == [2, 0, 0, 2] and offsets.tolist() == [0, 2, 2, 2, 4]
    assert perm[:4].tolist() == [0, 5, 2, 4] and inv.tolist() == [0, -1, 2, -1, 3, 1]


@pytest.mark.parametrize("name,N", [("tiny", 16), ("qwen", 1), ("qwen", 5), ("deepseek", 8), ("mixtral", 1), ("mixtral", 4),
                                    ("qwen", 512), ("qwen", 2047), ("deepseek", 1024), ("mixtral", 2048)])
def test_route_fused_equals_the_three_calls(name, N):
    cfg = SHAPES[name]
    x = gen_hidden(cfg, N, device=DEV)
    Wg, b = gen_gate(cfg, 0, device=DEV)
    Wg1, b1 = gen_gate(cfg, 1, device=DEV)
    E, k, m = cfg.E, cfg.k, cfg.m
    ws = torch.zeros(B.fate_route_fused_workspace(N, E), dtype=torch.uint8, device=DEV)
    mk = lambda *s, dt=torch.int32: torch.full(s, -3, dtype=dt, device=DEV)
    for rep in range(3):           # the workspace must come back clean
        ids, w = mk(N, k), mk(N, k, dt=torch.float32)
        pid, pw, pop = mk(N, m), mk(N, m, dt=torch.float32), mk(E)
        counts, offsets, perm, inv, order = mk(E), mk(E + 1), mk(N * k), mk(N * k), mk(E)
        B.fate_route_fused(x, Wg, b, Wg1, b1, k, m, cfg.renorm, ids, w, pid, pw, pop, counts, offsets, perm, inv,
                           order, ws)
        torch.cuda.synchronize()
        assert int(ws[:4].view(torch.int32)[0]) == 0
        sid, sw, _ = gpu_route(x, Wg, b, k, cfg.renorm, want_probs=False)
        spid, spw, spop = gpu_predict(x, Wg1, b1, k, m)
        sperm = gpu_permute(sid, E)
        torch.cuda.synchronize()
        for a, r in ((ids, sid), (w, sw), (pid, spid), (pw, spw), (pop, spop), (counts, sperm[0]),
                     (offsets, sperm[1]), (perm, sperm[2]), (inv, sperm[3]), (order, sperm[4])):
            assert torch.equal(a, r)
    # last layer: no next gate
    ids, w = mk(N, k), mk(N, k, dt=torch.float32)
    B.fate_route_fused(x, Wg, b, None, None, k, m, cfg.renorm, ids, w, None, None, None, counts, offsets, perm,
                       inv, order, ws)
    torch.cuda.synchronize()
    assert torch.equal(ids, sid) and torch.equal(w, sw)


@pytest.mark.parametrize("H,E,k,N", [(64, 8, 2, 512), (64, 8, 2, 513), (192, 60, 4, 1023), (1920, 16, 2, 2048), (64, 5, 5, 2049), (192, 200, 8, 2051)])
def test_gates_of_odd_sizes_over_many_tokens_match_oracle(H, E, k, N):
    """H no multiple of 1024: both sides of the lines between workgroups of 16 waves and of 4, a token and four tokens each."""
    cfg = dataclasses.replace(SHAPES["tiny"], H=H, E=E, k=k, gate_var=1.0 / H)
    x = gen_hidden(cfg, N, device=DEV)
    Wg, b = gen_gate(cfg, 0, device=DEV)
    ids, w, probs = gpu_route(x, Wg, b, k, False)
    rid, rw, rp, rz = O.gate_route(f32(x), f32(Wg), bias_np(b), k, False)
    assert check_routing(ids, w, rid, rw, rz, k, f"H={H} E={E} N={N}") <= max(1, N // 200)
    assert np.abs(probs.cpu().numpy().astype(np.float64) - rp).max() <= 1e-6


@pytest.mark.parametrize("E,k,N", [(8, 2, 3), (16, 4, 9), (17, 5, 12), (60, 4, 16), (64, 8, 8), (65, 8, 7), (128, 8, 5), (129, 6, 40),
                                   (200, 8, 64), (256, 8, 130)])
def test_equal_logits_and_equal_counts_go_to_the_lower_id(E, k, N):
    """Every third gate row is the row before it (equal logits in every token, whatever the order of summation), the last
    two rows are zero; sizes at both sides of the selection's blocks of 16 and 64 entries.  All calls that
    select agree with the oracle's order, and experts with equal counts are ordered by id."""
    H = 1024
    print(f"case E={E} k={k} N={N}", flush=True)
    cfg = dataclasses.replace(SHAPES["tiny"], H=H, E=E, k=k, gate_var=1.0 / H)
    x = gen_hidden(cfg, N, device=DEV)
    Wg, _ = gen_gate(cfg, 0, device=DEV)
    for e in range(2, E, 3):
        Wg[e] = Wg[e - 1]
    Wg[-2:] = 0.0
    m = min(E, k + 3)
    ids, w, _ = gpu_route(x, Wg, None, k, True, want_probs=False)
    pid, pw, pop = gpu_predict(x, Wg, None, k, m)
    z = np.zeros((N, E))
    z[:] = f32(x).astype(np.float64) @ f32(Wg).astype(np.float64).T
    for e in range(2, E, 3):
        if e < E - 2:
            z[:, e] = z[:, e - 1]
    z[:, -2:] = 0.0
    ref = np.argsort(-z, axis=1, kind="stable")
    gaps = np.sort(z, axis=1)[:, ::-1]
    d = gaps[:, :-1] - gaps[:, 1:]
    ok = ~((d[:, : m + 1] > 0) & (d[:, : m + 1] < 1e-5)).any(axis=1)       # (rows that are near-ties by accident)
    assert ok.sum() >= N - max(1, N // 20)
    assert np.array_equal(ids.cpu().numpy()[ok], ref[ok, :k]) and np.array_equal(pid.cpu().numpy()[ok], ref[ok, :m])
    got = gpu_permute(ids, E)
    for a, r, nm in zip(got, O.permute(ids.cpu().numpy(), E), ("counts", "offsets", "perm", "inv_perm", "expert_order")):
        assert np.array_equal(a.cpu().numpy(), r), nm
    assert np.array_equal(pop.cpu().numpy(), np.bincount(pid.cpu().numpy().ravel(), minlength=E))
    if N <= 16 or N >= 64:
        ws = torch.zeros(B.fate_route_fused_workspace(N, E), dtype=torch.uint8, device=DEV)
        mk = lambda *s, dt=torch.int32: torch.full(s, -3, dtype=dt, device=DEV)
        f = dict(ids=mk(N, k), w=mk(N, k, dt=torch.float32), pid=mk(N, m), pw=mk(N, m, dt=torch.float32), pop=mk(E))
        perm = (mk(E), mk(E + 1), mk(N * k), mk(N * k), mk(E))
        B.fate_route_fused(x, Wg, None, Wg, None, k, m, True, f["ids"], f["w"], f["pid"], f["pw"], f["pop"], *perm, ws)
        torch.cuda.synchronize()
        for a, r in zip((f["ids"], f["w"], f["pid"], f["pw"], f["pop"], *perm), (ids, w, pid, pw, pop, *got)):
            assert torch.equal(a, r)


@pytest.mark.parametrize("E,masked,k,m,N", [(64, 4, 4, 6, 13), (64, 4, 4, 6, 48), (64, 4, 4, 6, 130), (16, 8, 4, 12, 5), (130, 70, 8, 61, 20),
                                            (12, 11, 1, 2, 70)])
def test_masked_experts_and_tokens_without_input(E, masked, k, m, N):
    """Experts masked by a bias of -inf (all of them equal) behind the selection, across its end and inside it, and tokens
    whose x is zero (all logits equal): equal logits go to the lower id."""
    H = 1024
    print(f"case E={E} masked={masked} k={k} m={m} N={N}", flush=True)
    cfg = dataclasses.replace(SHAPES["tiny"], H=H, E=E, k=k, gate_var=1.0 / H)
    x = gen_hidden(cfg, N, device=DEV)
    x[1::3] = 0.0
    Wg, _ = gen_gate(cfg, 0, device=DEV)
    bias = torch.zeros(E, device=DEV)
    bias[torch.randperm(E, generator=torch.Generator().manual_seed(E))[:masked].to(DEV)] = float("-inf")
    ids, w, _ = gpu_route(x, Wg, bias, k, False, want_probs=False)
    pid, pw, pop = gpu_predict(x, Wg, bias, k, m)
    z = f32(x).astype(np.float64) @ f32(Wg).astype(np.float64).T + bias.cpu().numpy()
    ref = np.argsort(-z, axis=1, kind="stable")
    top = -np.sort(-z, axis=1)[:, : m + 1]
    with np.errstate(invalid="ignore"):
        d = top[:, :-1] - top[:, 1:]
    ok = ~((d > 0) & (d < 1e-5)).any(axis=1)               # (rows that are near-ties by accident)
    assert ok.sum() >= N - max(1, N // 20)
    assert np.array_equal(ids.cpu().numpy()[ok], ref[ok, :k]) and np.array_equal(pid.cpu().numpy()[ok], ref[ok, :m])
    assert np.array_equal(pop.cpu().numpy(), np.bincount(pid.cpu().numpy().ravel(), minlength=E))
    assert (pw.cpu().numpy()[np.isneginf(np.take_along_axis(z, pid.cpu().numpy().astype(np.int64), axis=1))] == 0).all()
