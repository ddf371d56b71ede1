"""Parity of the wide batched kernels (more than 16 tokens per weight set)
against the fp64 oracle at the edges of their token tiles (32, 64, 128
slots, several groups), row tiles, K padding and column slices, against the
one-pass kernels they replace, and the three-part MoE form at the
single-token kernels' tolerance (its x and Combined keep all 24 bits)."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import (TIGHT_SINGLE, assert_elementwise, check_ffn_output, compare_sets, ffn_inputs_to_dev, list_of,
                      moe_bound, rel_l2, to_dev)
from paper_2406_05955_amd import synth
from test_gpu_exact_batch import launches

pytestmark = pytest.mark.gpu

ts = pytest.importorskip("paper_2406_05955_amd.binding") if torch.cuda.is_available() else None


@pytest.mark.parametrize("B,H,I", [(17, 8, 1), (32, 1000, 65), (33, 4096, 130), (64, 264, 1500), (65, 512, 700),
                                   (128, 1032, 33), (129, 256, 513), (200, 2048, 300), (256, 520, 2100),
                                   (129, 136, 12289), (256, 64, 12300)])
def test_wide_ffn(B, H, I):
    inp = synth.make_ffn(B, H, I, gate_bias=-0.84, dtype=synth.BF16, seed=[71, B, H, I])
    ref = oracle.ffn(inp.x, inp.w_gate, inp.w_up, inp.w_down_t, inp.dtype)
    x, wg, wu, wd = ffn_inputs_to_dev(inp)
    ws = torch.empty(ts.ffn_workspace_bytes(B, H, I, ts.TS_BF16), dtype=torch.uint8, device="cuda")
    ws.fill_(0xFF)  # NaN in every type: nothing stale may be read
    out, st = ts.ffn_sparse(x, wg, wu, wd, stats=True, ws=ws)
    ws.fill_(0xFF)
    again = ts.ffn_sparse(x, wg, wu, wd, ws=ws)
    dense = ts.ffn_dense(x, wg, wu, wd, ws=ws)
    ts.tune_set("bx_wide", 1)
    try:
        narrow = ts.ffn_sparse(x, wg, wu, wd)
    finally:
        ts.tune_set("bx_wide", 0)
    torch.cuda.synchronize()
    assert torch.equal(out.view(torch.int32), again.view(torch.int32))
    for o, what in ((out, "sparse"), (dense, "dense")):
        check_ffn_output(o.cpu().numpy(), ref.y, inp.x, inp.w_gate, inp.w_up, inp.w_down_t, ref.g, ref.u,
                         batched=True, what=f"wide {what} B={B} H={H} I={I}")
    # either route is within 1e-4 of the oracle
    assert rel_l2(out.cpu().numpy(), narrow.cpu().numpy().astype(np.float64)) <= 2e-4
    for t in range(B):
        g, u = ref.g[t], ref.u[t]
        keep_g = np.abs(g) >= 1e-3
        keep_a = keep_g & (np.abs(u) >= 1e-3)
        assert compare_sets(list_of(st, "gate_idx", t, "n_gate"), g > 0, keep_g) == 0, t
        assert compare_sets(list_of(st, "active_idx", t, "n_active"), (g > 0) & (u > 0), keep_a) == 0, t


@pytest.fixture
def exact_route():
    ts.tune_set("bx_exact", 1)  # small shapes as well
    yield
    ts.tune_set("bx_exact", 0)
    ts.tune_set("down_chunks", 0)


@pytest.mark.parametrize("B,H,I,E,K,skew,chunks,wide", [
    (130, 520, 1205, 2, 2, False, 0, True), (200, 1032, 700, 4, 2, True, 0, True), (256, 264, 1300, 8, 4, True, 0, True),
    # every workgroup starts at another fold of rows this long
    (128, 4096, 700, 4, 2, False, 0, True), (130, 4104, 665, 2, 2, False, 0, True), (65, 3592, 640, 2, 2, False, 0, True),
    (65, 8, 600, 2, 2, False, 0, True),
    (130, 520, 2100, 2, 2, False, 1, True),  # a down chunk of 66 tiles
    # whose plan does not fit the workspace: the single-token kernels
    (65, 512, 700, 8, 2, False, 0, False), (128, 1032, 130, 4, 2, False, 0, False),
    (130, 256, 65, 8, 1, True, 0, False), (256, 264, 300, 64, 4, False, 0, False), (100, 128, 33, 1, 1, False, 0, False),
    (66, 4096, 130, 4, 2, False, 0, False), (70, 4104, 65, 2, 1, False, 0, False)])
def test_wide_moe(exact_route, B, H, I, E, K, skew, chunks, wide):
    """skew: every token routed to expert 0, which then takes several groups."""
    ts.tune_set("down_chunks", chunks)
    m = synth.make_moe(B, H, I, E, K, gate_bias=-0.84, dtype=synth.BF16, seed=[72, B, H, I, E, K])
    if skew:
        m.w_router[0, 0] = synth.f32_to_bf16_bits(np.float32([10.0]))[0]  # x[:, 0] = 1: a logit bias
    ref = oracle.moe(m.x, m.w_router, m.w_gate, m.w_up, m.w_down_t, m.dtype, K)
    args = [to_dev(m.x), to_dev(m.w_router), to_dev(m.w_gate), to_dev(m.w_up), to_dev(m.w_down_t)]
    ws = torch.empty(ts.moe_workspace_bytes(B, H, I, E, K, ts.TS_BF16), dtype=torch.uint8, device="cuda")
    ws.fill_(0xFF)
    out, idx, w, st = ts.moe_sparse(*args, K, stats=True, ws=ws)
    ws.fill_(0xFF)
    dense = ts.moe_dense(*args, K, ws=ws)[0]
    torch.cuda.synchronize()
    for call in (ts.moe_sparse, ts.moe_dense):
        assert launches(lambda: call(*args, K, ws=ws), "batch_down") == (1 if wide else 0)
    if skew:
        assert (ref.topk_idx[:, 0] == 0).all()
    p = np.sort(ref.probs, axis=1)[:, ::-1]
    keep = [t for t in range(B) if K == E or abs(p[t, K - 1] - p[t, K]) > 1e-6 * p[t, K - 1]]
    assert idx.cpu().numpy()[keep].tolist() == ref.topk_idx[keep].tolist()
    bound = moe_bound(m.x, m.w_router, m.w_gate, m.w_up, m.w_down_t, ref.topk_idx, ref.topk_w, ref.g, ref.u,
                      batched=True, tokens=keep)
    for o in (out.cpu().numpy(), dense.cpu().numpy()):
        assert rel_l2(o[keep], ref.y[keep]) <= TIGHT_SINGLE
        assert_elementwise(o[keep], ref.y[keep], bound[keep], f"wide moe B={B} H={H} I={I} E={E} K={K}")
    for t in keep:
        for k in range(K):
            n = int(st["n_active"][t * K + k])
            g, u = ref.g[t, k], ref.u[t, k]
            keep_a = (np.abs(g) >= 1e-4) & (np.abs(u) >= 1e-4)
            assert compare_sets(st["active_idx"][t * K + k, :n].cpu().numpy(), (g > 0) & (u > 0), keep_a) == 0
