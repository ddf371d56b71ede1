"""Parity of the HIP top-k MoE layer (ts_moe_sparse / ts_moe_dense through
the C ABI) against the fp64 oracle.  Routing is compared exactly except for
tokens whose k-th and (k+1)-th oracle probabilities are within 1e-6
(relative) of each other; outputs to relative L2 <= 1e-5 (fp32 weights) /
1e-2 (bf16 weights)."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import DEV, TIGHT_BATCH, TIGHT_SINGLE, assert_elementwise, compare_sets, moe_bound, rel_l2, to_dev
from paper_2406_05955_amd import synth

pytestmark = pytest.mark.gpu

ts = pytest.importorskip("paper_2406_05955_amd.binding") if torch.cuda.is_available() else None


def near_tie(probs_t, K):
    p = np.sort(probs_t)[::-1]
    return K < p.size and abs(p[K - 1] - p[K]) <= 1e-6 * p[K - 1]


def run_moe(m, stats=False, dense=False):
    args = [to_dev(m.x), to_dev(m.w_router), to_dev(m.w_gate), to_dev(m.w_up), to_dev(m.w_down_t)]
    if dense:
        return ts.moe_dense(*args, m.top_k)
    return ts.moe_sparse(*args, m.top_k, stats=stats)


def check_moe(m, dense=False):
    B, H, I, E, K = m.shape
    ref = oracle.moe(m.x, m.w_router, m.w_gate, m.w_up, m.w_down_t, m.dtype, K)
    res = run_moe(m, stats=not dense, dense=dense)
    torch.cuda.synchronize()
    out, idx, w = res[0], res[1].cpu().numpy(), res[2].cpu().numpy()
    ties = [near_tie(ref.probs[t], K) for t in range(B)]
    for t in range(B):
        if ties[t]:
            continue
        assert idx[t].tolist() == ref.topk_idx[t].tolist(), (t, idx[t], ref.topk_idx[t])
        assert np.allclose(w[t], ref.topk_w[t], rtol=1e-5, atol=1e-6)
    keep = [t for t in range(B) if not ties[t]]
    tol = 1e-5 if m.dtype == synth.F32 else 1e-2
    o = out.cpu().numpy()
    assert rel_l2(o[keep], ref.y[keep]) <= tol
    # several bf16 tokens take the matrix-core path
    batched = B > 1 and m.dtype == synth.BF16
    assert rel_l2(o[keep], ref.y[keep]) <= (TIGHT_BATCH if batched else TIGHT_SINGLE)
    if not dense:
        bound = moe_bound(m.x, m.w_router, m.w_gate, m.w_up, m.w_down_t, ref.topk_idx, ref.topk_w, ref.g, ref.u,
                          batched=batched, tokens=keep)
        assert_elementwise(o[keep], ref.y[keep], bound[keep], f"moe B={B} H={H} I={I} E={E} K={K}")
    if not dense:
        st = res[3]
        thr = 1e-6 if m.dtype == synth.F32 else 1e-4
        for t in keep:
            for k in range(K):
                s = t * K + k
                g, u = ref.g[t, k], ref.u[t, k]
                keep_a = (np.abs(g) >= thr) & (np.abs(u) >= thr)
                n = int(st["n_active"][s])
                got = st["active_idx"][s, :n].cpu().numpy()
                assert compare_sets(got, (g > 0) & (u > 0), keep_a) == 0
    return ref, res


@pytest.mark.parametrize("dtype", [synth.F32, synth.BF16])
@pytest.mark.parametrize("B,H,I,E,K", [(1, 512, 1024, 8, 2), (16, 512, 700, 8, 2), (3, 256, 130, 4, 4),
                                       (2, 1024, 333, 1, 1), (5, 640, 256, 64, 8), (1, 4096, 2048, 8, 2),
                                       (256, 128, 64, 8, 2),  # the largest batch
                                       # expert counts that do not divide the 8 waves or exceed
                                       # them (both routers read the rows in a rotated order)
                                       (1, 512, 700, 6, 3), (1, 384, 300, 12, 2), (9, 512, 500, 3, 2),
                                       (12, 256, 200, 12, 3)])
def test_moe_shapes(dtype, B, H, I, E, K):
    m = synth.make_moe(B, H, I, E, K, gate_bias=-1.5548, dtype=dtype, seed=[B, H, I, E, K])
    check_moe(m)


def test_moe_dense_matches():
    m = synth.make_moe(4, 512, 900, 8, 2, gate_bias=-0.5244, dtype=synth.BF16, seed=12)
    check_moe(m, dense=True)


@pytest.mark.parametrize("gate_bias,sparsity", [(-1.5548, 0.97), (-0.5244, 0.85)])
def test_moe_mixtral_shape_b1(gate_bias, sparsity):
    """E=8, H=4096, I=14336 per expert, bf16, drawn on the device like the
    benchmark's MoE layers, at 97% in-expert sparsity and at the paper's 85%
    per expert."""
    L = synth.make_moe_stack_torch(1, 1, 4096, 14336, 8, 2, gate_bias=gate_bias, dtype=synth.BF16, seed=0,
                                   device=DEV)
    h = lambda t: synth.tensor_to_host_array(t, synth.BF16)  # noqa: E731
    m = synth.MoEInputs(x=L["x"][0].cpu().numpy(), w_router=h(L["w_router"][0]), w_gate=h(L["w_gate"][0]),
                        w_up=h(L["w_up"][0]), w_down_t=h(L["w_down_t"][0]), dtype=synth.BF16, top_k=2,
                        gate_bias=gate_bias)
    ref, res = check_moe(m)
    n_act = res[3]["n_active"].cpu().numpy()
    assert np.all(np.abs(1.0 - n_act / 14336 - sparsity) < 0.02), n_act


@pytest.mark.parametrize("I", [14336, 14368])
@pytest.mark.parametrize("dense", [True, False])
def test_moe_long_down_lists(I, dense):
    """At 32 token slots per expert group (batch 64 over 8 experts, top 2) a
    down workgroup lists the active rows of up to 224 tiles of 32 (half a
    14336-neuron expert) at once.  The dense comparator makes every row
    active, so such an expert fills two lists exactly and 14368 neurons take
    a third, one-tile list; the sparse layer at the same shapes alongside."""
    m = synth.make_moe(64, 256, I, 8, 2, gate_bias=-1.5548, dtype=synth.BF16, seed=[13, I])
    check_moe(m, dense=dense)


@pytest.mark.parametrize("dtype,B,H,I,E,K,every", [(synth.BF16, 130, 520, 1205, 2, 2, 1),
                                                   (synth.BF16, 130, 520, 1205, 2, 2, 3),
                                                   (synth.BF16, 40, 264, 300, 4, 4, 1),
                                                   (synth.F32, 40, 128, 3300, 2, 2, 1),
                                                   (synth.BF16, 1, 264, 300, 8, 2, 1)])
def test_moe_non_finite_tokens(dtype, B, H, I, E, K, every):
    """Tokens whose router logits are NaN still take K distinct experts: an
    expert's groups have room for each token once, so one expert drawn twice
    by enough tokens (B K pairs against ceil(B / slots) groups: 260 against
    192, 160 against 64, 80 against 64) would leave pairs without a slot.
    Their outputs are NaN; the other tokens' are what they are without them."""
    m = synth.make_moe(B, H, I, E, K, gate_bias=-0.84, dtype=dtype, seed=[74, B, E, K])
    ref = oracle.moe(m.x, m.w_router, m.w_gate, m.w_up, m.w_down_t, m.dtype, K)
    bad = np.arange(0, B, every)
    x = m.x.copy()
    x[bad, 3] = np.nan
    args = [to_dev(m.w_router), to_dev(m.w_gate), to_dev(m.w_up), to_dev(m.w_down_t)]
    for dense in (False, True):
        out, idx, w = ts.moe_sparse(to_dev(x), *args, K, dense=dense)[:3]
        torch.cuda.synchronize()
        out, idx, w = out.cpu().numpy(), idx.cpu().numpy(), w.cpu().numpy()
        assert (idx[bad] == np.arange(K)).all()
        assert np.isnan(w[bad]).all() and np.isnan(out[bad]).all()
        good = [t for t in range(B) if t % every and not near_tie(ref.probs[t], K)]
        if good:
            assert idx[good].tolist() == ref.topk_idx[good].tolist()
            assert rel_l2(out[good], ref.y[good]) <= TIGHT_BATCH
