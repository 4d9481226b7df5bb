"""GPU parity of sparsek_attn_bwd (gradients with respect to q, k, v) against the CPU oracle.

Bars: |g - ref| <= 1e-2 max|ref| per tensor for bf16 storage (outputs are rounded to bf16, the
stored bf16 O enters D = dO.O with relative error 2^-9), <= 2e-4 max|ref| for fp32.  The reference
is computed from the oracle's own thresholds (rounded to fp32, the precision the kernels keep them in) and lifetimes.
"""
import numpy as np
import pytest
import torch

import paper_2406_16747_amd as spk
from paper_2406_16747_amd import synth
from gpu_util import check_mask_against, dev, host, kink_keys, oracle_mask32, require_gpu, say

pytestmark = pytest.mark.gpu


def run_bwd(oracle, inp, gate_mode, heads=None):
    B, H, n, d, k, w, Gu = (inp[x] for x in ("B", "H", "n", "d", "k", "w", "Gu"))
    bf16 = inp["dtype"] == "bf16"
    u = dev(inp["u"])
    Q, K, V, dO = (dev(inp[x], bf16) for x in ("Q", "K", "V", "dO"))
    tau, death = spk.sparsek_mask(u, k)
    o, lse = spk.sparsek_attn_fwd(Q, K, V, u, tau, death, k, w, gate_mode, inp["scale"])
    dq, dk, dv = spk.sparsek_attn_bwd(Q, K, V, u, tau, death, o, lse, dO, k, w, gate_mode, inp["scale"])
    torch.cuda.synchronize()
    got = [host(x) for x in (dq, dk, dv)]
    tau_r, death_r = oracle_mask32(oracle, inp["u"], k)
    check_mask_against(host(tau), host(death), tau_r, death_r)
    ref = oracle.attn_bwd(inp["Q32"], inp["K32"], inp["V32"], inp["u"], tau_r, death_r,
                          inp["dO32"], k, w, gate_mode, inp["scale"])
    worst = 0.0
    common = max(np.abs(r).max() for r in ref)
    for name, g, r in zip(("dq", "dk", "dv"), got, ref):
        assert np.isfinite(g).all(), name
        # a tensor whose exact gradient (nearly) vanishes, e.g. dq with a single key, is held to the others' scale
        scale = max(np.abs(r).max(), 1e-3 * common)
        err = np.abs(g - r).max()
        tol = (1e-2 if bf16 else 2e-4) * scale
        assert err <= tol + 1e-30, (name, err, scale, np.unravel_index(np.abs(g - r).argmax(), g.shape))
        worst = max(worst, err / max(scale, 1e-30))
    return worst


@pytest.mark.parametrize("n,d,k,w,Gu,dtype", [
    (200, 64, 12, 9, 1, "bf16"), (333, 128, 20, 0, 1, "bf16"), (520, 64, 30, 40, 2, "bf16"),
    (300, 32, 10, 7, 2, "fp32"), (90, 64, 100, 5, 1, "bf16"), (150, 64, 0, 5, 1, "bf16"), (64, 64, 3, 70, 1, "bf16"),
    (1, 64, 4, 4, 1, "bf16"), (257, 128, 16, 16, 1, "fp32"),
])
@pytest.mark.parametrize("gate_mode", [0, 1, 2, 3])
def test_attn_bwd_small(oracle, n, d, k, w, Gu, dtype, gate_mode):
    require_gpu()
    say("attn_bwd", n, d, k, w, Gu, dtype, gate_mode)
    inp = synth.make(3, Gu=Gu, seed=n + k, with_dO=True, B=2, H=2, n=n, d=d, k=k, w=w, dtype=dtype,
                     qk_div=float(np.sqrt(d)) / 4)
    run_bwd(oracle, inp, gate_mode)


def test_attn_bwd_config3_recipe_reduced(oracle):
    """Config 3 recipe (drifting scores, k=w=512 at n=8192 scaled down 4x), one batch, 2 heads."""
    require_gpu()
    say("attn_bwd config 3 reduced")
    inp = synth.make(3, with_dO=True, B=1, H=2, n=2048, k=128, w=128)
    run_bwd(oracle, inp, 0)


@pytest.mark.parametrize("n,d,k,w,Gu,gate_mode", [
    # a top-k list that spans two metadata segments of the dQ kernel and many blocks of selected keys
    (2600, 128, 1500, 256, 1, 0), (2600, 128, 1500, 256, 1, 1),
    # d = 64 with one score row per head, ragged tail, window narrower than a query tile
    (1500, 64, 300, 40, 2, 0), (1500, 64, 300, 40, 2, 3),
    # selection only (w = 0) and window only (k = 0) on the MFMA path
    (1100, 128, 200, 0, 1, 0), (1100, 64, 0, 300, 1, 2),
])
def test_attn_bwd_medium(oracle, n, d, k, w, Gu, gate_mode):
    require_gpu()
    say("attn_bwd medium", n, d, k, w, Gu, gate_mode)
    inp = synth.make(3, Gu=Gu, seed=3 * n + k, with_dO=True, B=1, H=2, n=n, d=d, k=k, w=w, dtype="bf16",
                     qk_div=float(np.sqrt(d)) / 2)
    run_bwd(oracle, inp, gate_mode)


@pytest.mark.parametrize("gate_mode", [0, 1, 3])
def test_one_call_backward_equals_the_two_parts(oracle, gate_mode):
    """sparsek_bwd = sparsek_attn_bwd + sparsek_mask_bwd, bit for bit (dq, dk, dv; du accumulates with atomics
    across heads, so it is compared to rounding), and all four gradients of the one call against the oracle."""
    require_gpu()
    say("one-call backward", gate_mode)
    inp = synth.make(3, seed=77, with_dO=True, B=2, H=2, n=700, d=64, k=40, w=30, dtype="bf16", qk_div=2.0)
    u = dev(inp["u"])
    Q, K, V, dO = (dev(inp[x], True) for x in ("Q", "K", "V", "dO"))
    tau, death = spk.sparsek_mask(u, 40)
    o, lse = spk.sparsek_attn_fwd(Q, K, V, u, tau, death, 40, 30, gate_mode, 1.0)
    dq, dk, dv = spk.sparsek_attn_bwd(Q, K, V, u, tau, death, o, lse, dO, 40, 30, gate_mode, 1.0)
    du = spk.sparsek_mask_bwd(Q, K, V, u, tau, death, o, lse, dO, 40, 30, gate_mode, 1.0)
    dq2, dk2, dv2, du2 = spk.sparsek_bwd(Q, K, V, u, tau, death, o, lse, dO, 40, 30, gate_mode, 1.0)
    torch.cuda.synchronize()
    for a, b in ((dq, dq2), (dk, dk2), (dv, dv2)):
        assert torch.equal(a, b)
    scale = float(du.abs().max())
    assert scale > 0 and float((du - du2).abs().max()) <= 1e-5 * scale
    tau_r, death_r = oracle_mask32(oracle, inp["u"], 40)
    check_mask_against(host(tau), host(death), tau_r, death_r)
    kink = kink_keys(inp["u"], tau_r, host(tau))
    assert kink.sum() <= 4
    args = (inp["Q32"], inp["K32"], inp["V32"], inp["u"], tau_r, death_r, inp["dO32"], 40, 30, gate_mode, 1.0)
    ref = list(oracle.attn_bwd(*args)) + [oracle.mask_bwd(*args)[0]]
    for name, g, r in zip(("dq", "dk", "dv", "du"), (dq2, dk2, dv2, du2), ref):
        rs = np.abs(r).max()
        diff = np.abs(host(g) - r)
        if name == "du":
            diff = diff[~kink]
        assert rs > 0 and diff.max() <= 1e-2 * rs, (name, diff.max(), rs)


# In the one call dK and dV are merged by groups of 8 workgroups among the score gradient's blocks.  A single block of a single head; one
# part per head and several, with a last group that is not full; a score row per head; more parts than one batch's heads.
@pytest.mark.parametrize("B,H,Gu,n,d,k,w", [
    (1, 1, 1, 100, 64, 10, 9), (1, 1, 1, 2600, 128, 150, 100), (1, 5, 5, 2300, 128, 150, 100), (2, 13, 13, 600, 128, 40, 30),
    (1, 11, 1, 2050, 64, 90, 64), (3, 7, 1, 2000, 128, 128, 128),
])
@pytest.mark.parametrize("gate_mode", [0, 3])
def test_one_call_backward_merges_every_row(B, H, Gu, n, d, k, w, gate_mode):
    """Bit for bit what sparsek_attn_bwd gives, whose merge is a launch of its own (that one against the oracle: above)."""
    require_gpu()
    say("one-call backward, merge", B, H, Gu, n, d, k, w, gate_mode)
    inp = synth.make(3, Gu=Gu, seed=n + H, with_dO=True, B=B, H=H, n=n, d=d, k=k, w=w, dtype="bf16", qk_div=2.0)
    u = dev(inp["u"])
    Q, K, V, dO = (dev(inp[x], True) for x in ("Q", "K", "V", "dO"))
    tau, death = spk.sparsek_mask(u, k)
    o, lse = spk.sparsek_attn_fwd(Q, K, V, u, tau, death, k, w, gate_mode, 1.0)
    two = spk.sparsek_attn_bwd(Q, K, V, u, tau, death, o, lse, dO, k, w, gate_mode, 1.0)
    torch.cuda.synchronize()
    poison = [torch.full_like(Q, float("nan")) for _ in range(4)]   # (what the results are allocated from: an unwritten row shows)
    torch.cuda.synchronize()
    del poison
    one = spk.sparsek_bwd(Q, K, V, u, tau, death, o, lse, dO, k, w, gate_mode, 1.0)
    torch.cuda.synchronize()
    for name, a, b in zip(("dq", "dk", "dv"), two, one):
        assert torch.isfinite(a.float()).all() and torch.equal(a, b), name


# Gate modes 2 and 3 at 64 columns have an instance for three workgroups per compute unit, taken with more than 512 blocks of queries
# (here 48 heads of 12 blocks, and of 11 in a chunk), and one for two, which the smaller tests hold against the oracle: the same bits.
@pytest.mark.parametrize("Gu,gate_mode", [(1, 2), (1, 3), (48, 3)])
def test_many_blocks_without_gates_equal_few(Gu, gate_mode):
    require_gpu()
    say("three workgroups per compute unit", Gu, gate_mode)
    H, n, d, k, w = 48, 1500, 64, 70, 90
    inp = synth.make(3, Gu=Gu, seed=1500 + Gu, with_dO=True, B=1, H=H, n=n, d=d, k=k, w=w, dtype="bf16", qk_div=2.0)
    Q, K, V, dO = (dev(inp[x], True) for x in ("Q", "K", "V", "dO"))
    u = dev(inp["u"])

    def run(hs):
        q, kk, v, g = (x[:, hs].contiguous() for x in (Q, K, V, dO))
        us = u if Gu == 1 else u[:, hs].contiguous()
        tau, death = spk.sparsek_mask(us, k)
        o, lse = spk.sparsek_attn_fwd(q, kk, v, us, tau, death, k, w, gate_mode, 1.0)
        out = [o, lse, *spk.sparsek_bwd(q, kk, v, us, tau, death, o, lse, g, k, w, gate_mode, 1.0)[:3]]
        st = spk.ChunkState(1, q.shape[1], us.shape[1], d, k, w, spk.BF16, 1400, gate_mode, 1.0, 0)
        for sl in (slice(0, 100), slice(100, n)):
            qc, kc, vc, gc, uc = (x[:, :, sl].contiguous() for x in (q, kk, v, g, us))
            oc = spk.sparsek_chunk_prefill(st, qc, kc, vc, uc)
            out += [oc, *spk.sparsek_chunk_bwd(st, qc, oc, gc)[:3]]
        return out

    many = run(slice(0, H))
    few = [torch.cat(pair, dim=1) for pair in zip(run(slice(0, H // 2)), run(slice(H // 2, H)))]
    torch.cuda.synchronize()
    for i, (a, b) in enumerate(zip(many, few)):
        assert torch.isfinite(a.float()).all() and torch.equal(a, b), i


def test_one_call_backward_fp32_generic_path(oracle):
    """sparsek_bwd on the generic (fp32) kernels against the oracle's two gradients."""
    require_gpu()
    say("one-call backward fp32")
    inp = synth.make(3, seed=91, with_dO=True, B=1, H=2, n=300, d=32, k=24, w=20, dtype="fp32", qk_div=2.0)
    u = dev(inp["u"])
    Q, K, V, dO = (dev(inp[x], False) for x in ("Q", "K", "V", "dO"))
    tau, death = spk.sparsek_mask(u, 24)
    o, lse = spk.sparsek_attn_fwd(Q, K, V, u, tau, death, 24, 20, 0, inp["scale"])
    got = [host(x) for x in spk.sparsek_bwd(Q, K, V, u, tau, death, o, lse, dO, 24, 20, 0, inp["scale"])]
    tau_r, death_r = oracle_mask32(oracle, inp["u"], 24)
    check_mask_against(host(tau), host(death), tau_r, death_r)
    assert not kink_keys(inp["u"], tau_r, host(tau)).any()
    ref = list(oracle.attn_bwd(inp["Q32"], inp["K32"], inp["V32"], inp["u"], tau_r, death_r, inp["dO32"], 24, 20, 0,
                               inp["scale"]))
    ref.append(oracle.mask_bwd(inp["Q32"], inp["K32"], inp["V32"], inp["u"], tau_r, death_r, inp["dO32"], 24, 20, 0,
                               inp["scale"])[0])
    for name, g, r in zip(("dq", "dk", "dv", "du"), got, ref):
        scale = np.abs(r).max()
        assert scale > 0 and np.abs(g - r).max() <= 2e-4 * scale, (name, np.abs(g - r).max(), scale)
