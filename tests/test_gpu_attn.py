"""GPU parity of stage 3 (sparsek_attn_fwd) against the CPU oracle.

Bars: bf16 outputs max abs err <= 1e-2 against the fp64 oracle, plus a self-imposed
relative bar max|err| <= 2^-7 max|ref| (the 1e-2 bar alone is looser than the signal for
the 1/sqrt(d)-scaled recipes); fp32 outputs <= 2e-5 relative to max|ref|.
A second pass with unscaled q,k (peaky softmax) makes wrong gates or indices visible.
"""
import numpy as np
import pytest
import torch

import paper_2406_16747_amd as spk
from paper_2406_16747_amd import synth
from gpu_util import dev, host, require_gpu, say

pytestmark = pytest.mark.gpu


def run_case(oracle, inp, gate_mode=0, scale=None, heads=None, rows=None, qk_boost=1.0):
    """Runs the GPU path on the whole input and the oracle on `heads` (list of (b,h)) and
    query rows `rows` (None = all)."""
    B, H, n, d, k, w, Gu = (inp[x] for x in ("B", "H", "n", "d", "k", "w", "Gu"))
    bf16 = inp["dtype"] == "bf16"
    scale = inp["scale"] if scale is None else scale
    u = inp["u"]
    ud = dev(u)
    tau_g, death_g = spk.sparsek_mask(ud, k)
    q, kk, v = (dev(inp[x], bf16) for x in ("Q", "K", "V"))
    q32, k32 = inp["Q32"], inp["K32"]
    if qk_boost != 1.0:  # exact in bf16 for powers of two
        q = (q.float() * qk_boost).to(q.dtype)
        q32 = q32 * np.float32(qk_boost)
    o_g, lse_g = spk.sparsek_attn_fwd(q, kk, v, ud, tau_g, death_g, k, w, gate_mode, scale)
    torch.cuda.synchronize()
    o_g, lse_g = host(o_g), host(lse_g)
    assert np.isfinite(o_g).all() and np.isfinite(lse_g).all()
    heads = heads if heads is not None else [(b, h) for b in range(B) for h in range(H)]
    worst = 0.0
    for (b, h) in heads:
        g = 0 if Gu == 1 else h
        tau_r = oracle.tau_prefixes(u[b, g], k)[0]
        death_r = oracle.death(u[b, g], k)
        np.testing.assert_array_equal(host(death_g)[b, g], death_r)
        spans = [(0, n)] if rows is None else rows
        for (a, e) in spans:
            o_r, lse_r = oracle.attn_rows(q32[b, h], k32[b, h], inp["V32"][b, h], u[b, g], tau_r, death_r, k, w,
                                          gate_mode, scale, a, e)
            err = np.abs(o_g[b, h, a:e] - o_r).max()
            ref = np.abs(o_r).max()
            if bf16:
                assert err <= 1e-2, (b, h, a, err)
                assert err <= ref * 2.0 ** -7 + 1e-6, (b, h, a, err, ref)
            else:
                assert err <= 2e-5 * max(ref, 1e-3), (b, h, a, err, ref)
            np.testing.assert_allclose(lse_g[b, h, a:e], lse_r, atol=2e-3 if bf16 else 1e-4, rtol=1e-4)
            worst = max(worst, err / max(ref, 1e-30))
    return worst


@pytest.mark.parametrize("gate_mode", [0, 1, 2, 3])
def test_config1_fp32(oracle, gate_mode):
    require_gpu()
    say("attn config 1 mode", gate_mode)
    inp = synth.make(1)
    run_case(oracle, inp, gate_mode)
    run_case(oracle, inp, gate_mode, qk_boost=8.0)


@pytest.mark.parametrize("n,d,k,w,Gu,dtype", [
    (1, 64, 4, 4, 1, "bf16"), (7, 64, 2, 3, 1, "bf16"), (300, 64, 16, 0, 1, "bf16"),
    (333, 128, 0, 40, 1, "bf16"), (700, 128, 50, 130, 2, "bf16"), (515, 64, 600, 5, 1, "bf16"),
    (450, 32, 20, 33, 2, "fp32"), (129, 128, 1, 1, 1, "fp32"),
    # windows just wider than a query block (edge and diagonal tile runs meet), a top-k list that
    # spans two metadata segments, and a long expiring tail of the list
    (1000, 128, 70, 150, 1, "bf16"), (900, 64, 100, 192, 1, "bf16"), (2600, 128, 1500, 256, 1, "bf16"),
    (1500, 64, 300, 64, 1, "bf16"),
])
@pytest.mark.parametrize("gate_mode", [0, 1, 2, 3])
def test_small_shapes(oracle, n, d, k, w, Gu, dtype, gate_mode):
    require_gpu()
    say("attn small", n, d, k, w, Gu, dtype, gate_mode)
    inp = synth.make(1, Gu=Gu, seed=n * 7 + k, B=2, H=2, n=n, d=d, k=k, w=w, dtype=dtype, qk_div=float(np.sqrt(d)))
    run_case(oracle, inp, gate_mode)
    run_case(oracle, inp, gate_mode, qk_boost=8.0)


# The generic kernel finds its own keys up to 4096 positions and 1024 of them; beyond, it takes the lists of blocks of 128 queries.
# Windows that are no multiple of its 16 queries, none at all, and prefixes that start in the middle of a workgroup's queries.
@pytest.mark.parametrize("n,d,k,w,Gu,dtype", [
    (4096, 32, 40, 30, 1, "fp32"), (4097, 32, 40, 30, 1, "fp32"), (2100, 32, 1024, 21, 2, "fp32"),
    (2100, 32, 1025, 21, 1, "fp32"), (17, 36, 3, 5, 1, "bf16"), (700, 64, 90, 0, 1, "fp32"), (300, 100, 0, 17, 1, "fp32"),
    (1100, 128, 70, 16, 2, "fp32"),
])
def test_generic_kernel_with_and_without_lists(oracle, n, d, k, w, Gu, dtype):
    require_gpu()
    say("generic kernel", n, d, k, w, Gu, dtype)
    run_case(oracle, synth.make(1, Gu=Gu, seed=n + k + w, B=1, H=2, n=n, d=d, k=k, w=w, dtype=dtype))


@pytest.mark.parametrize("k", [4095, 4096, 4100])
@pytest.mark.parametrize("Gu", [1, 24])   # a workgroup per block; runs of two blocks, whose lists grow past the limit
def test_lists_longer_than_lds_holds(oracle, k, Gu):
    """Up to 4096 entries of a block's list are put together in LDS, longer ones are written in place; blocks of a run then
    start anew instead of from the list before.  Queries around the first prefixes of k keys, and the last ones."""
    require_gpu()
    say("attn long lists", k, Gu)
    n, w = 5600, 70
    inp = synth.make(1, Gu=Gu, seed=k, B=1, H=Gu, n=n, d=64, k=k, w=w, dtype="bf16", qk_div=2.0)
    heads = [(0, 0)] if Gu == 1 else [(0, 5)]
    run_case(oracle, inp, 0, heads=heads, rows=[(4000, 4008), (4160, 4170), (4220, 4230), (4420, 4424), (n - 8, n)])


@pytest.mark.parametrize("dtype,d", [("fp32", 64), ("fp32", 100), ("bf16", 36)])
def test_generic_kernel_alignment_and_nonfinite_values(oracle, dtype, d):
    """Tensors that start at any element, and values that are not finite: those reach the queries that attend their key
    and nobody else."""
    require_gpu()
    say("attn generic", dtype, d)
    bf16, n, k, w = dtype == "bf16", 300, 20, 33
    inp = synth.make(1, Gu=1, seed=d, B=1, H=2, n=n, d=d, k=k, w=w, dtype=dtype, qk_div=float(np.sqrt(d)))
    u = dev(inp["u"])
    tau, death = spk.sparsek_mask(u, k)
    q, kk, v = (dev(inp[x], bf16) for x in ("Q", "K", "V"))
    want = spk.sparsek_attn_fwd(q, kk, v, u, tau, death, k, w, 0, inp["scale"])

    def shifted(t):
        buf = torch.empty(t.numel() + 1, dtype=t.dtype, device=t.device)
        out = buf[1:].view(t.shape)
        out.copy_(t)
        return out

    got = spk.sparsek_attn_fwd(shifted(q), shifted(kk), shifted(v), u, tau, death, k, w, 0, inp["scale"])
    for a, b in zip(want, got):
        np.testing.assert_array_equal(host(a), host(b))
    bad = v.clone()
    bad[:, :, 150, 3] = float("nan")
    bad[:, :, 201, :] = float("inf")
    o, lse = spk.sparsek_attn_fwd(q, kk, bad, u, tau, death, k, w, 0, inp["scale"])
    np.testing.assert_array_equal(host(lse), host(want[1]))
    i = np.arange(n)
    clean = np.ones(n, bool)
    for j in (150, 201):
        clean &= ~((i >= j) & (i <= w - 1 + host(death)[0, 0, j]))
    assert clean[:150].all() and not clean[150] and not clean[201]
    # the tiles that hold such a key add up in another order: a few units of the sums' last place
    np.testing.assert_allclose(host(o)[:, :, clean], host(want[0])[:, :, clean], atol=1e-2 if bf16 else 1e-5)
    other = np.arange(d) != 3   # (query 201 may still attend key 150)
    assert np.isnan(host(o)[:, :, 150, 3]).all() and np.isinf(host(o)[:, :, 201][..., other]).all()


def test_config2_shape_reduced_batch(oracle):
    """Config 2 recipe (scores from a linear scorer on a hidden state) at B=1, 3 heads."""
    require_gpu()
    say("attn config 2 (reduced batch)")
    inp = synth.make(2, B=1, H=3)
    run_case(oracle, inp, 0)
    run_case(oracle, inp, 1, qk_boost=8.0, heads=[(0, 1)])


@pytest.mark.parametrize("H", [8, 9, 11, 15, 17])
def test_heads_left_over_by_the_deal_to_partitions(oracle, H):
    """Of every 8 heads each partition of the chip gets one; the heads left over are dealt block by block.  Forward and all
    gradients of the last heads of the whole groups and of every head left over."""
    require_gpu()
    say("attn heads", H)
    inp = synth.make(3, with_dO=True, B=1, H=H, n=300, d=64, k=20, w=40, seed=H)
    heads = [(0, h) for h in range(H // 8 * 8 - 1, H)]
    run_case(oracle, inp, heads=heads)
    u = dev(inp["u"])
    tau, death = spk.sparsek_mask(u, 20)
    x = [dev(inp[name], True) for name in ("Q", "K", "V", "dO")]
    o, lse = spk.sparsek_attn_fwd(*x[:3], u, tau, death, 20, 40, 0, inp["scale"])
    got = spk.sparsek_bwd(*x[:3], u, tau, death, o, lse, x[3], 20, 40, 0, inp["scale"])
    tau_r, death_r = oracle.mask_all(inp["u"], 20)
    tau_r = tau_r.astype(np.float32).astype(np.float64)
    pick = [h for _, h in heads]
    ref = oracle.attn_bwd(inp["Q32"][:, pick], inp["K32"][:, pick], inp["V32"][:, pick], inp["u"], tau_r, death_r,
                          inp["dO32"][:, pick], 20, 40, 0, inp["scale"])
    for name, g, r in zip(("dq", "dk", "dv"), got, ref):
        assert np.abs(host(g)[:, pick] - r).max() <= 1e-2 * np.abs(r).max(), name
    du_r, _ = oracle.mask_bwd(inp["Q32"], inp["K32"], inp["V32"], inp["u"], tau_r, death_r, inp["dO32"], 20, 40, 0, inp["scale"])
    assert np.abs(host(got[3]) - du_r).max() <= 1e-2 * np.abs(du_r).max()
