"""GPU parity of the decode step (sparsek_decode_init/load/step/status) against the oracle.

The oracle's decode is "row t of the prefill attention over the whole history", so these
tests also check the paper's claim that incremental evaluation with a k+w cache gives
exactly the full-history result.
"""
import numpy as np
import pytest
import torch

import paper_2406_16747_amd as spk
from paper_2406_16747_amd import synth
from gpu_util import dev, host, require_gpu, say

pytestmark = pytest.mark.gpu


def history(rng, B, H, Gu, n, d, dtype, ties=False):
    div = np.float32(np.sqrt(d) / 4.0)  # moderately peaky softmax
    out = {}
    for name in ("Q", "K", "V"):
        x = rng.standard_normal((B, H, n, d), dtype=np.float32) / (div if name != "V" else np.float32(1))
        out[name], out[name + "32"] = synth._store(x, dtype)
    u = rng.standard_normal((B, Gu, n), dtype=np.float32)
    if ties:
        u = (np.round(u * 3) / 3).astype(np.float32)
    out["u"] = u
    return out


def run_decode(oracle, B, H, Gu, d, k, w, n_ctx, steps, dtype="bf16", gate_mode=0, ties=False, cand_cap=0,
               seed=0, check_heads=None):
    rng = np.random.default_rng(seed)
    n = n_ctx + steps
    hist = history(rng, B, H, Gu, n, d, dtype, ties)
    bf16 = dtype == "bf16"
    tdt = torch.bfloat16 if bf16 else torch.float32
    Q, K, V = (dev(hist[x], bf16) for x in ("Q", "K", "V"))
    u = dev(hist["u"])
    state = spk.DecodeState(B, H, Gu, d, k, w, tdt, gate_mode, 1.0, cand_cap)
    state.buf.fill_(255)  # NaN patterns everywhere: init/load must not rely on fresh memory
    if n_ctx == 0:
        spk.sparsek_decode_init(state)
    else:
        u_ctx = u[:, :, :n_ctx].contiguous()
        tau, death = spk.sparsek_mask(u_ctx, k)
        spk.sparsek_decode_load(state, K[:, :, :n_ctx].contiguous(), V[:, :, :n_ctx].contiguous(), u_ctx, tau, death)
    outs = []
    for s in range(steps):
        t = n_ctx + s
        o = spk.sparsek_decode_step(state, Q[:, :, t].contiguous(), K[:, :, t].contiguous(),
                                    V[:, :, t].contiguous(), u[:, :, t].contiguous())
        outs.append(o)
    torch.cuda.synchronize()
    og = np.stack([host(o) for o in outs], axis=2)  # [B,H,steps,d]
    flags = spk.sparsek_decode_status(state)
    heads = check_heads or [(b, h) for b in range(B) for h in range(H)]
    worst = 0.0
    for (b, h) in heads:
        g = 0 if Gu == 1 else h
        ref = oracle.decode_bydef(hist["Q32"][b, h, n_ctx:], hist["K32"][b, h], hist["V32"][b, h], hist["u"][b, g],
                                  n_ctx, k, w, gate_mode, 1.0)
        err = np.abs(og[b, h] - ref).max()
        scale = np.abs(ref).max()
        worst = max(worst, err / scale)
        if bf16:
            assert err <= 1e-2 * max(1.0, scale) and err <= scale * 2.0 ** -7, (b, h, err, scale)
        else:
            assert err <= 2e-5 * scale, (b, h, err, scale)
    return state, og, flags, hist


@pytest.mark.parametrize("Gu", [1, 2])
@pytest.mark.parametrize("k,w", [(8, 6), (5, 0), (0, 7), (1, 1), (40, 3)])
def test_decode_from_empty(oracle, k, w, Gu):
    require_gpu()
    say("decode from empty", k, w, Gu)
    _, _, flags, _ = run_decode(oracle, 2, 2, Gu, 64, k, w, 0, 90, ties=(k == 5), seed=k * 10 + w)
    assert not flags.any()


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("fp32", 32), ("bf16", 64)])
@pytest.mark.parametrize("gate_mode", [0, 1, 2, 3])
def test_decode_after_prefill(oracle, dtype, d, gate_mode):
    require_gpu()
    say("decode after prefill", dtype, d, gate_mode)
    _, _, flags, _ = run_decode(oracle, 1, 3, 3 if d == 64 else 1, d, 24, 20, 400, 60, dtype, gate_mode, seed=d)
    assert not flags.any()


@pytest.mark.parametrize("n_ctx", [1, 5, 19, 20, 21, 44, 45])
def test_decode_load_boundaries(oracle, n_ctx):
    """Contexts shorter than w, than k+w, and just past them."""
    require_gpu()
    say("decode boundaries", n_ctx)
    run_decode(oracle, 1, 2, 1, 64, 25, 20, n_ctx, 30, seed=n_ctx)


@pytest.mark.parametrize("B,H,Gu,d,k,w,n_ctx,steps,dtype,gate_mode,heads", [
    (1, 2, 1, 128, 300, 261, 700, 24, "bf16", 0, None),     # a head's slots in two uneven shares
    (1, 2, 2, 128, 1100, 950, 2100, 16, "bf16", 1, None),   # ... in eight, per-head selection, still filling up
    (1, 3, 1, 64, 500, 700, 1300, 12, "fp32", 2, None),
    (16, 64, 1, 32, 1200, 901, 2150, 2, "bf16", 0, [(0, 0), (7, 33), (15, 63)]),  # one workgroup per head, more slots than a slab
])
def test_decode_shares_and_slabs(oracle, B, H, Gu, d, k, w, n_ctx, steps, dtype, gate_mode, heads):
    require_gpu()
    say("decode shares", B, H, Gu, d, k, w, n_ctx, dtype, gate_mode)
    _, _, flags, _ = run_decode(oracle, B, H, Gu, d, k, w, n_ctx, steps, dtype, gate_mode, seed=k, check_heads=heads)
    assert not flags.any()


def test_decode_state_used_again(oracle):
    """A state that is set up again counts its steps from the start: partial results left in its memory with the step
    numbers of an earlier generation must not pass for those of the new one."""
    require_gpu()
    say("decode state used again")
    B, H, d, k, w, n_ctx = 1, 2, 128, 600, 500, 1200   # heads in several shares
    rng = np.random.default_rng(5)
    states, outs = [spk.DecodeState(B, H, 1, d, k, w, torch.bfloat16) for _ in range(2)], [[], []]
    states[0].buf.fill_(255)
    states[1].buf[: states[1].buf.numel() // 8 * 8].view(torch.int64).fill_(1 << 32)   # zeros of "step 1" everywhere
    for gen in range(3):
        hist = history(rng, B, H, 1, n_ctx + 1, d, "bf16")
        Q, K, V = (dev(hist[x], True) for x in ("Q", "K", "V"))
        u = dev(hist["u"])
        u_ctx = u[:, :, :n_ctx].contiguous()
        tau, death = spk.sparsek_mask(u_ctx, k)
        for st, out in zip(states, outs):
            if gen == 1 and st is states[0]:   # as new
                st.buf.fill_(255)
            spk.sparsek_decode_load(st, K[:, :, :n_ctx].contiguous(), V[:, :, :n_ctx].contiguous(), u_ctx, tau, death)
            assert not st.buf[-1024:-256].any().item()   # (the partial results are the last part of a state)
            out.append(host(spk.sparsek_decode_step(st, *(x[:, :, n_ctx].contiguous() for x in (Q, K, V, u)))))
            assert not spk.sparsek_decode_status(st).any()
    for a, b in zip(*outs):
        np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("k,w", [(20, 33), (600, 500)])   # one workgroup per head, several shares
@pytest.mark.parametrize("over", ["q", "k", "v"])
def test_decode_output_over_an_input(oracle, k, w, over):
    """The output may take the place of the new token's q, k or v."""
    require_gpu()
    say("decode output over", over, k, w)
    B, H, d, n_ctx, steps = 1, 4, 128, 1200, 6
    hist = history(np.random.default_rng(k), B, H, 1, n_ctx + steps, d, "bf16")
    Q, K, V = (dev(hist[x], True) for x in ("Q", "K", "V"))
    u = dev(hist["u"])
    u_ctx = u[:, :, :n_ctx].contiguous()
    tau, death = spk.sparsek_mask(u_ctx, k)
    states = [spk.DecodeState(B, H, 1, d, k, w, torch.bfloat16) for _ in range(2)]
    for st in states:
        spk.sparsek_decode_load(st, K[:, :, :n_ctx].contiguous(), V[:, :, :n_ctx].contiguous(), u_ctx, tau, death)
    for i in range(n_ctx, n_ctx + steps):
        new = [[x[:, :, i].contiguous() for x in (Q, K, V, u)] for _ in states]
        want = spk.sparsek_decode_step(states[0], *new[0])
        got = spk.sparsek_decode_step(states[1], *new[1], out=new[1]["qkv".index(over)])
        np.testing.assert_array_equal(host(got), host(want))


def test_decode_step_equals_prefill_row_on_gpu(oracle):
    """Sec. 3.4: recurrent evaluation gives the same result as the one-shot one."""
    require_gpu()
    B, H, Gu, d, k, w, n_ctx, steps = 1, 2, 1, 128, 32, 32, 700, 50
    state, og, _, hist = run_decode(oracle, B, H, Gu, d, k, w, n_ctx, steps, seed=3)
    Q, K, V = (dev(hist[x], True) for x in ("Q", "K", "V"))
    u = dev(hist["u"])
    tau, death = spk.sparsek_mask(u, k)
    o_pre = host(spk.sparsek_attn_fwd(Q, K, V, u, tau, death, k, w, 0, 1.0, return_lse=False))
    err = np.abs(o_pre[:, :, n_ctx:] - og).max()
    assert err <= 2.0 ** -7 * np.abs(og).max()


def test_decode_snapshot_and_replay(oracle):
    require_gpu()
    rng = np.random.default_rng(9)
    B, H, Gu, d, k, w = 2, 2, 1, 64, 10, 8
    hist = history(rng, B, H, Gu, 120, d, "bf16")
    Q, K, V = (dev(hist[x], True) for x in ("Q", "K", "V"))
    u = dev(hist["u"])
    state = spk.DecodeState(B, H, Gu, d, k, w, torch.bfloat16)
    spk.sparsek_decode_init(state)

    def go(a, b):
        return [spk.sparsek_decode_step(state, Q[:, :, t].contiguous(), K[:, :, t].contiguous(),
                                        V[:, :, t].contiguous(), u[:, :, t].contiguous()).clone() for t in range(a, b)]

    go(0, 70)
    snap = state.buf.clone()
    first = go(70, 120)
    state.buf.copy_(snap)
    second = go(70, 120)
    for a, b in zip(first, second):
        assert torch.equal(a, b)


def test_decode_candidate_overflow_sets_status(oracle):
    """All-equal scores keep every key above tau; a small candidate capacity must overflow,
    set bit 0 of the row's status word and keep running."""
    require_gpu()
    B, H, Gu, d, k, w = 1, 1, 1, 64, 4, 2
    state = spk.DecodeState(B, H, Gu, d, k, w, torch.bfloat16, cand_cap=8)
    spk.sparsek_decode_init(state)
    g = torch.Generator(device="cuda").manual_seed(1)
    for t in range(40):
        x = torch.randn(3, B, H, d, device="cuda", generator=g).bfloat16()
        o = spk.sparsek_decode_step(state, x[0], x[1], x[2], torch.full((B, Gu), 0.5, device="cuda"))
    torch.cuda.synchronize()
    assert torch.isfinite(o.float()).all()
    assert spk.sparsek_decode_status(state)[0] & 1


@pytest.mark.parametrize("k,w", [(200, 312), (100, 0)])
def test_decode_steps_of_several_states_at_once(k, w):
    """Steps of different states overlap on different streams as they like: no head waits for a workgroup that the other
    states' heads could keep from running."""
    require_gpu()
    say("decode states at once", k, w)
    B, H, d, n_ctx, steps, count = 8, 32, 128, 700, 8, 3
    g = torch.Generator(device="cuda").manual_seed(k)
    states = [spk.DecodeState(B, H, 1, d, k, w, torch.bfloat16) for _ in range(count)]
    new = []
    for st in states:
        u = torch.randn(B, 1, n_ctx, device="cuda", generator=g)
        kk, vv = (torch.randn(B, H, n_ctx, d, device="cuda", generator=g).bfloat16() for _ in range(2))
        spk.sparsek_decode_load(st, kk, vv, u, *spk.sparsek_mask(u, k))
        new.append([tuple(torch.randn(B, H, d, device="cuda", generator=g).bfloat16() for _ in range(3))
                    + (torch.randn(B, 1, device="cuda", generator=g),) for _ in range(steps)])
    before = [st.buf.clone() for st in states]
    want = [[spk.sparsek_decode_step(st, *x) for x in xs] for st, xs in zip(states, new)]
    for st, buf in zip(states, before):
        st.buf.copy_(buf)
    got = [[torch.empty_like(o) for o in os] for os in want]
    streams = [torch.cuda.Stream() for _ in states]
    torch.cuda.synchronize()
    for i in range(steps):
        for st, xs, os, stream in zip(states, new, got, streams):
            with torch.cuda.stream(stream):
                spk.sparsek_decode_step(st, *xs[i], out=os[i])
    torch.cuda.synchronize()
    for a, b, st in zip(want, got, states):
        assert all(torch.equal(x, y) for x, y in zip(a, b))
        assert not spk.sparsek_decode_status(st).any()


def test_decode_without_a_window_between_steps_with_one(oracle):
    """The update of a step is prepared by the one before it, except without a window: both, step by step, from a
    context that fills neither the selection nor the window."""
    require_gpu()
    say("decode prepared updates")
    for w in (0, 1, 2):
        for Gu in (1, 2):
            _, _, flags, _ = run_decode(oracle, 2, 2, Gu, 64, 6, w, 3, 40, ties=True, seed=w)
            assert not flags.any()


def test_decode_fork_of_a_copied_state(oracle):
    """Two generations continue from one state after copy.deepcopy, each as if it were alone; a chunked state as well."""
    import copy

    require_gpu()
    say("decode fork")
    B, H, d, k, w = 1, 2, 64, 10, 8
    hist = history(np.random.default_rng(4), B, H, 1, 60, d, "bf16")
    Q, K, V = (dev(hist[x], True) for x in ("Q", "K", "V"))
    u = dev(hist["u"])

    def go(state, a, b):
        return [spk.sparsek_decode_step(state, *(x[:, :, t].contiguous() for x in (Q, K, V, u))) for t in range(a, b)]

    state = spk.DecodeState(B, H, 1, d, k, w, torch.bfloat16)
    spk.sparsek_decode_init(state)
    go(state, 0, 30)
    fork = copy.deepcopy(state)
    for a, b in zip(go(state, 30, 60), go(fork, 30, 60)):
        assert torch.equal(a, b)
    chunked = spk.ChunkState(B, H, 1, d, k, w, spk.BF16, 64)
    first = [x[:, :, :30].contiguous() for x in (Q, K, V, u)]
    rest = [x[:, :, 30:60].contiguous() for x in (Q, K, V, u)]
    spk.sparsek_chunk_prefill(chunked, *first)
    fork = copy.deepcopy(chunked)
    assert torch.equal(spk.sparsek_chunk_prefill(chunked, *rest), spk.sparsek_chunk_prefill(fork, *rest))
