"""GPU parity of stages 1+2 (sparsek_mask, sparsek_materialize) against the CPU oracle.

Bars: lifetimes and index sets bit-exact; thresholds and masks within 1e-5 (relative to
max(1,|ref|); masks live in [0,1]).
"""
import numpy as np
import pytest
import torch

import paper_2406_16747_amd as spk
from paper_2406_16747_amd import synth
from gpu_util import dev, host, require_gpu, say

pytestmark = pytest.mark.gpu


def scores(kind, rng, rows, n):
    if kind == "normal":
        return rng.standard_normal((rows, n), dtype=np.float32)
    if kind == "ties":  # coarse grid: many exact ties
        return (np.round(rng.standard_normal((rows, n)) * 4) / 4).astype(np.float32)
    if kind == "equal":
        return np.full((rows, n), 0.5, np.float32)
    if kind == "rising":  # every newcomer enters the top-k
        return (np.arange(n, dtype=np.float32)[None] * 0.01 + rng.standard_normal((rows, 1), dtype=np.float32))
    if kind == "falling":
        return (-np.arange(n, dtype=np.float32)[None] * 0.01).repeat(rows, 0)
    if kind == "wide":  # gaps mostly above 1: hard top-k, flat tau
        return (rng.standard_normal((rows, n)) * 50).astype(np.float32)
    if kind == "drift":
        pos = np.arange(n, dtype=np.float32)
        return (rng.standard_normal((rows, n), dtype=np.float32) + 0.5 * np.sin(pos / 256)).astype(np.float32)
    raise ValueError(kind)


def check_rows(oracle, u, k, sample_t=None, every=1):
    """`every`: of many rows, look at the first, the last and each so many in between."""
    rows, n = u.shape
    ud = dev(u.reshape(rows, 1, n))
    ws = spk.sparsek_mask_workspace(ud, k)
    ws.fill_(0xFF)  # the call itself must clear its status word
    tau_g, death_g = spk.sparsek_mask(ud, k, ws=ws)
    assert spk.sparsek_mask_status(ud, k, ws) == 0  # every threshold solve converged
    tau_g, death_g = host(tau_g).reshape(rows, n), host(death_g).reshape(rows, n)
    looked_at = sorted({*range(0, rows, every), rows - 1})
    for r in looked_at:
        tau_r, us, ws = oracle.tau_prefixes(u[r], k)
        death_r = oracle.death(u[r], k)
        np.testing.assert_array_equal(death_g[r], death_r)
        err = np.abs(tau_g[r].astype(np.float64) - tau_r) / np.maximum(1.0, np.abs(tau_r))
        assert err.max() <= 1e-5, (r, int(err.argmax()), err.max())
    # explicit lists + gates on sampled prefixes
    ts = sample_t if sample_t is not None else sorted(set([0, min(n - 1, max(k - 1, 0)), min(n - 1, k), n // 2, n - 1]))
    for t in ts:
        idx, gate = spk.sparsek_materialize(ud, dev(tau_g.reshape(rows, 1, n)), dev(death_g.reshape(rows, 1, n)),
                                            k, t, t + 1)
        idx, gate = host(idx).reshape(rows, -1), host(gate).reshape(rows, -1)
        for r in looked_at:
            want = oracle.select_prefix(u[r], t, k)
            got = idx[r][idx[r] >= 0]
            np.testing.assert_array_equal(got, want)
            assert np.all(idx[r][len(want):] == -1)
            tau_t, p, _, _ = oracle.sparsek(u[r, : t + 1], k)
            np.testing.assert_allclose(gate[r][: len(want)], p[want], atol=1e-5, rtol=0)
    return tau_g, death_g


def route(rows, n, k):
    """The kernel and the deal that sparsek_mask takes, by the rule of its launch: "short" (a wave per prefix), or the length
    of the chunks, "+" how many of them are split, and "x2" where two workgroups share a compute unit (several rounds)."""
    if 1 <= k < n <= 2048 and rows * n * n <= 1 << 22 and (n <= 48 or rows * n <= 20 << 10):
        return "short"
    up = lambda a, b: -(-a // b)
    if rows * up(n, 32) <= 256:
        length, split, part = 32, 0, 32
    elif rows * (up(n, 64) + 2) <= 256:
        length, split, part = 64, 2, 32
    else:
        length, split, part = 128, 2, 64
    chunks = up(n, length)
    first = min(k // length, chunks)
    split = min(split, chunks - first)
    if split and first + split == chunks and n - (chunks - 1) * length <= part:
        split -= 1
    idle = min(k, n) // length

    def fits(s):
        total = rows * (chunks + s)
        if total > 256 + (32 if s else 0):
            return False
        load = [0] * 32
        for r in range(rows):
            for i in range(idle, chunks + s):
                load[(r * (chunks + s) + i) % 32] += 1
        return max(load) <= 8 - (total > 256 + (16 if rows <= 16 else 0))

    for s in range(split, -1, -1):
        if fits(s):
            return "%d+%d" % (length, s)
    whole, more = rows * (chunks - idle), rows * (chunks + split - idle)
    if whole <= 512 < more or whole <= 1024 < more or (whole > 1024 and 8 * split > chunks - idle):
        split = 0
    return "%d+%dx2" % (length, split)


@pytest.mark.parametrize("kind", ["normal", "ties", "equal", "rising", "falling", "wide", "drift"])
@pytest.mark.parametrize("n,k", [(1, 1), (5, 2), (130, 7), (1000, 64), (1024, 64), (2500, 300), (4500, 64)])
def test_mask_small(oracle, kind, n, k):
    require_gpu()
    say("mask", kind, n, k)
    rng = np.random.default_rng(n * 1000 + k)
    check_rows(oracle, scores(kind, rng, 3, n), k)


@pytest.mark.parametrize("n,k", [(300, 0), (300, 300), (300, 299), (300, 1000), (2049, 2048), (2300, 1)])
def test_mask_degenerate_k(oracle, n, k):
    require_gpu()
    say("mask degenerate", n, k)
    rng = np.random.default_rng(n + k)
    check_rows(oracle, scores("normal", rng, 2, n), k)


def test_mask_config1(oracle):
    require_gpu()
    inp = synth.make(1)
    say("mask config 1")
    check_rows(oracle, inp["u"].reshape(1, -1), inp["k"], sample_t=[63, 64, 100, 500, 1023])


@pytest.mark.parametrize("n,k,scale,offset", [
    (1500, 200, 1.0, 100.0),    # another histogram window over the whole range
    (1500, 200, 5.0, -40.0),    # a range too wide for one window: the window below the largest score
    (3000, 700, 0.02, 0.0),     # most scores between the bounds: more than one list or the breakpoint table holds
    (2200, 500, 0.2, 3.0),      # more breakpoints than the table of the parallel solution
    (1281, 1152, 1.0, 0.0),     # (a wave per prefix; in chunks: test_mask_edges_of_chunks)
    (1283, 1153, 1.0, 0.0),
])
def test_mask_ranges_and_clusters(oracle, n, k, scale, offset):
    require_gpu()
    say("mask range", n, k, scale, offset)
    rng = np.random.default_rng(n + k)
    check_rows(oracle, (rng.standard_normal((2, n)) * scale + offset).astype(np.float32), k)


@pytest.mark.parametrize("n,k,kind,x", [
    (1500, 200, "scale", 0.001), (1500, 200, "scale", 0.05), (2600, 300, "scale", 0.05), (1500, 200, "scale", 7.0),
    (2600, 300, "scale", 30.0), (1500, 200, "scale", 1e3), (1500, 200, "scale", 1e5), (2600, 130, "scale", 1e5),
    (1500, 200, "offset", 20.0), (1500, 200, "offset", -300.0), (1500, 200, "offset", 1e5),
    (1500, 200, "outlier", 1e3), (1500, 200, "outlier", -1e3),   # a few scores far from an offset of 20
    (1500, 200, "rising", 50.0), (2600, 300, "falling", 50.0),   # windows that move from chunk to chunk
    (1500, 200, "halves", 30.0), (1500, 900, "halves", 300.0),   # two clusters, the k-th largest score in either
    (1400, 600, "levels", 1.0),                                  # (a wave per prefix)
    (2600, 300, "levels", 9.0),                                  # few values: no window is fine enough; more than 512 sorted
])
def test_mask_windows(oracle, n, k, kind, x):
    """Histogram windows other than the first one, and what none of them suits."""
    require_gpu()
    say("mask window", n, k, kind, x)
    check_windows(oracle, 2, n, k, kind, x)


def check_windows(oracle, rows, n, k, kind, x, every=1):
    rng = np.random.default_rng(n + k)
    z = rng.standard_normal((rows, n))
    pos = np.arange(n) / n
    u = {"scale": z * x, "offset": z + x, "outlier": z + 20.0, "rising": 0.1 * z + x * pos, "falling": 0.1 * z - x * pos,
         "halves": 0.05 * z + x * (rng.random((rows, n)) < 0.5), "levels": np.round(z * 2) / 2 + x}[kind]
    if kind == "outlier":
        u[:, rng.integers(0, n, 3)] = x
    # (a threshold of 256 or more is rounded by up to 2^-16 in fp32, which is more than the lists' gates may be off)
    check_rows(oracle, u.astype(np.float32), k, sample_t=None if np.abs(u).max() < 256 else [], every=every)


@pytest.mark.parametrize("n,k,kind,x", [
    (1500, 200, "scale", 0.05), (1500, 200, "scale", 1e3), (1500, 200, "scale", 30.0), (1500, 200, "offset", 20.0),
    (1500, 200, "offset", 1e5), (1500, 200, "outlier", -1e3), (1500, 200, "rising", 50.0), (1500, 200, "falling", 50.0),
    (1500, 900, "halves", 300.0), (1400, 600, "levels", 1.0),
])
@pytest.mark.parametrize("rows,deal", [(12, "128+2"), (30, "128+2x2")])
def test_mask_windows_of_long_chunks(oracle, rows, deal, n, k, kind, x):
    """The same in chunks of 128 (two rows of these lengths have chunks of 32 or a wave per prefix), one workgroup and two
    per compute unit."""
    require_gpu()
    say("mask window, long chunks", rows, n, k, kind, x)
    assert route(rows, n, k) == deal
    check_windows(oracle, rows, n, k, kind, x, every=rows // 4)


@pytest.mark.parametrize("rows,n,k,deal", [
    (3, 1281, 1152, "32+0"), (3, 1283, 1153, "32+0"),         # the k-th prefix ends a chunk, and starts one
    (12, 1281, 1152, "128+1"), (12, 1283, 1153, "128+1"), (25, 1283, 1153, "128+1x2"),
    (3, 1400, 600, "32+0"), (47, 300, 299, "128+0"), (5, 1000, 64, "32+0"), (5, 1024, 64, "32+0"), (160, 130, 7, "128+1x2"),
])
@pytest.mark.parametrize("kind", ["normal", "ties", "equal", "rising", "wide"])
def test_mask_edges_of_chunks(oracle, kind, rows, n, k, deal):
    """Lengths that take a wave per prefix with fewer rows."""
    require_gpu()
    say("mask edges", kind, rows, n, k)
    assert route(rows, n, k) == deal
    check_rows(oracle, scores(kind, np.random.default_rng(n + k), rows, n), k, sample_t=[k - 1, k, n - 1], every=rows // 4 + 1)


@pytest.mark.parametrize("n,k,low", [
    (700, 200, [5]),                                # (a wave per prefix up to 900)
    (700, 200, [0, 1, 60, 127, 130, 199, 200, 500]),
    (900, 300, [3, 255, 256, 299, 300, 301]),
    (900, 300, list(range(0, 280, 2))),             # fewer than k finite scores until position 440
    (1500, 1153, [7, 1100, 1151, 1152]),
    (1500, 100, list(range(0, 700))),               # no finite score until position 700
])
def test_mask_scores_of_minus_infinity(oracle, n, k, low):
    """Padding scored -inf is selected while there are fewer than k other keys, and every lifetime is written.  The
    oracle gets a finite score below all others in its place: the order is the same, and so is every threshold that
    the finite scores determine (the others are -inf)."""
    require_gpu()
    say("mask -inf", n, k, len(low))
    check_minus_infinity(oracle, 2, n, k, low)


@pytest.mark.parametrize("rows,n,k,low,deal", [
    (9, 700, 200, [0, 1, 60, 127, 130, 199, 200, 500], "32+0"), (20, 700, 200, [0, 1, 60, 127, 130, 199, 200, 500], "128+2"),
    (60, 700, 200, [5], "128+2x2"),
    (6, 900, 300, list(range(0, 280, 2)), "32+0"), (16, 900, 300, [3, 255, 256, 299, 300, 301], "128+2"),
    (16, 900, 300, list(range(0, 280, 2)), "128+2"), (50, 900, 300, list(range(0, 280, 2)), "128+2x2"),
    (12, 1500, 1153, [7, 1100, 1151, 1152], "128+2"), (12, 1500, 100, list(range(0, 700)), "128+2"),
])
def test_mask_scores_of_minus_infinity_in_chunks(oracle, rows, n, k, low, deal):
    """The same where prefix k and the scores of -inf lie in chunks of 32 and of 128."""
    require_gpu()
    say("mask -inf in chunks", rows, n, k, len(low))
    assert route(rows, n, k) == deal
    check_minus_infinity(oracle, rows, n, k, low, every=rows // 3)


def check_minus_infinity(oracle, rows, n, k, low, every=1):
    u = np.random.default_rng(n + len(low)).standard_normal((rows, n)).astype(np.float32)
    stand_in = u.copy()
    u[:, low], stand_in[:, low] = -np.inf, np.float32(-1e30)
    ud = dev(u.reshape(rows, 1, n))
    tau = torch.full_like(ud, float("nan"))
    death = torch.full(ud.shape, -(2 ** 31), dtype=torch.int32, device="cuda")
    spk.sparsek_mask_static(ud, k, tau, death)
    for r in range(0, rows, every):
        np.testing.assert_array_equal(host(death)[r, 0], oracle.death(stand_in[r], k))
        tau_r, tau_g = oracle.tau_prefixes(stand_in[r], k)[0], host(tau)[r, 0].astype(np.float64)
        np.testing.assert_array_equal(tau_g == -np.inf, tau_r < -1e29)
        real = tau_r > -1e29
        np.testing.assert_allclose(tau_g[real], tau_r[real], rtol=1e-5, atol=1e-5)


@pytest.mark.parametrize("rows,n,k,share,deal", [
    (1, 1024, 8, 0.02, "short"), (1, 500, 64, 0.3, "short"), (1, 300, 20, 1.0, "short"),
    (8, 1024, 8, 0.02, "32+0"), (40, 500, 64, 0.3, "128+2"), (60, 300, 20, 1.0, "128+1"), (80, 500, 64, 0.3, "128+2x2"),
    (2, 5000, 300, 0.4, "64+2"),
])
def test_mask_scores_of_plus_infinity(oracle, rows, n, k, share, deal):
    """A threshold is +inf (the sup of all points) exactly from min(k, length) scores of +inf on, however many rows and
    however long they are; the others are those of finite scores above all others."""
    require_gpu()
    say("mask +inf", rows, n, k, share)
    assert route(rows, n, k) == deal
    rng = np.random.default_rng(n + k)
    u = rng.standard_normal(n).astype(np.float32)
    at = rng.random(n) < share
    stand_in = u.copy()
    u[at], stand_in[at] = np.inf, 100.0
    tau, death = spk.sparsek_mask(dev(np.repeat(u[None, None], rows, 1)), k)
    tau_r, death_r = oracle.tau_prefixes(stand_in, k)[0], oracle.death(stand_in, k)
    sup = np.cumsum(at) >= np.minimum(k, np.arange(n) + 1)
    assert sup.any()
    for r in {0, rows - 1}:
        tau_g = host(tau)[0, r].astype(np.float64)
        np.testing.assert_array_equal(host(death)[0, r], death_r)
        np.testing.assert_array_equal(tau_g == np.inf, sup)
        np.testing.assert_allclose(tau_g[~sup], tau_r[~sup], rtol=1e-5, atol=1e-5)


@pytest.mark.parametrize("rows,n,k,deal", [
    (2, 4096, 300, "32+0"), (2, 4097, 300, "64+2"),        # the last size of chunks of 32 prefixes, the first of 64
    (4, 3968, 200, "64+2"), (4, 3969, 200, "128+2"),       # the last size of chunks of 64, the first of 128
    (8, 4096, 256, "128+2"), (8, 4096, 255, "128+1"),      # one round: with both chunks around prefix k split, with one
    (16, 2048, 256, "128+1"), (9, 3500, 256, "128+0"),     # ... and none
    (8, 1050, 1030, "64+0"), (16, 1080, 1030, "128+0"),    # prefix k in the last chunk, which is too short to be split
    (16, 1100, 1030, "128+1"), (16, 1200, 1020, "128+2"),  # ... or not; split chunks ahead of the last one
    (6, 9000, 300, "128+2x2"), (20, 3500, 300, "128+2x2"),     # two workgroups per compute unit, in one round and in two
    (16, 4352, 300, "128+0x2"),                            # a split would take a second round
    (40, 3830, 300, "128+2x2"), (50, 3000, 100, "128+2x2"),    # several rounds: numbers of workgroups per row passed over
    (1100, 100, 12, "128+0x2"), (70, 2000, 200, "128+0x2"),    # ... without a split
    (160, 129, 60, "128+1x2"), (1100, 60, 40, "128+0x2"),      # many short rows that go to the chunks
])
def test_mask_deal_of_chunks(oracle, rows, n, k, deal):
    require_gpu()
    say("mask deal", rows, n, k)
    assert route(rows, n, k) == deal
    check_rows(oracle, scores("drift", np.random.default_rng(rows + n + k), rows, n), k, sample_t=[k - 1, k, n - 1],
               every=rows // 16 + 1)


@pytest.mark.parametrize("kind", ["normal", "ties", "equal", "wide", "huge", "minus_inf", "plus_inf"])
@pytest.mark.parametrize("rows,n,k", [
    (1, 2, 1), (3, 5, 4), (1, 64, 63), (2, 257, 1), (1, 2048, 100), (4, 1024, 1023), (4, 1024, 300), (1, 2047, 1500),
    (140, 64, 40), (600, 30, 9),         # more workgroups than have room at once: an odd number per row
    (1, 33, 32), (3, 97, 64),
])
def test_mask_of_short_rows(oracle, kind, rows, n, k):
    """A wave per prefix: edges of its groups of 4 and 256 positions, the longest row, and scores that are not finite
    (the oracle gets +-100 in their place: the order is the same, and so is every threshold that the others, all within
    +-6, determine)."""
    require_gpu()
    say("mask short rows", kind, rows, n, k)
    assert route(rows, n, k) == "short"
    rng = np.random.default_rng(n + k)
    u = (rng.standard_normal((rows, n)) * 1e30).astype(np.float32) if kind == "huge" else scores(
        kind if kind in ("normal", "ties", "equal", "wide") else "normal", rng, rows, n)
    at = rng.random((rows, n)) < (0.3 if kind == "minus_inf" else 0.01)
    odd = {"minus_inf": -np.inf, "plus_inf": np.inf}.get(kind)
    stand_in = u.copy()
    if odd is not None:
        u[at], stand_in[at] = odd, np.float32(np.copysign(100.0, odd))
    ud = dev(u.reshape(1, rows, n))
    ws = spk.sparsek_mask_workspace(ud, k)
    ws.fill_(0xFF)
    tau, death = spk.sparsek_mask(ud, k, ws=ws)
    assert spk.sparsek_mask_status(ud, k, ws) == 0
    tau, death = host(tau)[0], host(death)[0]
    for r in range(rows):
        np.testing.assert_array_equal(death[r], oracle.death(stand_in[r], k))
        tau_r, tau_g = oracle.tau_prefixes(stand_in[r], k)[0], tau[r].astype(np.float64)
        real = np.abs(tau_r) < (np.inf if odd is None else 50.0)   # (else the stand-ins determine it)
        np.testing.assert_allclose(tau_g[real], tau_r[real], rtol=1e-5, atol=1e-5)


@pytest.mark.parametrize("rows,n,k,offset", [
    (1, 2048, 1500, 1e5), (4, 1024, 300, 1e5), (16, 512, 64, 1e5), (16, 512, 64, -2e6), (64, 250, 16, 20.0),
])
def test_mask_of_short_rows_far_from_zero(oracle, rows, n, k, offset):
    """Scores whose fp32 spacing is coarse: the search for a starting point runs out of numbers between its ends, and
    f_t at a root is k up to rounding from either side.  The threshold is the root rounded to fp32 (half its spacing,
    beside which the fp64 error, n * 2^-53 * |offset|, is nothing)."""
    require_gpu()
    say("mask short rows far from zero", rows, n, k, offset)
    assert route(rows, n, k) == "short"
    u = (np.random.default_rng(n + k).standard_normal((rows, n)) + offset).astype(np.float32)
    tau, death = spk.sparsek_mask(dev(u[None]), k)
    for r in range(rows):
        np.testing.assert_array_equal(host(death)[0, r], oracle.death(u[r], k))
        tau_r = oracle.tau_prefixes(u[r], k)[0]
        half = 0.5 * np.spacing(np.abs(u).max())
        assert np.abs(host(tau)[0, r].astype(np.float64) - tau_r).max() <= 1.01 * half, r


def test_mask_candidate_overflow_fallback(oracle):
    """More scores above the threshold than the LDS list holds: the kernel must switch to
    its global-memory path and still be exact."""
    require_gpu()
    say("mask overflow")
    rng = np.random.default_rng(77)
    n, k = 12000, 5000
    u = (rng.standard_normal((1, n)) * 0.05).astype(np.float32)  # w* ~ n: everything is fractional
    check_rows(oracle, u, k, sample_t=[4999, 5000, 9000, n - 1])


def test_mask_is_deterministic(oracle):
    require_gpu()
    rng = np.random.default_rng(5)
    u = dev(rng.standard_normal((4, 1, 6000), dtype=np.float32))
    a = spk.sparsek_mask(u, 200)
    b = spk.sparsek_mask(u, 200)
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])


def test_many_rows_share_a_status_word(oracle):
    """With more than 2048 chunks all of them share one status word, which the call must clear itself (the workspace
    starts as garbage).  Rows of unit variance stay in the first histogram window, narrow scores (nearly every score in
    the support of the threshold) need others, and many equal scores are sorted: all must match the oracle."""
    require_gpu()
    rng = np.random.default_rng(11)
    rows, n, k = 20, 16384, 300   # 20 x 128 chunks > 2048
    u = rng.standard_normal((rows, n)).astype(np.float32)
    u[3] *= 0.02
    u[17] = (np.round(u[17] * 2) / 2).astype(np.float32) * 0.1   # narrow and full of ties
    ud = dev(u.reshape(1, rows, n))
    ws = spk.sparsek_mask_workspace(ud, k)
    for fill in (0xFF, 0x00):
        ws.fill_(fill)
        tau_g, death_g = spk.sparsek_mask(ud, k, ws=ws)
        assert spk.sparsek_mask_status(ud, k, ws) == 0
        tau_g, death_g = host(tau_g).reshape(rows, n), host(death_g).reshape(rows, n)
        for r in (0, 3, 17):
            say("  mask of many rows, row", r)
            tau_r = oracle.tau_incremental(u[r], k)   # pinned against the sort-based routine in the CPU tests
            np.testing.assert_array_equal(death_g[r], oracle.death(u[r], k))
            err = np.abs(tau_g[r].astype(np.float64) - tau_r) / np.maximum(1.0, np.abs(tau_r))
            assert err.max() <= 1e-5, (r, err.max())
