"""GPU parity of dbl_target_logprobs and dbl_early_determinism against the oracle.

The kept set of every row (which ids are finite) must be identical: both cuts are integer
decisions on binary32 values computed the same way on both sides. Log-probabilities of kept ids
agree within 2e-6 (binary64 normaliser summed in a different order, stored as binary32).
"""
import time

import numpy as np
import pytest
import torch

import synth
from oracle import target as TG

pytestmark = pytest.mark.gpu


def _logits(N, V, seed, ties=False):
    if ties == "flat":   # every logit equal: top-k keeps the whole row
        return np.zeros((N, V), np.float32)
    g = synth.make_uniform_logits((N, V), seed, scale=3.0).numpy()
    perm = np.random.default_rng(seed).permutation(V)
    g = g - 1.1 * np.log1p(perm)[None, :]
    if ties == "ulp":   # the 40 largest logits one ulp apart: fl32(x / T) merges neighbours
        g = g.astype(np.float32)
        for r in range(N):
            top = np.argsort(-g[r])[:40]
            g[r, top] = np.float32(7.0) + np.arange(40, dtype=np.float32) * np.spacing(np.float32(7.0))
    elif ties == "tail":   # one token at 0, the rest ~27.5 below it, where the integer masses
        # are 0, 1 or 2: a nucleus with p near 1 cuts there, in a bin past 2000 (the kernel then
        # computes the masses in every pass, not the bins alone)
        g = (-27.5 + 0.15 * synth.make_uniform_logits((N, V), seed).numpy()).astype(np.float32)
        g[:, 0] = 0.0
    elif ties in ("falling", "falling-noise"):   # logits that fall with the id, as in a vocabulary
        # ordered by frequency; without noise neighbours in the tail differ by 1e-5
        g = -1.1 * np.log1p(np.arange(V))[None, :] + np.zeros((N, 1))
        if ties == "falling-noise":
            g = g + 0.7 * np.random.default_rng(seed).standard_normal((N, V))
    elif ties == "bf16":   # logits of a bf16 head
        g = torch.from_numpy(g).to(torch.bfloat16).float().numpy()
    elif ties == "masked":   # the last quarter of the vocabulary is never allowed
        g = g.astype(np.float32)
        g[:, V - V // 4:] = -np.inf
    elif ties:   # coarse values: many equal logits at both cuts
        g = np.round(g * 2.0) / 2.0
    return g.astype(np.float32)


CASES = [
    # name, N, V, T, top_k, top_p, ties
    ("paper-t07-k20-p08", 6, 151936, 0.7, 20, 0.8, False),
    ("paper-t10-k20-p095", 6, 151936, 1.0, 20, 0.95, False),
    ("paper-t15-k20-p095", 6, 151936, 1.5, 20, 0.95, False),
    ("greedy", 5, 151936, 0.0, 20, 0.95, False),
    ("nucleus-only", 4, 151936, 1.0, 0, 0.9, False),
    ("top-k-only", 4, 50000, 1.0, 50, 1.0, False),
    ("no-filter", 3, 3001, 1.3, 0, 1.0, False),
    ("ties-at-both-cuts", 16, 2000, 1.0, 30, 0.7, True),
    ("ties-nucleus-only", 16, 2000, 1.0, 0, 0.5, True),
    ("tiny-vocab", 8, 7, 1.0, 3, 0.6, True),
    ("top-k-ragged-row", 4, 50001, 1.0, 50, 0.9, False),
    ("top-k-1000-ties", 4, 151936, 1.0, 1000, 0.9, True),
    ("top-k-1024", 3, 151936, 1.2, 1024, 0.95, False),
    ("top-k-1025", 3, 151936, 1.2, 1025, 0.95, False),
    ("flat-row-top-k", 2, 151936, 1.0, 20, 0.95, "flat"),
    ("one-ulp-neighbours-t15", 4, 30000, 1.5, 20, 0.95, "ulp"),
    ("one-ulp-neighbours-t07", 4, 30000, 0.7, 20, 0.95, "ulp"),
    ("temperature-3e4-merges-values", 4, 30000, 3e4, 20, 0.95, False),
    ("temperature-1e-3", 4, 30000, 1e-3, 20, 0.9, False),
    ("split-k256", 3, 151936, 1.0, 256, 0.95, False),
    ("split-k257", 3, 151936, 1.0, 257, 0.95, False),
    ("split-ties-overflow", 3, 151936, 1.0, 20, 0.95, True),
    ("split-smallest-vocab", 3, 16384, 1.0, 20, 0.95, False),
    ("split-ragged-vocab", 3, 16387, 1.0, 20, 0.95, False),
    ("nucleus-p0999", 3, 151936, 1.0, 0, 0.999, False),
    ("nucleus-p001", 3, 151936, 1.0, 0, 0.01, False),
    ("nucleus-high-T", 3, 151936, 5.0, 0, 0.9, False),
    ("nucleus-top-k-ge-V", 2, 3000, 1.0, 5000, 0.8, False),
    ("nucleus-ragged-vocab", 3, 50001, 0.7, 0, 0.8, False),
    ("flat-row-nucleus", 2, 151936, 1.0, 0, 0.95, "flat"),
    ("flat-row-nucleus-t07", 2, 40000, 0.7, 0, 0.95, "flat"),
    ("nucleus-cut-in-the-tail", 2, 151936, 1.0, 0, 0.9999999, "tail"),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_target_filter_parity(case):
    """Both launch forms (rows split over several workgroups through the workspace, and one
    workgroup per row) against the oracle, and bit-identical to each other."""
    from paper_2608_05448_amd import dblast as D
    name, N, V, T, k, p, ties = case
    print(f"[target] {name} N={N} V={V} T={T} k={k} p={p}", flush=True)
    lg = _logits(N, V, 7 + len(name), ties)
    lgd = torch.from_numpy(lg).cuda()
    got = D.dbl_target_logprobs(lgd, T, k, p)
    one = D.dbl_target_logprobs(lgd, T, k, p, split=False)
    torch.cuda.synchronize()
    assert torch.equal(got, one)
    got = got.cpu().numpy()
    want = TG.filter_logprobs(lg, T, k, p)
    assert np.array_equal(np.isfinite(got), np.isfinite(want))
    fin = np.isfinite(want)
    assert np.max(np.abs(got[fin] - want[fin])) < 2e-6
    print(f"[target] {name}: kept per row {np.isfinite(want).sum(1).tolist()}", flush=True)


def test_target_filter_benchmark_rows():
    """The Qwen3-8B verification rows (16 blocks x 17 positions) with the paper's filters."""
    from paper_2608_05448_amd import dblast as D
    N, V = 272, 151936
    lg = torch.from_numpy(_logits(N, V, 99)).cuda()
    out = torch.empty_like(lg)
    ws = torch.empty(D.dbl_workspace_bytes(D.DBL_OP_TARGET, N, 1, 1, 0, V), dtype=torch.uint8,
                     device="cuda")
    for T, k, p in ((0.7, 20, 0.8), (1.0, 20, 0.95), (1.5, 20, 1.0), (1.0, 0, 0.95)):
        for split in (True, False):
            D.dbl_target_logprobs(lg, T, k, p, out=out, ws=ws, split=split)
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            for _ in range(5):
                D.dbl_target_logprobs(lg, T, k, p, out=out, ws=ws, split=split)
            torch.cuda.synchronize()
            ms = (time.perf_counter() - t0) / 5 * 1e3
            print(f"[target] rows {N} x {V}, T={T} k={k} p={p} split={split}: {ms:.3f} ms "
                  f"({N * V * 8 / ms / 1e6:.0f} GB/s of logits in + logp out)", flush=True)
    rows = [0, 135, 271]
    want = TG.filter_logprobs(lg[rows].cpu().numpy(), 1.0, 0, 0.95)
    got = out[rows].cpu().numpy()
    assert np.array_equal(np.isfinite(got), np.isfinite(want))


def test_early_determinism_parity():
    from paper_2608_05448_amd import dblast as D
    M, b, V = 300, 8, 500
    lp = TG.filter_logprobs(_logits(M * b, V, 5), 1.0, 20, 0.9).reshape(M, b, V)
    rng = np.random.default_rng(6)
    p = np.exp(lp.astype(np.float64))
    cum = np.cumsum(p / p.sum(-1, keepdims=True), -1)
    x = np.minimum((cum < rng.random((M, b, 1))).sum(-1), V - 1).astype(np.int32)
    terms, mean = D.dbl_early_determinism(torch.from_numpy(x).cuda(), torch.from_numpy(lp).cuda())
    torch.cuda.synchronize()
    lpx = lp[np.arange(M)[:, None], np.arange(b)[None, :], x]
    want_terms = np.exp(np.cumsum(lpx.astype(np.float64), axis=1)).mean(1)
    np.testing.assert_allclose(terms.cpu().numpy(), want_terms, rtol=1e-6, atol=1e-9)
    assert abs(mean.item() - TG.early_determinism(lpx)) < 1e-6


# Rows split over workgroups, at the edges of their parts: two segments of 8192 ids exactly, one id
# and one group of four more, a third segment of one id, one and two mass parts of 32,768, the share
# counts' step at k = 128, and a quarter of the vocabulary masked (whole shares without a bound).
SPLIT_EDGES = [(f"{m}-{V}{'-' + t if t else ''}", 3, V, T, k, p, t)
               for V, t in ((16384, False), (16385, False), (16388, False), (24577, False),
                            (32768, False), (32771, False), (40000, "masked"))
               for m, T, k, p in (("scale", 0.7, 0, 1.0), ("nucleus", 1.3, 0, 0.9),
                                  ("k128", 0.7, 128, 0.95), ("k129", 1.0, 129, 1.0))]


@pytest.mark.parametrize("case", SPLIT_EDGES, ids=[c[0] for c in SPLIT_EDGES])
def test_target_split_edges(case):
    test_target_filter_parity(case)


def test_target_scale_normalises():
    """The temperature alone: every row's probabilities sum to one, in one and in many segments."""
    from paper_2608_05448_amd import dblast as D
    for V in (1, 5, 8192, 8193, 151936):
        lg = torch.from_numpy(_logits(2, V, 31)).cuda()
        for T in (0.6, 1.0, 5.0):
            out = D.dbl_target_logprobs(lg, T)
            assert torch.equal(out, D.dbl_target_logprobs(lg, T, split=False))
            # s = fl32(logit / T): divided on the host, where the division is correctly rounded
            s = torch.from_numpy(lg.cpu().numpy() / np.float32(T)).double()
            want = torch.log_softmax(s, -1)
            # binary32 results (half a unit of the value) of a binary64 normaliser, with slack
            err = (out.cpu().double() - want).abs()
            assert (err <= want.abs() * 2.0 ** -23 + 2.0 ** -30).all(), (V, T, err.max())


# Top-k rows whose shares list more tokens than they have room for: the smallest and ragged vocabularies
# (shares of 1024 ids, a last partial group of four) and the full one, both share counts, with lists that
# count (the first shares' or, with noise, most of them) and lists that do not (the tail's).
FALLING = [(f"{t}-{V}-k{k}", 3, V, T, k, p, t)
           for t in ("falling", "falling-noise", "bf16")
           for V, T, k, p in ((151936, 0.7, 5, 0.95), (151936, 1.0, 100, 1.0), (151936, 0.7, 128, 0.95),
                              (151935, 1.3, 256, 1.0), (40001, 0.7, 128, 0.9), (16384, 1.0, 128, 1.0),
                              (16387, 1.0, 256, 0.95))]

# Few allowed ids: fewer than k of them (the k-th largest is -inf and nothing is cut), just k and a few
# more, scattered and in one share alone; shares without a bound, with and without enough threads that
# hold an allowed id, and rows in which no share has one.
ALLOWED = [(f"{n}-allowed-{'one-share' if lo else 'scattered'}-k{k}-p{p}", n, lo, k, p)
           for n, lo in ((10, False), (10, True), (200, False), (200, True), (2500, True))
           for k, p in ((20, 1.0), (20, 0.9), (200, 0.95), (256, 1.0))]


@pytest.mark.parametrize("case", ALLOWED, ids=[c[0] for c in ALLOWED])
def test_target_few_allowed_ids(case):
    from paper_2608_05448_amd import dblast as D
    name, n, one_share, k, p = case
    N, V, T = 3, 40001, 0.7
    rng = np.random.default_rng(len(name) + n)
    lg = np.full((N, V), -np.inf, np.float32)
    for r in range(N):
        ids = 2600 + np.arange(n) if one_share else rng.permutation(V)[:n]
        lg[r, ids] = 3.0 * rng.standard_normal(n)
    lgd = torch.from_numpy(lg).cuda()
    got = D.dbl_target_logprobs(lgd, T, k, p)
    assert torch.equal(got, D.dbl_target_logprobs(lgd, T, k, p, split=False))
    got, want = got.cpu().numpy(), TG.filter_logprobs(lg, T, k, p)
    fin = np.isfinite(want)
    assert np.array_equal(np.isfinite(got), fin)
    assert np.max(np.abs(got[fin] - want[fin])) < 2e-6


# The rows' and temperatures' ranges in which the transform divides in full: T beyond 2^-20 and 2^20 (the
# logits scaled along, so that the distribution is the usual one), and a largest logit of 0.
@pytest.mark.parametrize("T", [2.0 ** -21, 2.0 ** 21, 0.7])
@pytest.mark.parametrize("p", [1.0, 0.9])
@pytest.mark.parametrize("top_zero", [False, True])
def test_target_division_ranges(T, p, top_zero):
    from paper_2608_05448_amd import dblast as D
    s = _logits(3, 40001, 17).astype(np.float64)
    if top_zero:
        s -= s.max(-1, keepdims=True)
    lg = (s * T).astype(np.float32)
    lgd = torch.from_numpy(lg).cuda()
    got = D.dbl_target_logprobs(lgd, T, 0, p)
    assert torch.equal(got, D.dbl_target_logprobs(lgd, T, 0, p, split=False))
    got, want = got.cpu().numpy(), TG.filter_logprobs(lg, T, 0, p)
    fin = np.isfinite(want)
    assert np.array_equal(np.isfinite(got), fin)
    assert np.max(np.abs(got[fin] - want[fin])) < 2e-6


@pytest.mark.parametrize("case", FALLING, ids=[c[0] for c in FALLING])
def test_target_falling_logits(case):
    test_target_filter_parity(case)


def _best_us(f, n=10, rounds=5):
    """The shortest of several runs of n calls, us per call."""
    for _ in range(3):
        f()
    best = 1e9
    for _ in range(rounds):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(n):
            f()
        torch.cuda.synchronize()
        best = min(best, (time.perf_counter() - t0) / n * 1e6)
    return best


def test_target_topk_time_in_any_order():
    """Top-k rows whose logits fall with the id take about as long as the same logits shuffled (24 times
    as long when a share's overflowing list sent the row to the general path)."""
    from paper_2608_05448_amd import dblast as D
    N, V = 16, 151936
    fall = torch.from_numpy(_logits(N, V, 3, "falling-noise")).cuda()
    mono = torch.from_numpy(_logits(N, V, 3, "falling")).cuda()
    mixed = fall[:, torch.randperm(V, device="cuda")].contiguous()
    for k in (20, 128, 256):
        us = [_best_us(lambda x=x: D.dbl_target_logprobs(x, 0.7, k, 0.95)) for x in (mixed, fall, mono)]
        print(f"[target] k={k}: shuffled {us[0]:.1f} us, falling {us[1]:.1f}, without noise {us[2]:.1f}",
              flush=True)
        assert max(us[1:]) < 4 * us[0]


# Nucleus rows by the number of tokens in the crossing bin: the former list's room and the present one's
# (4,090), the one-workgroup form's 4,096, and more, up to bins that are known from their mass not to fit.
@pytest.mark.parametrize("T", [1.0, 0.7])
@pytest.mark.parametrize("n", [1, 2030, 2100, 4089, 4090, 4091, 4096, 4097, 4200, 30000])
def test_target_crowded_nucleus_bin(n, T):
    from paper_2608_05448_amd import dblast as D
    N, V = 2, 40003
    rng = np.random.default_rng(n)
    s = np.full((N, V), -60.0)
    for r in range(N):
        ids = rng.permutation(V)[:n + 1]
        s[r, ids[0]] = 0.0
        s[r, ids[1:]] = -5.0 - 0.004 * rng.random(n)   # one bin: -5.0089 < s - m <= -4.9953
    lg = (s * T).astype(np.float32)
    p = float(np.float32((1.0 + 0.5 * n * np.exp(-5.002)) / (1.0 + n * np.exp(-5.002))))
    lgd = torch.from_numpy(lg).cuda()
    got = D.dbl_target_logprobs(lgd, T, 0, p)
    assert torch.equal(got, D.dbl_target_logprobs(lgd, T, 0, p, split=False))
    got, want = got.cpu().numpy(), TG.filter_logprobs(lg, T, 0, p)
    fin = np.isfinite(want)
    print(f"[target] n={n} T={T}: kept per row {fin.sum(1).tolist()}", flush=True)
    assert np.array_equal(np.isfinite(got), fin)
    assert np.max(np.abs(got[fin] - want[fin])) < 2e-6


@pytest.mark.parametrize("scale,most", [(1.0, 0.8), (0.01, 1.1)])
def test_target_wide_nucleus_is_no_slower_split(scale, most):
    """Rows at high temperature, split against one workgroup per row: a few thousand tokens in the crossing
    bin (1.22 times as long when their list overflowed), and nearly flat rows, which need the general
    path (1.31 times)."""
    from paper_2608_05448_amd import dblast as D
    lg = scale * torch.randn((16, 151936), device="cuda")
    a, b = (_best_us(lambda x=x: D.dbl_target_logprobs(lg, 5.0, 0, 0.9, split=x)) for x in (True, False))
    print(f"[target] noise {scale}: split {a:.1f} us, one workgroup per row {b:.1f}", flush=True)
    assert a < most * b


NAN_ROWS = [(V, T, k, p) for V, T, k, p in (
    (5, 1.0, 0, 1.0), (3001, 0.7, 0, 1.0), (16384, 1.3, 0, 1.0), (40001, 0.7, 0, 1.0), (40001, 1.0, 0, 1.0),
    (20000, 0.7, 0, 0.9), (40001, 0.7, 0, 0.9), (151936, 1.0, 0, 0.95), (40001, 0.7, 0, 0.01),
    (20001, 0.7, 20, 0.9), (40001, 1.0, 200, 1.0), (3001, 1.0, 20, 0.9))]


@pytest.mark.parametrize("V,T,k,p", NAN_ROWS)
def test_target_nan_logits(V, T, k, p):
    """A NaN logit of either sign shows: under the temperature alone the whole row is NaN, as in the
    oracle; under the filters both launch forms agree, and a NaN without the sign bit, the largest key,
    makes every kept value NaN. The call's other rows do not change."""
    from paper_2608_05448_amd import dblast as D
    at = sorted({0, V // 3, V // 2, V - 1})
    lg = _logits(2 * len(at) + 1, V, 41)
    for i, v in enumerate(at):
        lg[2 * i, v] = np.float32("nan")
        lg[2 * i + 1, v] = np.copysign(np.float32("nan"), np.float32(-1.0))
    assert np.signbit(lg[1, at[0]]) and not np.signbit(lg[0, at[0]])
    lgd = torch.from_numpy(lg).cuda()
    got = D.dbl_target_logprobs(lgd, T, k, p).cpu().numpy()
    one = D.dbl_target_logprobs(lgd, T, k, p, split=False).cpu().numpy()
    assert np.array_equal(got, one, equal_nan=True)
    want = TG.filter_logprobs(lg[-1:], T, k, p)[0]
    fin = np.isfinite(want)
    assert np.array_equal(np.isfinite(got[-1]), fin) and np.abs(got[-1][fin] - want[fin]).max() < 2e-6
    for i, v in enumerate(at):
        if k == 0 and p == 1.0:
            assert np.isnan(got[2 * i:2 * i + 2]).all(), v
        else:
            assert not np.isfinite(got[2 * i]).any() and np.isnan(got[2 * i, v]), v
            if k == 0 and p > 0.5:
                assert np.isnan(got[2 * i + 1, v]), v


@pytest.mark.parametrize("N,V", [(40000, 3), (20000, 7), (300, 3001), (3, 40001)])
def test_target_scale_rounds_correctly(N, V):
    """The temperature alone: a binary64 normaliser, so results are its correctly rounded binary32 values but
    for the odd one within 2^-50 or so of a midpoint (with sums good to
    2^-32 one in 12,000 differed, with few ids per row)."""
    from paper_2608_05448_amd import dblast as D
    lg = np.random.default_rng(V).standard_normal((N, V)).astype(np.float32)
    for T in (0.7, 1.0):
        got = D.dbl_target_logprobs(torch.from_numpy(lg).cuda(), T).cpu().numpy()
        s = (lg / np.float32(T)).astype(np.float64)
        d = s - s.max(-1, keepdims=True)
        want = (d - np.log(np.exp(d).sum(-1, keepdims=True))).astype(np.float32)
        bad = int((got != want).sum())
        print(f"[target] scale N={N} V={V} T={T}: {bad} of {got.size} rounded otherwise", flush=True)
        assert bad <= 2 + got.size // 10 ** 6
