"""GPU parity of dbl_expand_branches and dbl_prior_head against the oracle (Sec. "Architecture").

The expander output is bf16: the GPU rounds its fp32 result once, the oracle rounds the exact
binary64 value once. They agree except where the exact value lies within the fp32 error of a
bf16 rounding midpoint; every element must lie within half a bf16 ulp plus that error of the
exact value, and at least 99% must be identical. Prior logits are fp32 accumulations, compared
against binary64 within the accumulation error bound.
"""
import time

import numpy as np
import pytest
import torch

import synth
from oracle import expander as EX

pytestmark = pytest.mark.gpu


def _np(t):
    return t.detach().to("cpu", torch.float64).numpy()


EXPAND_CASES = [
    # name, B, K, R, d
    ("small", 2, 4, 3, 64),
    ("ragged-rows", 1, 7, 5, 96),
    ("qwen3-4b-paper-R", 1, 16, 4, 2560),
    ("qwen3-8b-R8", 16, 16, 8, 4096),
    ("max-categories", 1, 3, 64, 64),
    ("two-row-tiles-ragged", 2, 150, 2, 128),   # 300 trunk rows: a second, partial 256-row tile
]


def _expander_case(name, B, K, R, d):
    """One expander call at this shape against the oracle (all rows, or 48 sampled ones)."""
    from paper_2608_05448_amd import dblast as D
    print(f"[expander] {name} B={B} K={K} R={R} d={d}", flush=True)
    h = synth.make_uniform_logits((B, K, d), 11).to(torch.bfloat16)
    W = (synth.make_uniform_logits((R * d, d), 12) * (0.5 / d ** 0.5)).to(torch.bfloat16)
    c = (synth.make_uniform_logits((R * d,), 13) * 0.1).to(torch.bfloat16)
    hd, Wd, cd = h.cuda(), W.cuda(), c.cuda()
    out = D.dbl_expand_branches(hd, Wd, cd, R)
    torch.cuda.synchronize()
    if B * K * R * d >= 1 << 22:   # time the benchmark-sized case
        n = 10
        t0 = time.perf_counter()
        for _ in range(n):
            D.dbl_expand_branches(hd, Wd, cd, R, out=out)
        torch.cuda.synchronize()
        ms = (time.perf_counter() - t0) / n * 1e3
        print(f"[expander] {name}: {ms:.3f} ms, {2 * B * K * R * d * d / ms / 1e9:.1f} TFLOP/s",
              flush=True)
    got = _np(out)
    hh, WW, cc = _np(h), _np(W), _np(c)
    if B * K > 64:   # check a sample of rows at the large shape
        rows = np.random.default_rng(0).choice(B * K, 48, replace=False)
    else:
        rows = np.arange(B * K)
    exact = EX.expand_branches(hh.reshape(-1, d)[rows], WW, cc)          # [n, R, d]
    g = got.reshape(B * K, R, d)[rows]
    ulp = np.ldexp(1.0, np.frexp(exact)[1] - 8)
    err_bound = 0.5 * ulp + 1e-5 * np.abs(exact) + 1e-6
    assert np.all(np.abs(g - exact) <= err_bound)
    same = np.mean(g == EX.bf16_round(exact))
    assert same > 0.99, same


@pytest.mark.parametrize("case", EXPAND_CASES, ids=[c[0] for c in EXPAND_CASES])
def test_expander_parity(case):
    _expander_case(*case)


def test_expander_random_shapes():
    """A seeded sweep of random expander shapes: hidden sizes that are multiples of 32 (both the
    64-deep and the 32-deep kernels), odd category counts and ragged trunk-row tiles."""
    rng = np.random.default_rng(20261206)
    for i in range(10):
        B, K = int(rng.integers(1, 6)), int(rng.integers(1, 70))
        R, d = int(rng.integers(1, 20)), 32 * int(rng.integers(1, 21))
        _expander_case(f"random-{i}", B, K, R, d)


def test_zero_expander_copies_the_trunk_state():
    from paper_2608_05448_amd import dblast as D
    B, K, R, d = 3, 5, 4, 128
    h = synth.make_uniform_logits((B, K, d), 21).to(torch.bfloat16).cuda()
    W = torch.zeros((R * d, d), dtype=torch.bfloat16, device="cuda")
    c = torch.zeros(R * d, dtype=torch.bfloat16, device="cuda")
    out = D.dbl_expand_branches(h, W, c, R)
    torch.cuda.synchronize()
    for z in range(R):
        assert torch.equal(out[:, :, z], h)


def test_expander_feeds_the_head():
    """Expander -> head on the GPU against the oracle chain (rounded branch states -> binary64
    head) within the bf16 head tolerance."""
    from oracle import head as OH
    from paper_2608_05448_amd import dblast as D
    B, K, R, d, V = 1, 4, 3, 256, 3000
    h = synth.make_uniform_logits((B, K, d), 31).to(torch.bfloat16)
    W = (synth.make_uniform_logits((R * d, d), 32) * (0.5 / d ** 0.5)).to(torch.bfloat16)
    c = (synth.make_uniform_logits((R * d,), 33) * 0.1).to(torch.bfloat16)
    w = (synth.make_uniform_logits((V, d), 34) * (2.0 / d ** 0.5)).to(torch.bfloat16)
    hb = D.dbl_expand_branches(h.cuda(), W.cuda(), c.cuda(), R)
    tls, lmass, lse = D.dbl_head_logprobs(hb, w.cuda())
    torch.cuda.synchronize()
    branch = EX.expand_branches(_np(h), _np(W), _np(c), round_bf16=True).reshape(-1, d)
    want = OH.head_logq(branch, _np(w))
    from cases import flat_from_factored
    got = flat_from_factored(tls.cpu().numpy(), lmass.cpu().numpy(), lse.cpu().numpy())
    assert np.max(np.abs(got.reshape(-1, V) - want)) < 2e-3


PRIOR_CASES = [("small", 3, 4, 64), ("paper-R", 16, 4, 4096), ("many", 300, 64, 2560)]


@pytest.mark.parametrize("case", PRIOR_CASES, ids=[c[0] for c in PRIOR_CASES])
def test_prior_head_parity(case):
    from paper_2608_05448_amd import dblast as D
    name, B, R, d = case
    print(f"[prior head] {name} B={B} R={R} d={d}", flush=True)
    ha = synth.make_uniform_logits((B, d), 41).to(torch.bfloat16)
    U = (synth.make_uniform_logits((R, d), 42) * (1.0 / d ** 0.5)).to(torch.bfloat16)
    e = synth.make_uniform_logits((R,), 43).to(torch.bfloat16)
    ell = D.dbl_prior_head(ha.cuda(), U.cuda(), e.cuda())
    torch.cuda.synchronize()
    want = EX.prior_logits(_np(ha), _np(U), _np(e))
    bound = 1e-5 * (np.abs(_np(ha)) @ np.abs(_np(U)).T + np.abs(_np(e))) + 1e-6
    assert np.all(np.abs(ell.cpu().numpy() - want) <= bound)


# Hidden sizes at the edges of the 16-byte load path: one load of one thread, no multiple of 8 (the
# scalar path), just below and above one round of the workgroup's 2048 units, a ragged third round.
PRIOR_EDGES = [("one-load", 2, 1, 8), ("scalar", 2, 3, 77), ("below-a-round", 1, 5, 2040),
               ("past-a-round", 3, 2, 2056), ("third-round", 2, 64, 4104)]


@pytest.mark.parametrize("case", PRIOR_EDGES, ids=[c[0] for c in PRIOR_EDGES])
def test_prior_head_edges(case):
    test_prior_head_parity(case)


# One shape per tile of the expander's dispatch and at its edges: 64 x 32 (32 rows and few features),
# 64 x 64 (33 rows; any row count when d % 128 != 0), 128 x 64, 128 x 128 and 128 x 256 tiles with
# full and ragged last row tiles.
EXPAND_EDGES = [
    ("64x32-one-row", 1, 1, 1, 128), ("64x32-full", 1, 32, 4, 256), ("64x64-odd-blocks", 1, 5, 3, 192),
    ("64x64-rows", 1, 33, 40, 256), ("128x64-full", 1, 64, 40, 512), ("128x64-ragged", 1, 65, 20, 512),
    ("128x128-ragged", 1, 100, 40, 512), ("128x128-two", 3, 43, 40, 256), ("128x256", 1, 200, 60, 384),
    ("two-256-row-tiles", 1, 300, 30, 384),
]


@pytest.mark.parametrize("case", EXPAND_EDGES, ids=[c[0] for c in EXPAND_EDGES])
def test_expander_edges(case):
    _expander_case(*case)


# A trunk row's branch states do not depend on the other rows of the call: row counts that take every
# tile, up to the 256 x 256 ones, at hidden sizes whose sum starts at 0 (128, 192) and, from the second
# group of 1024 features on, further on (2048).
@pytest.mark.parametrize("R,d", [(48, 128), (32, 192), (3, 2048)])
def test_expander_rows_do_not_depend_on_the_batch(R, d):
    from paper_2608_05448_amd import dblast as D
    M = 2900
    h = synth.make_uniform_logits((1, M, d), 81).to(torch.bfloat16).cuda()
    W = (synth.make_uniform_logits((R * d, d), 82) * (0.5 / d ** 0.5)).to(torch.bfloat16).cuda()
    c = (synth.make_uniform_logits((R * d,), 83) * 0.1).to(torch.bfloat16).cuda()
    whole = D.dbl_expand_branches(h, W, c, R)
    for lo, n in ((5, 1), (0, 32), (9, 33), (64, 64), (70, 65), (0, 128), (33, 129), (300, 256),
                  (1000, 700)):
        print(f"[expander] R={R} d={d} rows {lo}..{lo + n} alone", flush=True)
        part = D.dbl_expand_branches(h[:, lo:lo + n].contiguous(), W, c, R)
        assert torch.equal(whole[:, lo:lo + n], part), (R, d, lo, n)
