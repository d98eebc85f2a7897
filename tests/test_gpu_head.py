"""GPU parity of dbl_head_logprobs against the oracle head (binary64 GEMM + log-softmax).

Tolerances: 2e-5 absolute on log-probabilities for fp32 inputs and 2e-3 for bf16 inputs with
fp32 accumulation (both sides read the identical bf16 values).
"""
import math
import time

import numpy as np
import pytest
import torch

import synth
from cases import flat_from_factored, np32
from oracle import head as OH

pytestmark = pytest.mark.gpu


def _run(h, w):
    from paper_2608_05448_amd import dblast as D
    out = D.dbl_head_logprobs(h.cuda(), w.cuda())
    torch.cuda.synchronize()
    return [t.cpu().numpy() for t in out]


def _check(h, w, tol, label):
    B, K, R, d = h.shape
    V = w.shape[0]
    print(f"[head] {label} B={B} K={K} R={R} d={d} V={V} dtype={h.dtype}", flush=True)
    tls, lmass, lse = _run(h, w)
    hh, ww = np32(h).reshape(-1, d), np32(w)
    ref = OH.head_logq(hh, ww)
    got = flat_from_factored(tls.reshape(-1, V), lmass.reshape(-1, lmass.shape[-1]),
                             lse.reshape(-1)).astype(np.float64)
    err = np.max(np.abs(got - ref))
    print(f"[head] {label} max |log q error| = {err:.3e}", flush=True)
    assert err < tol
    # The factored parts individually.
    r_tls, r_lm, r_lse = OH.factor_logits(OH.head_logits(hh, ww))
    assert np.max(np.abs(tls.reshape(-1, V) - r_tls)) < tol
    assert np.max(np.abs(lmass.reshape(-1, lmass.shape[-1]) - r_lm)) < tol
    assert np.max(np.abs(lse.reshape(-1) - r_lse)) < tol


def test_head_fp32_tiny_workload():
    wl = synth.WORKLOADS["tiny"]
    _check(synth.make_h(wl), synth.make_w(wl), 2e-5, "tiny")


@pytest.mark.parametrize("B,K,R,d,V", [
    (3, 2, 5, 100, 1000),    # d not a multiple of 8 (fp32 path allows it), ragged last tile
    (1, 1, 1, 1, 1),         # smallest problem
    (2, 3, 7, 40, 129),      # one id in the last tile
])
def test_head_fp32_ragged(B, K, R, d, V):
    h = synth.make_uniform_logits((B, K, R, d), 11).to(torch.float32)
    w = (synth.make_uniform_logits((V, d), 12) / math.sqrt(d)).to(torch.float32)
    _check(h, w, 2e-5, "fp32-ragged")


@pytest.mark.parametrize("B,K,R,d,V", [
    (3, 2, 5, 136, 1000),    # hidden size not a multiple of the 32-wide K step; ragged tiles
    (2, 10, 15, 512, 5000),  # several branch-row and vocabulary tiles, ragged on both
    (1, 4, 5, 64, 1001),     # V % 4 != 0: scalar stores
    (1, 1, 5, 8, 77),        # fewer ids than one tile
    (4, 16, 8, 256, 2048),   # exact tile multiples
    (2, 3, 5, 96, 3001),     # hidden size a multiple of 32 but not 64: direct-to-LDS kernel
    (1, 16, 8, 192, 4100),   # three 64-deep stages (odd count) in the register-staged kernel
    (9, 16, 8, 128, 3000),   # five branch-row tiles: more than one group of the tile order
    (9, 16, 8, 96, 3000),    # the same with the direct-to-LDS kernel
    (1, 1, 3, 64, 270000),   # more than 2048 tiles per row: the LSE pass reads the row twice
    (65, 16, 16, 64, 600),   # 65 branch-row tiles: the tile order's groups of 8, a partial last group
])
def test_head_bf16_ragged(B, K, R, d, V):
    h = synth.make_uniform_logits((B, K, R, d), 21).to(torch.bfloat16)
    w = (synth.make_uniform_logits((V, d), 22) * 0.05).to(torch.bfloat16)
    _check(h, w, 2e-3, "bf16-ragged")


def test_head_bf16_qwen3_8b_all_rows():
    """Full Qwen3-8B-shaped head (the benchmark's launch), every row against the oracle."""
    _full_size("qwen3_8b")


def test_head_bf16_qwen3_4b_all_rows():
    """Full Qwen3-4B-shaped head in the benchmark's launch, every row against the oracle."""
    _full_size("qwen3_4b")


def _full_size(name):
    from cases import oracle_full_head
    from paper_2608_05448_amd import dblast as D
    wl = synth.WORKLOADS[name]
    print(f"[head] full-size {name} M={wl.M} d={wl.d} V={wl.V}", flush=True)
    h = synth.make_h(wl, "cuda")
    w = synth.make_w(wl, "cuda")
    tls, lmass, lse = D.dbl_head_logprobs(h, w)
    torch.cuda.synchronize()
    M, V, nT = wl.M, wl.V, OH.n_tiles(wl.V)
    t2 = tls.view(M, V)
    # Identities at every row: each tile's probabilities sum to 1, tile masses sum to 1.
    tile_sums = torch.exp(t2.view(M, nT, 128).double()).sum(-1)   # V = 1187 * 128 exactly
    assert torch.max(torch.abs(tile_sums - 1.0)).item() < 1e-5
    mass = torch.exp((lmass.view(M, nT) - lse.view(M, 1)).double()).sum(-1)
    assert torch.max(torch.abs(mass - 1.0)).item() < 1e-5
    assert torch.max(t2).item() <= 1e-6
    del tile_sums, mass
    print(f"[head] full-size {name}: oracle head on all {M} rows", flush=True)
    ref = oracle_full_head(name, h, w)
    lm2, ls2 = lmass.view(M, nT), lse.view(M)
    err = 0.0
    for r0 in range(0, M, 256):
        got = flat_from_factored(t2[r0:r0 + 256].cpu().numpy(), lm2[r0:r0 + 256].cpu().numpy(),
                                 ls2[r0:r0 + 256].cpu().numpy())
        err = max(err, float(np.max(np.abs(got.astype(np.float64) - ref[r0:r0 + 256]))))
    print(f"[head] full-size {name} all rows max |log q error| = {err:.3e}", flush=True)
    assert err < 2e-3


def test_head_random_shapes():
    """A seeded sweep of random head shapes in both input precisions: hidden sizes that take each
    bf16 kernel (d % 64 = 0, d % 32 = 0 only, d % 8 = 0 only) and arbitrary fp32 ones, branch-row
    and vocabulary counts with ragged last tiles."""
    rng = np.random.default_rng(20261204)
    for i in range(12):
        bf16 = i % 3 != 2
        B, K, R = int(rng.integers(1, 25)), int(rng.integers(1, 9)), int(rng.integers(1, 9))
        if bf16:
            d = int(rng.choice([64 * int(rng.integers(1, 9)), 32 * int(rng.integers(1, 17)),
                                8 * int(rng.integers(1, 65))]))
        else:
            d = int(rng.integers(1, 300))
        V = int(rng.choice([int(rng.integers(1, 130)), int(rng.integers(130, 6000))]))
        dt = torch.bfloat16 if bf16 else torch.float32
        h = synth.make_uniform_logits((B, K, R, d), 300 + i).to(dt)
        w = (synth.make_uniform_logits((V, d), 400 + i) * (0.05 if bf16 else 1.0 / math.sqrt(d)))
        _check(h, w.to(dt), 2e-3 if bf16 else 2e-5, f"random-{i}")


# Few branch rows (up to 64 and up to 128 per launch, then the 256-row tiles): row counts at the edges
# of the 32-row blocks and of both tiles, 1 to 5 and 64 stages of 64 hidden units (fewer than the ring
# holds, and its wrap-around), vocabularies of one id, around one and two tiles and with every
# remainder mod 4 (unaligned rows of the output), on both sides of 160 tiles of 256 ids.
@pytest.mark.parametrize("M,d,V", [
    (1, 64, 1), (2, 64, 127), (31, 128, 129), (32, 192, 1001), (33, 256, 255), (63, 320, 1002),
    (64, 4096, 257), (65, 64, 1003), (95, 192, 259), (97, 128, 5000), (127, 320, 130),
    (128, 4096, 513), (129, 64, 1001), (33, 128, 40704), (64, 192, 40705), (5, 64, 41003),
])
def test_head_few_rows(M, d, V):
    from paper_2608_05448_amd import dblast as D
    h = synth.make_uniform_logits((1, 1, M, d) if M <= 64 else (M, 1, 1, d), 51).to(torch.bfloat16)
    w = (synth.make_uniform_logits((V, d), 52) * (2.0 / math.sqrt(d))).to(torch.bfloat16)
    _check(h, w, 2e-3, "few-rows")
    # The same with the argmax, into buffers with a guard behind the last row.
    hd, wd = h.cuda(), w.cuda()
    lead, nT = h.shape[:-1], OH.n_tiles(V)
    flat = [torch.full((M * n + 64,), 7.0, device="cuda") for n in (V, nT, 1)]
    views = [f[:M * n].view(*lead, *((n,) if i < 2 else ()))
             for i, (f, n) in enumerate(zip(flat, (V, nT, 1)))]
    plain = D.dbl_head_logprobs(hd, wd)
    got = D.dbl_head_logprobs(hd, wd, *views, argmax=True)
    torch.cuda.synchronize()
    for a, b, f in zip(plain, got, flat):
        assert torch.equal(a, b) and bool((f[-64:] == 7.0).all())
    lq = plain[0].view(M, V) + (plain[1] - plain[2][..., None]).view(M, nT).repeat_interleave(
        128, dim=1)[:, :V]
    at = lq.gather(1, got[3].view(M, 1).long())[:, 0]
    assert bool((at >= lq.max(1).values - 1e-5).all())


# The fp32 head: hidden sizes around one line of 32 units, around one chunk of 512 and in a second,
# odd multiples (unaligned rows), row counts around the tiles of 4 and 16 rows, and enough tiles for the
# 16-row form.
@pytest.mark.parametrize("M,d,V", [
    (1, 31, 130), (4, 32, 127), (5, 33, 129), (3, 512, 200), (9, 513, 300), (2, 1060, 128),
    (16, 160, 32769), (17, 161, 16500), (33, 545, 11100),
])
def test_head_fp32_edges(M, d, V):
    h = synth.make_uniform_logits((M, 1, 1, d), 61).to(torch.float32)
    w = (synth.make_uniform_logits((V, d), 62) / math.sqrt(d)).to(torch.float32)
    _check(h, w, 2e-5, "fp32-edges")


# A row's log-probabilities depend neither on the other rows of the call nor on its place among them:
# sharding a batch, or drafting one sequence of it alone, draws the same tokens. Row counts on both sides
# of every change of kernel and tile, hidden sizes whose sum starts at 0 and, in the second group of 4096
# ids, further on, vocabularies of fewer and of more than 160 tiles of 256 ids.
@pytest.mark.parametrize("d,V", [(64, 5003), (320, 5003), (2048, 5003), (4096, 5003), (2048, 41003)])
def test_head_rows_do_not_depend_on_the_batch(d, V):
    from paper_2608_05448_amd import dblast as D
    M = 2100
    h = synth.make_uniform_logits((M, 1, 1, d), 71).to(torch.bfloat16)
    h[1500] = h[3]
    w = (synth.make_uniform_logits((V, d), 72) * (2.0 / math.sqrt(d))).to(torch.bfloat16)
    hd, wd = h.cuda(), w.cuda()
    whole = D.dbl_head_logprobs(hd, wd, argmax=True)
    for out in whole:
        assert torch.equal(out[1500], out[3]), d
    for lo, n in ((3, 1), (0, 32), (40, 33), (7, 64), (100, 65), (0, 128), (50, 129), (600, 257),
                  (1000, 1100)):
        print(f"[head] d={d} rows {lo}..{lo + n} alone", flush=True)
        part = D.dbl_head_logprobs(hd[lo:lo + n].contiguous(), wd, argmax=True)
        for a, b in zip(whole, part):
            assert torch.equal(a[lo:lo + n], b), (d, lo, n)


def _best_us(f, n=20, rounds=5):
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


# Few rows do not pay for a tile of many: one and four rows against sixteen, which fill the 16-row tile
# that few rows would leave mostly empty (4 rows took 0.93 of the time of 16 in it; in tiles of 4 rows
# 0.4).
@pytest.mark.parametrize("M,d,V", [(1, 256, 151936), (4, 256, 151936), (4, 1024, 151936)])
def test_head_fp32_few_rows_cost_less_than_a_full_tile(M, d, V):
    from paper_2608_05448_amd import dblast as D
    w = torch.randn((V, d), device="cuda")
    h = torch.randn((16, 1, 1, d), device="cuda")
    few, full = (_best_us(lambda h=h[:m]: D.dbl_head_logprobs(h, w)) for m in (M, 16))
    print(f"[head] fp32 {M} rows {few:.1f} us, 16 rows {full:.1f} us (d={d})", flush=True)
    assert few < 0.85 * full


@pytest.mark.parametrize("M,d,V", [(12, 512, 38400), (11, 512, 38400), (61, 256, 9600),
                                   (64, 300, 32001), (128, 288, 4800)])
def test_head_fp32_tile_rule(M, d, V):
    h = synth.make_uniform_logits((M, 1, 1, d), 63).to(torch.float32)
    w = (synth.make_uniform_logits((V, d), 64) / math.sqrt(d)).to(torch.float32)
    _check(h, w, 2e-5, "fp32-tile-rule")


# The same for hidden sizes that 64 does not divide, and for fp32 rows in tiles of four and of sixteen.
@pytest.mark.parametrize("dt,d,V", [(torch.bfloat16, 96, 1003), (torch.bfloat16, 40, 1003),
                                    (torch.float32, 512, 38400), (torch.float32, 320, 38401)])
def test_other_head_rows_do_not_depend_on_the_batch(dt, d, V):
    from paper_2608_05448_amd import dblast as D
    M = 300
    h = synth.make_uniform_logits((M, 1, 1, d), 73).to(dt).cuda()
    w = (synth.make_uniform_logits((V, d), 74) * (2.0 / math.sqrt(d))).to(dt).cuda()
    whole = D.dbl_head_logprobs(h, w, argmax=True)
    for lo, n in ((4, 1), (0, 11), (20, 33), (40, 129)):
        part = D.dbl_head_logprobs(h[lo:lo + n].contiguous(), w, argmax=True)
        for a, b in zip(whole, part):
            assert torch.equal(a[lo:lo + n], b), (dt, d, lo, n)
