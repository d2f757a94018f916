"""GPU parity of the one-call layer where a run of scores that agree in their
top 24 bits lies across rank K: the routing keys do not order it, and the kernel
chooses its members for the ranks up to K by their exact scores and, between equal
ones, by the expert index.

Runs of 1 to E experts, from rank 0 on or below others, ending at rank K, one
past it or far past it, spread over the lanes of a row or crowded into a few, so
that a lane holds more of the run, or of the ranks above it, than its list.
"""
import numpy as np
import pytest

import workloads as W
from oracle import eqb_oracle as O
from test_gpu_fanouts import LANES
from test_gpu_layer import check, eqb, run_twice, say  # noqa: F401 (eqb is a fixture)
from timing import least_us

pytestmark = pytest.mark.gpu

ULP = 2.0 ** -22                      # of the scores near 3


def runs(E, K, mode, T, rng):
    """Logits and bias, and per row how many experts lie above its run and in it."""
    x = rng.uniform(-7.0, -4.0, (T, E)).astype(np.float32)
    lane = (np.arange(E) // 4) % LANES[E]
    above, run = np.zeros(T, int), np.zeros(T, int)
    for t in range(T):
        n = int(rng.integers(1, E + 1)) if t % 2 else int(rng.integers(1, min(E, 8) + 1))
        a = max(0, K + 1 - int(rng.integers(1, n + 1))) if t % 3 else max(0, K + 1 - n)
        n = min(n, E - a)
        order = rng.permutation(E)
        if t % 4 >= 2:
            order = order[np.argsort((lane[order] + t) % LANES[E], kind="stable")]   # lane by lane
        x[t, order[:a]] = 4.0 + 0.25 * rng.permutation(a)
        x[t, order[a:a + n]] = {"positive": 3.0, "negative": -3.0, "zero bias": -3.0, "zeros": 0.0}[mode]
        above[t], run[t] = a, n
    steps = rng.integers(0, 17, E)
    b = {"positive": steps * ULP, "negative": steps * -ULP, "zero bias": np.zeros(E), "zeros": np.zeros(E)}[mode]
    z, b = W._to_bf16_bits(x), b.astype(np.float32)
    if mode == "zeros":
        z = np.where((z == 0) & (rng.random((T, E)) < 0.5), np.uint16(0x8000), z)
        b = np.where(rng.random(E) < 0.5, np.float32(-0.0), b)
    return z, b, above, run


@pytest.mark.parametrize("mode", ["positive", "negative", "zero bias", "zeros"])
@pytest.mark.parametrize("E", [8, 16, 32, 64, 128, 256])
def test_runs_across_the_last_rank(eqb, E, mode):  # noqa: F811
    for K in sorted({min(K, E - 1) for K in (1, 4, 6, 8, 13, 14, 15, 16)}):
        T = 293
        z, b, above, run = runs(E, K, mode, T, np.random.default_rng(10 * E + K))
        # one run of equal top 24 bits per row, as long as meant, across rank K
        score = O.biased_scores(z, b) + np.float32(0.0)
        top = score.view(np.uint32) >> 8
        tau = -np.sort(-score, axis=1)[:, K:K + 1] + np.float32(0.0)
        np.testing.assert_array_equal((top == tau.view(np.uint32) >> 8).sum(1), run)
        past, most = above + run - (K + 1), E - (K + 1)  # members beyond rank K
        assert (past == 0).any() and (past == min(1, most)).any() and (2 * past >= most).any() and (above == 0).any()
        off = np.array([0, 100, T], np.int64)
        want = O.run_layer(z, b, K, off)
        say(f"runs E={E} K={K} {mode}")
        for got in run_twice(eqb, z, b, K, off):
            check(got, want, K)


@pytest.mark.parametrize("E,T", [(32, 65537), (32, 600000), (64, 4097)])
def test_ties_cost_no_more_than_the_generic_kernel(eqb, E, T):  # noqa: F811
    """Logits on a grid of quarters, a zero bias: half the rows have ties at a
    negative cutoff.  The widest fan-out of the fast kernel takes no longer than the
    next, which takes K + 1 rounds over 64-bit keys (5% for the timing; rows ordered one
    insertion after another, or sent to the 64-bit path, took 1.3 to 1.5 times as long)."""
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(E)
    z = (torch.randint(-16, 17, (T, E), generator=g, device="cuda") / 4).to(torch.bfloat16).view(torch.int16)
    b = torch.zeros(E, device="cuda")
    layers = {K: eqb.Layer(T, E, K) for K in (15, 16, 17)}
    us = dict(zip(layers, least_us([lambda lay=lay: lay.step(z, b) for lay in layers.values()])))
    say(f"ties E={E} T={T}: " + ", ".join(f"K={K} {t:.1f} us" for K, t in us.items()))
    assert max(us[15], us[16]) <= 1.05 * us[17]
