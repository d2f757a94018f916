"""GPU parity of the one-call layer where the run of equal leading score bits
around rank K is as long as the routing kernel's rank buffer, or longer.

Every third row holds `run` experts of one logit around rank K, their biases a
binary32 ulp or a few apart: the keys agree in their top 24 bits, and the exact
scores (or, between equal ones, the expert index) decide the order.
"""
import numpy as np
import pytest

import workloads as W
from oracle import eqb_oracle as O
from test_gpu_layer import check, eqb, run_twice, say  # noqa: F401 (eqb is a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("E", [32, 64, 128, 256])
def test_runs_around_the_last_rank(eqb, E):  # noqa: F811
    for K in (13, 14, 15, 16):
        rng = np.random.default_rng(10 * E + K)
        T = 301
        x = rng.uniform(-2.0, 1.0, (T, E)).astype(np.float32)
        for t in range(0, T, 3):
            run = 2 + (t // 3) % 12
            top = rng.permutation(E)
            above = max(0, K - rng.integers(0, run))     # experts above the run: rank K falls inside it
            x[t, top[:above]] = 4.0 + 0.25 * np.arange(above)
            x[t, top[above:above + run]] = 3.0
        b = (rng.integers(-8, 9, E) * 2.0 ** -22).astype(np.float32)
        z = W._to_bf16_bits(x)
        off = np.array([0, 100, T], np.int64)
        want = O.run_layer(z, b, K, off)
        say(f"runs E={E} K={K}")
        for got in run_twice(eqb, z, b, K, off):
            check(got, want, K)
