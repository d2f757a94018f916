"""Logits of -inf (experts masked for a token), in every routing kernel: such an
expert is never selected, and its margin is +inf.  Finite inputs are all that the
interface promises; this holds as long as every row keeps more than K finite logits."""
import numpy as np
import pytest

import workloads as W
from oracle import eqb_oracle as O
from test_gpu_fanouts import LANES
from test_gpu_layer import check, eqb, run_twice, say  # noqa: F401 (eqb is a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("E", [8, 16, 32, 64, 128, 256])
def test_masked_experts(eqb, E):  # noqa: F811
    for K in sorted({1, 2, 4, min(6, E // 2 - 1), min(9, E // 2 - 1), min(14, E // 2 - 1), min(16, E // 2 - 1),
                     min(20, E // 2 - 1)}):
        rng = np.random.default_rng(50 * E + K)
        T = 901
        x = rng.standard_normal((T, E)).astype(np.float32)
        mask = rng.random((T, E)) < 0.1
        if LANES[E] > 1:                       # all that one lane holds
            lane = (np.arange(E) // 4) % LANES[E]
            mask[::5] |= lane[None, :] == rng.integers(0, LANES[E], len(mask[::5]))[:, None]
        first = np.arange(E) < E // 4          # the lower experts
        mask[1::5] |= first[None, :]
        mask[mask.sum(1) >= E - K] = False     # K + 1 finite logits in every row
        x[mask] = -np.inf
        b = (rng.standard_normal(E) * 0.1).astype(np.float32) if K % 2 else np.zeros(E, np.float32)
        off = np.array([0, 300, T], np.int64)
        z = W._to_bf16_bits(x)
        # the lowest finite logit in place of -inf: its margin has the same high byte
        want = O.run_layer(np.where(z == 0xFF80, np.uint16(0xFF7F), z), b, K, off)
        assert want["tau"].min() > -100 and want["u"].max() < 0xFF     # no masked expert, no bin of such margins
        say(f"masked experts E={E} K={K}")
        for got in run_twice(eqb, z, b, K, off):
            check(got, want, K)
