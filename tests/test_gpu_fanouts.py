"""GPU parity of the one-call layer for every fan-out with a kernel of its own.

The routing kernels keep a sorted list of keys per lane whose depth depends on
the fan-out and on the lanes that share a row.  Each layer below mixes smooth
rows, rows of exact ties and rows whose largest scores all sit in one lane's
experts, so that its list runs dry.
"""
import numpy as np
import pytest

import workloads as W
from oracle import eqb_oracle as O
from test_gpu_layer import check, eqb, run_twice, say  # noqa: F401 (eqb is a fixture)

pytestmark = pytest.mark.gpu

LANES = {8: 1, 16: 2, 32: 4, 64: 4, 128: 8, 256: 8}     # lanes per row of the routing kernels


def layer(E, K, T):
    rng = np.random.default_rng(1000 * E + K)
    x = rng.standard_normal((T, E)).astype(np.float32)
    x[::3] = rng.integers(-16, 17, (len(x[::3]), E)) / 4.0
    lane = (np.arange(E) // 4) % LANES[E]
    crowd = rng.integers(0, LANES[E], T)
    x[1::3] += np.where(lane[None, :] == crowd[1::3, None], np.float32(5.0), np.float32(0.0))
    b = (rng.standard_normal(E) * 0.1).astype(np.float32) if K % 3 else np.zeros(E, np.float32)
    return W._to_bf16_bits(x), b


@pytest.mark.parametrize("E", [8, 16, 32, 64, 128, 256])
def test_every_fanout(eqb, E):  # noqa: F811
    for K in range(1, min(18, E)):
        T = 229 + 67 * K                   # not a multiple of any block step
        z, b = layer(E, K, T)
        off = np.array([0, T // 3, T], np.int64)
        want = O.run_layer(z, b, K, off)
        say(f"fan-out E={E} K={K} T={T}")
        for got in run_twice(eqb, z, b, K, off, cap=(0, 1, 3)[K % 3]):
            check(got, want, K)
