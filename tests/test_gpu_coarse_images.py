"""Coarse counts of the one-call layer inside and outside the window of bins that
its routing blocks hand over as images: margins below, across and above the window
(2^-11 .. 32), batches on both sides of the 65,535 rows a block's image can
count, blocks that cover several partitions, and one workspace used for all."""
import numpy as np
import pytest

import workloads as W
from oracle import eqb_oracle as O
from test_gpu_layer import check, eqb, run_twice, say  # noqa: F401 (eqb is a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("E,K", [(8, 2), (32, 4), (64, 6), (128, 5), (256, 8)])
@pytest.mark.parametrize("scale", [2.0 ** -13, 2.0 ** -5, 8.0, 2.0 ** 20])
def test_margins_in_and_outside_the_window(eqb, E, K, scale):  # noqa: F811
    rng = np.random.default_rng(E + K)
    T = 1501
    z = W._to_bf16_bits((rng.standard_normal((T, E)) * scale).astype(np.float32))
    b = (rng.standard_normal(E) * 0.1 * scale).astype(np.float32)
    off = np.array([0, 3, 3, 700, 701, T], np.int64)
    want = O.run_layer(z, b, K, off)
    for cap in (0, 1, 5):
        say(f"coarse images E={E} K={K} scale={scale} cap={cap}")
        for got in run_twice(eqb, z, b, K, off, cap):
            check(got, want, K)


@pytest.mark.parametrize("T", [65535, 65536])
def test_one_block_of_as_many_rows_as_an_image_counts(eqb, T):  # noqa: F811
    """One block; all rows alike, so that a counter of the image reaches T (or, one
    row more, the block falls back to the slabs)."""
    E, K = 8, 2
    z = W._to_bf16_bits(np.tile(np.array([4, 3, 2, 1.5, 1, 0.5, 0, -1], np.float32), (T, 1)))
    b = (np.arange(E) * 0.01).astype(np.float32)
    off = np.array([0, T // 2, T], np.int64)
    want = O.run_layer(z, b, K, off)
    say(f"coarse images, one block of {T} rows")
    for got in run_twice(eqb, z, b, K, off, 1):
        check(got, want, K)
