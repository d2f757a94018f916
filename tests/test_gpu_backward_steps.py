"""Router backward at the edges of its steps (batches of one row up to one past
a whole step of one block), on both sides of the line K = E/4 where a lane owns
one of a row's pairs, and across the logit |z| = 32 where sigmoid' changes form."""
import numpy as np
import pytest
import torch

from oracle import balance_oracle as B
from oracle import eqb_oracle as O
from test_gpu_balance import eqb, say  # noqa: F401 (eqb is a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("E", [8, 16, 32, 64, 128, 256])
def test_steps_pairs_and_large_logits(eqb, E):  # noqa: F811
    """Tolerance: sigmoid' is at most 2e-7 off (exponential 1 ulp and 1.3e-8,
    reciprocal 1 ulp, three roundings), the sum and product round once each."""
    step = 8 * 3 * (256 // E)              # rows of a block's step
    for K in sorted({1, max(E // 4, 1), min(E // 4 + 1, E - 1)}):
        for T in (1, step - 1, step, step + 1):
            rng = np.random.default_rng(E * 31 + K + T)
            x = (rng.standard_normal((T, E)) * 4).astype(np.float32)
            edge = np.array([0.0, -0.0, 31.875, -31.875, 32.0, -32.0, 32.25, 63.75, 64.0, -64.5, 80.0], np.float32)
            x.ravel()[rng.integers(0, x.size, 3)] = edge[rng.integers(0, edge.size, 3)]
            if T > 2:
                x[1, :] = edge[np.arange(E) % edge.size]
            z = O.f32_to_bf16_rne(x)
            idx = np.argsort(rng.random((T, E)), axis=1)[:, :K].astype(np.int32)
            gs = rng.standard_normal((T, K)).astype(np.float32)
            off = np.array([0, T // 2, T // 2, T], np.int64)
            inj = (rng.standard_normal((3, E)) * 1e-3).astype(np.float32)
            say(f"router backward steps E={E} K={K} T={T}")
            gz = torch.empty((T, E), dtype=torch.float32, device="cuda")
            eqb.eqb_lei_router_backward(torch.from_numpy(z.view(np.int16)).cuda(), torch.from_numpy(idx).cuda(),
                                        torch.from_numpy(gs).cuda(), gz, torch.from_numpy(inj).cuda(),
                                        [int(v) for v in off])
            got = gz.cpu().numpy().astype(np.float64)
            want = B.lei_router_backward(z, idx, gs, inj, off)
            # the sum g + inj may cancel: its rounding is relative to its terms
            scale = np.abs(B.lei_router_backward(z, idx, np.abs(gs), np.abs(inj), off))
            assert np.all(np.abs(got - want) <= 6e-7 * scale + 1e-37), (K, T)
