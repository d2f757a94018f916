"""Router backward on logits of every magnitude: sigmoid' over all BF16
values against binary64, and the time of a batch in which some logits are large."""
import numpy as np
import pytest
import torch

from test_gpu_balance import eqb, say  # noqa: F401 (eqb is a fixture)
from timing import least_us

pytestmark = pytest.mark.gpu


def test_every_logit(eqb):  # noqa: F811
    """grad_z = sigmoid'(z) where inj = 1 and no pair is selected.  Tolerance: an ulp
    of the exponential and 1.3e-8 of its correction, an ulp of the reciprocal and three
    roundings, 3e-7 in all; a subnormal result is rounded once more, by half of 2^-149."""
    E, T, K = 256, 256, 1
    bits = np.arange(1 << 16, dtype=np.uint32).astype(np.uint16)
    bits[(bits & 0x7FFF) > 0x7F80] = 0                  # infinities stay: masked experts
    z = np.random.default_rng(0).permutation(bits).reshape(T, E)
    say("router backward, every logit")
    gz = torch.empty((T, E), dtype=torch.float32, device="cuda")
    eqb.eqb_lei_router_backward(torch.from_numpy(z.view(np.int16)).cuda(),
                                torch.full((T, K), -1, dtype=torch.int32, device="cuda"),
                                torch.zeros((T, K), device="cuda"), gz, torch.ones((1, E), device="cuda"))
    e = np.exp(-np.abs((z.astype(np.uint32) << 16).view(np.float32).astype(np.float64)))
    want = e / (1.0 + e) ** 2
    assert np.all(np.abs(gz.cpu().numpy() - want) <= 3e-7 * want + 0.51 * 2.0 ** -149)


@pytest.mark.parametrize("E,K,T", [(256, 6, 147456), (128, 8, 300001), (64, 20, 300001)])
def test_large_logits_cost_no_more(eqb, E, K, T):  # noqa: F811
    """One logit in a hundred above 32 costs as much as none (the bound leaves a
    quarter for the timing; a wave that recomputed such logits one by one took 2.1 times as long)."""
    g = torch.Generator(device="cuda")
    g.manual_seed(E)
    x = torch.randn((T, E), generator=g, device="cuda")
    large = torch.where(torch.rand((T, E), generator=g, device="cuda") < 0.01, x + 40.0, x)
    idx = torch.rand((T, E), generator=g, device="cuda").topk(K, dim=1).indices.to(torch.int32)
    gs = torch.randn((T, K), generator=g, device="cuda")
    inj = torch.randn((1, E), generator=g, device="cuda")
    gz = torch.empty((T, E), device="cuda")
    zs = [v.to(torch.bfloat16).view(torch.int16) for v in (x, large)]
    us = least_us([lambda z=z: eqb.eqb_lei_router_backward(z, idx, gs, gz, inj) for z in zs])
    say(f"router backward E={E} K={K} T={T}: {us[0]:.1f} us, with large logits {us[1]:.1f} us")
    assert us[1] <= 1.25 * us[0]
