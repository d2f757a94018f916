"""eqb_route_topk without counts: the partitions bear on nothing it writes, and cost nothing."""
import numpy as np
import pytest
import torch

from test_gpu_layer import eqb, say  # noqa: F401 (eqb is a fixture)
from timing import least_us

pytestmark = pytest.mark.gpu


def route(eqb, T, E, K, P, seed=0):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    z = torch.randn((T, E), generator=g, device="cuda").to(torch.bfloat16).view(torch.int16)
    b = torch.randn(E, generator=g, device="cuda") * 0.1
    out = (torch.empty((T, K), dtype=torch.int32, device="cuda"), torch.empty((T, K), device="cuda"),
           torch.empty(T, device="cuda"))
    po = eqb.PartOffsets([T * p // P for p in range(P + 1)])
    return out, lambda: eqb.eqb_route_topk(z, b, K, *out, po)


@pytest.mark.parametrize("T,E,K", [(1021, 64, 6), (9, 8, 2), (70000, 32, 4), (3001, 256, 16), (5003, 128, 20)])
def test_partitions_do_not_matter(eqb, T, E, K):  # noqa: F811
    for cap in (0, 1):                       # one block: more rows than a segment holds
        eqb.eqb_set_max_blocks(cap)
        try:
            one, call = route(eqb, T, E, K, 1)
            call()
            many, call = route(eqb, T, E, K, 16)
            say(f"route alone T={T} E={E} K={K} cap={cap}")
            call()
        finally:
            eqb.eqb_set_max_blocks(0)
        for a, c in zip(one, many):
            assert np.array_equal(a.cpu().numpy().view(np.int32), c.cpu().numpy().view(np.int32))


def test_partitions_cost_nothing(eqb):  # noqa: F811
    """The bound leaves an eighth for the timing; swept one by one, 16 partitions took 1.3 times as long."""
    us = least_us([route(eqb, 1021, 64, 6, P)[1] for P in (1, 16)], passes=200)
    say(f"route alone, 1 and 16 partitions: {us[0]:.2f} and {us[1]:.2f} us")
    assert us[1] <= 1.125 * us[0]
