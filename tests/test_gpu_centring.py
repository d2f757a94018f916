"""The centring of Eq. 2 on the GPU, bit for bit, for quantiles whose exponents
span more or less than a binary64 sum of any order holds exactly."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def eqb():
    assert torch.cuda.is_available(), "GPU tests need a visible GPU"
    from paper_2609_28053_amd import eqb as binding
    return binding


def ascending(bhat):
    acc = np.float64(0.0)
    for x in bhat:
        acc += x
    return (bhat - acc / len(bhat)).astype(np.float32)


def centre(eqb, bits):
    """q_bf16 (checked) and b_next for quantiles of these BF16 patterns."""
    E = len(bits)
    key = np.where(bits & 0x8000, bits ^ 0xFFFF, bits ^ 0x8000)
    hist = np.zeros((1, E, 256), np.int32)
    hist[0, np.arange(E), key & 0xFF] = 1
    i32 = lambda a: torch.from_numpy(np.ascontiguousarray(a, np.int32)).cuda()
    rank = torch.ones(E, dtype=torch.int64, device="cuda")
    sel_lo = torch.empty(E, dtype=torch.int32, device="cuda")
    q = torch.empty(E, dtype=torch.int16, device="cuda")
    b_next = torch.empty(E, dtype=torch.float32, device="cuda")
    eqb.eqb_select_quantile(2, i32(hist), 1, i32(key >> 8), rank, sel_lo, q, b_next)
    assert np.array_equal(q.cpu().numpy().view(np.uint16), bits.astype(np.uint16))
    return b_next.cpu().numpy()


@pytest.mark.parametrize("E", [8, 64, 256])
@pytest.mark.parametrize("span", [0, 20, 35, 36, 37, 38, 60, 200])
def test_centring(eqb, E, span):
    rng = np.random.default_rng(100 * E + span)
    exp = rng.integers(20, 21 + span, E)               # biased BF16 exponents
    exp[:2] = (20, 20 + span)
    bits = (rng.integers(0, 2, E) << 15 | exp << 7 | rng.integers(0, 128, E)).astype(np.uint32)
    bits[3] = 0x8000                                   # a zero does not count to the span
    bhat = (bits << 16).astype(np.uint32).view(np.float32).astype(np.float64)
    assert np.array_equal(centre(eqb, bits).view(np.uint32), ascending(bhat).view(np.uint32))


@pytest.mark.parametrize("E", [8, 64, 128, 256])
@pytest.mark.parametrize("zeros", ["plus", "minus", "both"])
def test_centring_zeros(eqb, E, zeros):
    """Quantiles that are all zeros: the ascending sum is +0 whatever their signs."""
    bits = np.full(E, 0x8000 if zeros == "minus" else 0, np.uint32)
    if zeros == "both":
        bits[::2] = 0x8000
    bhat = (bits << 16).astype(np.uint32).view(np.float32).astype(np.float64)
    assert np.array_equal(centre(eqb, bits).view(np.uint32), ascending(bhat).view(np.uint32))
