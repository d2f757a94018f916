"""Fine counts on both sides of every line that decides how many experts a
block of the fine pass takes, against counts made with plain torch operations
from the same tau and selections."""
import sys

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def eqb():
    assert torch.cuda.is_available(), "GPU tests need a visible GPU"
    from paper_2609_28053_amd import eqb as binding
    return binding


def fine_counts(z, tau, sel, part, local):
    """[P,E,256] counts of the low key bytes of bf16(tau - z) inside each selected high byte."""
    E = z.shape[1]
    out = []
    for p, (a, b) in enumerate(zip(part, part[1:])):
        u = sel[p] if local else sel
        keep = torch.zeros(E * 256, dtype=torch.int64, device="cuda")
        for t0 in range(a, b, 1 << 15):
            t1 = min(b, t0 + (1 << 15))
            m = (tau[t0:t1, None] - z[t0:t1].view(torch.bfloat16).float()).to(torch.bfloat16)
            k = m.view(torch.int16).long() & 0xFFFF
            k = torch.where(k >= 0x8000, k ^ 0xFFFF, k ^ 0x8000)
            hit = (k >> 8) == u.long()
            cell = torch.arange(E, device="cuda") * 256 + (k & 0xFF)
            keep += torch.bincount(cell[hit], minlength=E * 256)
        out.append(keep.view(E, 256))
    return torch.stack(out)


# logits of the batch: 2^22 and 2^27 (the layer's images), 2^24 and 2^28 (slabs)
SIZES = [(256, 16384), (256, 16385), (128, 32768), (128, 32769), (64, 65536), (64, 65537),
         (256, 65536), (256, 65537), (64, 262144), (64, 262145), (256, 524288), (256, 524289),
         (128, 1048577), (256, 1048577), (128, 31), (256, 257), (64, 1)]


@pytest.mark.parametrize("E,T", SIZES)
@pytest.mark.parametrize("cap", [0, 5])
def test_fine_counts(eqb, E, T, cap):
    K = 4
    print(f"[gpu-fine] E={E} T={T} cap={cap}", flush=True)
    sys.stdout.flush()
    g = torch.Generator(device="cuda")
    g.manual_seed(E + T)
    z = torch.randn((T, E), generator=g, device="cuda").to(torch.bfloat16).view(torch.int16)
    b = torch.randn(E, generator=g, device="cuda") * 0.1
    part = [0, T // 5, T // 5, T]                     # unequal, one empty
    po = eqb.PartOffsets(part)
    lay = eqb.Layer(T, E, K, 3)
    try:
        eqb.eqb_set_max_blocks(cap)
        lay.run(z, b, po)
        lay.step(z, b, po, sums=False)
        lay.step(z, b, po, sums=True)
        assert int(lay.status.item()) == 0 and lay.counters_zero()
        want = fine_counts(z, lay.tau, lay.sel_hi, part, False)
        assert torch.equal(lay.hist_lo.long(), want)
        assert torch.equal(lay.L.long(), want.sum(0))
        sel = torch.stack([lay.sel_hi, lay.sel_hi, (lay.sel_hi + 1) % 256]).int().contiguous()
        hist = torch.zeros((3, E, 256), dtype=torch.int32, device="cuda")
        eqb.eqb_margin_hist_pass2_local(z, lay.tau, sel, hist, po)
        assert torch.equal(hist.long(), fine_counts(z, lay.tau, sel, part, True))
    finally:
        eqb.eqb_set_max_blocks(0)
    q = lay.q_bf16.cpu().numpy().view(np.uint16).astype(np.uint32)
    bhat = (q << 16).view(np.float32).astype(np.float64)
    mean = np.float64(0.0)
    for x in bhat:
        mean += x
    want_b = (bhat - mean / E).astype(np.float32)
    assert np.array_equal(lay.b_next.cpu().numpy().view(np.uint32), want_b.view(np.uint32))
