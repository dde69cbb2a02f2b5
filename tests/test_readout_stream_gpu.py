"""Streaming reductions of the read-out: pointers that allow only narrow
accesses, the smallest states, and both sides of the size from which a
work-group takes runs of rounds, against float64 sums of the same values."""
import math

import numpy as np
import pytest
import torch

from paper_1704_01127_amd import qsim

pytestmark = pytest.mark.gpu


def buffer(count, dtype, offset, gen):
    """`count` random values of `dtype` that start `offset` elements into an allocation."""
    real = torch.float32 if dtype == torch.complex64 else torch.float64
    v = torch.randn(count + offset, 2, dtype=real, device="cuda", generator=gen) / math.sqrt(2 * count)
    return torch.view_as_complex(v)[offset:]


# 11 to 14 qubits: one work-group alone (up to 2^12 units of two fp32 or one amplitude), single
# rounds and runs there; 16 to 18: both sides of the runs of many (from 2^17 units)
@pytest.mark.parametrize("n", [1, 2, 9, 10, 11, 12, 13, 14, 16, 17, 18, 26])
@pytest.mark.parametrize("dt,out_dt,ref_dt,offset", [
    (torch.complex64, torch.float32, torch.complex64, 0), (torch.complex64, torch.float32, torch.complex64, 1),
    (torch.complex64, torch.float64, torch.complex128, 0), (torch.complex64, torch.float64, torch.complex128, 1),
    (torch.complex128, torch.float64, torch.complex128, 0), (torch.complex128, torch.float32, torch.complex64, 1)])
def test_readout(n, dt, out_dt, ref_dt, offset):
    gen = torch.Generator(device="cuda").manual_seed(n)
    count = 1 << n
    psi = buffer(count, dt, offset, gen)
    ref = buffer(count, ref_dt, offset, gen)
    out = torch.zeros(count + offset, dtype=out_dt, device="cuda")[offset:]
    s = qsim.State(n, "c64" if dt == torch.complex64 else "c128")
    s.amps.copy_(psi)
    a, r = psi.to(torch.complex128), ref.to(torch.complex128)
    p = a.real.square() + a.imag.square()
    want = (p.sum().item(), p.square().sum().item(), -torch.special.xlogy(p, p).sum().item())
    for read in (s.probs, lambda out: qsim.probs_noalloc(psi, out=out)):
        out.zero_()
        got = read(out=out)
        # float64 sums over chains of at most 2^8 terms a lane; fp32 states take the mantissa's
        # logarithm in fp32: 2^-24 relative, of at most ln 2
        assert abs(got[0] - want[0]) <= 1e-13 * want[0]
        assert abs(got[1] - want[1]) <= 1e-13 * want[1]
        assert abs(got[2] - want[2]) <= 1e-12 * want[2] + (2.0 ** -23 if dt == torch.complex64 else 0) * want[0]
        # squares and sum in float64, one rounding to the output
        eps = 2.0 ** -23 if out_dt == torch.float32 else 2.0 ** -51
        assert (out.double() - p).abs().le(eps * p + 1e-40).all()
    fid, worst = s.compare(ref)
    dot = complex((r.conj() * a).sum())
    rr, aa = r.abs().square().sum().item(), p.sum().item()
    # the product's sum cancels: its error is relative to sqrt(rr aa)
    assert abs(fid - abs(dot) ** 2 / (rr * aa)) <= 1e-12
    assert worst == pytest.approx((a - r).abs().max().item(), rel=1e-14)
