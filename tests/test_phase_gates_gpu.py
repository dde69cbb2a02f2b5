"""T and CZ one by one on every place of their bits in a 16-byte unit, a half and
a whole 128-byte line and above, on states inside the caches, and on one of
512 MiB of which a gate touches what fits them: the amplitudes they select, and
no others, are changed."""
import math
import time

import pytest
import torch

from paper_1704_01127_amd import qsim

pytestmark = pytest.mark.gpu

SIZES = [("c64", 4), ("c64", 12), ("c64", 20), ("c64", 26), ("c128", 3), ("c128", 11), ("c128", 20), ("c128", 25)]


@pytest.mark.parametrize("dt,n", SIZES)
def test_only_selected_amplitudes_change(dt, n):
    gen = torch.Generator(device="cuda").manual_seed(n)
    real, eps = (torch.float32, 2.0 ** -23) if dt == "c64" else (torch.float64, 2.0 ** -52)
    psi = torch.view_as_complex(torch.randn(2 ** n, 2, generator=gen, device="cuda", dtype=real))
    index = torch.arange(2 ** n, device="cuda")
    phase = complex(math.sqrt(0.5), math.sqrt(0.5))
    places = [q for q in (0, 1, 2, 3, 4, 7, 8, 9, n - 2, n - 1) if 0 <= q < n]
    gates = [(q,) for q in sorted(set(places))]
    gates += [(a, b) for a in (0, 1, 2, 3, 8) for b in (1, 2, 3, 4, 9, n - 1) if a < b < n]
    for qs in gates:
        s = qsim.State(n, dt, init="keep", amps=psi.clone())
        s.apply_gate(("T" if len(qs) == 1 else "CZ", qs))
        on = torch.ones_like(index, dtype=torch.bool)
        for q in qs:
            on &= (index >> q & 1).bool()
        assert torch.equal(s.amps[~on], psi[~on]), qs
        if len(qs) == 2:
            assert torch.equal(s.amps[on], -psi[on]), qs
        else:  # one complex product, its factor rounded to the state's type
            want = psi[on].to(torch.complex128) * phase
            assert ((s.amps[on].to(torch.complex128) - want).abs() <= 3 * eps * psi[on].abs()).all(), qs


def best_us(f):
    f()
    torch.cuda.synchronize()
    best = math.inf
    for _ in range(10):
        t = time.perf_counter()
        for _ in range(20):
            f()
        torch.cuda.synchronize()
        best = min(best, (time.perf_counter() - t) / 20 * 1e6)
    return best


@pytest.mark.parametrize("dt,n,q", [("c64", 25, 3), ("c128", 24, 2)])
def test_half_lines_are_moved_alone_in_the_caches(dt, n, q):
    """A gate that selects half of every line of a cached state does not move the
    other half: it takes well less (0.75) than one that selects within half lines."""
    s = qsim.State(n, dt, init="uniform")
    half, whole = best_us(lambda: s.apply_gate(("T", (q,)))), best_us(lambda: s.apply_gate(("T", (q - 1,))))
    assert half <= 0.9 * whole, (half, whole)
