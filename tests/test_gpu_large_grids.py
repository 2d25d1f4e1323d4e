"""ACE application on grids whose orbital rows lie further apart than 32-bit byte
offsets reach (three rows of an xi^H phi transfer, two of an FP32 xi C transfer):
FP64 from 448^3, FP32 from 564^3 and from 2^29 points.  Reference: torch in
complex128, in pieces.  Random orbitals, so a contraction entry is a random sum of
N_g products: errors of a few eps relative to its size, FP32 with a factor for
the rounding of C and the sum over n; a row read from the wrong place is an error
of order one."""
import pytest

from _gpu import banner
from paper_2501_03061_amd import px

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fp32,n,orb", [(False, (448, 448, 448), 5), (True, (564, 564, 564), 5),
                                        (True, (1024, 1024, 514), 3)])
def test_ace_apply(px_ctx, fp32, n, orb):
    import torch
    banner(f"ace apply on a large grid {n} fp32={fp32} n={orb}")
    dt = torch.complex64 if fp32 else torch.complex128
    cell = px.Cell(tuple(0.3 * k for k in n), n)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    shape = (n[2], n[1], n[0])
    xi = torch.randn((orb,) + shape, dtype=dt, device="cuda", generator=gen)
    phi = torch.randn((1,) + shape, dtype=dt, device="cuda", generator=gen)
    xi *= (cell.ng * cell.dV) ** -0.5
    out = px_ctx.px_ace_apply(cell, xi, phi)
    torch.cuda.synchronize()
    x, p, y = xi.view(orb, -1), phi.view(-1), out.view(-1)
    step = 1 << 24
    pieces = [slice(a, min(a + step, cell.ng)) for a in range(0, cell.ng, step)]
    c = torch.zeros(orb, dtype=torch.complex128, device="cuda")
    for r in pieces:
        for a in range(orb):
            c[a] += (x[a, r].to(torch.complex128).conj() * p[r].to(torch.complex128)).sum() * cell.dV
    err = ref = 0.0
    for r in pieces:
        t = torch.zeros(r.stop - r.start, dtype=torch.complex128, device="cuda")
        for a in range(orb):
            t -= x[a, r].to(torch.complex128) * c[a]
        err += float(torch.linalg.vector_norm(y[r].to(torch.complex128) - t)) ** 2
        ref += float(torch.linalg.vector_norm(t)) ** 2
    e = (err / ref) ** 0.5
    print(f"relative error {e:.2e}", flush=True)
    assert e < (2e-6 if fp32 else 1e-12)
    del xi, phi, out, x, p, y, t
    torch.cuda.empty_cache()
