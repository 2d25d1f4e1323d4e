"""FP32 general form: the error of Vx does not grow with the columns of a chunk.
The same inputs with chunks of 16 columns (one running sum each, added to the output)
and with all columns in one chunk, both against the FP64 form.  Both add sums of at
most 16 pairs in FP32 to a few sums of sums, so their errors are equal up to the
roundings of those few additions: 10 %."""
import numpy as np
import pytest

from _gpu import banner
from paper_2501_03061_amd import inputs, px

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,orb,tgt", [((24, 24, 24), 100, 40), ((48, 48, 48), 130, 9), ((60, 60, 90), 113, 5)])
def test_row_sums(px_ctx, n, orb, tgt):
    import torch
    banner(f"FP32 row sums {n} {orb} x {tgt}")
    L = tuple(0.28 * k for k in n)
    cell = px.Cell(L, n)
    c = inputs.random_orbitals(n, L, orb + tgt, 10.0, np.random.default_rng(5))
    block = torch.from_numpy(c).cuda().to(torch.complex64)
    psi, phi = block[:orb].contiguous(), block[orb:].contiguous()
    occ = torch.sigmoid(torch.linspace(20.0, -20.0, orb, dtype=torch.float64, device="cuda"))
    kern = px_ctx.px_kernel_hse(cell, 0.106)
    ref = px_ctx.px_exchange_apply(cell, psi.to(torch.complex128), occ, phi.to(torch.complex128), kern)
    err = []
    try:
        for jc in (16, 128):
            px_ctx.set_tuning(cell, px.PX_PREC_FP32, 16, jc)
            out = px_ctx.px_exchange_apply(cell, psi, occ, phi, kern)
            err.append(float(torch.linalg.vector_norm(out.to(torch.complex128) - ref) / torch.linalg.vector_norm(ref)))
    finally:
        px_ctx.set_tuning(cell, px.PX_PREC_FP32, 0, 0)
    print(f"chunks of 16 {err[0]:.3e}, one chunk {err[1]:.3e}", flush=True)
    assert err[1] <= 1.1 * err[0]
