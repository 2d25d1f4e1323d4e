"""The blocked factorisation of the ACE construction (32-column blocks, panels
and inverse wavefronts) at sizes around its block edges: xi xi^H must reproduce
W (-M)^{-1} W^H, checked through V_ACE Psi = W (the exactness of the ACE form
on its own orbitals).  Tolerance 1e-10 (the condition of -M, at most about 1e4 here, times eps and the
accumulated roundings)."""
import pytest

import oracle
from paper_2501_03061_amd import inputs, px
from _gpu import banner, relerr, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_orb", [1, 31, 32, 33, 64, 65, 97])
def test_ace_exactness_at_block_edges(px_ctx, n_orb):
    banner(f"cholesky edges n={n_orb}")
    inst = inputs.make_instance(24, 10.0, n_orb, 0.05, seed=400 + n_orb)
    cell = px.Cell(inst.L, inst.n)
    psi, occ = to_dev(inst.psi), to_dev(inst.occ)
    kd = to_dev(oracle.kernel_hse(inst.n, inst.L, 0.106))
    xi, st = px_ctx.px_ace_build(cell, psi, occ, kd)
    px_ctx.px_sync()
    assert int(st.item()) == 0
    W = px_ctx.px_exchange_apply(cell, psi, occ, psi, kd)
    V = px_ctx.px_ace_apply(cell, xi, psi)
    err = relerr(to_host(V), to_host(W))
    print(f"n={n_orb} V psi - W {err:.2e}", flush=True)
    assert err < 1e-10

