"""The contractions of the ACE application (C = dV xi^H phi and out = -xi C) at
the edges of their tiles and stages, against numpy in complex128: orbital counts
around the 16-wide matrix tiles and the 64-wide workgroup tiles, sums shorter
than a stage and with every remainder class, odd N_g (FP64 form), few and many
splits.  Tolerances (relative Frobenius norm): FP64 1e-13 (sums of N_g terms of
random sign, Gauss products: about 10 eps times the root of a partial sum's
length); FP32 5e-6 (C summed in FP64 beyond 1024 terms; out sums up to 200
products, each within a few eps = 6e-8 of the operands' norms)."""
import numpy as np
import pytest

import oracle
from paper_2501_03061_amd import px
from _gpu import banner, relerr, to_dev, to_host

pytestmark = pytest.mark.gpu

CASES = [((5, 7, 9), 1, 1), ((5, 7, 9), 3, 17), ((3, 3, 3), 16, 15), ((16, 16, 16), 33, 64), ((24, 24, 24), 65, 31),
         ((24, 24, 24), 16, 16), ((24, 24, 24), 130, 1), ((48, 48, 48), 20, 200), ((11, 13, 17), 64, 48)]


@pytest.mark.parametrize("fp32", [False, True])
@pytest.mark.parametrize("n,n_xi,n_phi", CASES)
def test_ace_apply_edges(px_ctx, n, n_xi, n_phi, fp32):
    ng = n[0] * n[1] * n[2]
    if fp32 and ng % 2:
        pytest.skip("the FP32 form needs an even N_g")
    banner(f"ace apply grid {n} n={n_xi} n_phi={n_phi} fp32={fp32}")
    rng = np.random.default_rng(5)
    dt = np.complex64 if fp32 else np.complex128
    xi, phi = [(rng.standard_normal((k, ng)) + 1j * rng.standard_normal((k, ng))).astype(dt) for k in (n_xi, n_phi)]
    cell = px.Cell(tuple(0.28 * m for m in n), n)
    shape = (n[2], n[1], n[0])
    x, p = to_dev(xi.reshape(n_xi, *shape)), to_dev(phi.reshape(n_phi, *shape))
    dV = 0.28 ** 3
    x64, p64 = xi.astype(np.complex128), phi.astype(np.complex128)
    ref = -(dV * (x64.conj() @ p64.T)).T @ x64
    for f in (px_ctx.px_ace_apply, px_ctx.px_ace_apply_noalloc):
        out = to_host(f(cell, x, p)).reshape(n_phi, ng)
        err = relerr(out, ref)
        print(f"{f.__name__} {err:.2e}", flush=True)
        assert err < (5e-6 if fp32 else 1e-13)


@pytest.mark.parametrize("fp32", [False, True])
@pytest.mark.parametrize("n,n_xi,n_phi,iters", [((5, 7, 9), 4, 1, 1), ((16, 16, 16), 9, 17, 2), ((10, 12, 11), 33, 65, 3)])
def test_loop_edges(px_ctx, n, n_xi, n_phi, iters, fp32):
    """The fixed point's update in the contraction's stores: the first midpoint
    is phi_n itself, the last iteration leaves none; tolerances as above, the
    map being contracted with a norm below one (residuals to 1e-9, 1e-5)."""
    import torch
    ng = n[0] * n[1] * n[2]
    if fp32 and ng % 2:
        pytest.skip("the FP32 form needs an even N_g")
    banner(f"ptim loop grid {n} n={n_xi} n_phi={n_phi} iters={iters} fp32={fp32}")
    rng = np.random.default_rng(6)
    dt = np.complex64 if fp32 else np.complex128
    shape = (n[2], n[1], n[0])
    dV, dta = 0.28 ** 3, 0.25
    xi, phi = [((rng.standard_normal((k, *shape)) + 1j * rng.standard_normal((k, *shape))) / np.sqrt(dV * ng * n_xi)).astype(dt)
               for k in (n_xi, n_phi)]
    ref, rres = oracle.ptim_exchange_loop(xi.astype(np.complex128), phi.astype(np.complex128), dV, n_iter=iters, dt=dta, alpha=1.0)
    cell = px.Cell(tuple(0.28 * m for m in n), n)
    out, res = px_ctx.px_ptim_exchange_loop(cell, to_dev(xi), to_dev(phi), iters, dta)
    torch.cuda.synchronize()
    err = relerr(to_host(out), ref)
    rerr = np.abs(to_host(res) - np.array(rres)).max()
    print(f"loop {err:.2e} residuals {rerr:.2e}", flush=True)
    assert err < (5e-6 if fp32 else 1e-13)
    assert rerr < (1e-5 if fp32 else 1e-9)
