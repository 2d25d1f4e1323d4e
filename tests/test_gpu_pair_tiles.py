"""The pair pipeline at the edges of its tiles and groups, against the oracle:
grids whose planes the z tiles do not divide (60 x 60 x 90: 112.5 and 225 tiles)
or whose planes no 1 KiB transfer of whole rows divides (90 planes), chunks
with the orbitals short of, equal to and one past the groups whose sums pass 3
keeps (3 to 8 columns), in one chunk and in chunks of 2 or
3 in both tile configurations.  Tolerances as in the other grid tests: FP64
1e-11, FP32 2e-5 (E_x 1e-7)."""
import pytest

import oracle
from paper_2501_03061_amd import inputs, px
from _gpu import banner, relerr, to_dev, to_host

pytestmark = pytest.mark.gpu

FP64_TOL, FP32_TOL, FP32_EX_TOL = 1e-11, 2e-5, 1e-7
MU = 0.106
CASES = [((60, 60, 90), 1, 0, 0), ((60, 60, 90), 4, 4, 1), ((60, 60, 90), 16, 0, 0), ((24, 24, 24), 8, 0, 0), ((24, 24, 24), 9, 3, 1),
         ((32, 32, 32), 5, 3, 0), ((40, 40, 40), 13, 0, 0), ((72, 72, 72), 4, 4, 1), ((80, 80, 80), 3, 2, 0)]


@pytest.mark.parametrize("fp32", [False, True])
@pytest.mark.parametrize("n,n_orb,block,p2", CASES)
def test_pair_tiles(px_ctx, n, n_orb, block, p2, fp32, tmp_path):
    import torch
    banner(f"pair tiles grid {n} N={n_orb} block {block} p2={p2} fp32={fp32}")
    inst = inputs.make_instance(n, tuple(0.28 * m for m in n), n_orb, kT=0.04, seed=77)
    K = oracle.kernel_hse(inst.n, inst.L, MU)
    r = oracle.ace_build(inst.psi, inst.occ, K, inst.omega / inst.ng)
    vx = oracle.exchange_apply(inst.psi, inst.occ, inst.psi, K)
    ex = oracle.exchange_energy_gspace(inst.psi, inst.occ, K, inst.omega)
    cell = px.Cell(inst.L, inst.n)
    prec = px.PX_PREC_FP32 if fp32 else px.PX_PREC_FP64
    psi = to_dev(inst.psi)
    psi = px_ctx.px_convert_c128_to_c64(psi) if fp32 else psi
    occ, kd = to_dev(inst.occ), px_ctx.px_kernel_hse(cell, MU)
    tol, etol = (FP32_TOL, FP32_EX_TOL) if fp32 else (FP64_TOL, FP64_TOL)
    if block:
        tune = tmp_path / "tune.jsonl"
        tune.write_text(f'{{"n": {list(n)}, "prec": "{"fp32" if fp32 else "fp64"}", "block": {block}, "p2": {p2}}}\n')
        assert px_ctx.px_load_tuning(str(tune)) == 1
    try:
        e = torch.zeros(1, dtype=torch.float64, device="cuda")
        xi, st = px_ctx.px_ace_build(cell, psi, occ, kd, e_x=e)
        out = px_ctx.px_exchange_apply(cell, psi, occ, psi, kd)
        px_ctx.px_sync()
        assert int(st.item()) == 0
        err, verr = relerr(to_host(xi), r["xi"]), relerr(to_host(out), vx)
        eerr = abs(float(e.item()) - ex) / abs(ex)
        print(f"xi {err:.2e} vx {verr:.2e} e_x {eerr:.2e}", flush=True)
        assert err < tol and verr < tol and eerr < etol
    finally:
        px_ctx.set_tuning(cell, prec, 0, 0)
