"""px_sigma_diagonalize where eigenvalues coincide (projectors, occupations at 0
and 1: the rotations skip entries at the rounding level) and at scales whose
squares leave the normal range of the fast rotation formula.  Residual, orthogonality and
eigenvalues against numpy; tolerance 2e-14 n (error of the accumulated rotations:
a few eps per rotation of an index, about n of them a sweep, up to 20 sweeps,
random signs)."""
import numpy as np
import pytest

from _gpu import banner, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,kind,scale", [(5, "proj", 1.0), (33, "proj", 1.0), (256, "proj", 1.0), (200, "fd", 1.0),
                                          (40, "gue", 1e-143), (40, "gue", 1e143), (33, "proj", 1e-143)])
def test_clusters(px_ctx, n, kind, scale):
    import torch
    banner(f"eig clusters n={n} {kind} scale={scale}")
    rng = np.random.default_rng(11)
    h = rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n))
    w, q = np.linalg.eigh(h + h.conj().T)
    d = {"proj": (np.arange(n) < n // 2).astype(float), "gue": w,
         "fd": 1.0 / (1.0 + np.exp(np.clip((w - w[n // 2]) / 0.3, -700, 700)))}[kind]
    a = (q * d) @ q.conj().T
    a = 0.5 * (a + a.conj().T) * scale
    Q, dd, st = px_ctx.px_sigma_diagonalize(to_dev(a))
    torch.cuda.synchronize()
    Q, dd = to_host(Q), to_host(dd) / scale
    assert int(st.item()) == 0
    a /= scale
    tol = 2e-14 * n
    nrm = np.linalg.norm(a)
    res, orth = np.linalg.norm(a @ Q - Q * dd) / nrm, np.linalg.norm(Q.conj().T @ Q - np.eye(n))
    ev = np.abs(dd - np.linalg.eigvalsh(a)).max() / np.abs(d).max()
    print(f"res {res:.2e} orth {orth:.2e} ev {ev:.2e}", flush=True)
    assert res < tol and orth < tol and ev < tol
