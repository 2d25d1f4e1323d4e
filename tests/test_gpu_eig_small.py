"""px_sigma_diagonalize where a single rotation, or none, decides the result: 2 x 2
blocks, entries at the rounding level and scales at which squares leave the range of
FP64.  Residual |sigma Q - Q D| against the matrix's own rounding, computed in
extended precision."""
import numpy as np
import pytest

from _gpu import banner, to_dev, to_host

pytestmark = pytest.mark.gpu

EPS = np.finfo(np.float64).eps


def _residual(ctx, a):
    import torch
    Q, d, st = ctx.px_sigma_diagonalize(to_dev(a))
    torch.cuda.synchronize()
    assert int(st.item()) == 0
    al, Q = a.astype(np.clongdouble), to_host(Q).astype(np.clongdouble)
    r = np.sqrt((np.abs(al @ Q - Q * to_host(d)) ** 2).sum() / (np.abs(al) ** 2).sum())
    o = np.sqrt((np.abs(Q.conj().T @ Q - np.eye(len(a))) ** 2).sum())
    return float(r), float(o), to_host(d)


@pytest.mark.parametrize("ratio", [0.5, 0.1, 0.02])
def test_one_rotation(px_ctx, ratio):
    """2 x 2: after one rotation what is left are the roundings (half an eps each, random
    signs) of about six dependent operations, sqrt(6) eps at the most with all of them
    at their bound: 2.5 eps.  Roots and reciprocals of 4e-15 leave up to 3.4."""
    banner(f"eig one rotation, off-diagonal {ratio}")
    rng = np.random.default_rng(17)
    res = []
    for _ in range(32):
        z = ratio * np.exp(2j * np.pi * rng.random())
        a = np.array([[0.3 + rng.random(), z], [np.conj(z), 0.2 * rng.random()]])
        r, o, _ = _residual(px_ctx, a)
        res.append(r)
        assert o < 4 * EPS
    print(f"mean {np.mean(res) / EPS:.2f} eps, largest {np.max(res) / EPS:.2f} eps", flush=True)
    assert np.max(res) < 2.5 * EPS


@pytest.mark.parametrize("n", [2, 3, 8, 17, 33])
def test_entries_at_rounding_level(px_ctx, n):
    """The identity plus entries of 4.5 eps: within the convergence bound at the start,
    so one sweep rotates every entry and ends it.  The first rotations are by large
    angles (the diagonal entries are equal), and one sweep then leaves about half of the
    off-diagonal norm; entries that are not rotated at all would stay in the residual
    whole.  Bound half way between."""
    banner(f"eig entries at the rounding level n={n}")
    rng = np.random.default_rng(5)
    res = []
    for _ in range(16):
        h = rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n))
        a = np.eye(n) + 1e-15 * (h + h.conj().T) / 2
        np.fill_diagonal(a, 1.0)
        r, o, _ = _residual(px_ctx, a)
        res.append(r)
        assert o < 2 * n * EPS
    left = 1e-15 * np.sqrt(n - 1) / EPS  # norm of the entries over that of the matrix
    print(f"mean {np.mean(res) / EPS:.2f} eps, not rotated {left:.2f}", flush=True)
    assert np.mean(res) < 0.75 * left


@pytest.mark.parametrize("scale", [1e160, 1e-165])
def test_norm_outside_fp64(px_ctx, scale):
    """2 x 2 whose squared norm is infinite or zero in FP64: the first sweep rotates it
    all the same (residual as for any 2 x 2 matrix)."""
    banner(f"eig norm outside FP64, scale {scale}")
    a = np.array([[0.7, 0.3 - 0.2j], [0.3 + 0.2j, 0.1]]) * scale
    r, o, d = _residual(px_ctx, a)
    ev = np.abs(d / scale - np.linalg.eigvalsh(a / scale)).max()
    print(f"res {r / EPS:.2f} eps, ev {ev / EPS:.2f} eps", flush=True)
    assert r < 2.5 * EPS and o < 4 * EPS and ev < 4 * EPS
