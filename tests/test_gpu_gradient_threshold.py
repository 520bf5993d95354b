"""The gradient close to the threshold sqrt(s) = 1, where the photons are soft
and the electron barely moves."""
import numpy as np
import pytest
import torch

from oracle import qed_oracle_ld as LO
from paper_2511_19456_amd import inputs
from parity import C_FP64, EPS64, REL_FP64

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
LD = np.longdouble


def _rambo_ld(u, rs):
    """RAMBO in extended precision: momenta [N, n + 3, 4] of uniforms [4(n + 1)][N]."""
    q = []
    for j in range(u.shape[0] // 4):
        c, ph, e = 2 * u[4 * j] - 1, 2 * LD("3.14159265358979323846264") * u[4 * j + 1], -np.log(u[4 * j + 2] * u[4 * j + 3])
        st = np.sqrt(1 - c * c)
        q.append(e * np.stack([c * 0 + 1, st * np.cos(ph), st * np.sin(ph), c]))
    Q = sum(q)
    M = np.sqrt(Q[0] ** 2 - (Q[1:] ** 2).sum(0))
    b, x, gam = -Q[1:] / M, rs / M, Q[0] / M
    p = []
    for v in q:
        bq = (b * v[1:]).sum(0)
        p.append(np.concatenate([(x * (gam * v[0] + bq))[None], x * (v[1:] + b * (v[0] + bq / (1 + gam)))]))
    e2, rest = p[0][0] ** 2, sum(v[0] for v in p[1:])
    xi = np.full_like(e2, np.sqrt(1 - 1 / (rs * rs)))
    for _ in range(30):
        r = np.sqrt(1 + xi * xi * e2)
        xi = xi - (r + xi * rest - rs) / (xi * e2 / r + rest)
    k, o = (rs * rs - 1) / (2 * rs), np.ones_like(xi)
    mom = [np.stack([np.sqrt(1 + k * k) * o, 0 * o, 0 * o, -k * o]), np.stack([k * o, 0 * o, 0 * o, k * o]),
           np.concatenate([np.sqrt(1 + (xi * p[0][0]) ** 2)[None], xi * p[0][1:]])]
    return np.stack(mom + [xi * v for v in p[1:]]).transpose(2, 0, 1)


def _gradient_ld(u, rs):
    """Sixth-order differences of the extended-precision oracle: steps of 2^-12
    of the distance to the interval's end, so 1e-18 or less of truncation."""
    n = u.shape[0] // 4 - 1
    u, g = u.astype(LD), np.zeros(u.shape, dtype=LD)
    for r in range(u.shape[0]):
        h = LD(2) ** -12 * np.minimum(u[r], 1 - u[r])
        d = []
        for s in (1, 2, 4):
            y = []
            for x in (s, -s):
                w = u.copy()
                w[r] += x * h
                y.append(np.log(LO.m2_sum(_rambo_ld(w, LD(rs)), n)))
            d.append((y[0] - y[1]) / (2 * s * h))
        a, b = (4 * d[0] - d[1]) / 3, (4 * d[1] - d[2]) / 3
        g[r] = (16 * a - b) / 15
    return g


@pytest.mark.parametrize("delta", [1e-4, 1e-3])
def test_gradient_near_threshold_two_photons(delta):
    """Photon energies are differences of energies of order 1, so rounding
    reaches them as eps / delta; with the roundings of a product of currents
    (C_FP64, twice for |A|^2) half of the points stay below that."""
    from paper_2511_19456_amd.qedx import QedProcess
    n, rs = 2, 1.0 + delta
    u, _ = inputs.rambo_inputs(17, n, 24)
    _, g = QedProcess(n, "sum").eval_grad(torch.as_tensor(u, device=DEV), rs)
    ref = _gradient_ld(u, rs)
    err = np.sqrt(((g.cpu().numpy() - ref) ** 2).sum(0)) / np.sqrt((ref ** 2).sum(0))
    assert float(np.median(err)) < 2.0 * C_FP64 * EPS64 / delta, float(np.median(err))


@pytest.mark.parametrize("n", [1, 2, 3, 4])
def test_gradient_is_continuous_where_the_kernel_changes(n):
    """From sqrt(s) = 1.1 on another kernel takes the polarisation vectors'
    share: one bit below it the results are the same to the gradients'
    tolerance, for every size with the bits of the full set."""
    from paper_2511_19456_amd.qedx import QedProcess
    u, _ = inputs.rambo_inputs(18 + n, n, 131)
    ud = torch.as_tensor(u, device=DEV)
    p = QedProcess(n, "sum")
    below = float(np.nextafter(1.1, 0.0))
    v0, g0 = p.eval_grad(ud, below)
    v1, g1 = p.eval_grad(ud, 1.1)
    err = (g0 - g1).norm(dim=0) / g1.norm(dim=0)
    assert err.max().item() < REL_FP64 and (v0 - v1).abs().max().item() < REL_FP64 * max(1.0, v1.abs().max().item())
    for N in (1, 2, 5, 33, 130):
        v, g = p.eval_grad(ud[:, :N].contiguous(), below)
        assert torch.equal(v, v0[:N]) and torch.equal(g, g0[:, :N]), N
