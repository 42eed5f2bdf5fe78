"""Accuracy of the degree-pair contractions (FP64) at their longest segments, one order at
a time, against Legendre sums in extended precision on the library's own nodes.

Bar 1e-14, relative l2 over the degrees of an order (projection, unweighted sums over the
latitudes) or over the grid (synthesis). Derived: a segment has n = 66 rows at N = 511 and
every row rounds three times by 2^-53 of values that the difference forms do not amplify by
more than 1 / sin(45 degrees): 2^-53 sqrt(3 n) sqrt(2) = 2.2e-15, as much again from the rounding of
the node's square (n times 2^-54), and about 1e-15 each from the ring transform and from the
sums, so 1e-14 leaves a factor of two. A recurrence whose roots meet at the pole or the equator
amplifies by n there and misses it by a factor of three to five.

The derivative field's sums combine neighbouring rows that cancel to the order of 1 / l^2 near
the equator. Bar 2e-13 of the order's rms for each degree: a row's rounding there, 2^-53 of a
value l times the Legendre value's size on one latitude of 384, is l / (2 sqrt(192)) 2^-53 =
2e-15 of the rms for l = 511, thirty roundings of either sign behind it (one row in two of a
segment) times the three rows of the combination 1e-14 in the rms, 1e-13 at one degree in
several hundred; rows of two segments combined (one continued, one fresh) leave 1e-12.
"""
import math
import os

import numpy as np
import pytest
import torch

import paper_1009_3308_amd as pkg

pytestmark = pytest.mark.gpu
TOL = 1e-14
LD = np.longdouble


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    if not os.path.exists(pkg.LIB_PATH):
        from paper_1009_3308_amd import build
        build.build()
    torch.cuda.set_device(0)


def legendre(mu, m, lmax):
    """Pbar[l, m] at the nodes, l = m .. lmax, in extended precision: [l - m][node]."""
    x = mu.astype(LD)
    p = np.full(x.shape, np.sqrt(LD(1) / (16 * np.arctan(LD(1)))), dtype=LD)
    for k in range(1, m + 1):
        p = -p * np.sqrt(LD(2 * k + 1) / (2 * k)) * np.sqrt((1 - x) * (1 + x))
    out, prev, a_prev = [p], np.zeros_like(p), LD(1)
    for l in range(m + 1, lmax + 1):
        a = np.sqrt(LD(4 * l * l - 1) / LD(l * l - m * m))
        out.append(a * (x * out[-1] - prev / a_prev))
        prev, a_prev = out[-2], a
    return np.stack(out)


def rel(a, b):
    return float(np.sqrt((np.abs(a - b) ** 2).sum() / (np.abs(b) ** 2).sum()))


def slots(N, m):
    o = m * (2 * N + 3 - m) // 2
    return slice(o, o + N + 1 - m)


# two segmentations (N = 511: four of 66 rows; N = 300 and 255: eight), a group of members
CASES = [(511, 0, 1), (300, 0, 1), (255, 0, 1), (255, 0, 3)]


@pytest.mark.parametrize("N,nlat,members", CASES)
def test_projection_of_one_order(N, nlat, members):
    s = pkg.Sphere([(N, nlat, 0.0)] * members, omega=0.0, dt=1e-3)
    nl, M = s.nlat[0], 2 * s.nlat[0]
    mu, w = (np.asarray(v) for v in s.grid(0))
    rng = np.random.default_rng(N)
    phi = 2 * np.pi * np.arange(M) / M
    for m in (2, 4, 9):
        g = rng.standard_normal(nl)
        # u_phi = 0, u_theta = g cos(m phi): alpha[l, m] = lambda^-1/2 (-i m) sum_p c_p g_p P[l]
        u = np.stack([g[:, None] * np.cos(m * phi)[None], np.zeros((nl, M))])
        got = s.analyze_velocity([torch.as_tensor(u).cuda()] * members)
        got = got.cpu().numpy()[s.member_slice(members - 1)][slots(N, m)]
        x = mu.astype(LD)
        c = np.pi * LD(1) * w.astype(LD) / np.sqrt((1 - x) * (1 + x))  # (2 pi / M) w M / 2
        P = legendre(mu, m, N)
        l = np.arange(m, N + 1).astype(LD)
        ref = (-m * (P * (4 * np.arctan(LD(1)) / LD(np.pi) * c * g.astype(LD))).sum(1)
               / np.sqrt(l * (l + 1))).astype(np.float64)
        e = rel(got.imag, ref)
        print(f"case: projection N={N} members={members} m={m}: {e:.2e}", flush=True)
        assert e <= TOL
    s.close()


@pytest.mark.parametrize("N,nlat", [(511, 0), (420, 0), (340, 0)])
def test_projection_of_the_derivative_field(N, nlat):
    s = pkg.Sphere([(N, nlat, 0.0)], omega=0.0, dt=1e-3)
    nl, M = s.nlat[0], 2 * s.nlat[0]
    mu, w = (np.asarray(v) for v in s.grid(0))
    rng = np.random.default_rng(N)
    phi = 2 * np.pi * np.arange(M) / M
    x = mu.astype(LD)
    c = 4 * np.arctan(LD(1)) * w.astype(LD) / np.sqrt((1 - x) * (1 + x))
    for m in (1, 2, 16, 37, 119):
        g = rng.standard_normal(nl)
        # u_theta = 0, u_phi = g cos(m phi): alpha[l, m] = -lambda^-1/2 sum_p c_p g_p S P[l]
        # with S = sin(theta) d/dtheta, S P[l] = l e(l+1) P[l+1] - (l+1) e(l) P[l-1]
        u = np.stack([np.zeros((nl, M)), g[:, None] * np.cos(m * phi)[None]])
        got = s.analyze_velocity([torch.as_tensor(u).cuda()]).cpu().numpy()[slots(N, m)]
        T = (legendre(mu, m, N + 1) * (c * g.astype(LD))).sum(1)
        l = np.arange(m, N + 1).astype(LD)
        e = lambda d: np.sqrt((d * d - m * m) / (4 * d * d - 1))  # noqa: E731
        ref = l * e(l + 1) * T[1:]
        ref[1:] -= (l[1:] + 1) * e(l[1:]) * T[:-2]
        ref = (-ref / np.sqrt(l * (l + 1))).astype(np.float64)
        d = float(np.abs(got - ref).max() / np.sqrt((ref ** 2).mean()))
        print(f"case: derivative projection N={N} m={m}: {d:.2e}, l2 {rel(got, ref):.2e}", flush=True)
        assert d <= 2e-13
    s.close()


@pytest.mark.parametrize("N,nlat,members", CASES)
def test_vorticity_of_one_order(N, nlat, members):
    s = pkg.Sphere([(N, nlat, 0.0)] * members, omega=0.0, dt=1e-3)
    nl, M = s.nlat[0], 2 * s.nlat[0]
    mu = np.asarray(s.grid(0)[0])
    rng = np.random.default_rng(N + 1)
    cos = np.cos(2 * np.pi * np.arange(M) / M)
    for m in (0, 1):
        l = np.arange(m, N + 1).astype(LD)
        a = rng.standard_normal(N + 1 - m)
        a[l == 0] = 0.0
        host = np.zeros(pkg.coeff_count(N), dtype=np.complex128)
        host[slots(N, m)] = a
        alpha = s.new_state()
        alpha[s.member_slice(members - 1)] = pkg.to_device(host)
        got = s.synthesize(alpha)[members - 1][2].cpu().numpy()
        f = (legendre(mu, m, N) * (np.sqrt(l * (l + 1)) * a.astype(LD))[:, None]).sum(0)
        f = f.astype(np.float64)
        ref = f[:, None] * (np.ones(M) if m == 0 else 2 * cos)[None]
        e = rel(got, ref)
        print(f"case: vorticity N={N} members={members} m={m}: {e:.2e}", flush=True)
        assert e <= TOL
    s.close()
