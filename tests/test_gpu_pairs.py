"""The degree-pair contractions (FP64) where their tiling can go wrong: orders with one
pair, latitudes short of a tile of 16, odd rules, the size classes of both segmentations (few
members, and groups of at least four), more input sources than three, and the
adjoint and the projection on the same sizes, against the FP64 oracle.

Bar: relative l2 <= 1e-12 (two FP64 evaluations of the same sums: at most a few
hundred terms of either sign, 2^-53 each, and the 1e-13 the recurrence may grow to).
"""
import math
import os

import numpy as np
import pytest
import torch

import nse_inputs as I
import paper_1009_3308_amd as pkg
from oracle import nse_oracle as O

pytestmark = pytest.mark.gpu
OMEGA = 2.0 * math.pi
TOL = 1e-12


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    if not os.path.exists(pkg.LIB_PATH):
        from paper_1009_3308_amd import build
        build.build()
    torch.cuda.set_device(0)


def rel(a, b):
    return float(np.linalg.norm(np.asarray(a) - np.asarray(b)) / np.linalg.norm(np.asarray(b)))


# (N, nlat): one pair per order; 16 and 17 northern latitudes; the last nh of a size
# class (48, 96, 192) and the first of the next
SIZES = [(1, 3), (2, 0), (3, 9), (4, 32), (10, 27), (16, 30), (20, 32), (21, 36), (31, 96),
         (40, 100), (63, 192), (64, 200), (84, 384), (85, 400)]


@pytest.mark.parametrize("N,nlat", SIZES)
@pytest.mark.parametrize("members", [1, 5])
def test_pairs_nonlinear_adjoint_projection(N, nlat, members):
    print(f"case: pairs N={N} nlat={nlat} members={members}", flush=True)
    s = pkg.Sphere([(N, nlat, 1e-3)] * members, omega=OMEGA, dt=1e-3)
    S = O.Sphere(N, s.nlat[0])
    n = pkg.coeff_count(N)
    a = np.stack([I.flat_spectrum(N, i) for i in range(members)])
    c = np.stack([I.cotangent(N, i) for i in range(members)])
    ga, gc = pkg.to_device(a.reshape(-1)), pkg.to_device(c.reshape(-1))
    got = s.nonlinear(ga).cpu().numpy().reshape(members, n)
    bar = s.nonlinear_adjoint(ga, gc).cpu().numpy().reshape(members, n)
    u = [torch.as_tensor(I.grid_noise(50 + i, s.nlat[0], 2 * s.nlat[0])).cuda()
         for i in range(members)]
    pr = s.analyze_velocity(u).cpu().numpy().reshape(members, n)
    for i in range(members):
        t = O.to_tensor(a[i]).requires_grad_(True)
        ref = S.nonlinear(t, OMEGA)
        assert rel(got[i], ref.detach().numpy()) <= TOL
        w = O.to_tensor(c[i])
        (g,) = torch.autograd.grad((w.real * ref.real + w.imag * ref.imag).sum(), t)
        g = O.clean(g, N).numpy()
        assert rel(bar[i], g) <= TOL
        v = u[i].cpu()
        assert rel(pr[i], S.project(v[0], v[1]).numpy()) <= TOL
    s.close()


@pytest.mark.parametrize("order", [1, 4, 5])
@pytest.mark.parametrize("members", [1, 4])
def test_pairs_steps_of_high_order(order, members):
    # 4 and 5 read more than three predictor terms and history rows
    N, nu, dt = 33, 1e-3, 1e-3
    print(f"case: pairs steps order={order} members={members}", flush=True)
    s = pkg.Sphere([(N, 0, nu)] * members, omega=OMEGA, dt=dt, order=order)
    S = O.Sphere(N, s.nlat[0])
    h = s.new_history()
    a0 = [I.member_state(i, N) for i in range(members)]
    f = s.new_state()
    for i in range(members):
        h[0, s.member_slice(i)] = pkg.to_device(a0[i])
        f[s.member_slice(i)] = pkg.to_device(I.forcing(N))
    s.step(h, f, 0, 9)
    for i in range(members):
        ref = O.Stepper(S, nu, OMEGA, dt, order=order).run(O.to_tensor(a0[i]),
                                                          O.to_tensor(I.forcing(N)), 9)
        for j in range(order + 1):
            assert rel(h[j, s.member_slice(i)].cpu().numpy(), ref[j].numpy()) <= TOL
    s.close()


@pytest.mark.parametrize("N,nlat", [(2, 0), (21, 36), (100, 160), (64, 200)])
def test_pairs_grid_fields(N, nlat):
    print(f"case: pairs grid N={N} nlat={nlat}", flush=True)
    s = pkg.Sphere([(N, nlat, 0.0)], omega=OMEGA, dt=1e-3)
    S = O.Sphere(N, s.nlat[0])
    a = I.flat_spectrum(N, 3)
    t = O.to_tensor(a)
    ut, up = S.velocity(t)
    g = s.synthesize(pkg.to_device(a))[0].cpu().numpy()
    p = s.synthesize_psi(pkg.to_device(a))[0].cpu().numpy()
    for got, ref in ((g[0], ut), (g[1], up), (g[2], S.vorticity(t)), (p[0], ut),
                     (p[2], O.stream_function_psi(S, t))):
        assert rel(got, ref.numpy()) <= TOL
    s.close()
