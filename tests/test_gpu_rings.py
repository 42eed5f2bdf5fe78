"""The longitude transforms over their plans: two to four stages, every radix, LDS
padding of either kind, compile-time and run-time plans, odd rules (an equator ring, a
last workgroup with one ring of two), one and two rings per workgroup, each mode.

Bar: relative l2 <= 1e-12 against the FP64 oracle (as for the contractions: the transforms
add a few roundings per stage).
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


# (nlat, members): the largest N of the grid up to 40, so that small grids use every order
SIZES = [(3, 1), (5, 2), (6, 1), (12, 3), (25, 1), (27, 11), (45, 6), (48, 1), (48, 6), (75, 4),
         (81, 1), (96, 1), (96, 3), (125, 3), (128, 1), (135, 2), (144, 2), (160, 1), (192, 1),
         (192, 2), (243, 2), (250, 1), (324, 1), (375, 1), (384, 1), (384, 3), (405, 1),
         (480, 1), (500, 1), (512, 1), (600, 1), (625, 1), (729, 1), (750, 1), (768, 1)]


@pytest.mark.parametrize("nlat,members", SIZES)
def test_rings_all_modes(nlat, members):
    N, M = min(40, (2 * nlat - 2) // 3), 2 * nlat
    print(f"case: rings M={M} N={N} members={members}", flush=True)
    s = pkg.Sphere([(N, nlat, 1e-3)] * members, omega=OMEGA, dt=1e-3)
    S = O.Sphere(N, nlat)
    n = pkg.coeff_count(N)
    a = np.stack([I.flat_spectrum(N, i) for i in range(members)])
    c = np.stack([I.cotangent(N, i) for i in range(members)])
    ga, gc = pkg.to_device(a.reshape(-1)), pkg.to_device(c.reshape(-1))
    got = s.nonlinear(ga).cpu().numpy().reshape(members, n)
    bar = s.nonlinear_adjoint(ga, gc).cpu().numpy().reshape(members, n)
    u = [torch.as_tensor(I.grid_noise(50 + i, nlat, M)).cuda() for i in range(members)]
    pr = s.analyze_velocity(u).cpu().numpy().reshape(members, n)
    grid = s.synthesize(ga)
    for i in range(members):
        t = O.to_tensor(a[i]).requires_grad_(True)
        ref = S.nonlinear(t, OMEGA)
        assert rel(got[i], ref.detach().numpy()) <= TOL
        w = O.to_tensor(c[i])
        (g,) = torch.autograd.grad((w.real * ref.real + w.imag * ref.imag).sum(), t)
        assert rel(bar[i], O.clean(g, N).numpy()) <= TOL
        v = u[i].cpu()
        assert rel(pr[i], S.project(v[0], v[1]).numpy()) <= TOL
        t = t.detach()
        for j, r in enumerate((*S.velocity(t), S.vorticity(t))):
            assert rel(grid[i][j].cpu().numpy(), r.numpy()) <= TOL
    s.close()
