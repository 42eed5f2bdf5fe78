"""The split-bf16 contractions where their tiling can go wrong: degree counts about a
block (32), a group of four blocks (128) and a workgroup's tile, latitudes about a wave's 16,
64 and a workgroup's 128, odd rules, several members.

Bar: the mode's 1e-6 relative l2 against the FP64 oracle.
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


SIZES = [(1, 3), (2, 5), (9, 32), (30, 0), (31, 64), (32, 75), (62, 128), (63, 135), (94, 0),
         (126, 240), (127, 256), (128, 270), (130, 0), (160, 320)]


# (ten members: the analysis takes two tiles of degrees per wave from 160000 orders and degrees)
@pytest.mark.parametrize("N,nlat,members", [(n, l, b) for n, l in SIZES for b in (1, 3)]
                         + [(126, 240, 10), (128, 270, 10), (160, 320, 7)])
def test_split_bf16_tiles(N, nlat, members):
    print(f"case: bf16x3 N={N} nlat={nlat} members={members}", flush=True)
    s = pkg.Sphere([(N, nlat, 1e-3)] * members, omega=OMEGA, dt=1e-3, precision="bf16x3")
    S = O.Sphere(N, s.nlat[0])
    n = pkg.coeff_count(N)
    a = np.stack([I.flat_spectrum(N, i) for i in range(members)])
    ga = pkg.to_device(a.reshape(-1))
    got = s.nonlinear(ga).cpu().numpy().reshape(members, n)
    grid = s.synthesize(ga)
    for i in range(members):
        t = O.to_tensor(a[i])
        assert rel(got[i], S.nonlinear(t, OMEGA).numpy()) < 1e-6
        for j, r in enumerate((*S.velocity(t), S.vorticity(t))):
            assert rel(grid[i][j].cpu().numpy(), r.numpy()) < 1e-6
    s.close()
