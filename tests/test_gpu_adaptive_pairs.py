"""Device-controlled adaptive runs whose corrector sweep rides in the pair analysis: its
instances of three and four waves (several members on nh > 96, one member on nh >= 256), where
the norms that decide order and step meet from several waves, some without a degree, and
with the controller step in the synthesis (member blocks (0, 8)).

Bars as in test_gpu_adaptive.py: attempt logs exact in order, sweeps and outcome, t and h to
1e-9, the state to 1e-10 of its largest coefficient.
"""
import math
import os

import numpy as np
import pytest
import torch

import nse_inputs as I
import paper_1009_3308_amd as pkg
from oracle import nse_oracle as O
from test_gpu_adaptive import _compare_logs, _oracle_integrator

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


@pytest.mark.parametrize("N,nlat,members,blocks,T", [
    (40, 200, 2, None, 0.5),      # three waves, two of them without a degree
    (130, 200, 2, None, 0.1),     # three waves, the last with three degrees
    (40, 512, 1, None, 0.5),      # four waves of five groups
    (150, 512, 1, None, 0.1),
    (40, 768, 1, None, 0.3),      # four waves of six groups
    (60, 200, 2, (0, 8), 0.3),    # the controller step rides in the synthesis
    (31, 0, 3, (2, 0), 0.5),      # blocks in the synthesis only
])
def test_device_controlled_pair_analysis_matches_oracle(N, nlat, members, blocks, T):
    print(f"case: adaptive pairs N={N} nlat={nlat} members={members} blocks={blocks}", flush=True)
    nus = [1e-3, 3e-3, 2e-3][:members]
    a0 = np.concatenate([I.member_state(i, N) for i in range(members)])
    f = np.concatenate([(1.0 - 0.3 * i) * I.forcing(N) for i in range(members)])
    s = pkg.Sphere([(N, nlat, nu) for nu in nus], omega=OMEGA, dt=1e-3, order=2)
    if blocks:
        s.set_member_blocks(0, *blocks)
    nl = s.nlat[0]
    s.adaptive_begin(pkg.to_device(a0), 0.0, rtol=1e-4, atol=1e-6, forcing=pkg.to_device(f))
    out, stats = s.adaptive_advance(T)
    glog = s.adaptive_log()
    g = out.cpu()
    s.close()
    ft = O.to_tensor(f)
    integ = _oracle_integrator(N, nus, lambda t: ft, nlat=nl, rtol=1e-4, atol=1e-6)
    integ.begin(O.to_tensor(a0), 0.0)
    o = integ.advance(T)
    _compare_logs(glog, integ.log, f"N={N} nlat={nl}", (T,))
    diff, scale = float((g - o).abs().max()), float(o.abs().max())
    print(f"  attempts {len(glog)} state diff {diff / scale:.3e}", flush=True)
    assert stats["t"] == T and len(glog) > 8
    assert diff <= 1e-10 * scale
