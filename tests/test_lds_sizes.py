"""Every launch of every admissible member (N, nlat) fits the LDS of a compute unit, by the sizes
that nse_sphere_init checks (host code, no GPU)."""
import ctypes
import os

import pytest

import paper_1009_3308_amd as pkg

MAX_LDS, MAX_M = 160 * 1024, 1536


class Plan(ctypes.Structure):  # nse::FftPlan: four integers, then seven per-stage arrays of four
    _fields_ = [("head", ctypes.c_int * 4), ("stages", ctypes.c_int * 28)]


@pytest.fixture(scope="module")
def L():
    if not os.path.exists(pkg.LIB_PATH):
        from paper_1009_3308_amd import build
        build.build()
    lib = pkg.lib()
    lib._ZN3nse14pair_lds_bytesEii.restype = ctypes.c_size_t
    lib._ZN3nse14ring_lds_bytesEiRKNS_7FftPlanE.restype = ctypes.c_size_t
    lib._ZN3nse8fft_planEi.restype = Plan
    return lib


def _smooth(M):
    for p in (2, 3, 5):
        while M % p == 0:
            M //= p
    return M == 1


def test_admissible_members_fit_the_lds(L):
    pair, worst = L._ZN3nse14pair_lds_bytesEii, 0
    for nlat in range(3, MAX_M // 2 + 1):
        if not _smooth(2 * nlat):
            continue
        nh, top = (nlat + 1) // 2, (2 * nlat - 2) // 3
        sizes = [pair(N, nh) for N in range(1, top + 1)]
        assert 0 < max(sizes) <= MAX_LDS, nlat
        worst = max(worst, max(sizes))
        plan = L._ZN3nse8fft_planEi(2 * nlat)
        ring = L._ZN3nse14ring_lds_bytesEiRKNS_7FftPlanE(2 * nlat, ctypes.byref(plan))
        # (three arrays of M complex values at least, six for two rings)
        assert 16 * 3 * 2 * nlat < ring <= MAX_LDS, nlat
    # the largest are above the 64 KiB that other checks allow, so these are needed
    assert worst > 65536
    # two workgroups of the adjoint at N = 511 share a compute unit
    assert pair(511, 384) <= MAX_LDS // 2


def test_a_member_beyond_the_lds_would_be_seen(L):
    assert L._ZN3nse14pair_lds_bytesEii(1500, 1200) > MAX_LDS
