"""Python binding of libnse_sphere.so (include/nse_sphere.h).

Argument marshalling only: every step of the hot path runs in the HIP library.
Arrays are torch tensors on the GPU (complex128 states, float64 grids); the
library enqueues on the torch stream given at construction. If the library is
not built, every entry point raises; there is no CPU fallback.
"""
from __future__ import annotations

import ctypes
import os
from typing import Iterable, Sequence

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_HERE, "libnse_sphere.so")

NSE_OK = 0
NSE_ERR_ARG = 1
NSE_ERR_ALLOC = 2
NSE_ERR_HIP = 3
NSE_ERR_UNSUPPORTED = 4
NSE_ERR_NONFINITE = 5
NSE_ERR_STATE = 6

PREC_FP64 = 0
PREC_FP32 = 1
PREC_BF16X3 = 2
PRECISIONS = {"fp64": PREC_FP64, "fp32": PREC_FP32, "bf16x3": PREC_BF16X3}

FLAG_GRAPH = 1
FLAG_AUTOTUNE = 2
FLAG_CHECK_FINITE = 4

# Every function the header declares (checked against include/nse_sphere.h by the tests).
EXPORTS = (
    "nse_sphere_init", "nse_sphere_destroy", "nse_set_stream", "nse_coeff_count",
    "nse_state_count", "nse_member_grid", "nse_nonlinear", "nse_step",
    "nse_nonlinear_adjoint", "nse_step_adjoint", "nse_synthesize", "nse_legendre_values",
    "nse_sync", "nse_status_string", "nse_last_error", "nse_profile_enable", "nse_profile_read",
    "nse_analyze_velocity", "nse_get_member_blocks", "nse_set_member_blocks",
    "nse_adaptive_begin", "nse_adaptive_begin_scheduled", "nse_adaptive_advance",
    "nse_adaptive_log",
    "nse_energy_spectrum", "nse_synthesize_psi", "nse_inertial_manifold",
    "nse_nonlinear_adjoint_noalloc", "nse_step_trajectory", "nse_step_adjoint_trajectory",
    "nse_graph_counts",
)

ATTEMPT_ACCEPTED, ATTEMPT_ERROR_FAIL, ATTEMPT_NEWTON_FAIL = 0, 1, 2

KERNEL_KINDS = {"synthesis": 0, "ring": 1, "analysis": 2}


class NseError(RuntimeError):
    def __init__(self, status: int, message: str):
        super().__init__(message)
        self.status = status


class Member(ctypes.Structure):
    _fields_ = [("N", ctypes.c_int32), ("nlat", ctypes.c_int32), ("nu", ctypes.c_double)]


class Params(ctypes.Structure):
    _fields_ = [("omega", ctypes.c_double), ("dt", ctypes.c_double), ("order", ctypes.c_int32),
                ("newton_iters", ctypes.c_int32), ("precision", ctypes.c_int32),
                ("flags", ctypes.c_uint32)]


class AdaptiveParams(ctypes.Structure):
    _fields_ = [("rtol", ctypes.c_double), ("atol", ctypes.c_double), ("h0", ctypes.c_double),
                ("hmax", ctypes.c_double), ("max_order", ctypes.c_int32),
                ("max_newton", ctypes.c_int32)]


class AdaptiveRecord(ctypes.Structure):
    _fields_ = [("t", ctypes.c_double), ("h", ctypes.c_double), ("err", ctypes.c_double),
                ("order", ctypes.c_int32), ("sweeps", ctypes.c_int32),
                ("outcome", ctypes.c_int32), ("reserved", ctypes.c_int32)]


class AdaptiveStats(ctypes.Structure):
    _fields_ = [("t", ctypes.c_double), ("h", ctypes.c_double), ("order", ctypes.c_int32),
                ("reserved", ctypes.c_int32), ("accepted", ctypes.c_int64),
                ("error_failures", ctypes.c_int64), ("newton_failures", ctypes.c_int64),
                ("evaluations", ctypes.c_int64), ("waits", ctypes.c_int64),
                ("wait_seconds", ctypes.c_double)]

    def as_dict(self):
        return {name: getattr(self, name) for name, _ in self._fields_ if name != "reserved"}


class ForcingSchedule(ctypes.Structure):
    """Forcing scale evaluated on the device: s(t) = before for t <= t_on, else
    amp cos(omega t + phase) exp(-decay (t - t_on))."""
    _fields_ = [("t_on", ctypes.c_double), ("before", ctypes.c_double),
                ("amp", ctypes.c_double), ("omega", ctypes.c_double),
                ("phase", ctypes.c_double), ("decay", ctypes.c_double)]


FORCING_FN = ctypes.CFUNCTYPE(ctypes.c_double, ctypes.c_void_p, ctypes.c_double)

_lib = None


def lib():
    """Loads libnse_sphere.so (raises if it has not been built)."""
    global _lib
    if _lib is not None:
        return _lib
    if not os.path.exists(LIB_PATH):
        raise RuntimeError(f"{LIB_PATH} is not built: run __graft_entry__.build() "
                           "(python -m paper_1009_3308_amd.build)")
    L = ctypes.CDLL(LIB_PATH)
    vp, dp, i32, i64 = ctypes.c_void_p, ctypes.c_void_p, ctypes.c_int32, ctypes.c_int64
    st = ctypes.c_int
    sig = {
        "nse_sphere_init": (st, [ctypes.POINTER(Member), i32, ctypes.POINTER(Params), vp,
                                 ctypes.POINTER(vp)]),
        "nse_sphere_destroy": (st, [vp]),
        "nse_set_stream": (st, [vp, vp]),
        "nse_coeff_count": (i64, [i32]),
        "nse_state_count": (i64, [vp]),
        "nse_member_grid": (st, [vp, i32, ctypes.POINTER(i32), dp, dp]),
        "nse_nonlinear": (st, [vp, dp, dp]),
        "nse_step": (st, [vp, dp, dp, i64, i32]),
        "nse_nonlinear_adjoint": (st, [vp, dp, dp, dp]),
        "nse_nonlinear_adjoint_noalloc": (st, [vp, dp, dp, dp]),
        "nse_step_adjoint": (st, [vp, dp, dp, i64, dp]),
        "nse_step_trajectory": (st, [vp, dp, dp, i64, i32]),
        "nse_step_adjoint_trajectory": (st, [vp, dp, dp, i64, i32, dp]),
        "nse_synthesize": (st, [vp, dp, dp]),
        "nse_analyze_velocity": (st, [vp, dp, dp]),
        "nse_get_member_blocks": (st, [vp, i32, ctypes.POINTER(i32), ctypes.POINTER(i32)]),
        "nse_set_member_blocks": (st, [vp, i32, i32, i32]),
        "nse_graph_counts": (st, [vp, ctypes.POINTER(i64), ctypes.POINTER(i64)]),
        "nse_legendre_values": (st, [vp, i32, i32, dp]),
        "nse_sync": (st, [vp]),
        "nse_profile_enable": (st, [vp, i32]),
        "nse_profile_read": (st, [vp, i32, ctypes.POINTER(i64), ctypes.POINTER(ctypes.c_double)]),
        "nse_adaptive_begin": (st, [vp, dp, ctypes.c_double, ctypes.POINTER(AdaptiveParams), dp,
                                    FORCING_FN, vp]),
        "nse_adaptive_begin_scheduled": (st, [vp, dp, ctypes.c_double,
                                              ctypes.POINTER(AdaptiveParams), dp,
                                              ctypes.POINTER(ForcingSchedule)]),
        "nse_adaptive_advance": (st, [vp, ctypes.c_double, dp, ctypes.POINTER(AdaptiveStats)]),
        "nse_adaptive_log": (st, [vp, ctypes.POINTER(AdaptiveRecord), i64,
                                  ctypes.POINTER(i64)]),
        "nse_energy_spectrum": (st, [vp, dp, dp]),
        "nse_synthesize_psi": (st, [vp, dp, dp]),
        "nse_inertial_manifold": (st, [vp, dp, i32, i32, dp, dp]),
        "nse_status_string": (ctypes.c_char_p, [st]),
        "nse_last_error": (ctypes.c_char_p, [vp]),
    }
    for name, (res, args) in sig.items():
        fn = getattr(L, name)
        fn.restype = res
        fn.argtypes = args
    _lib = L
    return L


def coeff_count(N: int) -> int:
    return int(lib().nse_coeff_count(N))


def _check(status: int, ctx=None):
    if status != NSE_OK:
        L = lib()
        msg = L.nse_last_error(ctx).decode() if L.nse_last_error(ctx) else ""
        name = L.nse_status_string(status).decode()
        raise NseError(status, f"{name}: {msg}")


def _ptr(t, dtype, numel=None, name="array"):
    """Device pointer of a contiguous GPU tensor of the given dtype (None -> NULL)."""
    import torch
    if t is None:
        return None
    if not isinstance(t, torch.Tensor):
        raise TypeError(f"{name} must be a torch tensor")
    if t.device.type != "cuda":
        raise ValueError(f"{name} must be on the GPU")
    if t.dtype != dtype:
        raise TypeError(f"{name} must be {dtype}, got {t.dtype}")
    if not t.is_contiguous():
        raise ValueError(f"{name} must be contiguous")
    if numel is not None and t.numel() != numel:
        raise ValueError(f"{name} must have {numel} elements, got {t.numel()}")
    return ctypes.c_void_p(t.data_ptr())


class Sphere:
    """A context of one or more members (truncation N, latitudes nlat, viscosity nu).

    members: sequence of (N, nlat, nu) with nlat = 0 for the smallest alias-free grid.
    """

    def __init__(self, members: Sequence[tuple], omega: float, dt: float, order: int = 2,
                 newton_iters: int = 1, precision: str = "fp64", graph: bool = False,
                 check_finite: bool = False, autotune: bool = False, stream=None):
        import torch
        L = lib()
        self.member_specs = [(int(N), int(nlat), float(nu)) for (N, nlat, nu) in members]
        arr = (Member * len(self.member_specs))(*[Member(N, nl, nu) for (N, nl, nu) in
                                                   self.member_specs])
        if precision not in PRECISIONS:
            raise ValueError(f"precision must be one of {sorted(PRECISIONS)}")
        flags = ((FLAG_GRAPH if graph else 0) | (FLAG_CHECK_FINITE if check_finite else 0)
                 | (FLAG_AUTOTUNE if autotune else 0))
        self.params = Params(float(omega), float(dt), int(order), int(newton_iters),
                             PRECISIONS[precision], flags)
        self.order = int(order)
        if stream is None:
            stream = torch.cuda.current_stream()
        self.stream = stream
        h = ctypes.c_void_p()
        st = L.nse_sphere_init(arr, len(self.member_specs), ctypes.byref(self.params),
                               ctypes.c_void_p(stream.cuda_stream), ctypes.byref(h))
        _check(st, None)
        self._h = h
        self.state_count = int(L.nse_state_count(h))
        self.offsets, self.nlat = [], []
        off = 0
        for i, (N, _, _) in enumerate(self.member_specs):
            self.offsets.append(off)
            off += coeff_count(N)
            nl = ctypes.c_int32()
            _check(L.nse_member_grid(h, i, ctypes.byref(nl), None, None), h)
            self.nlat.append(nl.value)

    # -- helpers -------------------------------------------------------------
    def _handle(self):
        if self._h is None:
            raise NseError(NSE_ERR_STATE, "context is closed")
        return self._h

    def grid(self, member: int = 0):
        """(mu, w) of a member's Gauss-Legendre rule as float64 numpy arrays."""
        import numpy as np
        nl = self.nlat[member]
        mu = np.zeros(nl)
        w = np.zeros(nl)
        _check(lib().nse_member_grid(self._handle(), member, None,
                                     mu.ctypes.data_as(ctypes.c_void_p),
                                     w.ctypes.data_as(ctypes.c_void_p)), self._h)
        return mu, w

    def graph_counts(self):
        """(captured, launched): step and trajectory graphs of this context so far."""
        c, n = ctypes.c_int64(), ctypes.c_int64()
        _check(lib().nse_graph_counts(self._handle(), ctypes.byref(c), ctypes.byref(n)), self._h)
        return c.value, n.value

    def new_state(self):
        import torch
        return torch.zeros(self.state_count, dtype=torch.complex128, device="cuda")

    def new_history(self):
        import torch
        return torch.zeros(self.order + 1, self.state_count, dtype=torch.complex128,
                           device="cuda")

    # -- the hot path ----------------------------------------------------------
    def nonlinear(self, alpha, out=None):
        import torch
        if out is None:
            out = self.new_state()
        _check(lib().nse_nonlinear(self._handle(),
                                   _ptr(alpha, torch.complex128, self.state_count, "alpha"),
                                   _ptr(out, torch.complex128, self.state_count, "n_out")),
               self._h)
        return out

    def step(self, hist, forcing=None, step0: int = 0, nsteps: int = 1):
        import torch
        _check(lib().nse_step(self._handle(),
                              _ptr(hist, torch.complex128, (self.order + 1) * self.state_count,
                                   "hist"),
                              _ptr(forcing, torch.complex128, self.state_count, "forcing"),
                              int(step0), int(nsteps)), self._h)
        return hist

    def nonlinear_adjoint(self, alpha, n_bar, out=None):
        import torch
        if out is None:
            out = self.new_state()
        _check(lib().nse_nonlinear_adjoint(
            self._handle(), _ptr(alpha, torch.complex128, self.state_count, "alpha"),
            _ptr(n_bar, torch.complex128, self.state_count, "n_bar"),
            _ptr(out, torch.complex128, self.state_count, "alpha_bar")), self._h)
        return out

    def nonlinear_adjoint_noalloc(self, alpha, n_bar, out):
        """nse_nonlinear_adjoint_noalloc: the same product with the library's static
        scratch in place of allocated intermediates; `out` must be given (nothing is
        allocated here either)."""
        import torch
        _check(lib().nse_nonlinear_adjoint_noalloc(
            self._handle(), _ptr(alpha, torch.complex128, self.state_count, "alpha"),
            _ptr(n_bar, torch.complex128, self.state_count, "n_bar"),
            _ptr(out, torch.complex128, self.state_count, "alpha_bar")), self._h)
        return out

    def step_adjoint(self, hist, forcing, step: int, hist_bar):
        import torch
        n = (self.order + 1) * self.state_count
        _check(lib().nse_step_adjoint(
            self._handle(), _ptr(hist, torch.complex128, n, "hist"),
            _ptr(forcing, torch.complex128, self.state_count, "forcing"), int(step),
            _ptr(hist_bar, torch.complex128, n, "hist_bar")), self._h)
        return hist_bar

    def new_trajectory(self, nsteps: int):
        """A zeroed trajectory buffer of nsteps + order + 1 states (step_trajectory)."""
        import torch
        return torch.zeros(int(nsteps) + self.order + 1, self.state_count,
                           dtype=torch.complex128, device="cuda")

    def step_trajectory(self, traj, forcing, step0: int, nsteps: int):
        """nsteps steps on traj: traj[nsteps:] holds the starting history on entry,
        traj[nsteps - i:] the history before step step0 + i on return."""
        import torch
        n = (int(nsteps) + self.order + 1) * self.state_count
        _check(lib().nse_step_trajectory(
            self._handle(), _ptr(traj, torch.complex128, n, "traj"),
            _ptr(forcing, torch.complex128, self.state_count, "forcing"), int(step0),
            int(nsteps)), self._h)
        return traj

    def step_adjoint_trajectory(self, traj, forcing, step0: int, nsteps: int, hist_bar):
        import torch
        n = (int(nsteps) + self.order + 1) * self.state_count
        _check(lib().nse_step_adjoint_trajectory(
            self._handle(), _ptr(traj, torch.complex128, n, "traj"),
            _ptr(forcing, torch.complex128, self.state_count, "forcing"), int(step0),
            int(nsteps),
            _ptr(hist_bar, torch.complex128, (self.order + 1) * self.state_count, "hist_bar")),
            self._h)
        return hist_bar

    def synthesize(self, alpha):
        """[u_theta, u_phi, zeta] grids, one float64 tensor [3, nlat, M] per member."""
        import torch
        sizes = [3 * nl * 2 * nl for nl in self.nlat]
        out = torch.empty(sum(sizes), dtype=torch.float64, device="cuda")
        _check(lib().nse_synthesize(self._handle(),
                                    _ptr(alpha, torch.complex128, self.state_count, "alpha"),
                                    _ptr(out, torch.float64)), self._h)
        res, o = [], 0
        for nl, s in zip(self.nlat, sizes):
            res.append(out[o:o + s].view(3, nl, 2 * nl))
            o += s
        return res

    def member_blocks(self, member: int = 0):
        """(synthesis, analysis) member-block sizes of the member's group (0 = per member)."""
        sb, ab = ctypes.c_int32(), ctypes.c_int32()
        _check(lib().nse_get_member_blocks(self._handle(), member, ctypes.byref(sb),
                                           ctypes.byref(ab)), self._h)
        return sb.value, ab.value

    def set_member_blocks(self, member: int, synth_block: int, anal_block: int):
        _check(lib().nse_set_member_blocks(self._handle(), member, synth_block, anal_block),
               self._h)

    def analyze_velocity(self, grids, out=None):
        """alpha = (u, Z)_M from per-member grids [>=2, nlat, M] (u_theta, u_phi first)."""
        import torch
        if len(grids) != len(self.member_specs):
            raise ValueError("need one grid per member")
        parts = []
        for g, nl in zip(grids, self.nlat):
            if g.dim() != 3 or g.shape[0] < 2 or tuple(g.shape[1:]) != (nl, 2 * nl):
                raise ValueError(f"member grid must be [>=2, {nl}, {2 * nl}]")
            parts.append(g[:2].reshape(-1))
        flat = torch.cat(parts).to(torch.float64).contiguous()
        if out is None:
            out = self.new_state()
        _check(lib().nse_analyze_velocity(self._handle(), _ptr(flat, torch.float64),
                                          _ptr(out, torch.complex128, self.state_count,
                                               "alpha_out")), self._h)
        return out

    def legendre_values(self, member: int, m: int):
        """Pbar[l,m](mu_p), l = m..N+1, northern nodes: float64 tensor [N+2-m, ceil(nlat/2)]."""
        import torch
        N = self.member_specs[member][0]
        nh = (self.nlat[member] + 1) // 2
        out = torch.empty((N + 2 - m) * nh, dtype=torch.float64, device="cuda")
        _check(lib().nse_legendre_values(self._handle(), member, m, _ptr(out, torch.float64)),
               self._h)
        return out.view(N + 2 - m, nh)

    # -- diagnostics (Section 5.3) -----------------------------------------------
    def energy_spectrum(self, alpha, out=None):
        """E(L), L = 0..N, of every member: float64 [sum over members of N+1]."""
        import torch
        n = sum(spec[0] + 1 for spec in self.member_specs)
        if out is None:
            out = torch.empty(n, dtype=torch.float64, device="cuda")
        _check(lib().nse_energy_spectrum(
            self._handle(), _ptr(alpha, torch.complex128, self.state_count, "alpha"),
            _ptr(out, torch.float64, n, "E_out")), self._h)
        return out

    def synthesize_psi(self, alpha):
        """[(u_theta, u_phi, Psi_N) per member] on the grid (Psi_N of eq. (eq:vort_app))."""
        import torch
        sizes = [3 * nl * 2 * nl for nl in self.nlat]
        out = torch.empty(sum(sizes), dtype=torch.float64, device="cuda")
        _check(lib().nse_synthesize_psi(
            self._handle(), _ptr(alpha, torch.complex128, self.state_count, "alpha"),
            _ptr(out, torch.float64, None, "grid_out")), self._h)
        res, off = [], 0
        for nl, sz in zip(self.nlat, sizes):
            res.append(out[off:off + sz].view(3, nl, 2 * nl))
            off += sz
        return res

    def inertial_manifold(self, alpha_src, n_src: int, N1: int, forcing=None, out=None):
        """phi = (nu A + C)^-1 (P_N' - P_N1)[f - B(u1, u1)], u1 = P_N1 u (eq. (eq:p-p));
        alpha_src holds every member at truncation n_src."""
        import torch
        if out is None:
            out = self.new_state()
        nsrc = len(self.member_specs) * coeff_count(n_src)
        _check(lib().nse_inertial_manifold(
            self._handle(), _ptr(alpha_src, torch.complex128, nsrc, "alpha_src"), int(n_src),
            int(N1), _ptr(forcing, torch.complex128, self.state_count, "forcing"),
            _ptr(out, torch.complex128, self.state_count, "phi_out")), self._h)
        return out

    # -- adaptive integration ------------------------------------------------------
    def adaptive_begin(self, alpha0, t0: float = 0.0, rtol: float = 1e-3, atol: float = 1e-6,
                       h0: float = 0.0, hmax: float = 0.0, max_order: int = 5,
                       max_newton: int = 4, forcing=None):
        """Starts a variable-order, variable-step NDF integration at (t0, alpha0).

        forcing: None (zero), a state tensor (constant in time), a callable
        t -> state tensor (evaluated on the context stream at every time level), a
        pair (state tensor F, callable t -> float s) for f(t) = s(t) F, or a pair
        (F, ForcingSchedule) whose scale the device evaluates. Without a callback
        the step and order control runs on the device.
        """
        import torch
        self._ad_error = None
        fn = FORCING_FN()

        def guarded(body):
            def cb(_user, t):
                try:
                    return body(float(t))
                except BaseException as e:  # re-raised after the library call returns
                    if self._ad_error is None:
                        self._ad_error = e
                    return 0.0
            return FORCING_FN(cb)

        p = AdaptiveParams(float(rtol), float(atol), float(h0), float(hmax), int(max_order),
                           int(max_newton))
        a0 = _ptr(alpha0, torch.complex128, self.state_count, "alpha0")
        if isinstance(forcing, tuple) and isinstance(forcing[1], ForcingSchedule):
            self._ad_fbuf, sched = forcing
            self._ad_fn = None
            fptr = _ptr(self._ad_fbuf, torch.complex128, self.state_count, "forcing")
            _check(lib().nse_adaptive_begin_scheduled(self._handle(), a0, float(t0),
                                                      ctypes.byref(p), fptr,
                                                      ctypes.byref(sched)), self._h)
            return
        if isinstance(forcing, tuple):
            self._ad_fbuf, scale = forcing
            fn = guarded(lambda t: float(scale(t)))
            fptr = _ptr(self._ad_fbuf, torch.complex128, self.state_count, "forcing")
        elif callable(forcing):
            self._ad_fbuf = self.new_state()
            f = forcing

            def refresh(t):
                with torch.cuda.stream(self.stream):
                    self._ad_fbuf.copy_(f(t))
                return 1.0

            fn = guarded(refresh)
            fptr = _ptr(self._ad_fbuf, torch.complex128, self.state_count, "forcing")
        else:
            self._ad_fbuf = forcing
            fptr = _ptr(forcing, torch.complex128, self.state_count, "forcing")
        self._ad_fn = fn  # the library keeps the pointer
        st = lib().nse_adaptive_begin(self._handle(), a0, float(t0), ctypes.byref(p), fptr, fn,
                                      None)
        self._raise_callback_error()
        _check(st, self._h)

    def _raise_callback_error(self):
        e, self._ad_error = getattr(self, "_ad_error", None), None
        if e is not None:
            raise e

    def adaptive_advance(self, t_end: float, out=None):
        """Integrates to t_end (exactly); returns (alpha(t_end), stats dict)."""
        import torch
        if out is None:
            out = self.new_state()
        stats = AdaptiveStats()
        st = lib().nse_adaptive_advance(
            self._handle(), float(t_end), _ptr(out, torch.complex128, self.state_count, "alpha_out"),
            ctypes.byref(stats))
        self._raise_callback_error()
        _check(st, self._h)
        return out, stats.as_dict()

    def adaptive_log(self):
        """[(t, h, order, sweeps, outcome, err)] of every attempt since adaptive_begin."""
        n = ctypes.c_int64()
        _check(lib().nse_adaptive_log(self._handle(), None, 0, ctypes.byref(n)), self._h)
        buf = (AdaptiveRecord * max(1, n.value))()
        _check(lib().nse_adaptive_log(self._handle(), buf, n.value, ctypes.byref(n)), self._h)
        return [(r.t, r.h, r.order, r.sweeps, r.outcome, r.err) for r in buf[:n.value]]

    def profile(self, enable: bool = True, repeat: int = 1):
        """Starts (or stops) per-kernel event timing on the context stream; each
        launch is issued `repeat` times between its events (same results)."""
        _check(lib().nse_profile_enable(self._handle(), int(repeat) if enable else 0), self._h)

    def profile_read(self):
        """{kernel: (launches, total_ms)} since the last read; resets the counters."""
        out = {}
        for name, kind in KERNEL_KINDS.items():
            n = ctypes.c_int64()
            ms = ctypes.c_double()
            _check(lib().nse_profile_read(self._handle(), kind, ctypes.byref(n), ctypes.byref(ms)),
                   self._h)
            out[name] = (int(n.value), float(ms.value))
        return out

    def sync(self):
        _check(lib().nse_sync(self._handle()), self._h)

    def close(self):
        if getattr(self, "_h", None) is not None:
            lib().nse_sphere_destroy(self._h)
            self._h = None

    def __del__(self):
        try:
            self.close()
        except Exception:
            pass

    def member_slice(self, i: int):
        N = self.member_specs[i][0]
        return slice(self.offsets[i], self.offsets[i] + coeff_count(N))


def to_device(a, device="cuda"):
    """complex128 GPU tensor from a numpy array."""
    import torch
    return torch.as_tensor(a, dtype=torch.complex128).to(device).contiguous()
