"""ctypes marshalling for libba's C-ABI (include/ba.h).  Same names as the C
entry points, minus the ``ba_`` prefix.  Inputs and outputs are torch tensors
on the current HIP device; calls are enqueued on torch's current stream."""
from __future__ import annotations

import ctypes as ct
import os

import numpy as np
import torch

_HERE = os.path.dirname(os.path.abspath(__file__))
_LIB_PATH = os.path.join(_HERE, "libba.so")

MODE_MM = 0
MODE_COUPLED = 1
MODE_EXACT = 2
PREC_F64 = 0
PREC_F32 = 1

_STATUS = {0: "BA_OK", -1: "BA_E_ARG", -2: "BA_E_WORKSPACE", -3: "BA_E_HIP", -4: "BA_E_NOT_SPD",
           -5: "BA_E_UNSUPPORTED", -6: "BA_E_NOMEM", -7: "BA_E_BUDGET", -8: "BA_E_NOT_FOUND"}


class BAError(RuntimeError):
    def __init__(self, status: int, text: str):
        super().__init__(f"{_STATUS.get(status, status)}: {text}")
        self.status = status


class _Points(ct.Structure):
    _fields_ = [("n", ct.c_int64), ("x", ct.c_void_p), ("y", ct.c_void_p), ("z", ct.c_void_p),
                ("scan", ct.c_void_p), ("voxel", ct.c_void_p), ("n_scans", ct.c_int32), ("n_voxels", ct.c_int32)]


class _Sums(ct.Structure):
    _fields_ = [("n", ct.c_int64), ("voxel", ct.c_void_p), ("scan", ct.c_void_p), ("count", ct.c_void_p),
                ("sum", ct.c_void_p), ("sumsq", ct.c_void_p), ("n_scans", ct.c_int32), ("n_voxels", ct.c_int32)]


class _BuildOpts(ct.Structure):
    _fields_ = [("chunk_len", ct.c_int32), ("n_windows", ct.c_int32), ("scan_window", ct.c_void_p),
                ("precision", ct.c_int32), ("ref_poses", ct.c_void_p)]


class _Info(ct.Structure):
    _fields_ = [("n_points", ct.c_int64), ("n_clusters", ct.c_int64), ("n_voxels", ct.c_int32),
                ("n_scans", ct.c_int32), ("n_windows", ct.c_int32), ("max_m", ct.c_int32),
                ("device_bytes", ct.c_int64), ("n_wave_groups", ct.c_int32), ("n_pose_chunks", ct.c_int32),
                ("padded_clusters", ct.c_int64), ("precision", ct.c_int32), ("cluster_bytes", ct.c_int32)]


class _LMOpts(ct.Structure):
    _fields_ = [("mode", ct.c_int32), ("max_iters", ct.c_int32), ("mu0", ct.c_double), ("nu0", ct.c_double),
                ("tol_g", ct.c_double), ("max_rejects", ct.c_int32), ("rejects0", ct.c_int32),
                ("exact_below", ct.c_double), ("resume", ct.c_void_p)]


class _Tuning(ct.Structure):
    _fields_ = [("vox_split", ct.c_int32), ("vox_grid", ct.c_int32), ("pose_grid", ct.c_int32),
                ("chunk_len", ct.c_int32)]


class _ServerOpts(ct.Structure):
    _fields_ = [("hbm_budget", ct.c_int64), ("slots", ct.c_int32), ("precision", ct.c_int32),
                ("lm", _LMOpts), ("iters_per_check", ct.c_int32), ("batch", ct.c_int32)]


class _Request(ct.Structure):
    _fields_ = [("n", ct.c_int64), ("voxel", ct.c_void_p), ("scan", ct.c_void_p), ("count", ct.c_void_p),
                ("sum", ct.c_void_p), ("sumsq", ct.c_void_p), ("n_scans", ct.c_int32), ("n_voxels", ct.c_int32),
                ("poses_init", ct.c_void_p)]


class _LMReport(ct.Structure):
    _fields_ = [("iters", ct.c_int32), ("n_accepted", ct.c_int32), ("converged", ct.c_int32),
                ("last_info", ct.c_int32), ("cost_initial", ct.c_double), ("cost_final", ct.c_double),
                ("gnorm_final", ct.c_double), ("mu_final", ct.c_double), ("stalled", ct.c_int32),
                ("rejects_final", ct.c_int32), ("nu_final", ct.c_double)]


class _ReqStatus(ct.Structure):
    _fields_ = [("state", ct.c_int32), ("status", ct.c_int32), ("t_submit", ct.c_double), ("t_admit", ct.c_double),
                ("t_done", ct.c_double), ("footprint", ct.c_int64), ("report", _LMReport)]


_lib = None


VOXEL_MAX_LEVELS = 16


class _VoxOpts(ct.Structure):
    _fields_ = [("d", ct.c_double), ("levels", ct.c_int32), ("min_scans", ct.c_int32), ("tau", ct.c_double)]


class _StreamOpts(ct.Structure):
    _fields_ = [("alpha", ct.c_double), ("batch_points", ct.c_int64)]


class _VoxInfo(ct.Structure):
    _fields_ = [("n_points", ct.c_int64), ("n_clusters", ct.c_int64), ("n_voxels", ct.c_int32),
                ("levels", ct.c_int32), ("n_scans", ct.c_int32), ("n_batches", ct.c_int32),
                ("level_voxels", ct.c_int64 * VOXEL_MAX_LEVELS), ("level_clusters", ct.c_int64 * VOXEL_MAX_LEVELS),
                ("level_kept_voxels", ct.c_int64 * VOXEL_MAX_LEVELS),
                ("level_kept_clusters", ct.c_int64 * VOXEL_MAX_LEVELS), ("device_bytes", ct.c_int64)]


def lib_path() -> str:
    return _LIB_PATH


def load():
    """Load libba; raises if it has not been built."""
    global _lib
    if _lib is not None:
        return _lib
    if not os.path.exists(_LIB_PATH):
        raise RuntimeError(f"libba is not built ({_LIB_PATH} missing); run "
                           "`python -m paper_2608_14266_amd.build`")
    L = ct.CDLL(_LIB_PATH)
    P, i32, i64, dbl, sz = ct.c_void_p, ct.c_int32, ct.c_int64, ct.c_double, ct.c_size_t
    L.ba_status_str.restype = ct.c_char_p
    L.ba_status_str.argtypes = [i32]
    L.ba_last_error.restype = ct.c_char_p
    L.ba_last_error.argtypes = []
    L.ba_build_clusters.restype = i32
    L.ba_build_clusters.argtypes = [ct.POINTER(_Points), ct.POINTER(_BuildOpts), ct.POINTER(P), P]
    L.ba_build_clusters_from_sums.restype = i32
    L.ba_build_clusters_from_sums.argtypes = [ct.POINTER(_Sums), ct.POINTER(_BuildOpts), ct.POINTER(P), P]
    L.ba_problem_destroy.restype = i32
    L.ba_problem_destroy.argtypes = [P]
    L.ba_problem_get_info.restype = i32
    L.ba_problem_get_info.argtypes = [P, ct.POINTER(_Info)]
    L.ba_problem_export_clusters.restype = i32
    L.ba_problem_export_clusters.argtypes = [P, P, P, P, P, P, P]
    L.ba_eval_residual_grad_hessian.restype = i32
    L.ba_eval_residual_grad_hessian.argtypes = [P, P, i32, P, P, P, P, P]
    L.ba_solve_increment_workspace.restype = sz
    L.ba_solve_increment_workspace.argtypes = [i32, i32]
    L.ba_solve_increment.restype = i32
    L.ba_solve_increment.argtypes = [i32, i32, P, P, dbl, P, P, P, sz, P]
    L.ba_solve_increment_noalloc.restype = i32
    L.ba_solve_increment_noalloc.argtypes = [i32, i32, P, P, dbl, P, P, P]
    L.ba_profile_enable.restype = i32
    L.ba_profile_enable.argtypes = [i32]
    L.ba_profile_reset.restype = i32
    L.ba_profile_reset.argtypes = []
    L.ba_profile_query.restype = i32
    L.ba_profile_query.argtypes = [ct.c_char_p, ct.POINTER(ct.c_double), ct.POINTER(ct.c_int64)]
    L.ba_iterate.restype = i32
    L.ba_iterate.argtypes = [P, P, ct.POINTER(_LMOpts), ct.POINTER(_LMReport), P, P]
    L.ba_problem_get_tuning.restype = i32
    L.ba_problem_get_tuning.argtypes = [P, ct.POINTER(_Tuning)]
    L.ba_problem_set_tuning.restype = i32
    L.ba_problem_set_tuning.argtypes = [P, ct.POINTER(_Tuning)]
    L.ba_autotune.restype = i32
    L.ba_autotune.argtypes = [P, P, i32, ct.POINTER(_Tuning), P]
    L.ba_request_footprint.restype = i32
    L.ba_request_footprint.argtypes = [ct.POINTER(_Request), i32, i32, ct.POINTER(ct.c_int64)]
    L.ba_server_create.restype = i32
    L.ba_server_create.argtypes = [ct.POINTER(_ServerOpts), ct.POINTER(P)]
    L.ba_server_submit.restype = i32
    L.ba_server_submit.argtypes = [P, ct.POINTER(_Request), ct.POINTER(ct.c_int64)]
    L.ba_server_query.restype = i32
    L.ba_server_query.argtypes = [P, ct.c_int64, ct.POINTER(_ReqStatus)]
    L.ba_server_wait.restype = i32
    L.ba_server_wait.argtypes = [P, ct.c_int64, P, ct.POINTER(_ReqStatus)]
    L.ba_server_cancel.restype = i32
    L.ba_server_cancel.argtypes = [P, ct.c_int64]
    L.ba_server_destroy.restype = i32
    L.ba_server_destroy.argtypes = [P]
    L.ba_voxelize.restype = i32
    L.ba_voxelize.argtypes = [P, P, P, P, ct.c_int64, i32, P, ct.POINTER(_VoxOpts), ct.POINTER(P), P]
    L.ba_voxelize_host.restype = i32
    L.ba_voxelize_host.argtypes = [P, P, P, P, ct.c_int64, i32, P, ct.POINTER(_VoxOpts), ct.POINTER(_StreamOpts),
                                   ct.POINTER(P), P]
    L.ba_voxel_map_get_info.restype = i32
    L.ba_voxel_map_get_info.argtypes = [P, ct.POINTER(_VoxInfo)]
    L.ba_voxel_map_export.restype = i32
    L.ba_voxel_map_export.argtypes = [P, P, P, P, P, P, P, P, P]
    L.ba_voxel_map_destroy.restype = i32
    L.ba_voxel_map_destroy.argtypes = [P]
    L.ba_release_cached_memory.restype = i32
    L.ba_release_cached_memory.argtypes = []
    _lib = L
    return L


def _check(st: int):
    if st != 0:
        raise BAError(st, load().ba_last_error().decode(errors="replace"))


def _stream():
    return ct.c_void_p(torch.cuda.current_stream().cuda_stream)


def _dev(t: torch.Tensor, dtype, name: str) -> torch.Tensor:
    if not isinstance(t, torch.Tensor) or not t.is_cuda:
        raise TypeError(f"{name} must be a device tensor")
    if t.dtype != dtype:
        raise TypeError(f"{name} must be {dtype}, got {t.dtype}")
    return t.contiguous()


def _ptr(t):
    return ct.c_void_p(t.data_ptr()) if t is not None else ct.c_void_p(0)


class Problem:
    """A device-resident problem built by :func:`build_clusters`."""

    def __init__(self, handle: ct.c_void_p, n_voxels_input: int):
        self._h = handle
        self.n_voxels_input = int(n_voxels_input)

    @property
    def handle(self):
        return self._h

    def info(self) -> dict:
        inf = _Info()
        _check(load().ba_problem_get_info(self._h, ct.byref(inf)))
        return {k: getattr(inf, k) for k, _ in _Info._fields_}

    def export_clusters(self):
        """(voxel, scan, count, mu (C,3), S (C,6)) sorted by (voxel, scan)."""
        C = self.info()["n_clusters"]
        dev = torch.cuda.current_device()
        vox = torch.empty(C, dtype=torch.int32, device=dev)
        scan = torch.empty(C, dtype=torch.int32, device=dev)
        cnt = torch.empty(C, dtype=torch.float64, device=dev)
        mu = torch.empty((C, 3), dtype=torch.float64, device=dev)
        S = torch.empty((C, 6), dtype=torch.float64, device=dev)
        _check(load().ba_problem_export_clusters(self._h, _ptr(vox), _ptr(scan), _ptr(cnt), _ptr(mu), _ptr(S),
                                                 _stream()))
        return vox, scan, cnt, mu, S

    def close(self):
        if self._h:
            load().ba_problem_destroy(self._h)
            self._h = None

    def __del__(self):
        try:
            self.close()
        except Exception:
            pass


def _opts(chunk_len, n_windows, scan_window, precision=PREC_F64, ref_poses=None):
    o = _BuildOpts()
    o.chunk_len = int(chunk_len)
    o.n_windows = int(n_windows)
    keep = []
    if scan_window is not None:
        sw = np.ascontiguousarray(np.asarray(scan_window, dtype=np.int32))
        keep.append(sw)
        o.scan_window = sw.ctypes.data_as(ct.c_void_p)
    else:
        o.scan_window = None
    o.precision = int(precision)
    if ref_poses is not None:
        rp = _dev(ref_poses, torch.float64, "ref_poses")
        keep.append(rp)
        o.ref_poses = rp.data_ptr()
    else:
        o.ref_poses = None
    return o, keep


def build_clusters(x, y, z, scan, voxel, n_scans: int, n_voxels: int, chunk_len: int = 0, n_windows: int = 1,
                   scan_window=None, precision: int = PREC_F64, ref_poses=None) -> Problem:
    """ba_build_clusters: points (device tensors) -> problem.  Synchronous.
    precision=PREC_F32 builds the precision form; ref_poses (device [n_scans, 12])
    then place the per-voxel reference points."""
    x = _dev(x, torch.float64, "x"); y = _dev(y, torch.float64, "y"); z = _dev(z, torch.float64, "z")
    scan = _dev(scan, torch.int32, "scan"); voxel = _dev(voxel, torch.int32, "voxel")
    n = x.numel()
    if not (y.numel() == n and z.numel() == n and scan.numel() == n and voxel.numel() == n):
        raise ValueError("point arrays must have equal length")
    p = _Points(n, x.data_ptr(), y.data_ptr(), z.data_ptr(), scan.data_ptr(), voxel.data_ptr(), int(n_scans),
                int(n_voxels))
    o, keep = _opts(chunk_len, n_windows, scan_window, precision, ref_poses)
    h = ct.c_void_p()
    _check(load().ba_build_clusters(ct.byref(p), ct.byref(o), ct.byref(h), _stream()))
    return Problem(h, n_voxels)


def build_clusters_from_sums(voxel, scan, count, sums, sumsq, n_scans: int, n_voxels: int, chunk_len: int = 0,
                             n_windows: int = 1, scan_window=None, precision: int = PREC_F64,
                             ref_poses=None) -> Problem:
    """ba_build_clusters_from_sums: raw-sum clusters (device tensors) -> problem.  Synchronous."""
    voxel = _dev(voxel, torch.int32, "voxel"); scan = _dev(scan, torch.int32, "scan")
    count = _dev(count, torch.int64, "count")
    sums = _dev(sums, torch.float64, "sum"); sumsq = _dev(sumsq, torch.float64, "sumsq")
    n = voxel.numel()
    if not (scan.numel() == n and count.numel() == n and sums.numel() == 3 * n and sumsq.numel() == 6 * n):
        raise ValueError("cluster arrays have inconsistent sizes")
    s = _Sums(n, voxel.data_ptr(), scan.data_ptr(), count.data_ptr(), sums.data_ptr(), sumsq.data_ptr(),
              int(n_scans), int(n_voxels))
    o, keep = _opts(chunk_len, n_windows, scan_window, precision, ref_poses)
    h = ct.c_void_p()
    _check(load().ba_build_clusters_from_sums(ct.byref(s), ct.byref(o), ct.byref(h), _stream()))
    return Problem(h, n_voxels)


def eval_residual_grad_hessian(problem: Problem, poses, mode: int = MODE_MM, derivatives: bool = True,
                               voxel_eig: bool = False):
    """ba_eval_residual_grad_hessian.  Returns (cost[n_windows], grad (N,6) or None,
    hess ((N,6,6) for MM, dense per-window for COUPLED and EXACT) or None, eig (V_in,4) or None)."""
    poses = _dev(poses, torch.float64, "poses")
    inf = problem.info()
    N, W = inf["n_scans"], inf["n_windows"]
    if poses.numel() != 12 * N:
        raise ValueError("poses must hold 12 doubles per scan")
    dev = poses.device
    cost = torch.empty(W, dtype=torch.float64, device=dev)
    grad = hess = eig = None
    if derivatives:
        grad = torch.empty((N, 6), dtype=torch.float64, device=dev)
        if mode == MODE_MM:
            hess = torch.empty((N, 6, 6), dtype=torch.float64, device=dev)
        else:
            if W != 1:
                raise ValueError("dense coupled Hessian export supports one window")
            hess = torch.empty((6 * N, 6 * N), dtype=torch.float64, device=dev)
    if voxel_eig:
        eig = torch.full((problem.n_voxels_input, 4), float("nan"), dtype=torch.float64, device=dev)
    _check(load().ba_eval_residual_grad_hessian(problem.handle, _ptr(poses), int(mode), _ptr(cost), _ptr(grad),
                                                _ptr(hess), _ptr(eig), _stream()))
    return cost, grad, hess, eig


def solve_increment_workspace(mode: int, n_scans: int) -> int:
    return int(load().ba_solve_increment_workspace(int(mode), int(n_scans)))


def _solve_scans(mode: int, hess, grad) -> int:
    """Number of scans of an increment solve, checked against both operands:
    grad holds 6 N values, hess N 6x6 blocks (MM) or the (6N)^2 matrix."""
    if grad.numel() == 0 or grad.numel() % 6:
        raise ValueError(f"grad must hold 6 values per scan, got {grad.numel()}")
    N = grad.numel() // 6
    want = 36 * N if int(mode) == MODE_MM else (6 * N) ** 2
    if hess.numel() != want:
        raise ValueError(f"hess must hold {want} values for {N} scans in mode {int(mode)}, got {hess.numel()}")
    return N


def solve_increment_noalloc(mode: int, hess, grad, mu: float):
    """ba_solve_increment_noalloc: the same solve with the library's static
    device scratch as workspace (no device allocation by the library).
    Returns (dx (N,6), info (int32 device scalar))."""
    hess = _dev(hess, torch.float64, "hess"); grad = _dev(grad, torch.float64, "grad")
    N = _solve_scans(mode, hess, grad)
    dev = grad.device
    dx = torch.empty((N, 6), dtype=torch.float64, device=dev)
    info = torch.empty(1, dtype=torch.int32, device=dev)
    _check(load().ba_solve_increment_noalloc(int(mode), N, _ptr(hess), _ptr(grad), float(mu), _ptr(dx), _ptr(info),
                                             _stream()))
    return dx, info


def solve_increment(mode: int, hess, grad, mu: float):
    """ba_solve_increment: returns (dx (N,6), info (int32 device scalar))."""
    hess = _dev(hess, torch.float64, "hess"); grad = _dev(grad, torch.float64, "grad")
    N = _solve_scans(mode, hess, grad)
    dev = grad.device
    dx = torch.empty((N, 6), dtype=torch.float64, device=dev)
    info = torch.empty(1, dtype=torch.int32, device=dev)
    wsb = solve_increment_workspace(mode, N)
    ws = torch.empty(max(wsb, 1), dtype=torch.uint8, device=dev)
    _check(load().ba_solve_increment(int(mode), N, _ptr(hess), _ptr(grad), float(mu), _ptr(dx), _ptr(info),
                                     _ptr(ws), wsb, _stream()))
    return dx, info


def iterate(problem: Problem, poses, mode: int = MODE_MM, max_iters: int = 10, mu0: float = 1e-2,
            nu0: float = 2.0, tol_g: float = 0.0, trace: bool = True, max_rejects: int = 0,
            exact_below: float = 0.0, rejects0: int = 0, resume=None):
    """ba_iterate: LM on the device, poses updated in place.  Synchronous.
    resume: None, or per window (mu0, nu0, rejects0, skip) as an (n_windows, 4)
    array (a window's earlier report's mu_final, nu_final, rejects_final).
    Returns (reports: list of dicts per window, trace ndarray (iters, W, 8) or None)."""
    if not (poses.is_cuda and poses.dtype == torch.float64 and poses.is_contiguous()):
        raise TypeError("poses must be a contiguous float64 device tensor (updated in place)")
    W = problem.info()["n_windows"]
    o = _LMOpts(int(mode), int(max_iters), float(mu0), float(nu0), float(tol_g), int(max_rejects), int(rejects0),
                float(exact_below))
    if resume is not None:
        resume = np.ascontiguousarray(resume, dtype=np.float64)
        if resume.shape != (W, 4):
            raise ValueError(f"resume must be ({W}, 4), got {resume.shape}")
        o.resume = resume.ctypes.data_as(ct.c_void_p)
    reps = (_LMReport * W)()
    tr = np.zeros((max(int(max_iters), 1), W, 8)) if trace else None
    trp = tr.ctypes.data_as(ct.c_void_p) if trace else ct.c_void_p(0)
    _check(load().ba_iterate(problem.handle, _ptr(poses), ct.byref(o), reps, trp, _stream()))
    out = [{k: getattr(r, k) for k, _ in _LMReport._fields_} for r in reps]
    return out, (tr[: int(max_iters)] if trace else None)


def release_cached_memory():
    """ba_release_cached_memory: return the device and pinned memory the library
    keeps between calls to the driver."""
    _check(load().ba_release_cached_memory())


def profile_enable(on: bool = True):
    """ba_profile_enable: time later launches of the eval kernels with HIP events."""
    _check(load().ba_profile_enable(1 if on else 0))


def profile_reset():
    _check(load().ba_profile_reset())


def profile_query(kernel: str):
    """ba_profile_query: (total milliseconds, launches) of one kernel ("k_vox", "k_pose")."""
    ms = ct.c_double(0.0)
    n = ct.c_int64(0)
    _check(load().ba_profile_query(kernel.encode(), ct.byref(ms), ct.byref(n)))
    return ms.value, n.value


def problem_get_tuning(problem) -> dict:
    """ba_problem_get_tuning: the problem's launch choices."""
    t = _Tuning()
    _check(load().ba_problem_get_tuning(problem.handle, ct.byref(t)))
    return {k: getattr(t, k) for k, _ in _Tuning._fields_}


def problem_set_tuning(problem, tuning: dict):
    """ba_problem_set_tuning (synchronous)."""
    cur = problem_get_tuning(problem)
    cur.update({k: int(v) for k, v in tuning.items()})
    t = _Tuning(**cur)
    _check(load().ba_problem_set_tuning(problem.handle, ct.byref(t)))


def autotune(problem, poses, reps: int = 5) -> dict:
    """ba_autotune: time every launch choice at `poses`, apply and return the best."""
    poses = _dev(poses, torch.float64, "poses")
    t = _Tuning()
    _check(load().ba_autotune(problem.handle, _ptr(poses), int(reps), ct.byref(t), _stream()))
    return {k: getattr(t, k) for k, _ in _Tuning._fields_}


REQ_QUEUED, REQ_RUNNING, REQ_DONE, REQ_FAILED, REQ_CANCELLED = 0, 1, 2, 3, 4


def _request(voxel, scan, count, sums, sumsq, n_scans, n_voxels, poses_init):
    keep = [np.ascontiguousarray(voxel, dtype=np.int32), np.ascontiguousarray(scan, dtype=np.int32),
            np.ascontiguousarray(count, dtype=np.int64), np.ascontiguousarray(sums, dtype=np.float64),
            np.ascontiguousarray(sumsq, dtype=np.float64), np.ascontiguousarray(poses_init, dtype=np.float64)]
    n = keep[0].shape[0]
    if not (keep[1].shape[0] == n and keep[2].shape[0] == n and keep[3].size == 3 * n and keep[4].size == 6 * n
            and keep[5].size == 12 * int(n_scans)):
        raise ValueError("request arrays have inconsistent sizes")
    r = _Request(n, *[k.ctypes.data for k in keep[:5]], int(n_scans), int(n_voxels), keep[5].ctypes.data)
    return r, keep


def _status_dict(st: "_ReqStatus") -> dict:
    d = {k: getattr(st, k) for k, _ in _ReqStatus._fields_ if k != "report"}
    d["report"] = {k: getattr(st.report, k) for k, _ in _LMReport._fields_}
    return d


def request_footprint(voxel, scan, count, sums, sumsq, n_scans, n_voxels, poses_init, mode=MODE_MM,
                      precision=PREC_F64) -> int:
    """ba_request_footprint: device bytes reserved for a request (host arrays)."""
    r, keep = _request(voxel, scan, count, sums, sumsq, n_scans, n_voxels, poses_init)
    b = ct.c_int64(0)
    _check(load().ba_request_footprint(ct.byref(r), int(mode), int(precision), ct.byref(b)))
    return b.value


class Server:
    """ba_server_*: the served form.  Requests are host arrays of raw-sum
    clusters; results are host poses and an LM report."""

    def __init__(self, hbm_budget: int, slots: int = 4, precision: int = PREC_F64, mode: int = MODE_MM,
                 max_iters: int = 50, tol_g: float = 1e-6, mu0: float = 0.0, nu0: float = 0.0,
                 max_rejects: int = 10, iters_per_check: int = 0, batch: int = 0):
        o = _ServerOpts()
        o.hbm_budget = int(hbm_budget)
        o.slots = int(slots)
        o.precision = int(precision)
        o.lm = _LMOpts(int(mode), int(max_iters), float(mu0), float(nu0), float(tol_g), int(max_rejects), 0)
        o.iters_per_check = int(iters_per_check)
        o.batch = int(batch)
        h = ct.c_void_p()
        _check(load().ba_server_create(ct.byref(o), ct.byref(h)))
        self._h = h
        self._n_scans = {}

    def submit(self, voxel, scan, count, sums, sumsq, n_scans, n_voxels, poses_init) -> int:
        r, keep = _request(voxel, scan, count, sums, sumsq, n_scans, n_voxels, poses_init)
        rid = ct.c_int64(0)
        _check(load().ba_server_submit(self._h, ct.byref(r), ct.byref(rid)))
        self._n_scans[rid.value] = int(n_scans)
        return rid.value

    def submit_scene(self, sc) -> int:
        return self.submit(sc.voxel, sc.scan, sc.count, sc.sum, sc.sumsq, sc.n_scans, sc.n_voxels, sc.poses_init)

    def query(self, rid: int) -> dict:
        st = _ReqStatus()
        _check(load().ba_server_query(self._h, int(rid), ct.byref(st)))
        return _status_dict(st)

    def cancel(self, rid: int):
        """ba_server_cancel: stop request `rid` (queued: at once; running: at its
        next check).  wait() then raises BAError with status -9."""
        _check(load().ba_server_cancel(self._h, int(rid)))

    def wait_any(self, rid: int):
        """Like wait(), but a cancelled request returns (poses reached, status)
        instead of raising."""
        poses = np.empty((self._n_scans[rid], 12))
        st = _ReqStatus()
        rc = load().ba_server_wait(self._h, int(rid), poses.ctypes.data_as(ct.c_void_p), ct.byref(st))
        del self._n_scans[rid]
        if rc not in (0, -9):
            _check(rc)
        return poses, _status_dict(st)

    def wait(self, rid: int):
        """Block until request `rid` is done: (poses (n_scans, 12), status dict)."""
        poses = np.empty((self._n_scans[rid], 12))
        st = _ReqStatus()
        _check(load().ba_server_wait(self._h, int(rid), poses.ctypes.data_as(ct.c_void_p), ct.byref(st)))
        del self._n_scans[rid]
        return poses, _status_dict(st)

    def close(self):
        if getattr(self, "_h", None):
            _check(load().ba_server_destroy(self._h))
            self._h = None

    def __enter__(self):
        return self

    def __exit__(self, *a):
        self.close()

    def __del__(self):
        try:
            self.close()
        except Exception:
            pass


# ---------------------------------------------------------------- voxelization
class VoxelMap:
    """Kept planar cells of a multi-level voxelization (:func:`voxelize`)."""

    def __init__(self, handle: ct.c_void_p):
        self._h = handle

    def info(self) -> dict:
        inf = _VoxInfo()
        _check(load().ba_voxel_map_get_info(self._h, ct.byref(inf)))
        L = inf.levels
        return {"n_points": inf.n_points, "n_clusters": inf.n_clusters, "n_voxels": inf.n_voxels, "levels": L,
                "n_scans": inf.n_scans, "n_batches": inf.n_batches, "level_voxels": list(inf.level_voxels[:L]),
                "level_clusters": list(inf.level_clusters[:L]), "level_kept_voxels": list(inf.level_kept_voxels[:L]),
                "level_kept_clusters": list(inf.level_kept_clusters[:L]), "device_bytes": inf.device_bytes}

    def export(self) -> dict:
        """voxel, scan (C,) int32; count (C,) int64; sum (C,3), sumsq (C,6) f64;
        voxel_level (V,) int32; voxel_cell (V,3) int32 -- device tensors."""
        inf = self.info()
        C, V = inf["n_clusters"], inf["n_voxels"]
        dev = torch.cuda.current_device()
        out = {"voxel": torch.empty(C, dtype=torch.int32, device=dev),
               "scan": torch.empty(C, dtype=torch.int32, device=dev),
               "count": torch.empty(C, dtype=torch.int64, device=dev),
               "sum": torch.empty((C, 3), dtype=torch.float64, device=dev),
               "sumsq": torch.empty((C, 6), dtype=torch.float64, device=dev),
               "voxel_level": torch.empty(V, dtype=torch.int32, device=dev),
               "voxel_cell": torch.empty((V, 3), dtype=torch.int32, device=dev)}
        o = out
        _check(load().ba_voxel_map_export(self._h, _ptr(o["voxel"]), _ptr(o["scan"]), _ptr(o["count"]),
                                          _ptr(o["sum"]), _ptr(o["sumsq"]), _ptr(o["voxel_level"]),
                                          _ptr(o["voxel_cell"]), _stream()))
        return out

    def close(self):
        if self._h:
            load().ba_voxel_map_destroy(self._h)
            self._h = None

    def __del__(self):
        try:
            self.close()
        except Exception:
            pass


def voxelize(x, y, z, scan, poses, d: float, levels: int, tau: float, min_scans: int = 1,
             n_scans: int | None = None) -> VoxelMap:
    """ba_voxelize: body-frame points (device tensors) at the poses -> kept
    planar cells of every level.  Synchronous."""
    x = _dev(x, torch.float64, "x"); y = _dev(y, torch.float64, "y"); z = _dev(z, torch.float64, "z")
    scan = _dev(scan, torch.int32, "scan")
    poses = _dev(poses, torch.float64, "poses")
    n = x.numel()
    if not (y.numel() == n and z.numel() == n and scan.numel() == n):
        raise ValueError("point arrays have inconsistent sizes")
    N = poses.numel() // 12 if n_scans is None else int(n_scans)
    if poses.numel() != 12 * N:
        raise ValueError("poses must hold 12 doubles per scan")
    o = _VoxOpts(float(d), int(levels), int(min_scans), float(tau))
    h = ct.c_void_p()
    _check(load().ba_voxelize(_ptr(x), _ptr(y), _ptr(z), _ptr(scan), n, N, _ptr(poses), ct.byref(o), ct.byref(h),
                              _stream()))
    return VoxelMap(h)


def voxelize_host(x, y, z, scan, poses, d: float, levels: int, tau: float, min_scans: int = 1,
                  alpha: float = 0.5, batch_points: int = 0, n_scans: int | None = None) -> VoxelMap:
    """ba_voxelize_host: points in host memory (numpy arrays or CPU tensors,
    pinned or not) streamed to the device in batches, then the same
    voxelization as :func:`voxelize`.  Synchronous."""
    import numpy as np

    def host(a, dt, name):
        if isinstance(a, torch.Tensor):
            if a.is_cuda:
                raise TypeError(f"{name} must be in host memory")
            a = a.contiguous()
            if a.dtype != dt:
                raise TypeError(f"{name} must be {dt}")
            return a, a.data_ptr()
        npdt = {torch.float64: np.float64, torch.int32: np.int32}[dt]
        arr = np.ascontiguousarray(a, dtype=npdt)
        return arr, arr.ctypes.data
    xs, px = host(x, torch.float64, "x")
    ys, py = host(y, torch.float64, "y")
    zs, pz = host(z, torch.float64, "z")
    ss, ps = host(scan, torch.int32, "scan")
    n = len(xs)
    if not (len(ys) == n and len(zs) == n and len(ss) == n):
        raise ValueError("point arrays have inconsistent sizes")
    poses = _dev(poses, torch.float64, "poses")
    N = poses.numel() // 12 if n_scans is None else int(n_scans)
    o = _VoxOpts(float(d), int(levels), int(min_scans), float(tau))
    so = _StreamOpts(float(alpha), int(batch_points))
    h = ct.c_void_p()
    _check(load().ba_voxelize_host(ct.c_void_p(px), ct.c_void_p(py), ct.c_void_p(pz), ct.c_void_p(ps), n, N,
                                   _ptr(poses), ct.byref(o), ct.byref(so), ct.byref(h), _stream()))
    return VoxelMap(h)
