"""Workloads the framework's speed is measured on.

Each case is one call (or the short run of calls a program makes for one
window) through the public entry points of `paper_2608_14266_amd`, on inputs
drawn from a seed on the device:

  eval        cost, gradient and Hessian blocks at given poses
  iterate     a whole Levenberg-Marquardt run (MM or coupled form)
  solve       the damped increment of a given Hessian and gradient
  build       points or raw sums -> problem, its first residual, its clusters
  voxelize    unlabelled points -> planar voxels of every level (device or host)

Scenes follow two laws.  "loop": poses 4 m apart on a closed figure-eight,
every plane seen by a run of m poses around its anchor, m geometric(0.25) cut
at 20, 20-500 points per observation (the single-window and city workloads of
the benchmark).  "path": poses 2 m apart on a straight path, every plane seen
by 3-8 of the 16 poses nearest its anchor, 50 points per observation (the tiny
and the batch workloads).  Cluster sums are drawn from their sampling
distribution (mean normal, scatter Wishart by the Bartlett decomposition).
"""
import math

import torch

import paper_2608_14266_amd as ba

LOOP_P, LOOP_MAX = 0.25, 20
PATH_MIN, PATH_MAX, PATH_NEAR = 3, 8, 16
SIGMA = 0.03
MAP_CLUSTERS, MAP_VOXELS = 0.45, 0.22   # kept (cell, scan) clusters and cells per observation and level, at most


def listed():
    return [
        # the smallest call: one evaluation of a ten-scan window, where launches and host work are all of it
        {"name": "eval_tiny", "kind": "eval", "law": "path", "windows": 1, "poses": 10, "planes": 200, "f32": False,
         "derivatives": True},
        # the benchmark's single window, FP64: one evaluation of an optimizer outside the library
        {"name": "eval_window", "kind": "eval", "law": "loop", "windows": 1, "poses": 500, "planes": 200000,
         "f32": False, "derivatives": True},
        # city scale in the precision form
        {"name": "eval_city_f32", "kind": "eval", "law": "loop", "windows": 1, "poses": 2000, "planes": 1000000,
         "f32": True, "derivatives": True},
        # odometry: a small sliding window optimized again at every scan
        {"name": "iterate_tiny", "kind": "iterate", "law": "path", "windows": 1, "poses": 10, "planes": 200,
         "f32": False, "coupled": False, "iters": 10},
        # the benchmark's single window solved with the paper's MM form
        {"name": "iterate_window", "kind": "iterate", "law": "loop", "windows": 1, "poses": 500, "planes": 200000,
         "f32": False, "coupled": False, "iters": 20},
        # the benchmark's default: 256 windows of 20-400 poses, precision form, launch choices as the tuner caches them
        {"name": "iterate_batch_f32", "kind": "iterate", "law": "path", "windows": 256, "poses": 0, "planes": 0,
         "f32": True, "coupled": False, "iters": 10},
        # a served request in the coupled form (dense 3000 x 3000 systems)
        {"name": "iterate_coupled", "kind": "iterate", "law": "loop", "windows": 1, "poses": 500, "planes": 100000,
         "f32": False, "coupled": True, "iters": 5},
        # the largest dense system: 2000 scans, 12000 x 12000
        {"name": "solve_coupled", "kind": "solve", "coupled": True, "poses": 2000},
        # a labelled scan log turned into a problem
        {"name": "build_points", "kind": "build", "law": "loop", "windows": 1, "poses": 125, "planes": 50000,
         "f32": False, "points": True},
        # city scale from raw sums in the precision form
        {"name": "build_sums_f32", "kind": "build", "law": "loop", "windows": 1, "poses": 2000, "planes": 1000000,
         "f32": True, "points": False},
        # unlabelled points of a drive to planar voxels, three levels
        {"name": "voxelize", "kind": "voxelize", "poses": 500, "planes": 200000, "levels": 3, "host": False,
         "batches": 0},
        # the same from pageable host memory through the batched loader
        {"name": "voxelize_host", "kind": "voxelize", "poses": 60, "planes": 16001, "levels": 3, "host": True,
         "batches": 4},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["eval", "eval", "iterate", "iterate", "solve", "build", "build", "voxelize"])
    if kind == "solve":
        coupled = rng.random() < 0.6
        return {"kind": kind, "coupled": coupled, "poses": _log_int(rng, 5, 1900 if coupled else 20000)}
    if kind == "voxelize":
        host = rng.random() < 0.3
        n = _log_int(rng, 5, 100 if host else 400)
        return {"kind": kind, "poses": n, "planes": n * rng.randint(60, 250 if host else 450),
                "levels": rng.randint(1, 4), "host": host, "batches": rng.randint(1, 5) if host else 0}
    law = rng.choice(["loop", "path"])
    n = _log_int(rng, 7, 1900)
    windows = 1 if rng.random() < 0.6 else rng.randint(2, max(2, min(40, 1900 // n)))
    c = {"kind": kind, "law": law, "windows": windows, "poses": n, "planes": n * rng.randint(20, 500),
         "f32": rng.random() < 0.5}
    if windows > 1:
        c["planes"] = max(20, min(c["planes"], 950000 // windows))
    if kind == "eval":
        c["derivatives"] = rng.random() < 0.8
    elif kind == "iterate":
        c["coupled"] = windows == 1 and n <= 500 and rng.random() < 0.5
        c["iters"] = rng.randint(2, 5) if c["coupled"] else rng.randint(3, 15)
    else:
        c["points"] = windows == 1 and c["planes"] <= 50000 and rng.random() < 0.5
    return c


# ------------------------------------------------------------------ scenes
def _sizes(case):
    """Poses and planes of each window (the batch workload spreads them over 20-400 poses)."""
    W = case.get("windows", 1)
    if case["poses"]:
        return [case["poses"]] * W, [case["planes"]] * W
    n = [int(20 * 20 ** ((w + 0.5) / W)) for w in range(W)]
    return n, [min(80000, max(5000, 200 * k)) for k in n]


def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(0x5EED + int(seed))


def _rand(g, *shape):
    return torch.rand(*shape, generator=g, device="cuda", dtype=torch.float64)


def _randn(g, *shape):
    return torch.randn(*shape, generator=g, device="cuda", dtype=torch.float64)


def _quantiles(g, sizes):
    """(i + 1/2) / n, i < n, in random order within each part of n = sizes[w] values."""
    n = torch.repeat_interleave(sizes, sizes).cuda()
    part = torch.repeat_interleave(torch.arange(len(sizes), device=sizes.device), sizes).cuda()
    first = (torch.cumsum(sizes, 0) - sizes).cuda()
    i = torch.arange(len(n), device="cuda") - first[part]
    shuffled = torch.argsort(part + torch.rand(len(n), generator=g, device="cuda", dtype=torch.float64) * 0.999)
    return ((i + 0.5) / n)[shuffled]


def _rotations(a):
    """Rx(a0) Ry(a1) Rz(a2) of angle rows (n, 3)."""
    c, s = torch.cos(a), torch.sin(a)
    one, zero = torch.ones_like(c[:, 0]), torch.zeros_like(c[:, 0])
    rx = torch.stack([one, zero, zero, zero, c[:, 0], -s[:, 0], zero, s[:, 0], c[:, 0]], 1).view(-1, 3, 3)
    ry = torch.stack([c[:, 1], zero, s[:, 1], zero, one, zero, -s[:, 1], zero, c[:, 1]], 1).view(-1, 3, 3)
    rz = torch.stack([c[:, 2], -s[:, 2], zero, s[:, 2], c[:, 2], zero, zero, zero, one], 1).view(-1, 3, 3)
    mul = lambda p, q: (p[:, :, :, None] * q[:, None, :, :]).sum(2)  # noqa: E731
    return mul(mul(rx, ry), rz)


def _poses12(R, t):
    return torch.cat([R.reshape(-1, 9), t], 1).contiguous()


class _Scene:
    """Poses, planes and (voxel, scan) observations; voxel-major, scans rising."""

    def __init__(self, case, seed, loop):
        g = self.g = _generator(seed)
        n_w, v_w = _sizes(case)
        dev = "cuda"
        nw, vw = torch.tensor(n_w, device=dev), torch.tensor(v_w, device=dev)
        self.N, self.V, W = sum(n_w), sum(v_w), len(n_w)
        self.scan_window = torch.repeat_interleave(torch.arange(W), torch.tensor(n_w)).to(torch.int32).numpy()
        base = torch.cumsum(nw, 0) - nw
        win = torch.repeat_interleave(torch.arange(W, device=dev), nw)
        idx = (torch.arange(self.N, device=dev) - base[win]).double()
        if loop:
            th = 2 * math.pi * idx / nw[win]
            a = 4.0 * nw[win] / 6.1
            t = torch.stack([a * torch.sin(th), 0.5 * a * torch.sin(2 * th), torch.zeros_like(th)], 1)
        else:
            t = torch.stack([2.0 * idx, torch.zeros_like(idx), torch.zeros_like(idx)], 1)
        yaw = torch.zeros(self.N, 3, device=dev, dtype=torch.float64)
        yaw[:, 2] = 2 * math.pi * _rand(g, self.N)
        self.R, self.t = _rotations(yaw), t
        ang, off = (math.radians(1.0), 0.1) if loop else (math.radians(0.5), 0.05)

        def perturbed(scale):
            E = _rotations(scale * ang * (2 * _rand(g, self.N, 3) - 1))
            Rp = (E[:, :, :, None] * self.R[:, None, :, :]).sum(2)
            return _poses12(Rp, t + scale * off * (2 * _rand(g, self.N, 3) - 1))

        self.poses_init, self.poses_moved = perturbed(1.0), perturbed(0.5)
        vwin = torch.repeat_interleave(torch.arange(W, device=dev), vw)
        local = (_rand(g, self.V) * nw[vwin]).long().minimum(nw[vwin] - 1)
        d = _randn(g, self.V, 3)
        d = d / d.norm(dim=1, keepdim=True)
        self.centre = t[base[vwin] + local] + d * ((40.0 if loop else 30.0) * _rand(g, self.V, 1))
        nrm = _randn(g, self.V, 3)
        nrm = nrm / nrm.norm(dim=1, keepdim=True)
        ax = torch.zeros_like(nrm).scatter_(1, nrm.abs().argmin(1, keepdim=True), 1.0)
        e1 = torch.linalg.cross(nrm, ax)
        e1 = e1 / e1.norm(dim=1, keepdim=True)
        self.frame = torch.stack([e1, torch.linalg.cross(nrm, e1), nrm], 2)   # columns
        if loop:
            # the planes' observer counts are the law's quantiles in random order, so
            # the number of clusters is the case's and not the seed's
            m = (1 + torch.log(_quantiles(g, vw)) / math.log(1 - LOOP_P)).long()
            m = m.clamp(max=LOOP_MAX).minimum(nw[vwin])
            vox = torch.repeat_interleave(torch.arange(self.V, device=dev), m)
            k = torch.arange(vox.numel(), device=dev) - (torch.cumsum(m, 0) - m)[vox]
            obs = (local[vox] - m[vox] // 2 + k) % nw[vwin[vox]]
            order = torch.argsort(vox * (int(nw.max()) + 1) + obs)
            self.voxel, scan = vox[order], (base[vwin[vox]] + obs)[order]
        else:
            near = nw[vwin].clamp(max=PATH_NEAR)
            first = (local - PATH_NEAR // 2).clamp(min=0).minimum(nw[vwin] - near)
            m = (PATH_MIN + (PATH_MAX - PATH_MIN + 1) * _quantiles(g, vw)).long().clamp(max=PATH_MAX).minimum(near)
            r = torch.rand(self.V, PATH_NEAR, generator=g, device=dev)
            r = torch.where(torch.arange(PATH_NEAR, device=dev)[None] < near[:, None], r, 2.0)
            cut = torch.sort(r, 1).values.gather(1, (m - 1)[:, None])
            self.voxel, k = torch.nonzero(r <= cut, as_tuple=True)
            scan = base[vwin[self.voxel]] + first[self.voxel] + k
        self.scan = scan
        self.C = scan.numel()
        if loop:
            self.count = (20.0 * torch.exp(math.log(25.0) * _quantiles(g, torch.tensor([self.C])))).long()
        else:
            self.count = torch.full((self.C,), 50, device=dev, dtype=torch.int64)

    def sums(self):
        """Raw sums (voxel, scan, count, sum, sumsq) in the scans' body frames."""
        g, n = self.g, self.count.double()
        sd = torch.tensor([math.sqrt(1 / 12), math.sqrt(1 / 12), SIGMA], device="cuda", dtype=torch.float64)
        F, R = self.frame[self.voxel], self.R[self.scan]
        B = torch.empty(self.C, 3, 3, device="cuda", dtype=torch.float64)   # body axes of the plane frame: R^T F
        for i in range(3):
            for j in range(3):
                B[:, i, j] = R[:, 0, i] * F[:, 0, j] + R[:, 1, i] * F[:, 1, j] + R[:, 2, i] * F[:, 2, j]
        del F
        d = self.centre[self.voxel] - self.t[self.scan]
        mu = torch.stack([R[:, 0, i] * d[:, 0] + R[:, 1, i] * d[:, 1] + R[:, 2, i] * d[:, 2] for i in range(3)], 1)
        del R, d
        z = _randn(g, self.C, 3) * sd / n.sqrt()[:, None]
        for i in range(3):
            mu[:, i] += B[:, i, 0] * z[:, 0] + B[:, i, 1] * z[:, 1] + B[:, i, 2] * z[:, 2]

        def chi(df):   # square root of a chi-square (Wilson-Hilferty)
            return (df * (1 - 2 / (9 * df) + _randn(g, self.C) * torch.sqrt(2 / (9 * df))).clamp_min(0) ** 3).sqrt()
        w, q = _randn(g, self.C, 3), [None] * 6
        a00, a11, a22 = sd[0] * chi(n - 1), sd[1] * chi(n - 2), sd[2] * chi(n - 3)
        a10, a20, a21 = sd[1] * w[:, 0], sd[2] * w[:, 1], sd[2] * w[:, 2]
        L = [[B[:, i, 0] * a00 + B[:, i, 1] * a10 + B[:, i, 2] * a20, B[:, i, 1] * a11 + B[:, i, 2] * a21,
              B[:, i, 2] * a22] for i in range(3)]
        k = 0
        for i in range(3):
            for j in range(i, 3):
                q[k] = L[i][0] * L[j][0] + L[i][1] * L[j][1] + L[i][2] * L[j][2] + n * mu[:, i] * mu[:, j]
                k += 1
        return (self.voxel.int(), self.scan.int(), self.count, (mu * n[:, None]).contiguous(),
                torch.stack(q, 1).contiguous())

    def points(self):
        """Raw body-frame points, scan after scan (x, y, z, scan, voxel)."""
        g = self.g
        order = torch.argsort(self.scan * self.V + torch.randperm(self.V, generator=g, device="cuda")[self.voxel])
        c = torch.repeat_interleave(order, self.count[order])
        n = c.numel()
        v, s = self.voxel[c], self.scan[c]
        p = [_rand(g, n) - 0.5, _rand(g, n) - 0.5, SIGMA * _randn(g, n)]
        d = []
        for i in range(3):
            f = self.frame[:, i][v]
            d.append(self.centre[:, i][v] - self.t[:, i][s] + f[:, 0] * p[0] + f[:, 1] * p[1] + f[:, 2] * p[2])
        xyz = []
        for i in range(3):
            r = self.R[:, :, i][s]
            xyz.append(r[:, 0] * d[0] + r[:, 1] * d[1] + r[:, 2] * d[2])
        return xyz[0], xyz[1], xyz[2], s.int(), v.int()


def _build(s):
    f32 = ba.PREC_F32 if s["f32"] else ba.PREC_F64
    kw = {"precision": f32, "n_windows": s["W"], "scan_window": s["scan_window"] if s["W"] > 1 else None,
          "ref_poses": s["poses_init"] if s["f32"] else None}
    make = ba.build_clusters if s["points"] else ba.build_clusters_from_sums
    return make(*s["data"], s["N"], s["V"], **kw)


def _system(n, g):
    """A symmetric positive definite (6n)^2 matrix with the falling off of a pose
    graph's along the path (products of exponentials of pose distance and per-row
    scales), and a gradient."""
    rows = 6 * n
    scale = torch.exp(math.log(30.0) * _rand(g, rows)) * 10
    at = torch.arange(rows, device="cuda", dtype=torch.float64) / 6 + 0.3 * _rand(g, rows)
    at = torch.sort(at).values
    H = torch.exp(-(at[:, None] - at[None, :]).abs() / 8.0)
    H.diagonal().add_(0.5 + _rand(g, rows))
    H *= scale[:, None]
    H *= scale[None, :]
    return H, scale * _randn(g, rows)


def _blocks(n, g):
    """n 6x6 symmetric positive definite blocks and a gradient."""
    A = _randn(g, n, 6, 6) * torch.exp(2 * _rand(g, n, 6, 1))
    H = (A[:, :, None, :] * A[:, None, :, :]).sum(3)
    H.diagonal(dim1=1, dim2=2).add_(1.0)
    return H.contiguous(), _randn(g, n, 6)


def _map_buffers(C, levels):
    """A program's resident arrays for the kept cells, sized for the observations."""
    c, v = MAP_CLUSTERS * C * levels + 4096, MAP_VOXELS * C * levels + 4096
    new = lambda dt, *shape: torch.zeros(*[int(k) for k in shape], dtype=dt, device="cuda")  # noqa: E731
    return {"voxel": new(torch.int32, c), "scan": new(torch.int32, c), "count": new(torch.int64, c),
            "sum": new(torch.float64, c, 3), "sumsq": new(torch.float64, c, 6), "voxel_level": new(torch.int32, v),
            "voxel_cell": new(torch.int32, v, 3)}


def prepare(case, seed):
    kind = case["kind"]
    if kind == "solve":
        g = _generator(seed)
        H, b = _system(case["poses"], g) if case["coupled"] else _blocks(case["poses"], g)
        return {"kind": kind, "mode": ba.MODE_COUPLED if case["coupled"] else ba.MODE_MM, "H": H, "g": b}
    if kind == "voxelize":
        sc = _Scene({**case, "windows": 1}, seed, True)
        x, y, z, scan, _ = sc.points()
        s = {"kind": kind, "levels": case["levels"], "host": case["host"], "poses": sc.poses_init, "batch": 0}
        s["data"] = (x, y, z, scan)
        if case["host"]:
            s["data"] = tuple(a.cpu().numpy() for a in s["data"])
            s["batch"] = max(1024, -(-len(s["data"][0]) // case["batches"]))
        s["out"] = _map_buffers(sc.C, case["levels"])
        return s
    sc = _Scene(case, seed, case["law"] == "loop")
    s = {"kind": kind, "f32": case["f32"], "W": case["windows"], "N": sc.N, "V": sc.V, "scan_window": sc.scan_window,
         "poses_init": sc.poses_init, "points": case.get("points", False), "poses": sc.poses_moved}
    if s["points"]:
        x, y, z, scan, voxel = sc.points()
        s["data"] = (x, y, z, scan, voxel)
    else:
        s["data"] = sc.sums()
    if kind == "build":
        return s
    s["problem"] = _build(s)
    s["data"] = None
    if case["windows"] >= 64:   # the launch choices the tuner finds for many windows
        ba.problem_set_tuning(s["problem"], {"vox_split": 1, "vox_grid": 0, "pose_grid": 0, "chunk_len": 1024})
    if kind == "eval":
        s["derivatives"] = case["derivatives"]
    else:
        s["mode"] = ba.MODE_COUPLED if case["coupled"] else ba.MODE_MM
        s["iters"] = case["iters"]
        s["poses"] = sc.poses_init.clone()
    return s


def run(state):
    s = state
    kind = s["kind"]
    if kind == "eval":
        cost, grad, hess, _ = ba.eval_residual_grad_hessian(s["problem"], s["poses"], derivatives=s["derivatives"])
        return {"cost": cost, "grad": grad, "hess": hess}
    if kind == "iterate":
        s["poses"].copy_(s["poses_init"])
        rep, _ = ba.iterate(s["problem"], s["poses"], mode=s["mode"], max_iters=s["iters"], trace=False)
        return {"poses": s["poses"], "cost_initial": torch.tensor([r["cost_initial"] for r in rep], dtype=torch.float64),
                "cost_final": torch.tensor([r["cost_final"] for r in rep], dtype=torch.float64)}
    if kind == "solve":
        dx, info = ba.solve_increment(s["mode"], s["H"], s["g"], 1e-2)
        return {"dx": dx, "info": info}
    if kind == "build":
        p = _build(s)
        cost, _, _, _ = ba.eval_residual_grad_hessian(p, s["poses"], derivatives=False)
        voxel, scan, count, mu, S = p.export_clusters()
        p.close()
        return {"cost": cost, "voxel": voxel, "scan": scan, "count": count, "mu": mu, "S": S}
    if s["host"]:
        m = ba.voxelize_host(*s["data"], s["poses"], 0.5, s["levels"], 0.05, min_scans=2, batch_points=s["batch"])
    else:
        m = ba.voxelize(*s["data"], s["poses"], 0.5, s["levels"], 0.05, min_scans=2)
    new = m.export()
    m.close()
    for k, v in new.items():
        s["out"][k][:len(v)].copy_(v)
    return {**s["out"], "clusters": len(new["voxel"]), "voxels": len(new["voxel_level"])}


# ------------------------------------------------------------------ work
def _observers(case, n):
    if case.get("law", "loop") == "loop":
        cap = min(LOOP_MAX, n)
        return sum((1 - LOOP_P) ** k for k in range(cap))   # mean of the cut geometric
    near = min(PATH_NEAR, n)
    return sum(min(k, near) for k in range(PATH_MIN, PATH_MAX + 1)) / (PATH_MAX - PATH_MIN + 1)


def work(case):
    if case["kind"] == "solve":
        n = 6 * case["poses"]
        if case["coupled"]:
            return {"bytes": 4 * n * (n + 1) + 16 * n, "flops": n ** 3 / 3 + 2 * n * n}
        return {"bytes": case["poses"] * (288 + 96), "flops": case["poses"] * 250}
    n_w, v_w = _sizes(case)
    N, C = sum(n_w), sum(v * _observers(case, n) for n, v in zip(n_w, v_w))
    per_obs = 480 / math.log(25.0)   # mean of the log-uniform point counts
    if case["kind"] == "voxelize":
        n = C * per_obs
        return {"bytes": 28 * n + 96 * N, "flops": 40 * n}
    if case["kind"] == "build":
        inp = C * per_obs * 32 if case["points"] else C * 88
        return {"bytes": inp + C * 88 + 8, "flops": (20 * C * per_obs if case["points"] else 40 * C)}
    stored = C * (44 if case["f32"] else 84)
    if case["kind"] == "eval":
        full = case["derivatives"]
        return {"bytes": stored + 96 * N + (336 * N if full else 0) + 8, "flops": C * (350 if full else 150)}
    n = case["iters"]
    dense = n * (6 * N) ** 3 / 3 if case["coupled"] else 0
    return {"bytes": (n + 1) * (stored + 96 * N), "flops": n * C * 350 + dense}


# ------------------------------------------------------------------ exact
def _two_prod(a, b):
    def split(v):
        c = 134217729.0 * v
        h = c - (c - v)
        return h, v - h
    p = a * b
    ah, al = split(a)
    bh, bl = split(b)
    return p, ((ah * bh - p) + ah * bl + al * bh) + al * bl


def _centred(data, points, N):
    """(voxel, scan, count, mu, S) in (voxel, scan) order."""
    if points:
        x, y, z, scan, voxel = data
        key, inv, cnt = torch.unique(voxel.long() * N + scan.long(), return_inverse=True, return_counts=True)
        p, n = torch.stack([x, y, z], 1), cnt.double()
        first = torch.zeros(len(key), 3, device="cuda", dtype=torch.float64)
        first[inv] = p   # any one point of the cluster: the sums are formed about it
        q = p - first[inv]
        m = torch.zeros_like(first).index_add_(0, inv, q) / n[:, None]
        d = q - m[inv]
        prod = torch.stack([d[:, i] * d[:, j] for i in range(3) for j in range(i, 3)], 1)
        S = torch.zeros(len(key), 6, device="cuda", dtype=torch.float64).index_add_(0, inv, prod)
        return key // N, key % N, n, first + m, S
    voxel, scan, count, s1, s2 = data
    order = torch.argsort(voxel.long() * N + scan.long())
    voxel, scan, n, s, Q = voxel[order].long(), scan[order].long(), count[order].double(), s1[order], s2[order]
    out, k = torch.empty_like(Q), 0
    for i in range(3):
        for j in range(i, 3):
            ph, pl = _two_prod(s[:, i], s[:, j])
            qh = ph / n
            th, tl = _two_prod(qh, n)
            ql = (((ph - th) - tl) + pl) / n
            d = Q[:, k] - qh
            b = d - Q[:, k]
            out[:, k] = d + (((Q[:, k] - (d - b)) + (-qh - b)) - ql)
            k += 1
    return voxel, scan, n, s / n[:, None], out


def _sym(S):
    return S[:, [0, 1, 2, 1, 3, 4, 2, 4, 5]].view(-1, 3, 3)


def _mat(a, b):
    return (a[:, :, :, None] * b[:, None, :, :]).sum(2)


def _skew(v):
    z = torch.zeros_like(v[:, 0])
    return torch.stack([z, -v[:, 2], v[:, 1], v[:, 2], z, -v[:, 0], -v[:, 1], v[:, 0], z], 1).view(-1, 3, 3)


def _evaluate(cl, poses, V, N, W, scan_window, derivatives):
    voxel, scan, n, mu, S = cl
    R, t = poses[:, :9].view(-1, 3, 3)[scan], poses[:, 9:][scan]
    y = (R * mu[:, None, :]).sum(2)
    m = y + t
    St = _mat(_mat(R, _sym(S)), R.transpose(1, 2))
    add = lambda size, idx, v: torch.zeros((size,) + v.shape[1:], device="cuda", dtype=torch.float64).index_add_(0, idx, v)  # noqa: E731
    first = torch.zeros(V, 3, device="cuda", dtype=torch.float64)
    first[voxel] = m   # a reference point near each voxel
    Nv = add(V, voxel, n)
    seen = Nv > 0
    r = m - first[voxel]
    off = add(V, voxel, n[:, None] * r) / Nv.clamp_min(1)[:, None]
    d = r - off[voxel]
    A = add(V, voxel, St + n[:, None, None] * d[:, :, None] * d[:, None, :]) / Nv.clamp_min(1)[:, None, None]
    lam, vec = torch.linalg.eigh(A.cpu())
    lam, u = lam[:, 0].cuda(), vec[:, :, 0].cuda()
    u = u[voxel]
    win = torch.as_tensor(scan_window, device="cuda").long()
    vwin = torch.zeros(V, device="cuda", dtype=torch.long)
    vwin[voxel] = win[scan]
    cost = add(W, vwin[seen], lam[seen])
    if not derivatives:
        return cost, None, None
    sc, e = 2 / Nv[voxel], (u * d).sum(1)
    w = (n * e)[:, None] * y + (St * u[:, None, :]).sum(2)
    a = torch.linalg.cross(y, u)
    grad = add(N, scan, torch.cat([sc[:, None] * torch.linalg.cross(w, u), (sc * n * e)[:, None] * u], 1))
    U = _skew(u)
    uw = (u * w).sum(1)
    H = torch.empty(len(n), 6, 6, device="cuda", dtype=torch.float64)
    H[:, :3, :3] = (n[:, None, None] * a[:, :, None] * a[:, None, :] + _mat(_mat(U, St), U.transpose(1, 2))
                    + 0.5 * (u[:, :, None] * w[:, None, :] + w[:, :, None] * u[:, None, :])
                    - uw[:, None, None] * torch.eye(3, device="cuda", dtype=torch.float64))
    H[:, :3, 3:] = n[:, None, None] * a[:, :, None] * u[:, None, :]
    H[:, 3:, :3] = H[:, :3, 3:].transpose(1, 2)
    H[:, 3:, 3:] = n[:, None, None] * u[:, :, None] * u[:, None, :]
    return cost, grad, add(N, scan, sc[:, None, None] * H)


def _exact_voxels(s):
    x, y, z, scan = (torch.as_tensor(a).cuda() for a in s["data"])
    poses, N = s["poses"], s["poses"].shape[0]
    sl = scan.long()
    cell = []
    for r in range(3):
        P = [poses[:, c][sl] for c in (3 * r, 3 * r + 1, 3 * r + 2, 9 + r)]
        cell.append(torch.floor((((P[0] * x + P[1] * y) + P[2] * z) + P[3]) / 0.5).long())
    p = torch.stack([x, y, z], 1)
    out, base = [], 0
    for level in range(1, s["levels"] + 1):
        c = [k >> (level - 1) for k in cell]
        lo = [int(k.min()) for k in c]
        span = [int(k.max()) - a + 1 for k, a in zip(c, lo)]
        ck = ((c[0] - lo[0]) * span[1] + (c[1] - lo[1])) * span[2] + (c[2] - lo[2])
        key, inv, cnt = torch.unique(ck * N + sl, return_inverse=True, return_counts=True)
        sums = torch.zeros(len(key), 3, device="cuda", dtype=torch.float64).index_add_(0, inv, p)
        prod = torch.stack([p[:, i] * p[:, j] for i in range(3) for j in range(i, 3)], 1)
        sq = torch.zeros(len(key), 6, device="cuda", dtype=torch.float64).index_add_(0, inv, prod)
        cells, vi, ns = torch.unique(key // N, return_inverse=True, return_counts=True)
        cs = key % N
        _, _, n, mu, S = _centred((vi, cs, cnt, sums, sq), False, N)
        R, t = poses[:, :9].view(-1, 3, 3)[cs], poses[:, 9:][cs]
        m = (R * mu[:, None, :]).sum(2) + t
        V = len(cells)
        add = lambda v: torch.zeros((V,) + v.shape[1:], device="cuda", dtype=torch.float64).index_add_(0, vi, v)  # noqa: E731
        Nv = add(n)
        ref = torch.zeros(V, 3, device="cuda", dtype=torch.float64)
        ref[vi] = m
        r = m - ref[vi]
        d = r - (add(n[:, None] * r) / Nv[:, None])[vi]
        A = add(_mat(_mat(R, _sym(S)), R.transpose(1, 2)) + n[:, None, None] * d[:, :, None] * d[:, None, :])
        lam = torch.linalg.eigvalsh((A / Nv[:, None, None]).cpu()).cuda()
        keep = (Nv >= 3) & (lam[:, 1] > 1e-10 * lam[:, 2]) & (lam[:, 0] < 0.05 * lam[:, 1]) & (ns >= 2)
        rank = torch.cumsum(keep.long(), 0) - 1 + base
        k = keep[vi]
        out.append((rank[vi][k].int(), cs[k].int(), cnt[k], sums[k], sq[k]))
        base += int(keep.sum())
    for i, a in enumerate(("voxel", "scan", "count", "sum", "sumsq")):
        v = torch.cat([o[i] for o in out])
        s["out"][a][:len(v)] = v
    return {**s["out"], "voxel_level": None, "voxel_cell": None, "clusters": len(v), "voxels": base}


def exact(case, seed):
    kind = case["kind"]
    if kind == "iterate":
        return None   # a whole run: its poses have no value short of an optimizer of its own
    s = prepare(case, seed) if kind != "eval" else None
    if kind == "voxelize":
        return _exact_voxels(s)
    if kind == "solve":
        H, g = s["H"], s["g"].reshape(-1)
        if case["coupled"]:
            d = H.diagonal()
            d.add_(1e-2 * torch.maximum(d, 1e-12 * d.max()))
            L = torch.linalg.cholesky(H.cpu())
            return {"dx": -torch.cholesky_solve(g.cpu()[:, None], L).view(-1, 6), "info": None}
        d = H.diagonal(dim1=1, dim2=2)
        d.add_(1e-2 * torch.maximum(d, 1e-12 * d.max()))
        return {"dx": -torch.linalg.solve(H.cpu(), s["g"].cpu()), "info": None}
    sc = _Scene(case, seed, case["law"] == "loop")
    points = case.get("points", False)
    data = s["data"] if s else sc.sums()
    cl = _centred(data, points, sc.N)
    cost, grad, hess = _evaluate(cl, sc.poses_moved, sc.V, sc.N, case["windows"], sc.scan_window,
                                 case.get("derivatives", False))
    if kind == "eval":
        return {"cost": cost, "grad": grad, "hess": hess}
    voxel, scan, n, mu, S = cl
    return {"cost": cost, "voxel": None, "scan": None, "count": n, "mu": mu, "S": S}
