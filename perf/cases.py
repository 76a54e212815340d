"""The calls that a user of this library makes, as cases that can be timed and compared.

A case is one pass of a user's program over one batch that is resident on the GPU.  `call` names what the program does:

  serve     the pose stands (fs_precompute was called before), a batch of points arrives: fs_solve + fs_dedupe
  frame     a new pose and its batch of points: fs_precompute + fs_solve + fs_dedupe
  step      a training step on the C-ABI: fs_precompute + fs_solve + fs_grad, cell positions handed on, J~ kept inside
  exact     the same with the exact inverse Jacobian in the backward
  autograd  a training step through the torch.autograd hook
  two_call  initial states materialised by fs_init, J~ written out, and a backward that gets arrays only

`init` is the kind of initial state ("bone": one per bone, "voxel": candidates of the correspondence grid), `points` how
the query points lie: "scan" (half posed canonical samples, half uniform in the deformed box), "posed" (posed canonical
samples only) or "rays" (samples along rays through the deformed box).  Inputs are synthetic scenes of the shapes that
`paper_2211_15601_amd.workloads` builds, made on the GPU.
"""
import math

import numpy as np
import torch

from paper_2211_15601_amd import autograd, binding
from paper_2211_15601_amd import workloads as wl

DEV = "cuda:0"
F32, I32, U8 = torch.float32, torch.int32, torch.uint8
MIN_DIST = 1e-3            # roots closer than this are duplicates
RAY_SAMPLES = 256


def _case(name, call, init, points, n, dims, poses=1, bones=24, iters=50):
    return {"name": name, "call": call, "init": init, "points": points, "n": n, "nx": dims[0], "ny": dims[1], "nz": dims[2],
            "poses": poses, "bones": bones, "iters": iters}


def listed():
    return [
        # a handful of points of a standing pose, as an interactive probe asks for them: launches and latency
        _case("probe", "serve", "bone", "scan", 37, (64, 64, 16)),
        # the tiny configuration: one training step on a grid that fits the LDS
        _case("tiny_step", "step", "bone", "posed", 4096, (16, 16, 4)),
        # the SMPL-scale configuration: one training step of one scan
        _case("scan_step", "step", "bone", "scan", 65536, (64, 64, 16)),
        # the 200k-point batch on which the method is usually quoted: articulation of one frame
        _case("scan_frame", "frame", "bone", "scan", 200000, (64, 64, 16)),
        # several poses side by side, ragged, a grid of odd sizes
        _case("poses_frame", "frame", "bone", "scan", 40003, (61, 47, 13), poses=4),
        # ray samples of a standing pose in small ragged tiles, as a renderer asks for them
        _case("ray_tile", "serve", "voxel", "rays", 96 * RAY_SAMPLES + 7, (64, 64, 16), iters=30),
        # the ray-batch configuration: one frame of 4096 rays
        _case("ray_frame", "frame", "voxel", "rays", 1048576, (64, 64, 16), iters=30),
        # the training configuration
        _case("ray_step", "step", "voxel", "rays", 2097152, (64, 64, 16), iters=30),
        # the multi-pose configuration, the largest
        _case("multi_step", "step", "voxel", "scan", 8 * 524288, (128, 128, 32), poses=8),
        # training through the autograd hook, ragged
        _case("hook_step", "autograd", "voxel", "scan", 300007, (64, 64, 16)),
        # backward with the exact inverse Jacobian, odd grid
        _case("exact_step", "exact", "bone", "scan", 20011, (45, 39, 11)),
        # separate initialisation and a backward fed with arrays; bones that fill no 16-wide tile
        _case("two_call_step", "two_call", "bone", "posed", 30011, (32, 32, 8), bones=17),
    ]


def draw(rng):
    call = rng.choice(["serve", "serve", "frame", "frame", "step", "step", "step", "exact", "autograd", "two_call"])
    init = rng.choice(["bone", "voxel"])
    points = rng.choice(["scan", "scan", "posed"] if init == "bone" else ["scan", "rays", "rays"])
    bones = 24 if init == "voxel" or rng.random() < 0.6 else rng.choice([5, 12, 17, 33, 52, 64])
    poses = rng.choice([1, 1, 1, 2, 4, 8])
    scale = math.exp(rng.uniform(math.log(16), math.log(128 if poses <= 4 else 96)))
    dims = [max(4, int(round(scale * f * rng.uniform(0.85, 1.0)))) for f in (1.0, 1.0, 0.25)]
    # points: from a handful to what the largest listed case costs with this many states per point
    most = (1 << 21) if init == "voxel" else max(4096, 4_800_000 // bones)
    n = int(math.exp(rng.uniform(math.log(24), math.log(most))))
    return {"call": call, "init": init, "points": points, "n": max(n, poses), "nx": dims[0], "ny": dims[1], "nz": dims[2],
            "poses": poses, "bones": bones, "iters": rng.choice([30, 50])}


# ------------------------------------------------------------------------------------------------ inputs

def _weights(x, a, b):
    """Skinning weights of points x [m, 3]: normalised exp(-distance^2 / 0.02) to the bone segments, [m, bones]."""
    ab = b - a
    l2 = (ab * ab).sum(1).clamp_min(1e-12)
    t = ((x @ ab.T - (a * ab).sum(1)) / l2).clamp(0.0, 1.0)
    d2 = torch.zeros((x.shape[0], a.shape[0]), dtype=x.dtype, device=x.device)
    for c in range(3):
        e = x[:, c:c + 1] - a[:, c] - t * ab[:, c]
        d2 += e * e
    return torch.softmax(-d2 / wl.WEIGHT_SIGMA2, dim=1)


def _posed(x, a, b, B):
    """Canonical points moved by linear blend skinning under the continuous weights."""
    out = torch.empty_like(x)
    for s in range(0, x.shape[0], 1 << 19):
        xs = x[s:s + (1 << 19)]
        T = (_weights(xs, a, b) @ B).view(-1, 3, 4)
        out[s:s + (1 << 19)] = (T[:, :, :3] * xs[:, None, :]).sum(2) + T[:, :, 3]
    return out


def _ray_points(gen, n, lo, hi):
    """n samples along rays through the box [lo, hi], ray by ray, equally spaced between entry and exit."""
    rays = -(-n // RAY_SAMPLES)
    samples = RAY_SAMPLES if n >= RAY_SAMPLES else n
    d = torch.randn((rays, 3), generator=gen, device=DEV)
    org = 0.5 * (lo + hi) + 0.75 * (hi - lo).norm() * d / d.norm(dim=1, keepdim=True)
    tgt = lo + torch.rand((rays, 3), generator=gen, device=DEV) * (hi - lo)
    v = tgt - org
    v = v / v.norm(dim=1, keepdim=True)
    t0, t1 = (lo - org) / v, (hi - org) / v
    tn, tf = torch.minimum(t0, t1).amax(1), torch.maximum(t0, t1).amin(1)
    tf = torch.maximum(tf, tn)
    s = (torch.arange(samples, device=DEV, dtype=F32) + 0.5) / samples
    t = tn[:, None] + (tf - tn)[:, None] * s
    return (org[:, None, :] + t[..., None] * v[:, None, :]).reshape(-1, 3)[:n]


def _scene(case, seed):
    rng = np.random.default_rng(seed)
    gen = torch.Generator(device=DEV).manual_seed(int(seed))
    nb, P, N = case["bones"], case["poses"], case["n"]
    if nb == wl.N_BONES and case["points"] != "posed":
        sa, sb, parent = wl.human_skeleton(rng)
        Bs = [wl.chain_bone_transforms(rng, sa, parent, 45.0 if P == 1 else 60.0) for _ in range(P)]
    else:
        sa, sb = wl.random_segments(rng, nb)
        Bs = [wl.independent_bone_transforms(rng, nb) for _ in range(P)]
    up = lambda v: torch.from_numpy(np.ascontiguousarray(v, dtype=np.float32)).to(DEV)
    a, b, B = up(sa), up(sb), up(np.stack(Bs))
    lo, hi = up(wl.BOX_LO), up(wl.BOX_HI)
    dims = (case["nx"], case["ny"], case["nz"])
    axes = [torch.linspace(float(wl.BOX_LO[i]), float(wl.BOX_HI[i]), dims[i], device=DEV) for i in range(3)]
    nodes = torch.stack(torch.meshgrid(*axes, indexing="ij"), -1).reshape(-1, 3)
    W = _weights(nodes, a, b)
    xs, pose = [], []
    for p in range(P):
        m = N * (p + 1) // P - N * p // P
        T = (W @ B[p]).view(-1, 3, 4)
        y = (T[:, :, :3] * nodes[:, None, :]).sum(2) + T[:, :, 3]
        blo, bhi = y.amin(0), y.amax(0)
        if case["points"] == "rays":
            x = _ray_points(gen, m, blo, bhi)
        else:
            k = m if case["points"] == "posed" else m // 2
            x = _posed(lo + torch.rand((k, 3), generator=gen, device=DEV) * (hi - lo), a, b, B[p])
            x = torch.cat([x, blo + torch.rand((m - k, 3), generator=gen, device=DEV) * (bhi - blo)])
            x = x[torch.randperm(m, generator=gen, device=DEV)]
        xs.append(x)
        pose.append(torch.full((m,), p, dtype=I32, device=DEV))
    xq = torch.cat(xs).T.contiguous()
    return dims, W.view(*dims, nb).contiguous(), B.contiguous(), xq, (torch.cat(pose) if P > 1 else None), gen


def prepare(case, seed):
    dims, W, B, xq, pose, gen = _scene(case, seed)
    call, N = case["call"], case["n"]
    voxel = case["init"] == "voxel"
    fs = binding.Context(dims, case["bones"], wl.BOX_LO, wl.BOX_HI, n_poses=case["poses"], tol=1e-5, div_thresh=10.0,
                         max_iters=case["iters"], init_mode=binding.FS_INIT_VOXEL if voxel else binding.FS_INIT_BONE,
                         grad_mode=binding.FS_GRAD_EXACT_J if call == "exact" else binding.FS_GRAD_BROYDEN_J)
    K = fs.K
    new = lambda *shape, dtype=F32: torch.empty(shape, dtype=dtype, device=DEV)
    s = {"call": call, "fs": fs, "N": N, "K": K, "W": W, "B": B, "xq": xq, "pose": pose}
    if call == "autograd":
        s["W"], s["B"], s["xq"] = (t.requires_grad_(True) for t in (W, B, xq))
        s["gxc"] = torch.randn((K, 3, N), generator=gen, device=DEV)
        return s
    s["xc"], s["conv"], s["iters"] = new(K, 3, N), new(K, N, dtype=U8), new(K, N, dtype=U8)
    if call in ("serve", "frame"):
        s["keep"], s["offsets"] = new(K, N, dtype=U8), new(N + 1, dtype=I32)
        s["cap"] = K * N
        s["roots"] = torch.zeros((K * N, 3), dtype=F32, device=DEV)
        s["lane"] = torch.zeros((K * N,), dtype=I32, device=DEV)
    else:
        s["gxc"] = torch.randn((K, 3, N), generator=gen, device=DEV)
        s["gW"], s["gB"], s["gxq"] = torch.empty_like(W), torch.empty_like(B), new(3, N)
    if call in ("step", "exact"):
        s["slot"] = new(K, N, dtype=I32)
    if call == "two_call":
        s["x0"], s["J0"], s["v0"], s["J"] = new(K, 3, N), new(K, 9, N), new(K, N, dtype=U8), new(K, 9, N)
    if call == "serve":
        fs.precompute(W, B)
    return s


# ------------------------------------------------------------------------------------------------ the pass

def run(s):
    call, fs, N, K, W, B, xq, pose = (s[k] for k in ("call", "fs", "N", "K", "W", "B", "xq", "pose"))
    if call == "autograd":
        for t in (W, B, xq):
            t.grad = None
        xc, conv = autograd.CorrespondenceSearch.apply(fs, W, B, xq, pose)
        xc.backward(s["gxc"])
        return {"xc": xc, "conv": conv, "gW": W.grad, "gB": B.grad, "gxq": xq.grad}
    xc, conv, iters = s["xc"], s["conv"], s["iters"]
    if call != "serve":
        fs.precompute(W, B)
    if call in ("serve", "frame"):
        fs.solve(xq, pose, N, K, None, None, None, xc, conv, None, iters)
        fs.dedupe(xc, conv, N, K, MIN_DIST, s["keep"], s["offsets"], s["roots"], s["lane"], s["cap"])
        return {k: s[k] for k in ("xc", "conv", "iters", "keep", "offsets", "roots", "lane")}
    if call == "two_call":
        fs.init(xq, pose, N, s["x0"], s["J0"], s["v0"])
        fs.solve(xq, pose, N, K, s["x0"], s["J0"], s["v0"], xc, conv, s["J"], iters)
        fs.grad(W, xc, s["J"], conv, s["gxc"], pose, N, K, s["gW"], s["gB"], s["gxq"])
        return {k: s[k] for k in ("x0", "J0", "v0", "xc", "conv", "iters", "J", "gW", "gB", "gxq")}
    fs.solve(xq, pose, N, K, None, None, None, xc, conv, None, iters, s["slot"])
    fs.grad(W, xc, None, conv, s["gxc"], pose, N, K, s["gW"], s["gB"], s["gxq"], s["slot"])
    return {k: s[k] for k in ("xc", "conv", "iters", "gW", "gB", "gxq")}


def work(case):
    """Bytes: inputs read once, outputs written once.  Operations: field evaluations at 237 flop and Broyden steps at 81 for the
    pairs that have an initial state (every one with a state per bone; about one in seven of the candidates along rays,
    six in ten of those of scans), with the mean number of evaluations per pair that these scenes need."""
    N, P, nb = case["n"], case["poses"], case["bones"]
    voxel = case["init"] == "voxel"
    K = 3 if voxel else nb
    V = case["nx"] * case["ny"] * case["nz"]
    pairs = K * N * ((0.14 if case["points"] == "rays" else 0.62) if voxel else 1.0)
    flops = pairs * (6.0 if voxel else 7.5) * (237 + 81 * 0.85)
    points, roots = N * (12 + (4 if P > 1 else 0)), K * N * (12 + 1)
    grid, bones = V * nb * 4, P * nb * 48
    call = case["call"]
    if call == "serve":
        return {"bytes": points + roots + K * N * 2 + N * 4, "flops": flops}
    flops += V * P * nb * 24
    if call == "frame":
        return {"bytes": grid + bones + points + roots + K * N * 2 + N * 4, "flops": flops}
    flops += 2 * V * P * nb * 24 + pairs * (8 * 30 + 30)
    grads = K * N * 12 + grid + bones + N * 12
    if call == "two_call":
        return {"bytes": grid + bones + points + roots + K * N * (1 + 36 + 12 + 36 + 1) + grads, "flops": flops}
    return {"bytes": grid + bones + points + roots + (0 if call == "autograd" else K * N) + grads, "flops": flops}


def tolerance(case):
    """Roots, masks and counts are fixed to the bit by the documented order of operations; the gradients are 32-bit sums
    whose order is free."""
    if case["call"] in ("serve", "frame"):
        return "exact"
    return {"rel": 1e-5, "max": 1e-3, "differ": 0.0}
