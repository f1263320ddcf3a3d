"""Benchmark of the render-and-train step on one MI355X.

One step = the whole hot path over one frame of the avatar workload
(100k Gaussians, 7k-vertex / 14k-triangle body mesh, 24 joints, 16x32
environment = 512 light directions, visibility from 512 views at 128^2,
one 512x512 camera):
  skin the mesh -> visibility (raster + filters) -> skin the Gaussians ->
  shade -> splat forward -> L1 loss and gradient -> splat backward ->
  shade backward -> skinning backward.
Inputs are synthetic (seeded) and resident in HBM before timing starts.

Prints one JSON line.  `value` is the fwd+bwd time per step (ms/iter) of
the FP32 form; `render_fps` is the forward-only frame rate with visibility
recomputed per frame, `render_fps_no_vis` with visibility cached per pose.
The same figures for the BF16X3 form of the shading contraction (bf16 hi +
lo operands) sit under `bf16x3`; `shading_forward` names the kernel that each
form's forward ran on (the library chooses MFMA or the FP32 kernel; at this
workload both forms run on the latter).  `image_error_vs_fp64` gives each
form's image PSNR against the FP64 oracle (with the oracle's emulation of
plain bf16 operands beside it).
"""

from __future__ import annotations

import argparse
import json
import math
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

METRIC = ("fwd+bwd ms/iter and render fps at 512²/100k Gaussians; BF16-MFMA vs FP32 at PSNR")
PEAK_FP32_TFLOPS = 157.3       # MI355X vector FP32 (published, with packed issue)
PEAK_HBM_GBS = 8000.0


def parse():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=50)
    ap.add_argument("--warmup", type=int, default=10)
    ap.add_argument("--config", type=int, default=2)
    ap.add_argument("--precision", default="fp32", choices=["fp32", "bf16x3"])
    ap.add_argument("--kernel", default=None, help="kernel timed for the roofline entry")
    ap.add_argument("--no-cpu-baseline", action="store_true",
                    help="skip the oracle legs (CPU baseline and image error vs FP64)")
    ap.add_argument("--one-form", action="store_true",
                    help="time only the --precision form (by default the other form of the "
                         "shading contraction is timed beside it)")
    ap.add_argument("--all-kernels", action="store_true", help="time every kernel (diagnostic)")
    ap.add_argument("--copy-calibration", action="store_true",
                    help="also run a 256 MiB device copy (reference for HBM counters)")
    ap.add_argument("--graph", action="store_true",
                    help="capture one step in a HIP graph and replay it (no host launch cost)")
    ap.add_argument("--sequence", action="store_true",
                    help="animation x relighting sequence: step i renders frame i mod "
                         "(poses x maps), pose-major; visibility once per pose")
    return ap.parse_args()


# HBM traffic per launch of the roofline kernels, from rocprofv3 FETCH_SIZE /
# WRITE_SIZE passes scaled by a plain copy's readings; each summary records
# the SHA-256 of the kernel's source file at the time, and the figure is
# reported only while the source is unchanged.
TRAFFIC_PROFILES = {
    ("shade_bwd", 2): ("profiles/shade_bwd_avatar-100k-512px_hbm_counters.md",
                       "paper_2407_10707_amd/csrc/shade.hip"),
    ("blend_bwd", 2): ("profiles/blend_bwd_avatar-100k-512px_hbm_counters.md",
                       "paper_2407_10707_amd/csrc/splat.hip"),
}


def traffic_from_profile(kernel: str, config: int):
    import hashlib
    import re
    entry = TRAFFIC_PROFILES.get((kernel, config))
    if entry is None:
        return None
    prof, src = (os.path.join(ROOT, p) for p in entry)
    if not (os.path.exists(prof) and os.path.exists(src)):
        return None
    text = open(prof).read()
    m_sha = re.search(r"source_sha256:\s*([0-9a-f]{64})", text)
    m_val = re.search(r"traffic_bytes_per_launch:\s*([0-9]+)", text)
    if not (m_sha and m_val):
        return None
    sha = hashlib.sha256(open(src, "rb").read()).hexdigest()
    return int(m_val.group(1)) if sha == m_sha.group(1) else None


def shade_flops(live_pairs: float, tested_pairs: float, backward: bool,
                tested: bool = True) -> float:
    """Algorithmic FP32 operations of the shading sum: per tested (Gaussian,
    direction) pair the horizon and visibility test (n.w: 5, visibility
    interpolation: 5, compare: 1); per live pair the BRDF weights and the
    accumulation (forward 72, backward 171; counted from the formulas, an
    FMA as 2).  An adjoint that replays the forward's live-pair tape tests
    nothing (tested=False)."""
    per_live = 171.0 if backward else 72.0
    return (tested_pairs * 11.0 if tested else 0.0) + live_pairs * per_live


def shading_pairs(s, R, p, count):
    """Count (front-facing Gaussian, direction) pairs and the live ones
    (w.n > 0 and interpolated visibility > 0) of this frame -- bookkeeping for
    the roofline entry, outside the timed region."""
    import torch
    from paper_2407_10707_amd import rga
    xo, no, _ = rga.lbs_skin(R.d["skin"], R.d["jidx"], R.d["jw"], p["pos"], p["nrm"])
    _, front = rga.shade_gaussians(xo, no, p["albedo"], p["rough"], p["tint"], R.d["vidx"],
                                   R.d["vw"], count, s["kv"], s["he"], s["we"], s["hv"], s["wv"],
                                   p["env"], R.cam_pos)
    he, we, hv, wv = s["he"], s["we"], s["hv"], s["wv"]
    r = (torch.arange(he, device="cuda", dtype=torch.float64) + 0.5) * math.pi / he
    c = (torch.arange(we, device="cuda", dtype=torch.float64) + 0.5) * 2 * math.pi / we
    th, ph = torch.meshgrid(r, c, indexing="ij")
    dirs = torch.stack([th.sin() * ph.sin(), th.cos(), th.sin() * ph.cos()], -1).reshape(-1, 3)
    rr = torch.arange(he, device="cuda")[:, None].expand(he, we)
    cc = torch.arange(we, device="cuda")[None, :].expand(he, we)
    view = ((rr * hv) // he * wv + (cc * wv) // we).reshape(-1)
    live = 0
    tested = 0
    f = front.bool()
    for a in range(0, s["n"], 16384):
        b = min(s["n"], a + 16384)
        nn = no[:, a:b].T.double()
        nn = nn / nn.norm(dim=1, keepdim=True)
        ci = nn @ dirs.T
        anyv = (count[R.d["vidx"][:, a:b].long()] > 0).any(0)[:, view]
        m = (ci > 0) & anyv & f[a:b, None]
        live += int(m.sum())
        tested += int(f[a:b].sum()) * he * we
    return {"live": live, "tested": tested}


def blend_pairs(mean2d, conic, opac, sorted_ids, ranges, width: int, height: int,
                tiles_per_batch: int = 16):
    """Count the (pixel, splat) pairs of this frame's tile lists that the
    compositing walks -- every listed splat up to and including the one at
    which the pixel stops (or the whole list) -- and the applied ones among
    them (exponent <= 0, alpha >= 1/255, before the stop): bookkeeping for
    the blend adjoint's roofline entry, outside the timed region, in plain
    PyTorch on the device (the transmittance as a cumulative product, so a
    pixel within rounding of the 1e-4 threshold may count one entry more or
    less than the kernels' sequential walk).  mean2d [2][n], conic [3][n]
    (A, B, C), opac [n], sorted_ids [D], ranges [tiles][2]."""
    import torch
    dev = mean2d.device
    tx = (width + 15) // 16
    tiles = ranges.shape[0]
    ly = torch.arange(256, device=dev) // 16
    lx = torch.arange(256, device=dev) % 16
    walked = 0
    applied = 0
    for t0 in range(0, tiles, tiles_per_batch):
        t1 = min(tiles, t0 + tiles_per_batch)
        r = ranges[t0:t1].long()
        lens = (r[:, 1] - r[:, 0]).clamp(min=0)
        L = int(lens.max()) if lens.numel() else 0
        if L == 0:
            continue
        k = torch.arange(L, device=dev)
        ok = k[None, :] < lens[:, None]                                   # [b, L]
        e = (r[:, :1] + k[None, :]).clamp(max=max(int(sorted_ids.numel()) - 1, 0))
        g = sorted_ids[e].long()
        tid = torch.arange(t0, t1, device=dev)
        px = ((tid % tx) * 16)[:, None] + lx[None, :]                      # [b, 256]
        py = ((tid // tx) * 16)[:, None] + ly[None, :]
        inside = (px < width) & (py < height)
        dx = mean2d[0][g][:, None, :] - (px.float() + 0.5)[:, :, None]    # [b, 256, L]
        dy = mean2d[1][g][:, None, :] - (py.float() + 0.5)[:, :, None]
        A, B, C = (conic[i][g][:, None, :] for i in range(3))
        power = -0.5 * (A * dx * dx + C * dy * dy) - B * dx * dy
        alpha = torch.clamp(opac[g][:, None, :] * torch.exp(power), max=0.99)
        use = (power <= 0) & (alpha >= 1.0 / 255.0) & ok[:, None, :]
        Tafter = torch.cumprod(torch.where(use, 1.0 - alpha, torch.ones_like(alpha)), dim=-1)
        stop = use & (Tafter < 1e-4)
        first = torch.where(stop.any(-1), stop.float().argmax(-1), torch.full_like(
            stop[..., 0], L, dtype=torch.long))                           # [b, 256]
        n_walk = torch.minimum(first + 1, lens[:, None])
        before = k[None, None, :] < first[..., None]
        walked += int((n_walk * inside).sum())
        applied += int((use & before & inside[..., None]).sum())
    return {"walked": walked, "applied": applied}


def blend_bwd_flops(walked: float, applied: float) -> float:
    """Algorithmic FP32 operations of the blend adjoint (3DGS compositing,
    Sec. 3.1 last paragraph): per walked (pixel, splat) pair the offset,
    the exponent, its exp, alpha, the tests and the transmittance step (15,
    the exp as 1); per applied pair also the weight and the colour
    accumulation (7), d alpha from the three channels (20), d/d exponent,
    the mean, conic, opacity and colour partials (23) and their sums over
    the tile's pixels (9): 59.  An FMA counts 2."""
    return walked * 15.0 + applied * 59.0


def cpu_model() -> str:
    try:
        with open("/proc/cpuinfo") as f:
            for line in f:
                if line.startswith("model name"):
                    return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return "unknown"


def image_error(s, images, tiles_wanted: int = 8):
    """Image error of each form against the FP64 oracle's whole chain
    (skinning, shading, projection, compositing) on every pixel of 8 seeded
    lit tiles: PSNR (peak 1), relative L2 and max abs.  `images` maps a form
    to its GPU image; the FP64 oracle also renders the frame with its
    shading contraction's operands rounded to plain bfloat16 (and to the
    split hi + lo form), an emulation of what those operand precisions lose.
    The tiles (seeded, among those whose lists are at least the median
    length), the Gaussians that can reach them and the visibility counts
    come from the FP32 mirror (the oracle's own decisions)."""
    import numpy as np
    import torch
    from oracle import cpu, ref64
    cam = s["cam"]
    H, W = s["height"], s["width"]
    xo, no, Ao = cpu.lbs_f32(s["skin"], s["jidx"], s["jw"], s["pos"], s["nrm"])
    front = cpu.front_f32(xo, no, cam.centre.astype(np.float32))
    pre = cpu.splat_preprocess(cam, xo, Ao, s["quat"], s["log_s"], s["opac"], front)
    _, vals, ranges = cpu.splat_bin(cam, pre)
    TX = (W + 15) // 16
    # tiles whose lists are at least as long as the median non-empty list
    lens = ranges[:, 1] - ranges[:, 0]
    busy = np.nonzero(lens >= max(1, np.median(lens[lens > 0])))[0]
    rng = np.random.default_rng(13)
    tiles = np.sort(rng.choice(busy, tiles_wanted, replace=False))
    pix = []
    for t in tiles:
        ty, tx = divmod(int(t), TX)
        yy, xx = np.meshgrid(np.arange(ty * 16, min(H, ty * 16 + 16)),
                             np.arange(tx * 16, min(W, tx * 16 + 16)), indexing="ij")
        pix.append((yy * W + xx).reshape(-1))
    pix = np.sort(np.concatenate(pix))
    sub = np.unique(np.concatenate([vals[ranges[t, 0]:ranges[t, 1]] for t in tiles]))
    ss = dict(s)
    for k in ("pos", "nrm", "quat", "log_s", "albedo", "jidx", "jw", "vidx", "vw"):
        ss[k] = np.ascontiguousarray(s[k][:, sub])
    for k in ("opac", "rough", "tint"):
        ss[k] = np.ascontiguousarray(s[k][sub])
    vx = cpu.lbs_f32(s["skin"], s["mesh_jidx"], s["mesh_jw"], s["verts"])[0]
    _, cnt = cpu.mesh_visibility(vx, s["faces"], s["view_dirs"], s["vis_res"], s["knn_v"])

    def render(operands):
        p = {k: torch.tensor(np.asarray(ss[k], dtype=np.float64))
             for k in ("pos", "nrm", "quat", "log_s", "opac", "albedo", "rough", "tint", "env")}
        with torch.no_grad():
            xp, npr, A = ref64.lbs(ss["skin"], ss["jidx"], ss["jw"], p["pos"], p["nrm"])
            col, _ = ref64.shade(xp, npr, p["albedo"], p["rough"], p["tint"], ss["vidx"],
                                 ss["vw"], cnt, ss["kv"], ss["he"], ss["we"], ss["hv"], ss["wv"],
                                 p["env"], cam.centre, front[sub], operands=operands)
            proj = ref64.project(cam, xp, A, p["quat"], p["log_s"], p["opac"], front[sub])
            img, _ = ref64.composite(cam, proj, p["opac"], col, pixels=pix)
        return img.numpy()

    ref = render("exact")
    got = {f: np.asarray(im, dtype=np.float64).reshape(3, -1)[:, pix] for f, im in images.items()}
    got["bf16_operands_emulated"] = render("bf16")
    got["bf16x3_operands_emulated"] = render("bf16x3")
    out = {"pixels": int(len(pix)), "tiles": int(len(tiles)), "gaussians": int(len(sub))}
    for f, g in got.items():
        err = g - ref
        mse = float(np.mean(err ** 2))
        out[f] = {"psnr_db": round(10 * math.log10(1.0 / max(mse, 1e-300)), 2),
                  "rel_l2": float(f"{np.linalg.norm(err) / np.linalg.norm(ref):.3e}"),
                  "max_abs": float(f"{np.abs(err).max():.3e}")}
    return out


def cpu_baseline(s):
    """The oracle, as it stands, timed on the host on a bounded sample of one
    step: FP32-mirror skinning of mesh and Gaussians (all), visibility for
    16 of the views, FP64 shading forward+backward for 1000 Gaussians,
    FP32-mirror projection/binning/compositing of the whole frame, and FP64
    compositing forward+backward for 4096 of the pixels.  Each part's time
    is scaled to the full step."""
    import numpy as np
    import torch
    from oracle import cpu, ref64
    cam = s["cam"]
    n, H, W = s["n"], s["height"], s["width"]
    V = s["view_dirs"].shape[0]
    parts = {}
    t = time.perf_counter()
    vx, _, _ = cpu.lbs_f32(s["skin"], s["mesh_jidx"], s["mesh_jw"], s["verts"])
    xo, no, Ao = cpu.lbs_f32(s["skin"], s["jidx"], s["jw"], s["pos"], s["nrm"])
    parts["lbs"] = time.perf_counter() - t
    vs = 16
    t = time.perf_counter()
    cpu.mesh_visibility(vx, s["faces"], s["view_dirs"][:vs], s["vis_res"], s["knn_v"])
    parts["visibility"] = (time.perf_counter() - t) * V / vs
    # the FP64 shading oracle evaluates every (Gaussian, light) pair whatever
    # the visibility, so a constant count stands in for the full visibility
    campos = cam.centre.astype(np.float32)
    front = cpu.front_f32(xo, no, campos)
    ns = 1000
    idx = np.nonzero(front)[0][:ns]
    cnt_full = np.full((s["nv"], V), s["kv"] // 2, np.uint8)
    t = time.perf_counter()
    xs = torch.tensor(xo[:, idx].astype(np.float64), requires_grad=True)
    nsv = torch.tensor(no[:, idx].astype(np.float64), requires_grad=True)
    alb = torch.tensor(s["albedo"][:, idx].astype(np.float64), requires_grad=True)
    rough = torch.tensor(s["rough"][idx].astype(np.float64), requires_grad=True)
    tint = torch.tensor(s["tint"][idx].astype(np.float64), requires_grad=True)
    env = torch.tensor(s["env"].astype(np.float64), requires_grad=True)
    col, _ = ref64.shade(xs, nsv, alb, rough, tint, s["vidx"][:, idx], s["vw"][:, idx], cnt_full,
                         s["kv"], s["he"], s["we"], s["hv"], s["wv"], env, campos.astype(np.float64),
                         front[idx])
    col.sum().backward()
    parts["shading"] = (time.perf_counter() - t) * n / len(idx)
    colf = np.random.default_rng(0).random((3, n)).astype(np.float32)
    t = time.perf_counter()
    pre = cpu.splat_preprocess(cam, xo, Ao, s["quat"], s["log_s"], s["opac"], front)
    keys, vals, ranges = cpu.splat_bin(cam, pre)
    cpu.composite_tiles(cam, ranges, vals, pre, s["opac"], colf)
    parts["splat_fp32"] = time.perf_counter() - t
    npx = 4096
    pix = np.random.default_rng(1).choice(H * W, npx, replace=False)
    t = time.perf_counter()
    q = {k: torch.tensor(np.asarray(s[k], np.float64), requires_grad=True)
         for k in ("quat", "log_s", "opac")}
    xt = torch.tensor(xo.astype(np.float64), requires_grad=True)
    ct = torch.tensor(colf.astype(np.float64), requires_grad=True)
    proj = ref64.project(cam, xt, torch.tensor(Ao.astype(np.float64)), q["quat"], q["log_s"],
                         q["opac"], front)
    img, _ = ref64.composite(cam, proj, q["opac"], ct, pixels=pix)
    img.sum().backward()
    parts["splat_fp64_fwd_bwd"] = (time.perf_counter() - t) * (H * W) / npx
    total_ms = sum(parts.values()) * 1e3
    return {"value": round(total_ms, 1), "unit": "ms/iter", "cores": max(cpu.num_threads(),
                                                                          torch.get_num_threads()),
            "cpu_model": cpu_model(), "kind": "oracle",
            "sample": f"one step of the same workload, timed in parts and scaled: skinning (all), "
                      f"visibility {vs}/{V} views, FP64 shading fwd+bwd {len(idx)}/{n} Gaussians, "
                      f"FP32 projection+binning+compositing (all), FP64 compositing fwd+bwd "
                      f"{npx}/{H * W} pixels",
            "parts_s": {k: round(v, 3) for k, v in parts.items()}}


def knn_measure(s, d, reps: int = 20):
    """The neighbour search and the average of the interpolation equation
    (Sec. 3.1) at the workload's sizes, outside the timed step: K_g = 3
    nearest canonical vertices of every Gaussian, K_v = 19 of every vertex,
    and the average of 42 attribute channels (r 4, s 3, n 3, a 3, gamma,
    p, w 24, dx 3) with its adjoint.  Sums of kernel times from HIP events,
    per call."""
    import torch
    from paper_2407_10707_amd import rga
    n, nv = int(s["n"]), int(s["nv"])
    attr = torch.rand((42, nv), device="cuda")
    dout = torch.rand((42, n), device="cuda")
    index = rga.KnnIndex(d["verts"])
    idx, w = rga.knn(index, d["pos"], 3)

    def timed(fn):
        torch.cuda.synchronize()
        rga.timing_reset()
        rga.timing_filter(None)
        rga.timing_enable(True)
        for _ in range(reps):
            fn()
        torch.cuda.synchronize()
        rga.timing_enable(False)
        tot = 0.0
        for name in ("knn_bounds", "knn_count", "knn_scan", "knn_fill", "knn_qzero", "knn_qcell",
                     "knn_qscan", "knn_qfill", "knn_query", "knn_query_wide", "knn_interp",
                     "knn_interp_zero", "knn_interp_bwd"):
            tot += rga.timing_read(name)[0]
        return round(tot / reps, 4)

    return {"refs": nv, "queries": n, "k_g": 3, "k_v": 19, "channels": 42,
            "build_ms": timed(lambda: rga.KnnIndex(d["verts"])),
            "gaussian_query_ms": timed(lambda: rga.knn(index, d["pos"], 3)),
            "vertex_query_ms": timed(lambda: rga.knn(index, d["verts"], 19)),
            "interp_ms": timed(lambda: rga.knn_interpolate(idx, w, attr)),
            "interp_bwd_ms": timed(lambda: rga.knn_interpolate_backward(idx, w, dout, nv))}


def mlp_measure(d, reps: int = 20):
    """The displacement network d(x, theta) (Sec. 3.1 attributes, Sec. 3.5
    details) on the workload's canonical vertices and on a mesh of the
    paper's size (about 40K vertices), outside the timed step: forward (the
    operand packing included) and adjoint, sums of kernel times from HIP
    events per call, and the algorithmic rate (2 flops per multiply-add of
    the layer products; the split form issues three MFMAs per product)
    against the dense bf16 MFMA peak."""
    import numpy as np
    import torch
    from paper_2407_10707_amd import rga, synth
    inp = synth.mlp_inputs(0)
    theta = torch.as_tensor(inp["thetas"][0]).cuda()
    params = torch.as_tensor(inp["params"]).cuda()
    freqs = torch.as_tensor(inp["freqs"]).cuda()
    W = 256
    per_v_fwd = 2 * (128 * W + 3 * W * W + W * 3)
    per_v_bwd = 2 * (3 * W + 3 * W * W) + per_v_fwd

    def timed(fn, names):
        torch.cuda.synchronize()
        rga.timing_reset()
        rga.timing_filter(None)
        rga.timing_enable(True)
        for _ in range(reps):
            fn()
        torch.cuda.synchronize()
        rga.timing_enable(False)
        return sum(rga.timing_read(nm)[0] for nm in names) / reps

    def one(x):
        net = rga.Displacement(x, freqs)
        nv = net.nv
        ddx = torch.rand((3, nv), device="cuda")
        net.forward(theta, params)
        f = timed(lambda: net.forward(theta, params), ("mlp_pack", "mlp_fwd"))
        b = timed(lambda: net.backward(ddx),
                  ("mlp_bwd", "mlp_wgrad", "mlp_wgrad_io", "mlp_reduce", "mlp_dtheta"))
        tf, tb = per_v_fwd * nv / f / 1e9, per_v_bwd * nv / b / 1e9
        return {"vertices": nv, "fwd_ms": round(f, 4), "bwd_ms": round(b, 4),
                "fwd_tflops": round(tf, 2), "bwd_tflops": round(tb, 2),
                "fwd_frac_bf16_peak": round(tf / 2500.0, 4),
                "bwd_frac_bf16_peak": round(tb / 2500.0, 4)}

    verts, _ = synth.body_mesh(48, 46)
    big = torch.as_tensor(np.ascontiguousarray(verts.T), dtype=torch.float32).cuda()
    return {"workload_mesh": one(d["verts"]), "paper_size_mesh": one(big)}


def image_loss_measure(s, reps: int = 20):
    """The image loss of the training section ((1 - lambda) L1 + lambda
    D-SSIM, lambda = 0.2) with its adjoint at the workload's image size,
    outside the timed step (the step's loss is L1): kernel times per call
    and the rate of the algorithmic HBM bytes (forward: image and target
    read, three derivative maps written; adjoint: the maps, image and
    target read, the gradient written; 36 B per value) against 8 TB/s."""
    import numpy as np
    import torch
    from paper_2407_10707_amd import rga
    H, W = int(s["height"]), int(s["width"])
    rng = np.random.default_rng(3)
    x = torch.tensor(rng.random((3, H, W)), dtype=torch.float32).cuda()
    y = torch.tensor(rng.random((3, H, W)), dtype=torch.float32).cuda()
    rga.image_loss(x, y)
    torch.cuda.synchronize()
    rga.timing_reset()
    rga.timing_filter(None)
    rga.timing_enable(True)
    for _ in range(reps):
        rga.image_loss(x, y)
    torch.cuda.synchronize()
    rga.timing_enable(False)
    ms = sum(rga.timing_read(nm)[0] for nm in ("ssim_fwd", "ssim_final", "ssim_bwd")) / reps
    gbs = 36.0 * 3 * H * W / (ms * 1e-3) / 1e9
    return {"image": [3, H, W], "lambda": 0.2, "fwd_bwd_ms": round(ms, 4),
            "gb_per_s": round(gbs, 1), "frac_hbm_peak": round(gbs / 8000.0, 4)}


def densify_measure(s, d, reps: int = 20):
    """Density-based densification (App. B, Alg. 1) over the workload's
    Gaussians and mesh, outside the timed step (it runs every hundred
    iterations): the paper's d0 = 1, p0 = 0.02, and a threshold at the
    densities' 70th percentile with p0 = 0.5 (thousands of draws).  Kernel
    times per call; algorithmic bytes: the K_g lists read (12 B per
    Gaussian), per triangle its indices, three counts, d_f and the
    cumulative weight (36 B), per draw about 40 B."""
    import numpy as np
    import torch
    from paper_2407_10707_amd import rga
    sg = torch.as_tensor(np.ascontiguousarray(s["vidx"])).cuda()
    verts, faces = d["verts"], torch.as_tensor(np.ascontiguousarray(s["faces"])).cuda()
    base = rga.densify(sg, verts, faces)
    q70 = float(torch.quantile(base["df"].double(), 0.7))
    out = {"gaussians": int(s["n"]), "triangles": int(s["nf"])}
    for tag, d0, p0 in (("paper", 1.0, 0.02), ("q70", q70, 0.5)):
        r = rga.densify(sg, verts, faces, d0=d0, p0=p0, seed=1, cap=1 << 16)
        torch.cuda.synchronize()
        rga.timing_reset()
        rga.timing_filter(None)
        rga.timing_enable(True)
        for _ in range(reps):
            rga.densify(sg, verts, faces, d0=d0, p0=p0, seed=1, cap=1 << 16, sync=False)
        torch.cuda.synchronize()
        rga.timing_enable(False)
        ms = sum(rga.timing_read(nm)[0] for nm in ("densify_clear", "densify_count",
                                                      "densify_faces", "densify_draw")) / reps
        nbytes = 12 * int(s["n"]) + 36 * int(s["nf"]) + 40 * r["n_added"]
        out[tag] = {"d0": round(d0, 4), "p0": p0, "added": r["n_added"], "ms": round(ms, 4),
                    "gb_per_s": round(nbytes / (ms * 1e-3) / 1e9, 1)}
    return out


def kernel_times(step, names, reps=5):
    """{name: ms per launch} of those of the named kernels that step() launches."""
    import torch

    from paper_2407_10707_amd import rga
    out = {}
    for name in names:
        rga.timing_reset()
        rga.timing_filter(name)
        rga.timing_enable(True)
        for _ in range(reps):
            step()
        torch.cuda.synchronize()
        rga.timing_enable(False)
        ms, cnt = rga.timing_read(name)
        if cnt:
            out[name] = ms / cnt
    return out


def measure_form(args, s, d, precision: str, capacity=None):
    """Time the step of one precision form: sizes the splat workspace to the
    frame's duplicates, runs the warm-up, times exactly `args.steps` steps
    (and the shading adjoint inside them with HIP events on its stream),
    then the forward-only frame rates.  Returns (result, renderer, step)."""
    import numpy as np
    import torch

    from paper_2407_10707_amd import render, rga, synth
    cfg = s["cfg"]
    R = render.Renderer(s, d, precision=precision, capacity=capacity)
    p = {k: d[k] for k in render.TRAINABLE}
    target = d["target"]

    frames = cfg.n_pose * cfg.n_env if args.sequence else 1
    if args.sequence:
        skins = [torch.as_tensor(synth.pose_skin(args.config, k).reshape(-1, 12)
                                 .astype(np.float32)).cuda() for k in range(cfg.n_pose)]
        envs = [torch.as_tensor(synth.env_map(args.config, e).astype(np.float32)).cuda()
                for e in range(cfg.n_env)]
        env0 = p["env"]
        skin0 = R.d["skin"]
    seq = {"frame": 0, "count": None}

    def step():
        if not args.sequence:
            # the visibility of the pose is computed inside the frame,
            # beside the binning of the splats
            loss, grads = R.train_step(p, None, target, check=False)
            return loss
        k, e = divmod(seq["frame"] % frames, cfg.n_env)
        seq["frame"] += 1
        if e == 0 or seq["count"] is None:
            R.d["skin"] = skins[k]
            seq["count"] = R.visibility()
        p["env"] = envs[e]
        loss, grads = R.train_step(p, seq["count"], target, check=False)
        return loss

    def fwd(with_vis, count=None):
        # a frame for display: no tape for an adjoint
        _, _, ctx = R.forward(p, None if with_vis else count, for_backward=False)
        return ctx["count"]

    # size the splat workspace to the real duplicate count (every pose of a
    # sequence), then start the sequence again at frame 0
    Ds = []
    for _ in range(frames):
        step()
        while R.ensure_capacity():
            seq["frame"] -= 1
            step()
        Ds.append(R.ws.count())
    D = max(Ds)
    seq["frame"] = 0
    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()

    run = step
    if args.graph:
        # capture one whole step; replays re-run every kernel of the step
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            for _ in range(3):
                step()
        torch.cuda.current_stream().wait_stream(side)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            step()
        torch.cuda.synchronize()
        run = graph.replay

    # the roofline entries are the blend adjoint and the shading kernel of
    # the form (the FP32 adjoint, or the BF16X3 form's forward: both forms'
    # adjoints replay the tape), which is timed on a few eager steps after
    # the timed region; the longer of the two becomes the entry
    if args.kernel:
        kernels = [args.kernel]
    elif precision == "bf16x3":
        kernels = ["blend_bwd", "shade_fwd", "shade_fwd_bf16x3"]   # (one of the two runs)
    else:
        kernels = ["blend_bwd", "shade_bwd"]
    kernel = kernels[0]
    rga.timing_reset()
    rga.timing_filter(None if args.all_kernels else kernel)
    rga.timing_enable(not args.graph)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(args.steps):
        run()
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    rga.timing_enable(False)
    ms_step = (t1 - t0) * 1e3 / args.steps
    k_ms, k_n = rga.timing_read(kernel)
    if k_n == 0:          # graph replay: time the kernel on a few eager steps instead
        rga.timing_filter(kernel)
        rga.timing_enable(True)
        for _ in range(5):
            step()
        torch.cuda.synchronize()
        rga.timing_enable(False)
        k_ms, k_n = rga.timing_read(kernel)
    if k_n == 0:
        raise SystemExit(f"bench.py: kernel {kernel!r} was not launched in the timed steps")
    per_kernel = {}
    if args.all_kernels:
        for name in ("lbs_fwd", "vis_frame", "vis_raster", "vis_transpose", "vis_majority",
                     "vis_count", "shade_fwd", "shade_fwd_bf16x3", "splat_fill", "back_face",
                     "splat_preprocess", "radix_upsweep", "radix_binscan", "radix_downsweep",
                     "touched_sum", "rank_sort", "splat_duplicate", "tile_ranges",
                     "blend", "l1_partial", "l1_final", "blend_bwd", "preprocess_bwd", "shade_bwd",
                     "shade_bwd_bf16x3", "shade_denv", "lbs_bwd"):
            ms, cnt = rga.timing_read(name)
            if cnt:
                per_kernel[name] = round(ms / args.steps, 4)
        per_kernel["sum_of_kernels"] = round(sum(per_kernel.values()), 4)
    k_avg = {kernel: k_ms / k_n}
    timed_where = {kernel: "timed region"}
    others = kernel_times(step, kernels[1:])
    k_avg.update(others)
    timed_where.update({kn: "5 eager steps after the timed region" for kn in others})
    forward = list(kernel_times(step, ["shade_fwd", "shade_fwd_bf16x3"], 1))

    # forward-only frame rates (visibility per frame, and cached per pose;
    # a sequence recomputes visibility once per pose)
    seq["frame"] = 0
    if args.sequence:
        R.d["skin"] = skins[0]
        p["env"] = envs[0]
    count = R.visibility()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for i in range(args.steps):
        if args.sequence:
            k, e = divmod(i % frames, cfg.n_env)
            R.d["skin"] = skins[k]
            p["env"] = envs[e]
            count = fwd(e == 0, count)
        else:
            fwd(True)
    torch.cuda.synchronize()
    fps = args.steps / (time.perf_counter() - t0)
    if args.sequence:
        R.d["skin"] = skins[0]
        p["env"] = envs[0]
        count = R.visibility()
    t0 = time.perf_counter()
    for _ in range(args.steps):
        fwd(False, count)
    torch.cuda.synchronize()
    fps_nv = args.steps / (time.perf_counter() - t0)

    # algorithmic work of the timed kernels: (Gaussian, direction) pairs of
    # the shading, (pixel, splat) pairs of the compositing; the splat state
    # read here is that of the last fwd+bwd step
    wl = shading_pairs(s, R, p, count)
    st = R.ws.state()
    D = R.ws.count()
    n = s["n"]
    tiles = int(st.tiles_x) * int(st.tiles_y)
    bp = blend_pairs(R.ws.view(st.mean2d, (2, n), torch.float32),
                     R.ws.view(st.conic, (3, n), torch.float32), p["opac"],
                     R.ws.view(st.sorted, (max(D, 1),), torch.int32),
                     R.ws.view(st.ranges, (tiles, 2), torch.int32), R.cam.width, R.cam.height)

    def roofline_of(kn):
        if kn.startswith("shade_bwd") or kn.startswith("shade_fwd"):
            # the renderer's adjoint replays the forward's tape
            replay = kn == "shade_bwd" and R.tape is not None
            flops = shade_flops(wl["live"], wl["tested"], kn.startswith("shade_bwd"),
                                tested=not replay)
            work = {"tested_pairs": 0 if replay else wl["tested"], "live_pairs": wl["live"]}
        elif kn == "blend_bwd":
            flops = blend_bwd_flops(bp["walked"], bp["applied"])
            work = {"walked_pixel_splat_pairs": bp["walked"],
                    "applied_pixel_splat_pairs": bp["applied"]}
        else:
            return None
        ach = flops / (k_avg[kn] * 1e-3) / 1e12
        work["flops_per_launch"] = flops
        return {"bound": "alu", "achieved": round(ach, 3), "peak": PEAK_FP32_TFLOPS,
                "unit": "TFLOP/s", "frac": round(ach / PEAK_FP32_TFLOPS, 4),
                "traffic": traffic_from_profile(kn, args.config),
                "kernel": kn, "kernel_ms": round(k_avg[kn], 4), "timed": timed_where[kn],
                "work": work}

    roofs = sorted((r for r in (roofline_of(kn) for kn in k_avg) if r is not None),
                   key=lambda r: -r["kernel_ms"])
    roof = roofs[0] if roofs else None
    roof_other = roofs[1] if len(roofs) > 1 else None
    # this frame's image (pose 0, map 0) for the image-error report
    image, _, _ = R.forward(p, count)
    torch.cuda.synchronize()
    if args.sequence:
        R.d["skin"] = skin0
        p["env"] = env0
    out = {"ms_per_step": round(ms_step, 4), "render_fps": round(fps, 2),
           "render_fps_no_vis": round(fps_nv, 2), "duplicates": D,
           "sequence_frames": frames if args.sequence else None, "roofline": roof,
           "roofline_other": roof_other, "shading_forward": forward[0]}
    if per_kernel:
        out["per_kernel_ms_per_step"] = per_kernel
    return out, R, p, step, image.cpu().numpy()


def main():
    args = parse()
    if args.gpus != 1:
        print(f"bench.py runs on one GPU only (asked for {args.gpus}): the library has no "
              "multi-GPU path", file=sys.stderr)
        sys.exit(2)
    import numpy as np
    import torch

    from paper_2407_10707_amd import render, rga, synth

    assert torch.cuda.is_available(), "bench.py needs a GPU"
    torch.cuda.set_device(0)
    rga.lib()
    s = synth.make_scene(args.config)
    cfg = s["cfg"]
    # the Gaussians stored grouped by nearest vertex (on the device, before
    # the timed region; the host mirror follows the same order)
    d, order = render.layout_by_vertex(render.upload(s))
    s = render.scene_in_order(s, order)
    target = d["target"]

    if args.copy_calibration:
        # a plain copy of known size (256 MiB read, 256 MiB written): its
        # FETCH_SIZE / WRITE_SIZE counters calibrate the path kernels' counters
        src = torch.ones(64 * 1024 * 1024, dtype=torch.float32, device="cuda")
        dst = torch.empty_like(src)
        for _ in range(3):
            dst.copy_(src)
        torch.cuda.synchronize()
        del src, dst

    head, R, p, step, image = measure_form(args, s, d, args.precision)
    images = {args.precision: image}
    other = None
    if not args.one_form:
        # the other precision form of the shading contraction, same frame
        oform = "bf16x3" if args.precision == "fp32" else "fp32"
        okw = argparse.Namespace(**vars(args))
        okw.kernel = None
        okw.all_kernels = False
        other, R2, _, _, oimage = measure_form(okw, s, d, oform, capacity=R.ws.capacity)
        images[oform] = oimage
        del R2

    # the same step with the image loss of the training section in place of
    # L1 (outside the timed region above; the metric keeps the L1 step)
    R.image_loss = True
    for _ in range(3):
        step()
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    for _ in range(args.steps):
        step()
    torch.cuda.synchronize()
    img_loss_step_ms = (time.perf_counter() - t1) * 1e3 / args.steps

    # a whole training iteration: the step with the image loss and an Adam
    # update of every trained tensor (a tiny learning rate; the parameters
    # are restored afterwards, so the figures above are unaffected)
    saved = {k: t.clone() for k, t in p.items()}
    mom = {k: (torch.zeros_like(t), torch.zeros_like(t)) for k, t in p.items()}

    def train_iter(it):
        _, grads = R.train_step(p, None, target, check=False)
        for k, (m1, m2) in mom.items():
            if k in grads:
                rga.adam_step(p[k], grads[k], m1, m2, 1e-7, it)

    for it in range(1, 4):
        train_iter(it)
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    for it in range(4, 4 + args.steps):
        train_iter(it)
    torch.cuda.synchronize()
    full_iter_ms = (time.perf_counter() - t1) * 1e3 / args.steps
    for k, t in saved.items():
        p[k].copy_(t)

    # the same iteration in the paper's parametrisation: materials and the
    # network's displacement on the vertices, interpolated to the Gaussians
    # (K_g = 3 search every iteration), skinning from the pose, and the
    # adjoint back to theta, the network and the vertex attributes
    skin0 = R.d["skin"].clone()
    vin = synth.mlp_inputs(0)
    vparams = vin["params"].copy()
    vparams[-(3 * 256 + 3):] *= 0.01
    M = render.VertexModel(R, torch.as_tensor(vin["freqs"]).cuda(),
                           torch.as_tensor(synth.JOINTS_REST, dtype=torch.float32).cuda(),
                           torch.as_tensor(synth.PARENTS, dtype=torch.int32).cuda())
    vrng = np.random.default_rng(21)
    nvert = int(d["verts"].shape[1])
    vv = dict(theta=torch.as_tensor(0.2 * vrng.standard_normal((24, 3)), dtype=torch.float32).cuda(),
              mlp=torch.as_tensor(vparams).cuda(),
              v_albedo=torch.as_tensor(vrng.random((3, nvert)), dtype=torch.float32).cuda(),
              v_rough=torch.as_tensor(vrng.uniform(0.2, 0.9, nvert), dtype=torch.float32).cuda(),
              v_tint=torch.as_tensor(vrng.random(nvert), dtype=torch.float32).cuda(),
              pos=p["pos"], nrm=p["nrm"], quat=p["quat"], log_s=p["log_s"], opac=p["opac"],
              env=p["env"])

    def vertex_iter():
        # the total loss of Sec. 3.3: the image loss plus the weighted
        # regularisers, whose gradients the library adds to the image loss's
        image, _, ctx = M.forward(vv, None)
        loss, dimage = R.loss(image, target)
        M.backward(vv, ctx, dimage, loss=loss)

    vertex_iter()
    R.ensure_capacity()
    for _ in range(2):
        vertex_iter()
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    for _ in range(args.steps):
        vertex_iter()
    torch.cuda.synchronize()
    vertex_iter_ms = (time.perf_counter() - t1) * 1e3 / args.steps
    R.d["skin"] = skin0
    R.image_loss = False

    knn = knn_measure(s, d)
    mlp = mlp_measure(d)
    img_loss = image_loss_measure(s)
    dens = densify_measure(s, d)

    cpu = None
    err = None
    if not args.no_cpu_baseline:
        cpu = cpu_baseline(s)
        if not args.sequence:
            err = image_error(s, images)

    out = {
        "metric": METRIC,
        "value": head["ms_per_step"],
        "unit": "ms/iter",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": head["ms_per_step"],
        "higher_is_better": False,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f32",
        "data": "synthetic",
        "config": {"workload": cfg.name, "gaussians": s["n"], "mesh_vertices": s["nv"],
                   "mesh_triangles": s["nf"], "joints": 24, "light_directions": cfg.he * cfg.we,
                   "vis_views": cfg.hv * cfg.wv, "vis_res": cfg.vis_res,
                   "image": [s["height"], s["width"]], "precision": args.precision,
                   "layout": "gaussians grouped by nearest vertex"},
        "graph": bool(args.graph),
        "render_fps": head["render_fps"],
        "render_fps_no_vis": head["render_fps_no_vis"],
        "duplicates": head["duplicates"],
        "sequence_frames": head["sequence_frames"],
        "roofline": head["roofline"],
        "roofline_other": head["roofline_other"],
        "shading_forward": head["shading_forward"],
        "cpu_baseline": cpu,
    }
    if other is not None:
        oform = "bf16x3" if args.precision == "fp32" else "fp32"
        out[oform] = {k: other[k] for k in ("ms_per_step", "render_fps", "render_fps_no_vis",
                                            "roofline", "roofline_other", "shading_forward")}
    out["image_error_vs_fp64"] = err
    out.update({
        "knn": knn,
        "displacement_mlp": mlp,
        "image_loss": dict(img_loss, step_ms_with_image_loss=round(img_loss_step_ms, 4)),
        "densify": dens,
        "training_iteration_ms": round(full_iter_ms, 4),
        "vertex_model_iteration_ms": round(vertex_iter_ms, 4),
    })
    if "per_kernel_ms_per_step" in head:
        out["per_kernel_ms_per_step"] = head["per_kernel_ms_per_step"]
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
