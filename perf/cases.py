"""Performance cases of the detector library: whole frames over the range of
workloads the library is configured for, and rotated NMS on caller records.

A frame case is what a perception server does per frame: begin the frame,
release the branches (one by one as their inputs arrive, all at once, or at
the barrier), join, and read the detections back.  The sizes are those of the
repository's workload descriptions (two agents on a 64 x 64 grid up to eight
agents with 100,000 points each on a 512 x 512 grid) and the ranges between
them, with every option a server uses in earnest: release rule, input location,
executor, HIP graphs, fusion rule, placement of the warp, multi-scale fusion.

bf16 frames return the raw head outputs (the logits and box residuals; the
whole map, as rtcc_get_tensor gives it) and the set of kept anchors as a mask;
the float32 frames return the detections themselves.  NMS cases return the
caller's output buffer, the kept records first.
"""

import math
import time

import numpy as np
import torch

from paper_2608_08330_amd import rtcc as R

# PointPillars networks: point-feature channels, (stride, channels, convs) of
# every stage, upsampling channels (0: the slot is the last stage's output)
NETS = {
    "tiny": (32, ((1, 32, 2),), 0),
    "small": (64, ((2, 64, 2), (2, 128, 2), (2, 256, 2)), 128),
    "pp64": (64, ((2, 64, 3), (2, 128, 5), (2, 256, 5)), 128),
    "pp128": (64, ((2, 128, 3), (2, 256, 5), (2, 256, 5)), 128),
}
# class-logit threshold of drawn frames; with these weights it passes between
# a few anchors and some per cent of them (the listed frames state their own,
# which about 1% pass, as in the repository's workloads)
THRESHOLD = {"tiny": 0.85, "small": 1.3, "pp64": 0.42, "pp128": 0.85}
ANCHOR = dict(w=1.6, l=3.9, h=1.5, z=-1.0, yaw=(0.0, math.pi / 2.0))
Z_RANGE = (-3.0, 1.0)
MAX_PTS = 32
NMS_CAP = 4096
NMS_IOU = 0.15


def _frame(**kw):
    c = dict(kind="frame", net="pp64", agents=4, points=20000, x_half=51.2, y_half=51.2, pillar=0.4,
             precision="bf16", fusion="attn", release="batch", inputs="device", executor="streams",
             graphs=False, warp_in_branch=False, multiscale=False)
    c.update(kw)
    c.setdefault("threshold", THRESHOLD[c["net"]])
    return c


def listed():
    return [
        # two agents, float32, max fusion, 64 x 64 cells: the smallest
        # workload, where launches and the host path are all there is;
        # inputs already in pinned staging, released as they arrive
        _frame(name="frame_2x2k_fp32", net="tiny", agents=2, points=2000, x_half=25.6, y_half=25.6, pillar=0.8,
               precision="fp32", fusion="max", release="each", inputs="staged", threshold=0.9),
        # four agents around a 44 x 60 ragged grid (partial tiles and a
        # cropped upsampling everywhere), graphs, released as they arrive
        _frame(name="frame_4x6k_ragged", net="small", agents=4, points=6000, x_half=12.0, y_half=8.8,
               release="each", inputs="staged", graphs=True, threshold=1.55),
        # three agents, max fusion, 256 x 256 cells, inputs on the device
        _frame(name="frame_3x20k_max", agents=3, points=20000, fusion="max", graphs=True, threshold=0.4),
        # five agents on the 352 x 100 road strip, each released by its own
        # completion event from host memory: the uplink-triggered use
        _frame(name="frame_5x40k_each", agents=5, points=40000, x_half=70.4, y_half=20.0, release="each",
               inputs="staged", threshold=0.62),
        # six agents with about 64 KiB of points each, the barrier baseline
        # on the single-stream executor (the measured-DAG sweep)
        _frame(name="frame_6x4k_barrier", agents=6, points=4027, x_half=70.4, y_half=20.0, release="barrier",
               inputs="host", executor="serial", threshold=0.18),
        # three agents, odd point count, the warp as each branch's last node
        _frame(name="frame_3x33k_prewarp", agents=3, points=33333, x_half=70.4, y_half=20.0,
               warp_in_branch=True, inputs="host", threshold=0.63),
        # four agents, the multi-scale fusion shape on a 312 x 248 grid
        _frame(name="frame_4x30k_multiscale", agents=4, points=30011, x_half=62.4, y_half=49.6, multiscale=True,
               graphs=True, threshold=0.51),
        # eight agents, 512 x 512 cells, 100,000 points each: the stress
        # workload, all inputs resident and released together (throughput)
        _frame(name="frame_8x100k", net="pp128", agents=8, points=100000, pillar=0.2, graphs=True),
        # the same frame branch by branch from pinned staging (latency use)
        _frame(name="frame_8x100k_each", net="pp128", agents=8, points=100000, pillar=0.2, release="each",
               inputs="staged", graphs=True),
        # rotated NMS of caller records: a sparse scene, a usual frame's
        # decoded boxes, and a dense low-threshold scene
        dict(name="nms_90", kind="nms", records=90, cap=NMS_CAP, per_object=3, entry="noalloc"),
        dict(name="nms_1400", kind="nms", records=1400, cap=NMS_CAP, per_object=6, entry="noalloc"),
        dict(name="nms_30000", kind="nms", records=30000, cap=NMS_CAP, per_object=24, entry="alloc"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges: a fifth NMS sizes, the rest frames
    from the tiny network up to seven agents on the stress network."""
    r = rng.random()
    if r < 0.2:
        return dict(kind="nms", records=_log(rng, 40, 60000), cap=rng.choice((512, 1000, NMS_CAP)),
                    per_object=rng.randint(1, 30), entry=rng.choice(("alloc", "noalloc")))
    common = dict(release=rng.choice(("batch", "each", "barrier")), inputs=rng.choice(("device", "host", "staged")),
                  executor=rng.choice(("streams", "streams", "serial")), graphs=rng.random() < 0.5,
                  fusion=rng.choice(("attn", "max")))
    if r < 0.35:
        return _frame(net="tiny", agents=rng.randint(1, 8), points=_log(rng, 200, 20000),
                      x_half=0.8 * rng.randint(12, 64), y_half=0.8 * rng.randint(12, 64), pillar=0.8,
                      **dict(common, precision="fp32", fusion="max"))
    shape = rng.choice(("post", "post", "warp", "multi"))
    common.update(warp_in_branch=shape == "warp", multiscale=shape == "multi")
    if r < 0.5:
        return _frame(net="small", agents=rng.randint(1, 8), points=_log(rng, 500, 20000),
                      x_half=0.4 * rng.randint(20, 80), y_half=0.4 * rng.randint(20, 80), **common)
    if r < 0.85:
        return _frame(net="pp64", agents=rng.randint(1, 8), points=_log(rng, 1500, 60000),
                      x_half=0.4 * rng.randint(64, 180), y_half=0.4 * rng.randint(48, 128), **common)
    return _frame(net="pp128", agents=rng.randint(1, 7), points=_log(rng, 10000, 100000),
                  x_half=0.2 * rng.randint(160, 256), y_half=0.2 * rng.randint(100, 256), pillar=0.2, **common)


# ------------------------------------------------------------------ shapes

def _grid(case):
    return (int(round(2 * case["y_half"] / case["pillar"])), int(round(2 * case["x_half"] / case["pillar"])))


def _counts(case):
    """Points of every agent: no two alike, the last a few per cent fewer."""
    n, K = case["points"], case["agents"]
    return [max(1, n - (k * n) // 200) for k in range(K)]


def _layers(case):
    """(conv layers, stage grids): (Hi, Wi, Ci, Ho, Wo, Co, stride) each."""
    c_pfn, stages, _up = NETS[case["net"]]
    h, w = _grid(case)
    c, convs, out = c_pfn, [], []
    for stride, co, n in stages:
        for l in range(n):
            s = stride if l == 0 else 1
            ho, wo = -(-h // s), -(-w // s)
            convs.append((h, w, c, ho, wo, co, s))
            h, w, c = ho, wo, co
        out.append((h, w, c))
    return convs, out


def work(case):
    if case["kind"] == "nms":
        n = case["records"]
        m = min(n, case["cap"])
        # records read once, about one in per_object written; one IoU (about
        # 400 operations) per suppressed candidate is the least a greedy walk does
        return {"bytes": 36.0 * n + 36.0 * m / case["per_object"], "flops": 400.0 * m}
    elt = 2 if case["precision"] == "bf16" else 4
    c_pfn, stages, up = NETS[case["net"]]
    K = case["agents"]
    convs, grids = _layers(case)
    H2, W2 = grids[0][0], grids[0][1]
    C = up * len(stages) if up else grids[-1][2]
    flops = sum(2.0 * 4 * c_pfn * n for n in _counts(case))
    flops += K * sum(2.0 * ho * wo * co * 9 * ci for (_h, _w, ci, ho, wo, co, _s) in convs)
    if up:
        flops += (1 if case["multiscale"] else K) * sum(2.0 * H2 * W2 * cs * up for (_h, _w, cs) in grids)
    flops += 2.0 * H2 * W2 * C * 16
    cells = sum(h * w * c for h, w, c in grids) if case["multiscale"] else H2 * W2 * C
    flops += cells * K * (8.0 + (4.0 if case["fusion"] == "attn" else 1.0))
    weights = sum(9 * ci * co for (_h, _w, ci, _ho, _wo, co, _s) in convs)
    if up:
        u = 1
        for s, (_h, _w, cs) in enumerate(grids):
            u *= stages[s][0] if s else 1
            weights += u * u * cs * up
    weights += 16 * C
    return {"bytes": 16.0 * sum(_counts(case)) + elt * weights + 64.0 * H2 * W2, "flops": flops}


# ------------------------------------------------------------------ inputs

def _points(rng, n, case):
    """A LiDAR-like cloud: 70% ground returns, 30% on objects; the tiny
    network's recipe is a uniform cloud."""
    xh, yh = case["x_half"], case["y_half"]
    p = np.empty((n, 4), dtype=np.float32)
    p[:, 0] = rng.uniform(-xh, xh, n)
    p[:, 1] = rng.uniform(-yh, yh, n)
    p[:, 3] = rng.random(n)
    if case["net"] == "tiny":
        p[:, 2] = rng.uniform(Z_RANGE[0], Z_RANGE[1], n)
        return p
    p[:, 2] = rng.normal(-1.7, 0.05, n)
    objects = max(1, -(-(n - int(0.7 * n)) // 200))
    at = np.stack([rng.uniform(-xh, xh, objects), rng.uniform(-yh, yh, objects), rng.uniform(-1.7, 0.0, objects)], 1)
    hit = rng.random(n) < 0.3
    m = int(hit.sum())
    p[hit, :3] = at[rng.integers(0, objects, m)] + rng.normal(0.0, 0.5, (m, 3))
    return p


def _scene(case, seed):
    rng = np.random.default_rng([seed, 11])
    K = case["agents"]
    poses = np.zeros((K, 3))
    poses[1:, 0] = rng.uniform(-math.pi, math.pi, K - 1)
    poses[1:, 1:] = rng.uniform(-5.0, 5.0, (K - 1, 2))
    return [_points(rng, n, case) for n in _counts(case)], poses


def _weights(case):
    """The network's parameters by name: He-normal matrices, small biases;
    one fixed draw per network, as a trained network is fixed."""
    c_pfn, stages, up = NETS[case["net"]]
    rng = np.random.default_rng([20260830, sorted(NETS).index(case["net"])])
    w = {}

    def put(name, shape, fan):
        w[name + "_w"] = rng.standard_normal(shape, dtype=np.float32) * np.float32(math.sqrt(2.0 / fan))
        w[name + "_b"] = rng.standard_normal(shape[-1], dtype=np.float32) * np.float32(0.1)

    put("pfn", (4, c_pfn), 4)
    c = c_pfn
    for s, (_stride, co, n) in enumerate(stages):
        for l in range(n):
            ci = c if l == 0 else co
            put("s%dc%d" % (s, l), (3, 3, ci, co), 9 * ci)
        c = co
    u = 1
    for s, (stride, co, _n) in enumerate(stages):
        u *= stride if s else 1
        if up:
            put("up%d" % s, (u, u, co, up), co)
    C = up * len(stages) if up else c
    put("head", (C, 16), C)
    return w


def _config(case):
    """The library's workload description of a frame case."""
    c_pfn, stages, up = NETS[case["net"]]
    return dict(K=case["agents"], n_points=case["points"], x_range=(-case["x_half"], case["x_half"]),
                y_range=(-case["y_half"], case["y_half"]), z_range=Z_RANGE, pillar=case["pillar"], max_pts=MAX_PTS,
                c_pfn=c_pfn, precision=case["precision"], stages=stages, up_channels=up, fusion=case["fusion"],
                n_anchors=2, anchor_w=ANCHOR["w"], anchor_l=ANCHOR["l"], anchor_h=ANCHOR["h"], anchor_z=ANCHOR["z"],
                anchor_yaws=ANCHOR["yaw"], logit_threshold=case["threshold"], nms_max_candidates=NMS_CAP,
                nms_iou_threshold=NMS_IOU, warp_in_branch=case["warp_in_branch"], multiscale=case["multiscale"])


def _records(case, seed):
    """Decoded boxes of a scene: per object a few jittered boxes, scores
    spread, in anchor order."""
    rng = np.random.default_rng([seed, 12])
    n = case["records"]
    objects = max(1, n // case["per_object"])
    at = rng.uniform(-51.2, 51.2, (objects, 2))
    yaw = rng.uniform(-math.pi, math.pi, objects)
    who = rng.integers(0, objects, n)
    rec = np.empty((n, 9), dtype=np.float32)
    rec[:, 0:2] = at[who] + rng.normal(0.0, 0.4, (n, 2))
    rec[:, 2] = rng.normal(-1.0, 0.2, n)
    rec[:, 3] = 1.6 * np.exp(rng.normal(0.0, 0.1, n))
    rec[:, 4] = 3.9 * np.exp(rng.normal(0.0, 0.1, n))
    rec[:, 5] = 1.5 * np.exp(rng.normal(0.0, 0.1, n))
    rec[:, 6] = yaw[who] + rng.normal(0.0, 0.1, n)
    rec[:, 7] = rng.uniform(0.5, 1.0, n)
    rec[:, 8] = np.sort(rng.choice(4 * n + 64, n, replace=False)).astype(np.int32).view(np.float32)
    return rec


def prepare(case, seed):
    if case["kind"] == "nms":
        rec = torch.from_numpy(_records(case, seed)).cuda()
        out = torch.zeros((case["cap"], 9), dtype=torch.float32, device="cuda")
        return dict(case=case, rec=rec, out=out)
    cfg = _config(case)
    opts = R.rtcc_runtime_opts()
    opts.exec = R.RTCC_EXEC_SERIAL if case["executor"] == "serial" else R.RTCC_EXEC_PER_BRANCH_STREAMS
    opts.use_graphs = int(case["graphs"])
    opts.premature_tol_s = 1e-6
    ctx = R.rtcc_create(R.model_desc(cfg), R.weights_blob(cfg, _weights(case)), opts)
    R.rtcc_set_mode(ctx, R.RTCC_MODE_BARRIER if case["release"] == "barrier" else R.RTCC_MODE_RELEASE)
    points, poses = _scene(case, seed)
    state = dict(case=case, ctx=ctx, points=points, poses=[tuple(p) for p in poses],
                 anchors=2 * int(np.prod(_layers(case)[1][0][:2])),
                 # fixed-capacity detections, as handed on to a tracker
                 boxes=np.zeros((NMS_CAP, 8), dtype=np.float32), anchor_idx=np.zeros(NMS_CAP, dtype=np.int32))
    if case["inputs"] == "device":
        state["points"] = [torch.from_numpy(p).cuda() for p in points]
        torch.cuda.synchronize()
    elif case["inputs"] == "staged":
        # the receiver filled the pinned buffers while the payload arrived
        state["points"] = []
        for k, p in enumerate(points):
            s = R.rtcc_staging_buffer(ctx, k)
            s[:len(p)] = p
            state["points"].append(s[:len(p)])
    return state


# ------------------------------------------------------------------ run

def run(state):
    case = state["case"]
    if case["kind"] == "nms":
        rec, out = state["rec"], state["out"]
        if case["entry"] == "noalloc":
            kept = R.rtcc_rotated_nms_noalloc(rec.data_ptr(), len(rec), case["cap"], NMS_IOU, out.data_ptr(),
                                              torch.cuda.current_stream().cuda_stream)
        else:
            kept = R.rtcc_rotated_nms(rec.data_ptr(), len(rec), case["cap"], NMS_IOU, out.data_ptr())
        return {"kept": kept, "records": out[:, :8], "anchor_idx": out.view(torch.int32)[:, 8]}
    ctx, points, poses = state["ctx"], state["points"], state["poses"]
    device = case["inputs"] == "device"
    R.rtcc_begin_frame(ctx, time.monotonic() - 1.0)
    if case["release"] == "batch":
        R.rtcc_release_branches(ctx, [
            dict(agent=k, device=1, points=p.data_ptr(), n=len(p), pose=poses[k], arrival_t=0.0) if device else
            dict(agent=k, points=p, pose=poses[k], arrival_t=0.0) for k, p in enumerate(points)])
    else:
        for k, p in enumerate(points):
            if device:
                R.rtcc_release_branch_device(ctx, k, p.data_ptr(), len(p), poses[k], 0.0)
            else:
                R.rtcc_release_branch(ctx, k, p, poses[k], 0.0)
    det = R.rtcc_join_and_detect(ctx)
    if case["precision"] == "fp32":
        n, boxes, idx = det["count"], state["boxes"], state["anchor_idx"]
        boxes[:n, :7] = det["boxes"]
        boxes[:n, 7] = det["scores"]
        idx[:n] = det["anchor_idx"]
        return {"count": n, "decoded": det["count_decoded"], "boxes": boxes, "anchor_idx": idx}
    kept = np.zeros(state["anchors"], dtype=np.uint8)
    kept[det["anchor_idx"]] = 1
    return {"head": R.rtcc_get_tensor(ctx, R.RTCC_T_HEAD, 0, np.float32), "kept": kept}


def tolerance(case):
    if case["kind"] == "nms":
        return "exact"  # records are copied, the decisions are taken in 64 bits
    if case["precision"] == "fp32":
        return {"rel": 1e-6, "max": 2e-5}
    # the head of a bf16 network: roundings of up to 17 layers; a few anchors
    # next to the threshold, or suppressed by one that is, change sides
    return {"rel": 1.2e-2, "max": 0.2, "differ": 2e-3}


# ------------------------------------------------------------------ 64 bits

def _bf16(w, case):
    t = torch.from_numpy(w).cuda()
    return (t.bfloat16() if case["precision"] == "bf16" else t).double()


def _canvas64(p, w, case):
    """Pillars and point-feature net of one cloud."""
    H, W = _grid(case)
    f32 = np.float32
    x0, y0, v = f32(-case["x_half"]), f32(-case["y_half"]), f32(case["pillar"])
    ok = ((p[:, 0] >= x0) & (p[:, 0] < f32(case["x_half"])) & (p[:, 1] >= y0) & (p[:, 1] < f32(case["y_half"])) &
          (p[:, 2] >= f32(Z_RANGE[0])) & (p[:, 2] < f32(Z_RANGE[1])))
    cx, cy = np.floor((p[:, 0] - x0) / v), np.floor((p[:, 1] - y0) / v)
    ok &= (cx < W) & (cy < H)
    q, cell = p[ok], (cy[ok] * W + cx[ok]).astype(np.int64)
    order = np.argsort(cell, kind="stable")
    sc = cell[order]
    rank = np.arange(len(sc)) - np.searchsorted(sc, sc, side="left")
    use = order[rank < MAX_PTS]  # the lowest point indices of every cell
    f = q[use].astype(np.float64)
    feat = np.stack([f[:, 0] / case["x_half"], f[:, 1] / case["y_half"],
                     (f[:, 2] - Z_RANGE[0]) / (Z_RANGE[1] - Z_RANGE[0]), f[:, 3]], 1)
    # the point-feature net's parameters stay float32 in every workload
    h = torch.relu(torch.from_numpy(feat).cuda() @ torch.from_numpy(w["pfn_w"]).cuda().double() +
                   torch.from_numpy(w["pfn_b"]).cuda().double())
    idx = torch.from_numpy(cell[use]).cuda()[:, None].expand(-1, h.shape[1])
    out = torch.zeros(H * W, h.shape[1], dtype=torch.float64, device="cuda")
    return out.scatter_reduce_(0, idx, h, "amax").view(H, W, -1)


def _conv64(x, w, b, s):
    H, W, C = x.shape
    ho, wo = -(-H // s), -(-W // s)
    pad = torch.zeros(H + 3, W + 3, C, dtype=torch.float64, device="cuda")
    pad[1:H + 1, 1:W + 1] = x
    acc = b.expand(ho * wo, -1).clone()
    for dy in range(3):
        for dx in range(3):
            t = pad[dy:dy + s * (ho - 1) + 1:s, dx:dx + s * (wo - 1) + 1:s]
            acc += t.reshape(ho * wo, C) @ w[dy, dx]
    return torch.relu(acc).view(ho, wo, -1)


def _up64(x, w, b, H2, W2):
    h, wd, c = x.shape
    u = w.shape[0]
    y = x.reshape(h * wd, c) @ w.permute(2, 0, 1, 3).reshape(c, -1)
    y = y.view(h, wd, u, u, -1).permute(0, 2, 1, 3, 4).reshape(h * u, wd * u, -1)[:H2, :W2]
    return torch.relu(y + b)


def _warp64(x, pose, case):
    """x on the ego grid: cells sampled bilinearly at R^T (p - t), zero outside."""
    H, W, C = x.shape
    dx, dy = 2 * case["x_half"] / W, 2 * case["y_half"] / H
    j = torch.arange(W, dtype=torch.float64, device="cuda")[None, :].expand(H, W)
    i = torch.arange(H, dtype=torch.float64, device="cuda")[:, None].expand(H, W)
    px, py = (j + 0.5) * dx - case["x_half"] - pose[1], (i + 0.5) * dy - case["y_half"] - pose[2]
    c, s = math.cos(pose[0]), math.sin(pose[0])
    u = (c * px + s * py + case["x_half"]) / dx - 0.5
    v = (-s * px + c * py + case["y_half"]) / dy - 0.5
    u0, v0 = torch.floor(u), torch.floor(v)
    out = torch.zeros_like(x)
    for a in (0, 1):
        for b in (0, 1):
            yy, xx = (v0 + a).long(), (u0 + b).long()
            wt = (v - v0 if a else 1 - (v - v0)) * (u - u0 if b else 1 - (u - u0))
            wt = torch.where((yy >= 0) & (yy < H) & (xx >= 0) & (xx < W), wt, torch.zeros_like(wt))
            out += wt[..., None] * x[yy.clamp(0, H - 1), xx.clamp(0, W - 1)]
    return out


def _fuse64(maps, case):
    x = torch.stack(maps)
    if case["fusion"] == "max":
        return x.amax(0)
    p = torch.softmax((x * x[:1]).sum(-1) / math.sqrt(x.shape[-1]), 0)
    return (p[..., None] * x).sum(0)


def _head64(case, seed):
    points, poses = _scene(case, seed)
    poses = np.float32(poses).astype(np.float64)
    raw = _weights(case)
    w = {n: _bf16(a, case) if n.endswith("_w") else torch.from_numpy(a).cuda().double() for n, a in raw.items()}
    _c, stages, up = NETS[case["net"]]
    H2, W2 = _layers(case)[1][0][:2]
    outs = []
    for p in points:
        x, got = _canvas64(p, raw, case), []
        for s, (stride, _co, n) in enumerate(stages):
            for l in range(n):
                x = _conv64(x, w["s%dc%d_w" % (s, l)], w["s%dc%d_b" % (s, l)], stride if l == 0 else 1)
            got.append(x)
        outs.append(got)

    def cat(got):
        if not up:
            return got[-1]
        return torch.cat([_up64(x, w["up%d_w" % s], w["up%d_b" % s], H2, W2) for s, x in enumerate(got)], -1)

    def fuse(maps):
        return _fuse64([_warp64(x, poses[k], case) for k, x in enumerate(maps)], case)

    if case["multiscale"]:
        fused = cat([fuse([g[s] for g in outs]) for s in range(len(stages))])
    else:
        fused = fuse([cat(g) for g in outs])
    return fused @ w["head_w"] + w["head_b"]


def _corners(b):
    c, s = math.cos(b[6]), math.sin(b[6])
    return [(b[0] + p * b[4] / 2 * c - q * b[3] / 2 * s, b[1] + p * b[4] / 2 * s + q * b[3] / 2 * c)
            for p, q in ((1, 1), (-1, 1), (-1, -1), (1, -1))]


def _iou(a, b):
    poly, clip = _corners(a), _corners(b)
    for k in range(4):
        (x0, y0), (x1, y1) = clip[k], clip[(k + 1) % 4]
        side = [(x1 - x0) * (y - y0) - (y1 - y0) * (x - x0) for x, y in poly]
        new = []
        for i in range(len(poly)):
            j = (i + 1) % len(poly)
            if side[i] >= 0:
                new.append(poly[i])
            if (side[i] >= 0) != (side[j] >= 0):
                t = side[i] / (side[i] - side[j])
                new.append((poly[i][0] + t * (poly[j][0] - poly[i][0]), poly[i][1] + t * (poly[j][1] - poly[i][1])))
        poly = new
        if not poly:
            return 0.0
    inter = 0.5 * sum(poly[i - 1][0] * poly[i][1] - poly[i][0] * poly[i - 1][1] for i in range(len(poly)))
    return inter / (a[3] * a[4] + b[3] * b[4] - inter)


def _nms64(rec, cap):
    """Rows kept: greedy by score (ties to the lower row), IoU at most the threshold."""
    order = np.argsort(-rec[:, 7], kind="stable")[:cap]
    thr, kept = float(np.float32(NMS_IOU)), []
    r = 0.5 * np.hypot(rec[:, 3], rec[:, 4])
    xy = np.empty((len(order), 3))
    for i in order:
        k = xy[:len(kept)]
        near = np.nonzero((k[:, 0] - rec[i, 0]) ** 2 + (k[:, 1] - rec[i, 1]) ** 2 <= (k[:, 2] + r[i]) ** 2)[0]
        if all(_iou(rec[i], rec[kept[j]]) <= thr for j in near):
            xy[len(kept)] = rec[i, 0], rec[i, 1], r[i]
            kept.append(i)
    return sorted(kept)


def _padded(rows, n):
    out = np.zeros((n,) + rows.shape[1:])
    out[:len(rows)] = rows
    return out


def exact(case, seed):
    if case["kind"] == "nms":
        if case["records"] > 4000 and case["per_object"] < 3:
            return None  # too many kept boxes for the plain walk
        rec = _records(case, seed)
        kept = _nms64(rec[:, :8].astype(np.float64), case["cap"])
        return {"kept": len(kept), "records": _padded(rec[kept, :8], case["cap"]), "anchor_idx": None}
    head = _head64(case, seed)
    if case["precision"] != "fp32":
        return {"head": head.reshape(-1), "kept": None}
    H2, W2 = head.shape[:2]
    z = head.cpu().numpy().reshape(-1, 8)
    idx = np.nonzero(z[:, 0] > float(np.float32(case["threshold"])))[0]
    z, cell = z[idx], idx // 2
    A = ANCHOR
    diag = math.hypot(A["w"], A["l"])
    xa = (cell % W2 + 0.5) * 2 * case["x_half"] / W2 - case["x_half"]
    ya = (cell // W2 + 0.5) * 2 * case["y_half"] / H2 - case["y_half"]
    rec = np.stack([xa + z[:, 1] * diag, ya + z[:, 2] * diag, A["z"] + z[:, 3] * A["h"], A["w"] * np.exp(z[:, 4]),
                    A["l"] * np.exp(z[:, 5]), A["h"] * np.exp(z[:, 6]),
                    np.where(idx % 2, A["yaw"][1], A["yaw"][0]) + z[:, 7], 1 / (1 + np.exp(-z[:, 0]))], 1)
    kept = _nms64(rec, NMS_CAP)
    return {"count": len(kept), "decoded": len(idx), "boxes": _padded(rec[kept], NMS_CAP),
            "anchor_idx": _padded(idx[kept], NMS_CAP).astype(np.int32)}
