"""The work that a program using this library has it do, as measurable cases.

Every case goes through the public entry points (`Elas.process`,
`Elas.process_batch`, `Server.submit` / `wait`) on image pairs resident on the
GPU and returns both disparity maps of every pair. Outputs are whole numbers,
decided by integer arithmetic and two FP32 expressions of fixed order.

The scenes follow the repository's synthetic recipe (piecewise slanted planes
over Voronoi cells, box-blurred byte noise, textureless patches, a z-buffer
warp with Gaussian noise on the right view), built here on the device so that
large batches are quick to make.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1802_07210_amd as elas

# Parameter sets: the plain path and the variants that the benchmark reports.
VARIANTS = {
    "plain": {},
    "census_9x9_5x5": dict(descriptor=1, census_support_window=9, census_dense_window=5),
    "census_13x13_7x7": dict(descriptor=1, census_support_window=13, census_dense_window=7),
    "shiftsum_eq3": dict(ambiguity=1),
    "past_only_redundancy": dict(redundancy=1),
    "support_1_of_8": dict(support_subsample=8),
    "median_5x5": dict(median_window=5),
    "embedded_best": dict(descriptor=1, census_support_window=9, census_dense_window=5,
                          ambiguity=1, redundancy=1, support_subsample=8, median_window=5),
}

# The four workload shapes: width, height, disparity count, planes, flat share.
SHAPES = {
    "320x240": (320, 240, 64, 8, 0.10),
    "640x480": (640, 480, 128, 24, 0.10),
    "1242x375": (1242, 375, 256, 32, 0.15),
    "1280x720": (1280, 720, 192, 32, 0.10),
}


def _case(name, kind, w, h, D, pairs=1, streams=1, variant="plain", pad=0, dmin=0, mixed=False):
    return {"name": name, "kind": kind, "w": w, "h": h, "D": D, "pairs": pairs,
            "streams": streams, "variant": variant, "pad": pad, "dmin": dmin, "mixed": mixed}


def listed():
    return [
        # one camera, one frame at a time: the smallest frame the repository
        # runs (its smoke test), where launches and latency are everything
        _case("frame_160x96", "frame", 160, 96, 32),
        # a small robot camera
        _case("frame_320x240", "frame", 320, 240, 64),
        # the paper's New Tsukuba shape: the headline frame
        _case("frame_640x480", "frame", 640, 480, 128),
        # the paper's KITTI shape: odd sides (ragged tiles), every disparity
        _case("frame_1242x375", "frame", 1242, 375, 256),
        # HD video
        _case("frame_1280x720", "frame", 1280, 720, 192),
        # a crop with odd sides, padded rows and a disparity offset
        _case("frame_451x333_padded", "frame", 451, 333, 100, pad=13, dmin=3),
        # the paper's most accurate embedded configuration: census, shift-sum,
        # past-only redundancy, down-sampled support, median
        _case("frame_640x480_embedded", "frame", 640, 480, 128, variant="embedded_best"),
        # one request through the batching server and back (camera latency)
        _case("served_640x480", "served", 640, 480, 128),
        # a small multi-camera rig in one batched call
        _case("batch8_640x480", "batch", 640, 480, 128, pairs=8),
        # eight HD cameras in one batched call
        _case("batch8_1280x720", "batch", 1280, 720, 192, pairs=8),
        # cameras of all four shapes and ranges in one batched call
        _case("batch32_mixed", "batch", 640, 480, 128, pairs=32, mixed=True),
        # the benchmark's throughput setting: 32 pairs per call on each of two
        # streams, both batches in flight together
        _case("batch32_640x480_two_streams", "batch", 640, 480, 128, pairs=32, streams=2),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["frame", "frame", "frame", "served", "batch", "batch"])
    w, h = _log_int(rng, 96, 1440), _log_int(rng, 72, 800)
    D = min(_log_int(rng, 16, 256), max(16, w // 3))
    variant = rng.choice(list(VARIANTS)) if rng.random() < 0.5 else "plain"
    pad = rng.choice([0, 0, 1, 6, 64])
    dmin = rng.choice([0, 0, 0, 2, 9]) if D <= 240 else 0
    pairs, streams, mixed = 1, 1, False
    if kind == "batch":
        # at most the pixels of the listed 32-pair mixed call
        most = max(2, min(32, int(14e6 / (w * h))))
        pairs = _log_int(rng, 2, most)
        streams = rng.choice([1, 1, 2]) if pairs * w * h < 6e6 else 1
        mixed = rng.random() < 0.2 and pairs <= 16
    c = _case("", kind, w, h, D, pairs, streams, variant, pad, dmin, mixed)
    del c["name"]
    return c


def _shapes_of(case):
    """(w, h, D, planes, flat share) of each pair of one call."""
    n = case["pairs"]
    if case["mixed"]:
        names = list(SHAPES)
        return [SHAPES[names[(5 * i + i // 4) % 4]] for i in range(n)]
    w, h, D = case["w"], case["h"], case["D"]
    for s in SHAPES.values():
        if s[:3] == (w, h, D):
            return [s] * n
    return [(w, h, D, max(4, min(32, w * h // 12800)), 0.10)] * n


def _scene(rng, shape, dmin, pad, dev):
    """One stereo pair as uint8 [h, w] device tensors (rows `pad` bytes longer)."""
    w, h, D, planes, flat = shape
    su = rng.random(planes) * w
    sv = rng.random(planes) * h
    slope = 0.08 if D == 256 else 0.05
    a = rng.uniform(-slope, slope, planes)
    b = rng.uniform(-slope, slope, planes)
    c = dmin + rng.uniform(min(4.0, D / 4), D - min(5.0, D / 4), planes)
    noise = rng.integers(0, 256, (3, h, w), dtype=np.uint8)
    gauss = rng.standard_normal((h, w), dtype=np.float32)
    patches = []
    ps, covered = min(48, w, h), 0.0
    while covered < flat * w * h:
        patches.append((int(rng.integers(0, w - ps + 1)), int(rng.integers(0, h - ps + 1)),
                        int(rng.integers(0, 256))))
        covered += 0.9 * ps * ps  # patches overlap a little
    T = lambda x: torch.from_numpy(np.asarray(x)).to(dev)  # noqa: E731
    u = torch.arange(w, device=dev, dtype=torch.float64)[None, :]
    v = torch.arange(h, device=dev, dtype=torch.float64)[:, None]
    tu, tv = T(su), T(sv)
    label = ((u[None] - tu[:, None, None]) ** 2 + (v[None] - tv[:, None, None]) ** 2).argmin(0)
    disp = T(c)[label] + T(a)[label] * (u - tu[label]) + T(b)[label] * (v - tv[label])
    gt = torch.floor(disp + 0.5).clamp(dmin, dmin + D - 1).to(torch.int64)
    tex = T(noise)
    p = torch.nn.functional.pad(tex[0].float()[None, None], (1, 1, 1, 1), mode="replicate")
    left = torch.floor((torch.nn.functional.avg_pool2d(p, 3, 1) * 9 + 4.5) / 9)[0, 0]
    left = left.clamp(0, 255).to(torch.uint8)
    for x0, y0, val in patches:
        left[y0:y0 + ps, x0:x0 + ps] = val
    # right view: the larger disparity wins, holes keep fresh noise
    ui = torch.arange(w, device=dev)[None, :].expand(h, w)
    vi = torch.arange(h, device=dev)[:, None].expand(h, w)
    ut = ui - gt
    ok = ut >= 0
    z = torch.full((h * w,), -1, dtype=torch.int64, device=dev)
    z.scatter_reduce_(0, (vi * w + ut)[ok], (gt * 65536 + ui)[ok], "amax")
    hit = z >= 0
    right = tex[1].reshape(-1).clone()
    src = (torch.arange(h * w, device=dev) // w * w + (z & 65535))[hit]
    right[hit] = left.reshape(-1)[src]
    sigma = 3.0 if D == 256 else 2.0
    right = torch.floor(right.reshape(h, w).float() + sigma * T(gauss) + 0.5)
    right = right.clamp(0, 255).to(torch.uint8)
    if not pad:
        return left.contiguous(), right.contiguous()
    out = []
    for img in (left, right):
        rows = torch.full((h, w + pad), 7, dtype=torch.uint8, device=dev)
        rows[:, :w] = img
        out.append(rows[:, :w])
    return tuple(out)


def prepare(case, seed):
    """Image pairs and outputs on the GPU, and the handles (or server) that a
    program keeps from frame to frame: they have already seen one call of this
    shape, so buffers, tile variants and captured launches exist."""
    dev = torch.device("cuda:0")
    rng = np.random.default_rng([int(seed), case["w"], case["h"], case["D"], case["pairs"]])
    shapes = _shapes_of(case)
    handles, calls, outs = {}, [], []
    for _ in range(case["streams"]):
        # the maps of all pairs of one shape in one tensor: [pair, view, h, w]
        maps = {s: torch.empty((shapes.count(s), 2, s[1], s[0]), dtype=torch.int16, device=dev)
                for s in dict.fromkeys(shapes)}
        outs.extend(maps.values())
        taken = dict.fromkeys(maps, 0)
        items = []
        for s in shapes:
            if s[2] not in handles:
                handles[s[2]] = elas.Elas(disp_min=case["dmin"], disp_max=case["dmin"] + s[2] - 1,
                                          **VARIANTS[case["variant"]])
            L, R = _scene(rng, s, case["dmin"], case["pad"], dev)
            m = maps[s][taken[s]]
            taken[s] += 1
            items.append((L, R, m[0], m[1], handles[s[2]]))
        calls.append(items)
    state = {"kind": case["kind"], "calls": calls, "outs": outs, "handle": handles[shapes[0][2]],
             "streams": [torch.cuda.Stream(dev) for _ in calls] if len(calls) > 1 else [None]}
    if case["kind"] == "served":
        state["server"] = elas.Server(state["handle"])
    # one call on another view of the scenes (upside down), so that the program
    # is past its start-up when the first of these frames arrives
    flipped = dict(state, calls=[[(_flip(L), _flip(R), oL, oR, h) for L, R, oL, oR, h in items]
                                 for items in calls])
    torch.cuda.synchronize()
    run(flipped)
    torch.cuda.synchronize()
    return state


def _flip(img):
    """The image upside down, in rows of the same pitch."""
    rows = torch.empty((img.shape[0], img.stride(0)), dtype=img.dtype, device=img.device)
    view = rows[:, :img.shape[1]]
    view.copy_(img.flip(0))
    return view


def run(state):
    """One frame, one served request, or one batched call on each stream; the
    maps of every pair."""
    if state["kind"] == "frame":
        L, R, oL, oR, h = state["calls"][0][0]
        h.process(L, R, oL, oR)
    elif state["kind"] == "served":
        L, R, oL, oR, _ = state["calls"][0][0]
        server = state["server"]
        server.wait(server.submit(L, R, oL, oR))
    else:
        for items, stream in zip(state["calls"], state["streams"]):
            state["handle"].process_batch(items, stream=stream)
    return state["outs"]


def work(case):
    """Bytes: both images read, both maps written. Operations: the byte
    absolute differences (one subtraction and one addition each) of the forward
    support search over the lattice and of five candidates per pixel and view."""
    nbytes = flops = 0
    for w, h, D, _, _ in _shapes_of(case):
        nbytes += 2 * w * h + 2 * 2 * w * h
        lattice = max(1, (w - 5) // 5) * max(1, (h - 5) // 5)
        flops += 2 * (64 * lattice * min(D, w) + 2 * w * h * 5 * 16)
    return {"bytes": nbytes * case["streams"], "flops": flops * case["streams"]}
