"""The work that users of this package have it do, as measurable cases: triplet builds, the layers of an inference
pass and of a training step, through the public calls of paper_2511_23227_amd.

A case is a dict of plain values:
  mode        infer      build (forward plan) + forward pass of one layer on a cloud that has just arrived
              build      triplets and the plan of a training step (forward and input-gradient side)
              strided    down-sampling to one point per voxel, then the build of the strided layer onto those points
              forward    one layer on a plan that is kept (several layers share one build)
              backward   input gradient and weight gradient of one layer
              train      forward, input gradient and weight gradient of one layer
  cloud       uniform (in a cube), surface (noisy rectangles, random order), lidar (spinning sensor, ring order),
              ground (ground plane and walls, random order)
  layer       same (outputs at the inputs), down (outputs = one input per voxel, about a quarter), up (the decoder's
              layer back to the original points)
  n, neighbours, t, batch    points (of all clouds of a batch), mean inputs within the radius of an output, kernel
                             resolution per axis, clouds held back to back
  c_in, c_out, dtype, out    channels, storage type of features and weights, type of `out` / `dx`
  spatial     the plan groups its centres along a space-filling curve (what wide layers ask for)
"""
import math

import numpy as np
import torch

import paper_2511_23227_amd as pcpp

# Neighbourhood radius by kind of cloud, metres.  The density follows from it and the mean neighbour count.
RADIUS = {"uniform": 0.1, "surface": 0.05, "lidar": 0.4, "ground": 0.186}
RINGS = 64                        # of the spinning sensor; 0.2 degrees between azimuths (1800 a turn) is its full rate
LIDAR_NEIGHBOURS = 148.0          # mean within RADIUS["lidar"] at 1800 azimuths
# kernel cells that the neighbourhood of a point on a surface reaches, by t; a ball of volume reaches nearly all
CELLS_ON_SURFACE = {1: 1.0, 2: 5.5, 3: 12.5, 4: 17.5, 5: 23.0, 6: 30.0}


def _case(name, mode, cloud, n, neighbours, t, c_in=0, c_out=0, dtype="bf16", out="f32", layer="same", spatial=False,
          batch=1):
    d = {"mode": mode, "cloud": cloud, "layer": layer, "n": n, "neighbours": neighbours, "t": t, "batch": batch,
         "c_in": c_in, "c_out": c_out, "dtype": dtype, "out": out, "spatial": spatial}
    return dict(d, name=name) if name else d


def listed():
    return [
        # a small cloud answered at once (an object, a crop around a point): launches and the host count
        _case("infer_tiny_f32", "infer", "uniform", 2048, 8.6, 3, 16, 16, "f32"),
        # the points and triplets of an encoder stage: down-sampling, then the strided layer's build
        _case("strided_build", "strided", "surface", 200_000, 92.0, 3),
        # a training batch of indoor clouds built in one call
        _case("batched_build", "build", "surface", 800_000, 24.3, 3, batch=8),
        # an early layer of an indoor network in fp32
        _case("train_indoor_f32", "train", "surface", 100_000, 24.3, 3, 32, 32, "f32"),
        # an early layer of an outdoor network: crowded neighbourhoods near the sensor, few far away
        _case("train_lidar_bf16", "train", "lidar", 115_200, LIDAR_NEIGHBOURS, 3, 64, 64),
        # the strided layer that doubles the channels
        _case("train_strided_bf16", "train", "surface", 200_000, 92.0, 3, 64, 128, layer="down"),
        # the decoder's layer back to more points and fewer channels, activations in bf16
        _case("train_upsample_bf16", "train", "surface", 99_991, 92.0, 3, 128, 64, out="bf16", layer="up"),
        # a residual block's layer in the middle of a network, where points are fewer and channels more
        _case("train_residual_bf16", "train", "surface", 40_009, 24.3, 3, 128, 128, out="bf16"),
        # channel counts that are no power of two (input features, concatenated skips)
        _case("train_ragged_f32", "train", "surface", 20_011, 24.3, 3, 20, 36, "f32"),
        # the largest layer: a million points, 5 x 5 x 5 cells, 256 channels
        _case("forward_large_bf16", "forward", "ground", 1_000_000, 32.0, 5, 256, 256, spatial=True),
        _case("backward_large_bf16", "backward", "ground", 1_000_000, 32.0, 5, 256, 256, spatial=True),
        _case("build_large", "build", "ground", 1_000_000, 32.0, 5, spatial=True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    mode = rng.choice(["infer", "build", "strided", "forward", "backward", "train", "train"])
    cloud = rng.choice(["uniform", "surface", "surface", "lidar", "ground"])
    t = rng.choice([2, 3, 3, 3, 4, 5])
    layer = "same"
    if mode == "strided":
        cloud = "surface"
    elif mode != "build" and cloud == "surface":
        layer = rng.choice(["same", "down", "up"])
    # channels: mostly a power of two that stays, doubles or halves; otherwise whatever a user's features have
    dtype = rng.choice(["f32", "bf16", "bf16"])
    if rng.random() < 0.75:
        c_in = rng.choice([16, 32, 64, 128, 256])
        c_out = max(16, min(256, rng.choice([c_in // 2, c_in, c_in, c_in * 2])))
    else:
        c_in, c_out = rng.randint(4, 130), rng.randint(6, 130)
    out = rng.choice(["f32", "bf16"]) if dtype == "bf16" else "f32"
    spatial = rng.random() < 0.2 or min(c_in, c_out) >= 256
    batch = rng.choice([1, 1, 2, 3, 8]) if mode == "build" and cloud == "surface" else 1
    # points and density, within the triplets and the arithmetic of the largest listed layer (fp32: a sixteenth of
    # the arithmetic; all shapes but the widest: a quarter)
    n = _log_int(rng, 2_000, 1_000_000)
    neighbours = round(math.exp(rng.uniform(math.log(8.0), math.log(100.0 if layer != "same" or mode == "strided" else 50.0))), 1)
    per = 1.0
    if mode in ("infer", "forward", "backward", "train"):
        per = c_in * c_out / 65536.0 * (16.0 if dtype == "f32" else 1.0) * (1.0 if min(c_in, c_out) >= 256 else 4.0)
        per = max(per, 0.5) * (3.0 if mode == "train" else 2.0 if mode == "backward" else 1.0)
    most = 30e6 / per
    if cloud == "lidar":
        azimuths = max(32, min(1800, n // RINGS))
        while RINGS * azimuths * LIDAR_NEIGHBOURS * azimuths / 1800 > most and azimuths > 32:
            azimuths = azimuths * 4 // 5
        n, neighbours = RINGS * azimuths, round(LIDAR_NEIGHBOURS * azimuths / 1800, 1)
    else:
        n = max(2_000, min(n, int(most / neighbours)))
    if mode == "build" or mode == "strided":
        c_in = c_out = 0
        dtype, out = "bf16", "f32"
    return _case(None, mode, cloud, n, neighbours, t, c_in, c_out, dtype, out, layer, spatial, batch)


# ---- inputs ------------------------------------------------------------------------------------------------------

def _rand(g, *shape):
    return torch.rand(*shape, generator=g, device="cuda")


def _randn(g, *shape):
    return torch.randn(*shape, generator=g, device="cuda")


def _rectangles(g, n, n_rect, area, room, noise, upright):
    """n points on n_rect rectangles that share `area`, placed in a room of side `room`."""
    sides = 0.6 + 0.8 * _rand(g, n_rect, 2)
    sides = sides * torch.sqrt(area / (sides[:, 0] * sides[:, 1]).sum())
    centres = room * _rand(g, n_rect, 3)
    if upright:
        angle = 2 * math.pi * _rand(g, n_rect)
        u = torch.stack([torch.cos(angle), torch.sin(angle), torch.zeros_like(angle)], 1)
        v = torch.tensor([0.0, 0.0, 1.0], device="cuda").expand(n_rect, 3)
        centres[:, 2] = 0.5 * sides[:, 1]
    else:
        u = torch.nn.functional.normalize(_randn(g, n_rect, 3), dim=1)
        v = torch.nn.functional.normalize(torch.linalg.cross(u, _randn(g, n_rect, 3)), dim=1)
    share = (sides[:, 0] * sides[:, 1]).cumsum(0)
    which = torch.searchsorted(share / share[-1], _rand(g, n)).clamp_(max=n_rect - 1)
    s = (_rand(g, n, 2) - 0.5) * sides[which]
    return centres[which] + s[:, :1] * u[which] + s[:, 1:] * v[which] + noise * _randn(g, n, 3)


def _lidar(g, azimuths):
    """One turn of a sensor with RINGS beams 1.8 m above the ground among boxes; ring-major order."""
    elev = torch.deg2rad(torch.linspace(-25.0, -1.5, RINGS, device="cuda"))
    az = torch.arange(azimuths, device="cuda") * (2 * math.pi / azimuths)
    d = torch.stack([torch.cos(elev)[:, None] * torch.cos(az), torch.cos(elev)[:, None] * torch.sin(az),
                     torch.sin(elev)[:, None].expand(RINGS, azimuths)], -1).reshape(-1, 3)
    sensor = torch.tensor([0.0, 0.0, 1.8], device="cuda")
    dist = -1.8 / d[:, 2]
    size = 1.0 + 4.0 * _rand(g, 30, 3)
    at = 100.0 * _rand(g, 30, 2) - 50.0
    near = at.norm(dim=1) < 6.0
    at[near] += 8.0 * torch.sign(at[near])
    lo = torch.cat([at - 0.5 * size[:, :2], torch.zeros(30, 1, device="cuda")], 1)
    a, b = (lo - sensor)[:, None] / d, (lo + size - sensor)[:, None] / d
    enter, leave = torch.minimum(a, b).amax(2), torch.maximum(a, b).amin(2)
    hit = torch.where((leave >= enter) & (enter > 0), enter, torch.inf).amin(0)
    dist = torch.minimum(dist, hit) + 0.02 * _randn(g, len(d))
    return sensor + dist[:, None] * d


def _cloud(g, c, n):
    r, m = RADIUS[c["cloud"]], c["neighbours"]
    if c["cloud"] == "uniform":
        p = _rand(g, n, 3) * (n * 4 / 3 * math.pi * r ** 3 / m) ** (1 / 3)
    elif c["cloud"] == "surface":
        area = n * math.pi * r * r / m
        p = _rectangles(g, n, max(4, n // 2500), area, 1.8 * math.sqrt(area), r / 10, False)
    elif c["cloud"] == "lidar":
        p = _lidar(g, n // RINGS)
    else:
        ground = int(0.7 * n)
        side = math.sqrt(1.05 * ground * math.pi * r * r / m)
        flat = torch.cat([side * _rand(g, ground, 2), torch.zeros(ground, 1, device="cuda")], 1)
        flat = flat + 0.005 * _randn(g, ground, 3)
        walls = _rectangles(g, n - ground, max(4, n // 5000), side * side * 3 / 7, side, 0.005, True)
        p = torch.cat([flat, walls])[torch.randperm(n, generator=g, device="cuda")]
    return p.float().contiguous()


def _pitch(c):
    """Voxel pitch that keeps about a quarter of the points of a surface cloud."""
    return math.sqrt(5.5 * math.pi / c["neighbours"]) * RADIUS[c["cloud"]]


def _coarse(points, c):
    """A quarter of the points, one to a voxel as far as there are that many voxels, in ascending order."""
    kept = pcpp.pcpp_voxel_subsample(points, 0.85 * _pitch(c)).long()
    chosen = torch.full((len(points),), 2.0, device="cuda")
    chosen[kept] = torch.linspace(0.0, 1.0, len(kept), device="cuda").mul_(7919.0).frac_()
    return points[torch.sort(torch.argsort(chosen, stable=True)[:len(points) // 4])[0]].contiguous()


def _flags(c):
    return (pcpp.PLAN_FWD | (0 if c["mode"] in ("infer", "forward") else pcpp.PLAN_BWD_INPUT)
            | (pcpp.PLAN_SPATIAL if c["spatial"] else 0))


def _sizes(c):
    """Inputs and outputs of the case's layer."""
    n, quarter = c["n"], c["n"] // 4
    return (quarter, n) if c["layer"] == "up" else (n, quarter) if c["layer"] == "down" or c["mode"] == "strided" else (n, n)


def prepare(case, seed):
    c = case
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    per = [len(a) for a in np.array_split(np.arange(c["n"]), c["batch"])]
    points = torch.cat([_cloud(g, c, n) for n in per]) if c["batch"] > 1 else _cloud(g, c, c["n"])
    s = {"case": c, "points": points, "radius": RADIUS[c["cloud"]], "flags": _flags(c)}
    if c["batch"] > 1:
        s["offsets"] = torch.tensor(np.concatenate([[0], np.cumsum(per)]), dtype=torch.int32, device="cuda")
    other = points if c["layer"] == "same" else _coarse(points, c)
    s["in"], s["out"] = (other, points) if c["layer"] == "up" else (points, other)
    if c["mode"] in ("infer", "build", "strided"):
        # a program that builds clouds of one kind all the time keeps lists with room for them
        s["room"] = int(min(_sizes(c)) * (1.5 * c["neighbours"] + 8)) + 4096
        s["lists"] = {k: torch.zeros(s["room"], dtype=torch.int32, device="cuda") for k in ("tri_o", "tri_i", "tri_k")}
        if c["mode"] == "strided":
            s["coarse"] = torch.zeros_like(points)
    if c["c_in"]:
        dt = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
        k = c["t"] ** 3
        s["out_dtype"] = torch.bfloat16 if c["out"] == "bf16" else torch.float32
        s["w"] = (_randn(g, k, c["c_out"], c["c_in"]) / math.sqrt(k * c["c_in"])).to(dt)
        if c["mode"] != "infer":
            s["T"] = pcpp.pcpp_build_triplets(s["in"], s["out"], s["radius"], c["t"], plan_flags=s["flags"])
        s["x"] = _randn(g, len(s["in"]), c["c_in"]).to(dt)
        if c["mode"] in ("backward", "train"):
            s["dy"] = _randn(g, len(s["out"]), c["c_out"]).to(dt)
    return s


# ---- one pass ----------------------------------------------------------------------------------------------------

def _build(s, points_in, points_out):
    return pcpp.pcpp_build_triplets(points_in, points_out, s["radius"], s["case"]["t"], plan_flags=s["flags"],
                                    capacity=s["room"], buffers=s["lists"], in_offsets=s.get("offsets"),
                                    out_offsets=s.get("offsets"))


def run(state):
    s, c = state, state["case"]
    mode = c["mode"]
    if mode in ("infer", "build", "strided"):
        points_in, points_out = s["in"], s["out"]
        if mode == "strided":
            kept = pcpp.pcpp_voxel_subsample(s["points"], _pitch(c))
            points_out = torch.index_select(s["points"], 0, kept, out=s["coarse"][:len(kept)])
        T = _build(s, points_in, points_out)
        got = dict(s["lists"], segments=T.seg_offsets, triplets=T.n_triplets)
        if mode == "strided":
            got["coarse"] = s["coarse"]
        if mode == "infer":
            got["y"] = pcpp.pcpp_mvmr_fwd(s["x"], s["w"], T, out_dtype=s["out_dtype"])
        return got
    T, got = s["T"], {}
    if mode in ("forward", "train"):
        got["y"] = pcpp.pcpp_mvmr_fwd(s["x"], s["w"], T, out_dtype=s["out_dtype"])
    if mode in ("backward", "train"):
        got["dx"] = pcpp.pcpp_mvmr_bwd_input(s["dy"], s["w"], T, out_dtype=s["out_dtype"])
        got["dw"] = pcpp.pcpp_mvmr_bwd_weight(s["x"], s["dy"], T)
    return got


# ---- what a pass cannot do without -------------------------------------------------------------------------------

def work(case):
    c = case
    n_in, n_out = _sizes(c)
    # triplets: every output of a down-sampling layer has `neighbours` inputs; an up-sampling layer is its mirror
    triplets = c["neighbours"] * min(n_in, n_out)
    k = c["t"] ** 3
    bytes_ = flops = 0.0
    if c["mode"] in ("infer", "build", "strided"):
        sides = 0 if c["mode"] == "infer" else 1
        # coordinates in; the three lists, and the neighbour list of each further side of the plan, out
        bytes_ += 12.0 * (n_in + (n_out if n_out != n_in else 0)) + triplets * (12.0 + 4.0 * sides + (4.0 if c["spatial"] else 0.0))
    if c["c_in"]:
        e = 2 if c["dtype"] == "bf16" else 4
        eo = 2 if c["out"] == "bf16" else 4
        x, y, w = n_in * c["c_in"], n_out * c["c_out"], k * c["c_in"] * c["c_out"]
        # one product per (cell, centre) that holds a neighbour, after the neighbours' rows have been added up
        cells = 0.9 * min(k, 27) if c["cloud"] == "uniform" else 8.0 * c["t"] ** 2 / 9 if c["cloud"] == "lidar" else CELLS_ON_SURFACE[c["t"]]

        def one(centres):
            per = triplets / centres
            return 2.0 * centres * cells * (1 - math.exp(-per / cells)) * c["c_in"] * c["c_out"]
        if c["mode"] in ("infer", "forward", "train"):
            bytes_ += x * e + w * e + y * eo + 4.0 * triplets
            flops += one(n_out)
        if c["mode"] in ("backward", "train"):
            bytes_ += y * e + w * e + x * eo + 4.0 * triplets       # input gradient
            bytes_ += x * e + y * e + w * 4 + 8.0 * triplets        # weight gradient
            flops += one(n_in) + one(n_out)
    return {"bytes": bytes_, "flops": flops}


def tolerance(case):
    if not case["c_in"]:
        return "exact"
    # fp32: sums of up to a few thousand products in another order; bf16: the inputs' own rounding, 2^-9, applied once
    # more to the sums that enter the matrix products and to a bf16 result
    return {"rel": 1e-5} if case["dtype"] == "f32" else {"rel": 1e-2}
