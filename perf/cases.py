"""The work that users of this estimator have it do, as measurable cases.

Each case goes through the package's public entry points with the buffers that a
program estimating frame after frame keeps.  Sizes are those of the repository's
own workloads (``paper_2012_12618_amd/synth.py``, the tests and ``bench.py``):

* ``frame``      one frame in GPU memory, ``rv_estimate_velocity``;
* ``prepared``   the same through ``PreparedEstimate`` (buffers held, one C call);
* ``paper``      the paper-literal variant, ``rv_estimate_velocity_paper``;
* ``batch``      many frames in one launch sequence, as a captured graph, in
                 float32 or in the FP16 residual form (``fp16_min``);
* ``pipelined``  one frame from pinned host memory, copied and estimated in parts;
* ``server``     frames in host memory submitted to ``RVServer``, all results taken.

Inputs follow the generative model of ``synth.py`` (rigid-body velocity profile,
N(0, 0.05) noise, uniform and micro-Doppler-band outliers), drawn on the GPU.
"""
import math

import numpy as np
import torch

from paper_2012_12618_amd import binding as rv

TAU = 0.15        # m/s, the inlier threshold of every workload of the repository
SIGMA = 0.05      # m/s, inlier noise
V_MAX = 30.0      # m/s
FOV = 60.0        # degrees, azimuth field of view +/-
SPAN = 40.0       # m/s, uniform outliers


def _case(name, kind, clusters, lo, hi, hyp, frames=1, pu=0.2, pb=0.0, law="log", spread=0.0,
          bits=False, fp16_min=0, parts=0):
    """One case: ``frames`` frames of ``clusters`` clusters each (a batch's frames
    vary between half and one and a half times that), sizes in [lo, hi] points
    (``law``: "log" log-uniform, "uni" uniform), ``hyp`` hypotheses per cluster,
    outlier fractions ``pu`` and ``pb``; ``spread``: azimuth window of a cluster
    in degrees (0: the whole field of view); ``bits``: the frame-wide inlier mask
    is asked for."""
    d = dict(kind=kind, clusters=clusters, lo=lo, hi=hi, hyp=hyp, frames=frames, pu=pu, pb=pb,
             law=law, spread=spread, bits=bits, fp16_min=fp16_min, parts=parts)
    if name:
        d["name"] = name
    return d


def listed():
    return [
        # The smallest call in earnest: one frame of 64 clusters, estimated as it
        # arrives; latency and launches count.
        _case("frame-small", "prepared", 64, 20, 200, 256, law="uni"),
        # The paper's own largest timing-table shape, through its own inlier test.
        _case("paper-table", "paper", 64, 150, 150, 256, law="uni"),
        # The paper-literal variant on an ordinary frame, with the frame-wide mask.
        _case("paper-mask", "paper", 512, 8, 2048, 512, bits=True),
        # One radar's frame in the served shape, mask wanted: an ordinary call by
        # a program that does not keep its output buffers.
        _case("frame-served", "frame", 700, 8, 1024, 512, pu=0.25, bits=True),
        # The benchmark's dense frame: 4096 clusters, half of the outliers in a
        # micro-Doppler band.
        _case("frame-dense", "prepared", 4096, 8, 4096, 1024, pu=0.15, pb=0.15),
        # Distant objects: every cluster inside a 3-degree azimuth window (the
        # ill-conditioned clusters of the tests), an odd number of hypotheses.
        _case("frame-narrow", "prepared", 1021, 8, 3000, 999, pu=0.2, spread=3.0),
        # 64 radars' frames of one tick, one captured graph.
        _case("batch-served", "batch", 700, 8, 1024, 512, frames=64, pu=0.25),
        # The batched workload: 256 frames of U{100..1500} clusters.
        _case("batch-frames", "batch", 800, 8, 2048, 512, frames=256),
        # Very long clusters (the precision-stress shape, fewer clusters), float32.
        _case("long-f32", "batch", 64, 65536, 65536, 4096, pu=0.0, pb=0.4, law="uni"),
        # The same in the FP16 residual form.
        _case("long-fp16", "batch", 64, 65536, 65536, 4096, pu=0.0, pb=0.4, law="uni",
              fp16_min=1024),
        # The dense frame from pinned host memory in three parts, results to
        # pinned host memory: copies and estimates overlap.
        _case("pipelined-dense", "pipelined", 4096, 8, 4096, 1024, pu=0.15, pb=0.15, parts=3),
        # The frame server: one tick of 32 radars submitted, every result taken.
        _case("server-tick", "server", 700, 8, 1024, 512, frames=32, pu=0.25),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["prepared", "frame", "paper", "batch", "batch", "fp16", "pipelined", "server"])
    pu = round(rng.uniform(0.0, 0.4), 3)
    pb = round(rng.uniform(0.0, 0.3), 3)
    lo = _log(rng, 2, 64)
    spread = round(rng.uniform(1.0, 120.0), 1) if rng.random() < 0.25 else 0.0
    bits = rng.random() < 0.3
    hyp = _log(rng, 64, 2048)
    if kind == "paper":
        return _case(None, kind, _log(rng, 8, 1024), lo, _log(rng, 64, 4096), _log(rng, 64, 1024),
                     pu=pu, bits=bits)
    if kind in ("prepared", "frame"):
        return _case(None, kind, _log(rng, 8, 6000), lo, _log(rng, 80, 8192), hyp, pu=pu, pb=pb,
                     spread=spread, bits=bits and kind == "frame")
    if kind == "pipelined":
        return _case(None, kind, _log(rng, 500, 5000), lo, _log(rng, 256, 4096), hyp, pu=pu, pb=pb,
                     parts=rng.randint(2, 4))
    if kind == "server":
        return _case(None, kind, _log(rng, 64, 1200), lo, _log(rng, 128, 1024), _log(rng, 64, 512),
                     frames=rng.randint(4, 32), pu=pu)
    if rng.random() < 0.4:  # few, very long clusters
        return _case(None, "batch", _log(rng, 8, 64), 2000, _log(rng, 4096, 65536),
                     _log(rng, 256, 4096), pu=pu, pb=pb, fp16_min=1024 if kind == "fp16" else 0)
    return _case(None, "batch", _log(rng, 64, 1200), lo, _log(rng, 128, 2048), _log(rng, 64, 700),
                 frames=rng.randint(2, 128), pu=pu, pb=pb, bits=bits,
                 fp16_min=_log(rng, 256, 1024) if kind == "fp16" else 0)


def _mean_size(case):
    lo, hi = case["lo"], case["hi"]
    if case["law"] == "uni" or hi <= lo:
        return 0.5 * (lo + hi)
    return (hi + 1 - lo) / math.log((hi + 1) / lo) - 0.5


def work(case):
    """Bytes: azimuth and Doppler read once, offsets read, results written (and
    the mask).  Operations: four per hypothesis and point (two fused
    multiply-adds of a residual), the path's nominal evaluations."""
    k = case["clusters"] * case["frames"]
    n = k * _mean_size(case)
    return {"bytes": 8.0 * n + (4 + 21) * k + (n / 8 if case["bits"] else 0),
            "flops": 4.0 * n * case["hyp"]}


# ---- inputs -----------------------------------------------------------------

def _inputs(case, seed):
    """theta, vd (GPU), cluster offsets and frame offsets (numpy), frame seeds.
    Cluster counts and sizes follow from the case, so that every seed's outputs
    have one shape; points, outliers and hypothesis seeds from the seed."""
    rng = np.random.default_rng([case["clusters"], case["lo"], case["hi"], case["frames"]])
    f, k = case["frames"], case["clusters"]
    counts = rng.integers(max(1, k // 2), k + k // 2 + 1, size=f) if f > 1 else np.array([k])
    total = int(counts.sum())
    lo, hi = case["lo"], max(case["lo"], case["hi"])
    if case["law"] == "uni":
        sizes = rng.integers(lo, hi + 1, size=total)
    else:
        sizes = np.clip(np.floor(np.exp(rng.uniform(math.log(lo), math.log(hi + 1), total))), lo, hi)
    offsets = np.zeros(total + 1, np.int64)
    np.cumsum(sizes, out=offsets[1:])
    n = int(offsets[-1])
    frame_offsets = np.zeros(f + 1, np.int64)
    np.cumsum(counts, out=frame_offsets[1:])
    rng = np.random.default_rng(seed)
    seeds = rng.integers(0, 1 << 62, size=f)

    dev = torch.device("cuda")
    g = torch.Generator(device=dev).manual_seed(int(rng.integers(1 << 62)))
    cid = torch.repeat_interleave(torch.arange(total, device=dev),
                                  torch.from_numpy(sizes.astype(np.int64)).to(dev), output_size=n)

    def uniform(count, a, b):
        return torch.rand(count, generator=g, device=dev) * (b - a) + a

    vx, vy = uniform(total, -V_MAX, V_MAX), uniform(total, -V_MAX, V_MAX)
    if case["spread"]:
        half = 0.5 * case["spread"]
        deg = uniform(n, -half, half)
        deg += uniform(total, -FOV + half, FOV - half)[cid]
    else:
        deg = uniform(n, -FOV, FOV)
    theta = torch.deg2rad(deg)
    vd = vx[cid] * torch.cos(theta)
    vd += vy[cid] * torch.sin(theta)
    pick = torch.rand(n, generator=g, device=dev)
    if case["pb"]:
        band = uniform(n, 0.5, 2.0) * torch.hypot(vx, vy)[cid]
        band *= (torch.rand(n, generator=g, device=dev) < 0.5) * 2.0 - 1.0
        band += vd
    vd += torch.randn(n, generator=g, device=dev) * SIGMA
    if case["pu"]:
        vd = torch.where(pick < case["pu"], uniform(n, -SPAN, SPAN), vd)
    if case["pb"]:
        vd = torch.where((pick >= case["pu"]) & (pick < case["pu"] + case["pb"]), band, vd)
    return theta, vd, offsets, frame_offsets, seeds


class _State:
    pass


def prepare(case, seed):
    theta, vd, offsets, frame_offsets, seeds = _inputs(case, seed)
    s = _State()
    s.kind, s.hyp, s.bits = case["kind"], case["hyp"], case["bits"]
    n, k = int(theta.numel()), len(offsets) - 1
    dev = theta.device
    s.theta, s.vd, s.seed = theta, vd, int(seeds[0])
    s.offsets = torch.from_numpy(offsets.astype(np.int32)).to(dev)
    if s.kind == "prepared":
        s.call = rv.PreparedEstimate(s.theta, s.vd, s.offsets, s.hyp, TAU,
                                     rv.allocate_outputs(k, n, s.hyp, dev, want_bits=s.bits))
    elif s.kind == "paper":
        s.out = rv.allocate_paper_outputs(k, n, s.hyp, dev, want_bits=s.bits)
    elif s.kind == "batch":
        s.out = rv.allocate_batch_outputs(case["frames"], k, n, s.hyp, dev, want_bits=s.bits)
        tuning = rv.rv_tuning_default()
        tuning.fp16_min_points = case["fp16_min"]
        s.graph = rv.rv_graph_capture_batch(
            s.theta, s.vd, s.offsets, torch.from_numpy(frame_offsets.astype(np.int32)).to(dev),
            torch.from_numpy(seeds).to(dev), s.hyp, TAU, s.out, tuning=tuning)
        s.results = {name: v for name, v in s.out.items() if name != "workspace"}
    elif s.kind == "pipelined":
        s.device_inputs = (torch.empty_like(theta), torch.empty_like(vd), torch.empty_like(s.offsets))
        s.theta, s.vd, s.offsets = theta.cpu().pin_memory(), vd.cpu().pin_memory(), s.offsets.cpu().pin_memory()
        s.out = {name: (v if name == "workspace" else torch.empty(v.shape, dtype=v.dtype, pin_memory=True))
                 for name, v in rv.allocate_outputs(k, n, s.hyp, dev).items()}
        s.parts = case["parts"]
        s.copy_stream = torch.cuda.Stream()
    elif s.kind == "server":
        t, v = theta.cpu(), vd.cpu()
        s.frames = []
        for f in range(case["frames"]):
            c0, c1 = int(frame_offsets[f]), int(frame_offsets[f + 1])
            p0, p1 = int(offsets[c0]), int(offsets[c1])
            s.frames.append((t[p0:p1].clone().pin_memory(), v[p0:p1].clone().pin_memory(),
                             torch.from_numpy((offsets[c0:c1 + 1] - p0).astype(np.int32)).pin_memory(),
                             int(seeds[f])))
        s.theta = s.vd = s.offsets = None
        s.server = rv.RVServer(n_hyp=s.hyp, tau=TAU, hbm_budget_bytes=4 << 30)
    return s


def run(s):
    if s.kind == "prepared":
        return s.call(s.seed)
    if s.kind == "frame":
        return rv.rv_estimate_velocity(s.theta, s.vd, s.offsets, s.hyp, TAU, s.seed, want_bits=s.bits)
    if s.kind == "paper":
        return rv.rv_estimate_velocity_paper(s.theta, s.vd, s.offsets, s.hyp, s.seed, out=s.out)
    if s.kind == "batch":
        s.graph.launch()
        return s.results
    if s.kind == "pipelined":
        return rv.rv_estimate_velocity_pipelined(
            s.theta, s.vd, s.offsets, s.parts, s.hyp, TAU, s.seed, device_inputs=s.device_inputs,
            out=s.out, copy_stream=s.copy_stream)
    tickets = [s.server.submit_pinned(*frame) for frame in s.frames]
    results = [s.server.result(t) for t in tickets]
    return {name: np.concatenate([r[name] for r in results])
            for name in ("vx", "vy", "heading", "n_inliers", "status", "n_near_tau", "best_hyp")}


# ---- the same in 64 bits, in plain torch ----------------------------------------

def _philox(c0, c1, key0, key1):
    """First two words of Philox4x32-10 (Salmon et al., SC'11) of the counters
    (c0, c1, 0, 0); int64 tensors holding 32-bit values."""
    mask = 0xFFFFFFFF
    x = [c0, c1, torch.zeros_like(c0), torch.zeros_like(c0)]
    for _ in range(10):
        p0, p1 = x[0] * 0xD2511F53, x[2] * 0xCD9E8D57
        x = [((p1 >> 32) & mask) ^ x[1] ^ key0, p1 & mask, ((p0 >> 32) & mask) ^ x[3] ^ key1, p0 & mask]
        key0, key1 = (key0 + 0x9E3779B9) & mask, (key1 + 0xBB67AE85) & mask
    return x[0], x[1]


def _paper_fit(theta, vd, valid, n, i, j):
    """Alg. 1 on padded clusters [B, n]: per-cluster threshold and, per trial, the
    line through the normalised seeds."""
    inf = float("inf")

    def unit(a):
        low = torch.where(valid, a, inf).amin(1, keepdim=True)
        span = torch.where(valid, a, -inf).amax(1, keepdim=True) - low
        return torch.where(span > 0, (a - low) / span, torch.zeros_like(a))

    def median(a):
        a = torch.where(valid, a, inf).sort(1).values
        hi = a.gather(1, (n // 2)[:, None])
        lo = a.gather(1, (n // 2 - (n % 2 == 0).long())[:, None])
        return torch.where((n % 2 == 1)[:, None], hi, (lo + hi) / 2)

    x, y = unit(theta), unit(vd)
    thresh = median((y - median(y)).abs())
    xi, yi, xj, yj = x.gather(1, i), y.gather(1, i), x.gather(1, j), y.gather(1, j)
    m = (yj - yi) / (xj - xi)
    c = yi - m * xi
    return x, y, thresh, m, c


def exact(case, seed):
    theta_all, vd_all, offsets, frame_offsets, seeds = _inputs(case, seed)
    dev, hyp, paper = theta_all.device, case["hyp"], case["kind"] == "paper"
    tau = float(np.float32(TAU))
    k_all = len(offsets) - 1
    frame = np.searchsorted(frame_offsets, np.arange(k_all), side="right") - 1
    local = np.arange(k_all) - frame_offsets[frame]
    sizes = np.diff(offsets)
    out = {name: torch.full((k_all,), float("nan"), dtype=torch.float64, device=dev)
           for name in ("vx", "vy", "heading") + (("thresh",) if paper else ())}
    budget = 1 << 27  # elements of one temporary
    order = np.argsort(sizes, kind="stable")
    at = 0
    while at < k_all:
        # Clusters of about one size, padded to the largest of them.
        limit = max(16, int(sizes[order[at]] * 1.2))
        end = at
        while end < k_all and sizes[order[end]] <= limit and \
                (end + 1 - at) * hyp * int(sizes[order[end]]) <= max(budget, hyp * int(sizes[order[end]])):
            end += 1
        ks = order[at:end]
        at = end
        width = int(sizes[ks].max())
        if width < 2:
            continue
        kt = torch.from_numpy(ks).to(dev)
        n = torch.from_numpy(sizes[ks]).to(dev)
        low = torch.from_numpy(offsets[:-1][ks]).to(dev)
        span = torch.arange(width, device=dev)
        valid = span[None] < n[:, None]
        points = torch.where(valid, low[:, None] + span, low[:, None]).clamp(max=theta_all.numel() - 1)
        theta, vd = theta_all[points].double(), vd_all[points].double()
        key = seeds[frame[ks]]
        key0 = torch.from_numpy(key & 0xFFFFFFFF).to(dev)[:, None]
        key1 = torch.from_numpy(key >> 32).to(dev)[:, None]
        h = torch.arange(hyp, device=dev)[None].expand(len(ks), hyp)
        u0, u1 = _philox(h.clone(), torch.from_numpy(local[ks]).to(dev)[:, None].expand_as(h).clone(),
                         key0, key1)
        n2 = n[:, None].clamp(min=2)
        i = (u0 * n2) >> 32
        j = (u1 * (n2 - 1)) >> 32
        j = j + (j >= i)
        j = torch.minimum(j, n2 - 1)
        ok = ((theta.gather(1, j) - theta.gather(1, i)).abs() >= 1e-3) & (n[:, None] >= 2)
        cos, sin = torch.cos(theta), torch.sin(theta)
        if paper:
            x, y, thresh, a, b = _paper_fit(theta, vd, valid, n, i, j)
            scale = torch.sqrt(a * a + 1.0)
        else:
            ci, si, vi = cos.gather(1, i), sin.gather(1, i), vd.gather(1, i)
            cj, sj, vj = cos.gather(1, j), sin.gather(1, j), vd.gather(1, j)
            inv = 1.0 / (ci * sj - si * cj)
            a, b = (vi * sj - vj * si) * inv, (ci * vj - cj * vi) * inv
        count = torch.zeros(len(ks), hyp, dtype=torch.int64, device=dev)
        step = max(1, budget // (len(ks) * width))
        for h0 in range(0, hyp, step):
            a0, b0 = a[:, h0:h0 + step, None], b[:, h0:h0 + step, None]
            if paper:
                r = ((-a0 * x[:, None] + y[:, None]) - b0).abs_()
                inside = r.div_(scale[:, h0:h0 + step, None]) <= thresh[:, :, None]
            else:
                r = (a0 * cos[:, None]).sub_(vd[:, None])
                inside = r.add_(b0 * sin[:, None]).abs_() < tau
            count[:, h0:h0 + step] = (inside & valid[:, None]).sum(2)
        best = torch.where(ok, count * hyp + (hyp - 1 - h), -1).amax(1)
        kept = torch.where(best >= 0, hyp - 1 - best % hyp, 0)[:, None]
        ak, bk = a.gather(1, kept), b.gather(1, kept)
        if paper:
            r = ((-ak * x + y) - bk).abs() / scale.gather(1, kept)
            inlier = (r <= thresh) & valid
        else:
            inlier = ((vd - ak * cos - bk * sin).abs() < tau) & valid
        w = inlier.double()
        scc, scs, sss = (w * cos * cos).sum(1), (w * cos * sin).sum(1), (w * sin * sin).sum(1)
        scv, ssv = (w * cos * vd).sum(1), (w * sin * vd).sum(1)
        det = scc * sss - scs * scs
        good = (best >= 0) & (inlier.sum(1) >= 2) & (det > 0)
        nan = torch.full_like(det, float("nan"))
        vx = torch.where(good, (sss * scv - scs * ssv) / det, nan)
        vy = torch.where(good, (scc * ssv - scs * scv) / det, nan)
        out["vx"][kt], out["vy"][kt], out["heading"][kt] = vx, vy, torch.atan2(vy, vx)
        if paper:
            out["thresh"][kt] = torch.where(n >= 2, thresh[:, 0], nan)
    # Whole-number outputs (counts, status, masks) are compared as they are.
    return out
