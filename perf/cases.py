"""Workloads for timing the clustering library through its public entry points.

A case is a dict of plain values. ``prepare`` builds what a program holds
before it clusters (hits on the GPU, or in pinned host memory for the
host-resident form, and a context), ``run`` makes one pass, ``work`` gives the
bytes and operations a pass cannot do without, and ``exact`` the densities in
64 bits where a pass returns densities.

The events follow ``paper_2001_09761_amd.gen`` (same shapes, orders and
parameters) but are drawn on the GPU, so that 32M hits take well under a
second. ``layer-major`` order is the generators' own: each layer's hits
together, cluster by cluster, noise last. ``shuffled`` permutes the hits of
every event.
"""
import math
import random

import torch

import paper_2001_09761_amd as clue
from paper_2001_09761_amd import autotune, gen

# clustering parameters by name: the benchmark configurations', the paper's
# performance study's and those of the noise-rejection sweep
PARAMS = {
    "default": dict(gen.DEFAULT_PARAMS),
    "dc1": dict(gen.DEFAULT_PARAMS, dc=1.0),
    "dc3": dict(gen.DEFAULT_PARAMS, dc=3.0),
    "paper": dict(gen.PAPER_PARAMS),
    "sweep": dict(gen.NOISE_SWEEP_PARAMS, delta_o=gen.NOISE_SWEEP_DELTA_O[1]),
}

BASE = dict(entry="run", events=1, layers=100, hits_lo=10000, hits_hi=10000, extent=200.0, shape="gauss",
            noise=0.05, cluster=20, params="default", kernel="flat", order="layer-major", tile=0.0, tuned=False,
            keep=False, followers=False)


def _case(name, **kw):
    return dict(BASE, name=name, **kw)


def listed():
    return [
        # the smallest call: one layer of 1,000 hits (config 1), where launches are all the time there is
        _case("event_1k", layers=1, hits_lo=1000, hits_hi=1000, extent=100.0, cluster=19),
        # a small event of odd size through the form that allocates nothing
        _case("noalloc_10k", entry="run_noalloc", layers=10, hits_lo=1003, hits_hi=1003),
        # one point of the noise-rejection sweep: few hits, all windows crowded (hundreds of neighbours each)
        _case("noise_sweep_4k", layers=1, hits_lo=4000, hits_hi=4000, extent=500.0, shape="ellipses", noise=0.3,
              cluster=400, params="sweep", order="shuffled"),
        # the low end of the occupancy sweep, read out in full: densities, nearest-higher and follower lists
        _case("event_100k_full", hits_lo=1000, hits_hi=1000, keep=True, followers=True),
        # the middle of the sweep with the hits in no order
        _case("event_500k_shuffled", hits_lo=5000, hits_hi=5000, order="shuffled"),
        # one full event (config 2), the single-event latency of the benchmark
        _case("event_1M", tuned=True),
        # the paper's own performance study: unit weights, wide clusters, three-tile windows at its 5 cm bin
        _case("paper_1M", shape="unit", cluster=50, params="paper", tile=gen.PAPER_BIN),
        # what a serving slot runs at low load: one event of uneven layers out of a device-resident pool
        _case("served_event", entry="run_batch_range", hits_lo=1000, hits_hi=10000, tuned=True),
        # what a serving slot runs under load: a batch of such events (config 4)
        _case("batch_16_uneven", entry="run_batch", events=16, hits_lo=1000, hits_hi=10000, tuned=True),
        # densities with a Gaussian kernel over a batch, kept for the caller
        _case("batch_4x1M_gaussian", entry="run_batch", events=4, kernel="gaussian", keep=True),
        # the headline batch: 32 full events in one call
        _case("batch_32x1M", entry="run_batch", events=32, tuned=True),
        # a batch that lives in pinned host memory, streamed through a context a quarter of its size
        _case("host_16x500k", entry="run_batch_host", events=16, hits_lo=5000, hits_hi=5000),
    ]


MAX_DRAWN_HITS = 8_000_000


def draw(rng):
    shape, noise, cluster, params, tile, extent = rng.choice([
        ("gauss", 0.05, 20, "default", 0.0, 200.0),
        ("gauss", 0.05, 20, "default", 0.0, 200.0),
        ("gauss", 0.05, 19, "default", 0.0, 100.0),
        ("rings", 0.20, 20, rng.choice(["dc1", "default", "dc3"]), 0.0, 200.0),
        ("unit", 0.05, 50, "paper", gen.PAPER_BIN, 200.0),
        ("unit", 0.05, 50, "paper", 0.0, 200.0),
    ])
    layers = rng.choice([1, rng.randint(2, 99), 100, 100])
    # the density of a full layer is 10,000 hits in 200 x 200 cm
    top = 10000.0 * (extent / 200.0) ** 2
    hi = int(round(math.exp(rng.uniform(math.log(200.0), math.log(top)))))
    lo = rng.choice([hi, max(1, hi // 10)])
    entry = rng.choice(["run", "run", "run_noalloc", "run_batch", "run_batch", "run_batch_range", "run_batch_host"])
    events = 1
    if entry in ("run_batch", "run_batch_host"):
        most = max(1, min(64, MAX_DRAWN_HITS // (hi * layers)))
        events = int(round(math.exp(rng.uniform(0.0, math.log(most)))))
    if entry == "run_noalloc":
        layers = min(layers, 1_000_000 // hi)
    keep = entry in ("run", "run_batch") and rng.random() < 0.3
    return dict(BASE, entry=entry, events=events, layers=layers, hits_lo=lo, hits_hi=hi, extent=extent, shape=shape,
                noise=noise, cluster=cluster, params=params, tile=tile,
                kernel=rng.choice(["flat", "flat", "flat", "gaussian", "exponential"]),
                order=rng.choice(["layer-major", "layer-major", "layer-major", "shuffled"]),
                tuned=tile == 0.0 and rng.random() < 0.5, keep=keep, followers=keep and rng.random() < 0.5)


# --------------------------------------------------------------------------
# Inputs.
# --------------------------------------------------------------------------
def _unit_hits(case):
    """Hits of every (event, layer) unit, a list of events x layers counts; the
    same for every seed, so that a case has one size."""
    rng = random.Random(17 + case["hits_lo"] + case["hits_hi"])
    return [rng.randint(case["hits_lo"], case["hits_hi"]) for _ in range(case["events"] * case["layers"])]


def _hits(case, seed):
    """Device tensors x, y, energy (float32), layer, event (int32), and the events' offsets (host)."""
    dev = torch.device("cuda")
    g = torch.Generator(device=dev)
    g.manual_seed(int(seed) * 1000003 + 12345)
    ext = case["extent"]

    def uniform(n, lo, hi):
        return torch.rand(n, generator=g, device=dev, dtype=torch.float64) * (hi - lo) + lo

    def normal(n):
        return torch.randn(n, generator=g, device=dev, dtype=torch.float64)

    host_counts = _unit_hits(case)
    counts = torch.tensor(host_counts, device=dev)
    n = sum(host_counts)
    units = counts.numel()
    unit = torch.repeat_interleave(torch.arange(units, device=dev), counts, output_size=n)
    first = torch.cumsum(counts, 0) - counts
    pos = torch.arange(n, device=dev) - first[unit]
    # each unit: its clusters of about `cluster` hits one after the other, then its noise
    noise = torch.round(counts * case["noise"]).long()
    in_cl = counts - noise
    ncl = torch.clamp((in_cl + case["cluster"] - 1) // case["cluster"], min=1)
    size, extra = in_cl // ncl, in_cl % ncl
    head = (extra * (size + 1))[unit]
    su = torch.clamp(size[unit], min=1)
    cl = torch.where(pos < head, pos // (su + 1), extra[unit] + (pos - head) // su)
    clustered = pos < in_cl[unit]
    base = torch.cumsum(ncl, 0) - ncl
    k = torch.where(clustered, base[unit] + cl, torch.zeros_like(cl))
    nk = sum(max(1, (h - round(h * case["noise"]) + case["cluster"]) // case["cluster"] + 1) for h in host_counts)
    del pos, head, su, cl
    if case["shape"] in ("gauss", "unit"):
        sigma = 1.0 if case["shape"] == "gauss" else 3.0
        cx, cy = uniform(nk, 0.0, ext), uniform(nk, 0.0, ext)
        ox, oy = sigma * normal(n), sigma * normal(n)
        e = 10.0 * torch.exp(-(ox * ox + oy * oy) / (2.0 * sigma * sigma))
    elif case["shape"] == "rings":  # every second cluster a half circle
        cx, cy = uniform(nk, 0.0, ext), uniform(nk, 0.0, ext)
        radius, phase = uniform(nk, 3.0, 8.0), uniform(nk, 0.0, 2.0 * math.pi)
        span = torch.where(torch.arange(nk, device=dev) % 2 == 1, math.pi, 2.0 * math.pi)
        jitter = 0.5 * normal(n)
        theta = phase[k] + uniform(n, 0.0, 1.0) * span[k]
        ox, oy = (radius[k] + jitter) * torch.cos(theta), (radius[k] + jitter) * torch.sin(theta)
        e = 10.0 * torch.exp(-(jitter * jitter) / 2.0)
    else:  # ellipses of any orientation, away from the edges
        cx, cy = uniform(nk, 60.0, ext - 60.0), uniform(nk, 60.0, ext - 60.0)
        sx, sy, th = uniform(nk, 10.0, 30.0), uniform(nk, 10.0, 30.0), uniform(nk, 0.0, math.pi)
        u, v = sx[k] * normal(n), sy[k] * normal(n)
        ox, oy = u * torch.cos(th[k]) - v * torch.sin(th[k]), u * torch.sin(th[k]) + v * torch.cos(th[k])
        e = torch.ones(n, device=dev, dtype=torch.float64)
    x = torch.where(clustered, cx[k] + ox, uniform(n, 0.0, ext))
    y = torch.where(clustered, cy[k] + oy, uniform(n, 0.0, ext))
    if case["shape"] in ("unit", "ellipses"):
        e = torch.ones(n, device=dev, dtype=torch.float64)
    else:
        e = torch.where(clustered, e, uniform(n, 0.0, 1.0))
    layer, event = (unit % case["layers"]).int(), (unit // case["layers"]).int()
    out = dict(x=x.float(), y=y.float(), energy=e.float(), layer=layer, event=event)
    if case["order"] == "shuffled":  # within each event
        order = torch.argsort(event.double() + 0.999 * uniform(n, 0.0, 1.0))
        out = {key: t[order].contiguous() for key, t in out.items()}
    offsets = [0]
    for i in range(case["events"]):
        offsets.append(offsets[-1] + sum(host_counts[i * case["layers"]:(i + 1) * case["layers"]]))
    return out, offsets


def _params(case):
    return dict(PARAMS[case["params"]], extent=case["extent"], n_layers=case["layers"])


def _shipped_tuning(case, n):
    """The tuning the package ships for this workload, as set_tuning arguments; {} if it ships none."""
    if not case["tuned"]:
        return {}
    t = autotune.load_cached(autotune.cache_key(_params(case), n, case["events"]), autotune.SHIPPED_CACHE)
    if t is None:
        return {}
    return dict(tile_size=t["tile_size"], threads_per_query=t["threads_per_query"], block_x=t["block"][0],
                block_y=t["block"][1], lds_cap=t["lds_cap"], nh_first_radius=t["nh_first_radius"],
                density_quads=t["density_quads"], expansion=t.get("expansion", 1),
                plain_lds_cap=t.get("plain_lds_cap", 0))


def prepare(case, seed):
    hits, offsets = _hits(case, seed)
    n, p = offsets[-1], _params(case)
    scale = 0.0 if case["kernel"] == "flat" else 1.0
    st = dict(case=case, n=n, tuning=_shipped_tuning(case, n))
    if case["entry"] == "run_noalloc":
        st.update(hits, cluster_id=torch.empty(n, dtype=torch.int32, device="cuda"),
                  is_seed=torch.empty(n, dtype=torch.uint8, device="cuda"), scale=scale)
        return st
    max_hits, max_events = n, case["events"]
    if case["entry"] == "run_batch_host":
        # a context of about a quarter of the batch, in whole events
        max_events = max(1, case["events"] // 4)
        max_hits = max(offsets[i + max_events] - offsets[i] for i in range(case["events"] - max_events + 1))
        hits = {key: torch.empty(t.shape, dtype=t.dtype, pin_memory=True).copy_(t) for key, t in hits.items()}
        st.update(cluster_id=torch.empty(n, dtype=torch.int32, pin_memory=True),
                  is_seed=torch.empty(n, dtype=torch.uint8, pin_memory=True))
    elif case["entry"] != "run":  # a pool's or a batch's own outputs
        st.update(cluster_id=torch.empty(n, dtype=torch.int32, device="cuda"),
                  is_seed=torch.empty(n, dtype=torch.uint8, device="cuda"))
    if case["entry"] == "run_batch_range":  # the event's id in its pool
        hits["event"] += 3
    flags = clue.KEEP_INTERMEDIATES if case["keep"] else 0
    ctx = clue.Context(p["dc"], p["rho_c"], p["delta_c"], p["delta_o"], max_hits=max_hits, max_events=max_events,
                       extent=p["extent"], n_layers=p["n_layers"], tile_size=case["tile"], flags=flags,
                       kernel=case["kernel"], kernel_scale=scale)
    if st["tuning"]:
        ctx.set_tuning(**st["tuning"])
    if case["followers"]:
        st["flist"] = torch.full((n,), -1, dtype=torch.int32, device="cuda")
    st.update(hits, ctx=ctx)
    return st


# --------------------------------------------------------------------------
# One pass.
# --------------------------------------------------------------------------
def run(st):
    case = st["case"]
    x, y, layer, energy = st["x"], st["y"], st["layer"], st["energy"]
    if case["entry"] == "run_noalloc":
        p = _params(case)
        cid, seed = clue.run_noalloc(p["dc"], p["rho_c"], p["delta_c"], p["delta_o"], x, y, layer, energy,
                                     st["cluster_id"], st["is_seed"], extent=p["extent"], n_layers=p["n_layers"],
                                     tile_size=case["tile"], kernel=case["kernel"], kernel_scale=st["scale"],
                                     tuning=st["tuning"] or None)
        return dict(cluster_id=cid, is_seed=seed)
    ctx = st["ctx"]
    if case["entry"] == "run":
        cid, seed = ctx.run(x, y, layer, energy)
    elif case["entry"] == "run_batch":
        cid, seed = ctx.run_batch(st["event"], case["events"], x, y, layer, energy, st["cluster_id"], st["is_seed"])
    elif case["entry"] == "run_batch_range":
        cid, seed = ctx.run_batch_range(3, case["events"], st["event"], x, y, layer, energy, st["cluster_id"],
                                        st["is_seed"])
    else:
        cid, seed = ctx.run_batch_host(st["event"], case["events"], x, y, layer, energy, st["cluster_id"],
                                       st["is_seed"])
    out = dict(cluster_id=cid, is_seed=seed)
    if case["keep"]:
        out.update(ctx.intermediates())
    if case["followers"]:
        out["fstart"], flist = ctx.followers()
        # how many there are depends on the hits: they go to the front of the program's own array
        st["flist"][:flist.numel()].copy_(flist)
        out["flist"] = st["flist"]
    return out


def work(case):
    """Bytes: every input read once and every output written once. Operations:
    the six of a distance and its sum for each neighbour within dc, for the
    density, and as many for the nearest-higher search."""
    mean = 0.5 * (case["hits_lo"] + case["hits_hi"])
    n = mean * case["layers"] * case["events"]
    per_hit = 16.0 + 5.0 + (12.0 if case["keep"] else 0.0) + (8.0 if case["followers"] else 0.0)
    if case["entry"] not in ("run", "run_noalloc"):
        per_hit += 4.0
    dc = PARAMS[case["params"]]["dc"]
    uniform = mean * math.pi * dc * dc / (case["extent"] ** 2)
    sigma = {"gauss": 1.0, "unit": 3.0, "ellipses": 20.0}.get(case["shape"])
    if sigma is None:  # a ring of mean radius 5.5 cm
        near = min(1.0, 2.0 * dc / (2.0 * math.pi * 5.5))
    else:  # two hits of one Gaussian cluster within dc of each other
        near = 1.0 - math.exp(-dc * dc / (4.0 * sigma * sigma))
    neighbours = uniform + case["cluster"] * near
    return {"bytes": n * per_hit, "flops": n * neighbours * 12.0}


def exact(case, seed):
    """rho with 64-bit distances, kernel and sums; no other output is a computed number of its own."""
    if not case["keep"]:
        return None
    counts = _unit_hits(case)
    if sum(c * c for c in counts) > 2e11:
        return None
    hits, _ = _hits(case, seed)
    p = PARAMS[case["params"]]
    n = hits["x"].numel()
    rho = torch.empty(n, dtype=torch.float64, device="cuda")
    unit = hits["event"].long() * case["layers"] + hits["layer"].long()
    order = torch.argsort(unit, stable=True)
    x, y, e = (hits[k].double()[order] for k in ("x", "y", "energy"))
    at = 0
    for c in counts:
        xu, yu, eu = x[at:at + c], y[at:at + c], e[at:at + c]
        parts = []
        for a in range(0, c, 2500):
            d2 = (xu[a:a + 2500, None] - xu[None, :]) ** 2 + (yu[a:a + 2500, None] - yu[None, :]) ** 2
            if case["kernel"] == "flat":
                chi = torch.ones_like(d2)
            elif case["kernel"] == "gaussian":
                chi = torch.exp(d2 * -0.5)  # scale 1 cm
            else:
                chi = torch.exp(-torch.sqrt(d2))
            parts.append(torch.where(d2 < p["dc"] * p["dc"], chi * eu[None, :], 0.0).sum(1))
        if parts:
            rho[order[at:at + c]] = torch.cat(parts)
        at += c
    out = dict(cluster_id=None, is_seed=None, rho=rho, nh=None, delta2=None)
    if case["followers"]:
        out.update(fstart=None, flist=None)
    return out
