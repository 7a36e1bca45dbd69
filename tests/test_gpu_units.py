"""The unit path, with the units' hits together and apart, and the general path
it falls back to: bit for bit against the oracle with units empty, of one hit, of
the sizes around a workgroup's 1,024 lanes and around the largest unit it takes,
with layers out of order, and with contexts that meet both kinds of run."""
import os

import numpy as np
import pytest

import oracle
from gpu_helpers import assert_parity, gpu_run
from oracle_cases import adversarial_event

pytestmark = pytest.mark.gpu
NT = min(16, os.cpu_count() or 1)
P = dict(dc=2.0, rho_c=5.0, delta_c=2.0, delta_o=4.0, bounds=(0, 0, 60, 60))


def _ref(ev, p, **kw):
    return oracle.run(ev["x"], ev["y"], ev["layer"], ev["energy"], dc=p["dc"], rho_c=p["rho_c"],
                      delta_c=p["delta_c"], delta_o=p["delta_o"], bounds=p["bounds"], n_layers=p["n_layers"],
                      event=ev.get("event"), n_events=ev.get("n_events"), n_threads=NT, **kw)


def _layers(sizes, seed, extent=60.0):
    """One event with sizes[l] hits on layer l, in layer order."""
    parts = []
    for i, n in enumerate(sizes):
        e = adversarial_event(1000 * seed + i, n=max(n, 20), n_layers=1, extent=extent)
        parts.append({k: v[:n] for k, v in e.items()})
        parts[-1]["layer"] = np.full(n, i, np.int32)
    return {k: np.concatenate([q[k] for q in parts]) for k in ("x", "y", "layer", "energy")}


SIZES = {
    "uneven": [0, 1, 1023, 1024, 1025, 0, 2049, 3000, 64, 0],
    "first and last empty": [0, 5000, 0, 4097, 0],
    "largest": [11264, 1, 300],
    "too large by one": [11265, 40, 300],
    "too large": [300, 13000, 300],
}


@pytest.mark.parametrize("name", list(SIZES))
@pytest.mark.parametrize("batched", [False, True])
def test_unit_sizes(name, batched):
    ev = _layers(SIZES[name], 1)
    p = dict(P, n_layers=len(SIZES[name]))
    print(f"unit path, {name}: {ev['x'].size} hits", flush=True)
    got = gpu_run(ev, p, batched=batched, tuning=dict(threads_per_query=2))
    assert_parity(got, _ref(ev, p), where=name)


@pytest.mark.parametrize("order", ["last two layers swapped", "one hit out of place", "reversed", "shuffled"])
@pytest.mark.parametrize("batched", [False, True])
def test_hits_not_grouped(order, batched):
    ev = _layers([3000, 2000, 1500, 2500], 2)
    n = ev["x"].size
    q = np.arange(n)
    if order == "last two layers swapped":
        q = np.r_[q[:5000], q[6500:], q[5000:6500]]
    elif order == "one hit out of place":
        q[[2999, 3000]] = q[[3000, 2999]]
    elif order == "reversed":
        q = q[::-1]
    else:
        q = np.random.default_rng(3).permutation(n)
    ev = {k: np.ascontiguousarray(v[q]) for k, v in ev.items()}
    p = dict(P, n_layers=4)
    assert_parity(gpu_run(ev, p, batched=batched), _ref(ev, p), where=order)


@pytest.mark.parametrize("sizes", [[12900, 300, 0, 11000], [11264, 11265, 1, 40, 0], [0, 0, 9000]])
@pytest.mark.parametrize("batched", [False, True])
def test_large_units_apart(sizes, batched):
    """Units over and at what LDS holds, their hits interleaved; one crowded in a single tile."""
    ev = _layers(sizes, 7)
    n = ev["x"].size
    ev["x"][:400] = 10.0 + 0.001 * np.arange(400, dtype=np.float32)
    ev["y"][:400] = 10.0
    q = np.random.default_rng(n).permutation(n)
    ev = {k: np.ascontiguousarray(v[q]) for k, v in ev.items()}
    p = dict(P, n_layers=len(sizes))
    got = gpu_run(ev, p, batched=batched, tuning=dict(threads_per_query=2))
    assert_parity(got, _ref(ev, p), where=f"{sizes}")


def _batch(sizes_per_event, ids, n_events):
    evs = [_layers(s, 10 + i) for i, s in enumerate(sizes_per_event)]
    b = {k: np.concatenate([e[k] for e in evs]) for k in ("x", "y", "layer", "energy")}
    b["event"] = np.concatenate([np.full(e["x"].size, i, np.int32) for i, e in zip(ids, evs)])
    b["n_events"] = n_events
    return b


@pytest.mark.parametrize("tuning", [None, dict(lds_cap=128), dict(tile_size=2.1, block_x=4, block_y=4)])
def test_batch_with_empty_events(tuning):
    """Events 0, 3 and the last have no hits; crowded units go through the spill queues too."""
    b = _batch([[4000, 0, 900], [0, 0, 2500], [1200, 3100, 0], [10, 20, 30]], [1, 2, 4, 5], 7)
    p = dict(P, n_layers=3)
    assert_parity(gpu_run(b, p, batched=True, n_events=7, tuning=tuning), _ref(b, p), where=f"{tuning}")


def test_one_context_meets_grouped_and_other_runs():
    import paper_2001_09761_amd as clue
    p = dict(P, n_layers=3)
    runs = []
    for k, shuffled in enumerate((False, True, False, True, False)):
        b = _batch([[3000 + 100 * k, 500, 2000], [100, 4000, 800]], [0, 1], 2)
        if shuffled:
            rng = np.random.default_rng(k)
            q = np.argsort(b["event"] + 0.9 * rng.random(b["x"].size), kind="stable")
            b = {key: (v[q] if isinstance(v, np.ndarray) else v) for key, v in b.items()}
        runs.append(b)
    with clue.Context(p["dc"], p["rho_c"], p["delta_c"], p["delta_o"], max_hits=20000, max_events=2,
                      bounds=p["bounds"], n_layers=3, flags=clue.KEEP_INTERMEDIATES) as ctx:
        for k, b in enumerate(runs):
            assert_parity(gpu_run(b, p, batched=True, n_events=2, ctx=ctx), _ref(b, p), where=f"run {k}")


def test_no_followers_and_strict():
    import paper_2001_09761_amd as clue
    ev = _layers([4000, 3000, 2500], 5)
    p = dict(P, n_layers=3)
    got = gpu_run(ev, p, flags=clue.NO_FOLLOWERS | clue.KEEP_INTERMEDIATES)
    assert_parity(got, _ref(ev, p), keys=("cluster_id", "is_seed", "rho", "nh", "delta2"), where="no followers")
    got = gpu_run(ev, p, flags=clue.KEEP_INTERMEDIATES | clue.TIE_PAPER_STRICT)
    assert_parity(got, _ref(ev, p, paper_strict=True), where="strict")


def test_long_chain_and_one_owner():
    """The deepest links and the longest list of a unit."""
    n = 9000
    p = dict(P, n_layers=2, bounds=(0, 0, 200, 200))
    k = np.arange(n)
    row, col = k // 100, k % 100  # a snake through the layer, 1.9 cm a step
    chain = dict(x=(1.9 * np.where(row % 2 == 0, col, 99 - col)).astype(np.float32), y=(2.1 * row).astype(np.float32),
                 layer=np.ones(n, np.int32), energy=np.linspace(3.0, 400.0, n).astype(np.float32))
    assert_parity(gpu_run(chain, p), _ref(chain, p), where="chain")
    star = dict(x=np.full(n, 30.0, np.float32), y=np.full(n, 30.0, np.float32), layer=np.ones(n, np.int32),
                energy=np.ones(n, np.float32))
    assert_parity(gpu_run(star, p), _ref(star, p), where="coincident hits")


@pytest.mark.parametrize("tuning", [dict(), dict(lds_cap=64), dict(density_quads=2), dict(density_quads=3, tile_size=5.0),
                                    dict(expansion=2), dict(tile_size=2.5, nh_first_radius=0.0)])
@pytest.mark.parametrize("order", ["grouped", "shuffled"])
def test_small_runs_of_many_items_by_the_graph(tuning, order):
    """Batches of up to 4M hits run by sized launches unless they have over
    65,536 work items: here 160 events of 3 layers in one-tile blocks, so that the
    captured graph's persistent kernels meet empty events, units of one hit,
    crowded tiles (the spill queues at the low cap) and hits out of order."""
    sizes = [[30 + 7 * (i % 5), i % 3, 100] if i % 11 else [0, 0, 0] for i in range(160)]
    sizes[7] = [900, 500, 1025]
    ids = list(range(160))
    b = _batch(sizes, ids, 160)
    if order == "shuffled":
        q = np.argsort(b["event"] + 0.9 * np.random.default_rng(1).random(b["x"].size), kind="stable")
        b = {k: (v[q] if isinstance(v, np.ndarray) else v) for k, v in b.items()}
    p = dict(P, n_layers=3)
    t = dict(dict(block_x=1, block_y=1, tile_size=4.03125), **tuning)
    assert_parity(gpu_run(b, p, batched=True, n_events=160, tuning=t), _ref(b, p), where=f"{tuning} {order}")


@pytest.mark.parametrize("n_per_layer", [700, 3000], ids=["all pairs", "tiles"])
@pytest.mark.parametrize("warm", [False, True])
def test_small_batch_under_capture(n_per_layer, warm):
    """A small batch captured by the caller, as a context's first run and after one, in a context with room
    for batches that replay the context's own graph. Replayed over grouped and shuffled hits in turn, with
    eager runs between, every replay equals the oracle."""
    import torch
    import paper_2001_09761_amd as clue
    dev = torch.device("cuda", 0)
    p = dict(P, n_layers=3)

    def draw(seed, shuffled):
        ev = _layers([n_per_layer] * 3, seed)
        if shuffled:
            q = np.random.default_rng(seed).permutation(ev["x"].size)
            ev = {k: v[q] for k, v in ev.items()}
        return ev

    first = draw(50, False)
    n = first["x"].size
    t = {k: torch.from_numpy(v).to(dev) for k, v in first.items()}
    ids = torch.zeros(n, dtype=torch.int32, device=dev)
    cid = torch.empty(n, dtype=torch.int32, device=dev)
    seed_out = torch.empty(n, dtype=torch.uint8, device=dev)
    with clue.Context(2.0, 5.0, 2.0, 4.0, max_hits=6_000_000, max_events=2, bounds=p["bounds"], n_layers=3) as ctx:
        args = (ids, 1, t["x"], t["y"], t["layer"], t["energy"], cid, seed_out)
        if warm:
            ctx.run_batch(*args)
            torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            ctx.run_batch(*args)
        for i in range(4):
            ev = draw(60 + i, i % 2 == 1)
            for k in t:
                t[k].copy_(torch.from_numpy(ev[k]))
            graph.replay()
            torch.cuda.synchronize()
            ref = _ref(ev, p)
            for when in ("replay", "eager"):
                assert np.array_equal(cid.cpu().numpy(), ref["cluster_id"]), (i, when)
                assert np.array_equal(seed_out.cpu().numpy(), ref["is_seed"].astype(np.uint8)), (i, when)
                cid.fill_(-9)
                if when == "replay":
                    ctx.run_batch(*args)
                    torch.cuda.synchronize()
