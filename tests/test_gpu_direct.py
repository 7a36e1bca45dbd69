"""The all-pairs form that small untuned runs take (up to 8,192 hits): bit
for bit against the oracle at the edges of its candidate chunks (64), blocks
(1,024), workgroups' queries (16) and of its range, over layers, events, order,
kernels and flags, and on a context whose runs alternate between the forms."""
import os

import numpy as np
import pytest

import oracle
from gpu_helpers import assert_parity, gpu_run
from golden_cases import load_cases
from oracle_cases import adversarial_event
from paper_2001_09761_amd import gen

pytestmark = pytest.mark.gpu
NT = min(16, os.cpu_count() or 1)
P = dict(dc=2.0, rho_c=5.0, delta_c=2.0, delta_o=4.0, bounds=(0, 0, 20, 20), n_layers=3)


def _ref(ev, p, **kw):
    return oracle.run(ev["x"], ev["y"], ev["layer"], ev["energy"], dc=p["dc"], rho_c=p["rho_c"],
                      delta_c=p["delta_c"], delta_o=p["delta_o"], extent=p.get("extent"), bounds=p.get("bounds"),
                      n_layers=p["n_layers"], event=ev.get("event"), n_events=ev.get("n_events"),
                      kernel=p.get("kernel", "flat"), kernel_scale=p.get("kernel_scale", 0.0), n_threads=NT, **kw)


@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 63, 64, 65, 100, 1008, 1023, 1024, 1025, 2047, 2049, 8191, 8192,
                               8193])
def test_sizes(n):
    extent = 20.0 if n < 3000 else 100.0
    p = dict(P, n_layers=1 + n % 3, bounds=(0, 0, extent, extent))
    ev = adversarial_event(n, n=n, n_layers=p["n_layers"], extent=extent) if n >= 20 else \
        {k: v[:n] for k, v in adversarial_event(n, n=40, n_layers=p["n_layers"]).items()}
    ref = _ref(ev, p)
    print(f"all-pairs form: n = {n}", flush=True)
    assert_parity(gpu_run(ev, p), ref, where=f"n={n} plain")
    assert_parity(gpu_run(ev, p, batched=True), ref, where=f"n={n} batched")


@pytest.mark.parametrize("kernel", ["flat", "gaussian", "exponential"])
@pytest.mark.parametrize("layers", [1, 7, 100])
def test_kernels_and_layers_crowded(kernel, layers):
    """Hundreds of neighbours a query: its term list is summed several times."""
    rng = np.random.default_rng(layers)
    n = 5000
    ev = dict(x=rng.normal(10.0, 0.8, n).astype(np.float32), y=rng.normal(10.0, 0.8, n).astype(np.float32),
              layer=np.sort(rng.integers(0, layers, n)).astype(np.int32),
              energy=rng.uniform(0.0, 1.0, n).astype(np.float32))
    p = dict(P, n_layers=layers, kernel=kernel, kernel_scale=0.0 if kernel == "flat" else 1.0)
    assert_parity(gpu_run(ev, p), _ref(ev, p), where=f"{kernel}, {layers} layers")


def test_events_of_uneven_sizes_some_empty():
    evs = [adversarial_event(30 + i, n=n, n_layers=3) for i, n in enumerate([700, 20, 1300, 64, 2000, 21])]
    ids = [0, 2, 3, 4, 8, 9]  # events 1, 5, 6 and 7 have no hits, nor has the last
    b = {k: np.concatenate([e[k] for e in evs]) for k in ("x", "y", "layer", "energy")}
    b["event"] = np.concatenate([np.full(e["x"].size, i, np.int32) for i, e in zip(ids, evs)])
    b["n_events"] = 11
    assert_parity(gpu_run(b, P, batched=True, n_events=11), _ref(b, P), where="uneven events")


def test_one_owner_of_every_hit_and_a_long_chain():
    """The longest follower list and the longest chain of links."""
    n = 6000
    star = dict(x=np.full(n, 5.0, np.float32), y=np.full(n, 5.0, np.float32), layer=np.zeros(n, np.int32),
                energy=np.ones(n, np.float32))
    p = dict(P, n_layers=1)
    assert_parity(gpu_run(star, p), _ref(star, p), where="coincident hits")
    chain = dict(x=(np.arange(n) * 1.9).astype(np.float32), y=np.zeros(n, np.float32), layer=np.zeros(n, np.int32),
                 energy=np.linspace(3.0, 4.0, n).astype(np.float32))
    p = dict(P, n_layers=1, bounds=(0, 0, 1.9 * n, 20.0))
    assert_parity(gpu_run(chain, p), _ref(chain, p), where="chain")


def test_flags():
    import paper_2001_09761_amd as clue
    ev = adversarial_event(51, n=1500, n_layers=3, unit_weights=True)
    got = gpu_run(ev, P, flags=clue.KEEP_INTERMEDIATES | clue.TIE_PAPER_STRICT)
    assert_parity(got, _ref(ev, P, paper_strict=True), where="strict")
    got = gpu_run(ev, P, flags=clue.NO_FOLLOWERS)
    assert_parity(got, _ref(ev, P), keys=("cluster_id", "is_seed"), where="no followers")


def test_forms_alternate_on_one_context():
    import paper_2001_09761_amd as clue
    big, p = gen.config3_sweep(1)
    small, _ = gen.config2(n_layers=100, hits_per_layer=81)  # 8,100 hits
    with clue.Context(p["dc"], p["rho_c"], p["delta_c"], p["delta_o"], max_hits=big["x"].size, max_events=2,
                      extent=p["extent"], n_layers=p["n_layers"], flags=clue.KEEP_INTERMEDIATES) as ctx:
        refs = {id(e): _ref(e, p) for e in (big, small)}
        for ev, batched in ((small, False), (big, False), (small, True), (big, True), (small, False)):
            assert_parity(gpu_run(ev, p, batched=batched, ctx=ctx), refs[id(ev)], where=f"{ev['x'].size} {batched}")


@pytest.mark.parametrize("case", load_cases(), ids=lambda c: c["name"])
@pytest.mark.parametrize("batched", [False, True])
def test_hand_cases_through_the_tiled_kernels(case, batched):
    """A set tuning selects the tiled kernels at every size."""
    got = gpu_run(case["event"], dict(case["params"]), batched=batched, tuning=dict(threads_per_query=1))
    for k in ("nh", "cluster_id", "is_seed", "fstart", "flist"):
        assert np.array_equal(got[k], case[k]), k
    assert np.array_equal(got["rho"].view(np.uint32), case["rho"].view(np.uint32))
