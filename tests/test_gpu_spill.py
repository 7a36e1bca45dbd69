"""Tiles too crowded for LDS, whose queries go through the spill kernels: the
lists around a tile of every size against the staging rounds (one short of a
round, just over it, many rounds), hit indices interleaved between the tiles or
one tile after the other, few and many queries a tile, the density kernels and
the strict tie rule, all outputs against the oracle."""
import os

import numpy as np
import pytest

import oracle
from gpu_helpers import assert_parity, gpu_run

pytestmark = pytest.mark.gpu
KW = dict(dc=2.0, rho_c=5.0, delta_c=2.0, delta_o=4.0, bounds=(0, 0, 40, 40), n_layers=2)


def _event(counts, order, seed):
    """Hits of layer 0 within the tiles around (14.1, 14.1): counts[k] in tile k
    of 3 x 3 tiles of 4.03125 cm; a few hits elsewhere and on layer 1."""
    rng = np.random.default_rng(seed)
    t = 4.03125
    xs, ys, layer = [], [], []
    for k, c in enumerate(counts):
        xs.append((2 + k % 3 + rng.uniform(0.02, 0.98, c)) * t)
        ys.append((2 + k // 3 + rng.uniform(0.02, 0.98, c)) * t)
        layer.append(np.zeros(c, np.int32))
    xs.append(rng.uniform(0, 40, 200))
    ys.append(rng.uniform(0, 40, 200))
    layer.append(rng.integers(0, 2, 200).astype(np.int32))
    x, y, layer = np.concatenate(xs).astype(np.float32), np.concatenate(ys).astype(np.float32), np.concatenate(layer)
    p = {"tiles": np.arange(x.size), "reversed": np.arange(x.size)[::-1], "mixed": rng.permutation(x.size)}[order]
    e = np.round(rng.uniform(0.1, 1.0, x.size) * 8) / 8  # ties in density
    return dict(x=x[p], y=y[p], layer=layer[p], energy=e.astype(np.float32))


COUNTS = {
    "one round less one": (100, 100, 100, 100, 223, 100, 100, 100, 100),
    "one round": (100, 100, 100, 100, 224, 100, 100, 100, 100),
    "one hit over": (100, 100, 100, 100, 225, 100, 100, 100, 100),
    "one full tile": (1, 0, 2, 0, 5000, 0, 33, 1, 0),
    "few queries": (1200, 31, 0, 1300, 1, 32, 33, 2, 1100),
    "even": (700,) * 9,
    "257 queries": (900, 0, 0, 0, 257, 0, 0, 900, 0),
}


@pytest.mark.parametrize("counts", list(COUNTS), ids=lambda s: s.replace(" ", "-"))
@pytest.mark.parametrize("order", ["tiles", "reversed", "mixed"])
def test_spilled_tiles(counts, order):
    ev = _event(COUNTS[counts], order, len(counts))
    for kernel, batched in (("flat", False), ("gaussian", True)):
        ref = oracle.run(ev["x"], ev["y"], ev["layer"], ev["energy"], kernel=kernel, kernel_scale=1.0,
                         n_threads=min(16, os.cpu_count() or 1), **KW)
        p = dict(KW, kernel=kernel, kernel_scale=1.0)
        # a cap below any crowded region, with blocks that halve down to single tiles
        tuning = dict(tile_size=4.03125, lds_cap=256, plain_lds_cap=256)
        assert_parity(gpu_run(ev, p, batched=batched, tuning=tuning), ref, where=f"{counts} {order} {kernel}")


def test_spilled_tiles_strict():
    import paper_2001_09761_amd as clue
    ev = _event(COUNTS["even"], "mixed", 3)
    ref = oracle.run(ev["x"], ev["y"], ev["layer"], ev["energy"], paper_strict=True,
                     n_threads=min(16, os.cpu_count() or 1), **KW)
    assert_parity(gpu_run(ev, KW, flags=clue.KEEP_INTERMEDIATES | clue.TIE_PAPER_STRICT, tuning=dict(lds_cap=256,
                  plain_lds_cap=256)), ref, where="strict")


@pytest.mark.parametrize("order", ["layers", "one layer at both ends", "shuffled"])
@pytest.mark.parametrize("batched", [False, True])
def test_events_beyond_the_packed_index(order, batched):
    """An event of more than 2**21 hits: regions whose hits span less than that are staged, counted from their
    first hit, and the others are searched by the spill kernel."""
    from paper_2001_09761_amd import gen
    ev, p = gen.config2(seed=31, event_index=3, n_layers=110, hits_per_layer=20000)
    n = ev["x"].size
    assert n > 2 ** 21
    q = np.arange(n)
    if order == "one layer at both ends":
        q = np.concatenate([q[10000:], q[:10000]])  # half of the first layer's hits come last
    elif order == "shuffled":
        q = np.random.default_rng(1).permutation(n)
    ev = {k: np.ascontiguousarray(ev[k][q]) for k in ("x", "y", "layer", "energy")}
    ref = oracle.run(ev["x"], ev["y"], ev["layer"], ev["energy"], dc=p["dc"], rho_c=p["rho_c"], delta_c=p["delta_c"],
                     delta_o=p["delta_o"], extent=p["extent"], n_layers=p["n_layers"],
                     n_threads=min(16, os.cpu_count() or 1))
    assert_parity(gpu_run(ev, p, batched=batched), ref, where=f"{order} batched {batched}")
