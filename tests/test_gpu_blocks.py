"""Blocks whose region overflows the LDS cap are halved down to single tiles:
every shape of block, at caps where it overflows once, several times and down
to tiles that are queued for the spill kernels, bit for bit against the oracle."""
import os

import numpy as np
import pytest

import oracle
from gpu_helpers import assert_parity, gpu_run
from oracle_cases import adversarial_event

pytestmark = pytest.mark.gpu
P = dict(dc=2.0, rho_c=5.0, delta_c=2.0, delta_o=4.0, bounds=(0, 0, 70, 50), n_layers=2)


@pytest.fixture(scope="module")
def event():
    a = adversarial_event(61, n=3000, n_layers=2, extent=70.0)
    a["y"] = (a["y"] * np.float32(50.0 / 70.0)).astype(np.float32)
    ref = oracle.run(a["x"], a["y"], a["layer"], a["energy"], dc=2.0, rho_c=5.0, delta_c=2.0, delta_o=4.0,
                     bounds=P["bounds"], n_layers=2, n_threads=min(16, os.cpu_count() or 1))
    return a, ref


@pytest.mark.parametrize("block", [(1, 1), (16, 16), (13, 7), (2, 16), (16, 1), (5, 3)])
@pytest.mark.parametrize("cap", [64, 200, 700])
@pytest.mark.parametrize("batched", [False, True])
def test_block_shapes_over_the_cap(event, block, cap, batched):
    ev, ref = event
    tuning = dict(block_x=block[0], block_y=block[1], lds_cap=cap, plain_lds_cap=cap)
    assert_parity(gpu_run(ev, P, batched=batched, tuning=tuning), ref, where=f"{block} cap {cap}")


@pytest.mark.parametrize("bounds", [(0, 0, 200, 200), (-30, 10, 170, 60), (0, 0, 9, 400)], ids=str)
@pytest.mark.parametrize("per_layer", [60, 700, 2500])
@pytest.mark.parametrize("spot", [0.0, 0.9])
def test_sparse_layers_take_large_blocks(bounds, per_layer, spot):
    """Untuned runs of sparse layers take blocks of up to 22 tiles a side and grown tiles; with most
    hits of a layer in one spot, the blocks are halved from there down to single tiles."""
    rng = np.random.default_rng(per_layer)
    n_layers = 9000 // per_layer + 2
    n = n_layers * per_layer
    x0, y0, x1, y1 = bounds
    x, y = rng.uniform(x0, x1, n), rng.uniform(y0, y1, n)
    s = rng.random(n) < spot
    x[s], y[s] = rng.normal(x0 + 6, 2.0, s.sum()), rng.normal(y1 - 20, 2.0, s.sum())
    ev = dict(x=x.astype(np.float32), y=y.astype(np.float32), layer=np.repeat(np.arange(n_layers, dtype=np.int32), per_layer),
              energy=rng.uniform(0.1, 2.0, n).astype(np.float32))
    p = dict(P, bounds=bounds, n_layers=n_layers)
    ref = oracle.run(ev["x"], ev["y"], ev["layer"], ev["energy"], dc=2.0, rho_c=5.0, delta_c=2.0, delta_o=4.0,
                     bounds=bounds, n_layers=n_layers, n_threads=min(16, os.cpu_count() or 1))
    for batched in (False, True):
        assert_parity(gpu_run(ev, p, batched=batched), ref, where=f"{bounds} {per_layer} {spot} {batched}")
