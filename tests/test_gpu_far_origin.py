"""Grids far from the origin, where the rounding of the coordinates widens the
density windows to three tiles at tiles that are otherwise large enough for two:
every run stays within the arena of the requested grid and equals the oracle bit
for bit."""
import os

import numpy as np
import pytest

import oracle
from gpu_helpers import assert_parity, gpu_run

pytestmark = pytest.mark.gpu
NT = min(16, os.cpu_count() or 1)
P = dict(dc=0.01, rho_c=12.0, delta_c=0.01, delta_o=0.03, bounds=(4200.0, 4200.0, 4201.0, 4201.0), n_layers=3)


def _event(n, order, seed=5):
    rng = np.random.default_rng(seed)
    c = rng.uniform(4200.0, 4201.0, (n // 20, 2))[rng.integers(0, n // 20, n)]
    xy = (c + rng.normal(0.0, 0.008, (n, 2))).astype(np.float32)
    ev = dict(x=xy[:, 0], y=xy[:, 1], layer=np.sort(rng.integers(0, 3, n)).astype(np.int32),
              energy=rng.uniform(0.5, 5.0, n).astype(np.float32))
    q = np.arange(n) if order == "grouped" else rng.permutation(n)
    return {k: np.ascontiguousarray(v[q]) for k, v in ev.items()}


def _ref(ev):
    return oracle.run(ev["x"], ev["y"], ev["layer"], ev["energy"], dc=P["dc"], rho_c=P["rho_c"], delta_c=P["delta_c"],
                      delta_o=P["delta_o"], bounds=P["bounds"], n_layers=P["n_layers"], n_threads=NT)


@pytest.mark.parametrize("order", ["grouped", "shuffled"])
@pytest.mark.parametrize("n", [9000, 20000])
def test_far_origin(n, order):
    import torch
    import paper_2001_09761_amd as clue
    ev = _event(n, order)
    ref = _ref(ev)
    print(f"far origin: {n} hits, {order}", flush=True)
    for batched in (False, True):
        assert_parity(gpu_run(ev, P, batched=batched), ref, where=f"batched {batched}")
    t = {k: torch.from_numpy(v).cuda() for k, v in ev.items()}
    cid = torch.full((n,), -9, dtype=torch.int32, device="cuda")
    seed = torch.full((n,), 9, dtype=torch.uint8, device="cuda")
    clue.run_noalloc(P["dc"], P["rho_c"], P["delta_c"], P["delta_o"], t["x"], t["y"], t["layer"], t["energy"], cid, seed,
                     bounds=P["bounds"], n_layers=P["n_layers"])
    torch.cuda.synchronize()
    assert np.array_equal(cid.cpu().numpy(), ref["cluster_id"])
    assert np.array_equal(seed.cpu().numpy(), ref["is_seed"].astype(np.uint8))
