"""Runs whose hits are not grouped by layer, sparse enough that most hits are alone
in their tiles, in two contexts on two streams at once: workgroups of one run then
start late, and every one has to come to the same verdict on the unit path. Bit for
bit against the oracle."""
import os

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu
NT = min(16, os.cpu_count() or 1)
LAYERS, EXTENT = 100, 200.0
RUNS = 12  # of each context, enqueued together


def _event(n, order, seed):
    rng = np.random.default_rng(seed)
    ev = dict(x=rng.uniform(0, EXTENT, n).astype(np.float32), y=rng.uniform(0, EXTENT, n).astype(np.float32),
              layer=np.sort(rng.integers(0, LAYERS, n)).astype(np.int32),
              energy=rng.uniform(0.5, 8.0, n).astype(np.float32))
    if order == "shuffled":
        q = rng.permutation(n)
    else:  # one hit in another layer's place: a single workgroup sees it
        q = np.arange(n)
        a, b = n // 3, n // 3 + 2 * n // LAYERS
        q[a], q[b] = q[b], q[a]
    return {k: np.ascontiguousarray(v[q]) for k, v in ev.items()}


@pytest.mark.parametrize("order", ["shuffled", "one hit out of place"])
@pytest.mark.parametrize("n", [9000, 20000, 40000])
def test_two_streams_of_ungrouped_sparse_runs(n, order):
    import torch
    import paper_2001_09761_amd as clue
    dev = torch.device("cuda", 0)
    lanes = []
    for k in range(2):
        ev = _event(n, order, 10 * n + k)
        ref = oracle.run(ev["x"], ev["y"], ev["layer"], ev["energy"], dc=2.0, rho_c=5.0, delta_c=2.0, delta_o=4.0,
                         bounds=(0, 0, EXTENT, EXTENT), n_layers=LAYERS, n_threads=NT)
        t = {key: torch.from_numpy(v).to(dev) for key, v in ev.items()}
        ctx = clue.Context(2.0, 5.0, 2.0, 4.0, max_hits=n, extent=EXTENT, n_layers=LAYERS)
        outs = [(torch.full((n,), -9, dtype=torch.int32, device=dev), torch.full((n,), 9, dtype=torch.uint8, device=dev))
                for _ in range(RUNS)]
        lanes.append((ctx, torch.cuda.Stream(), t, outs, ref))
    torch.cuda.synchronize()
    print(f"ungrouped sparse runs: {n} hits, {order}", flush=True)
    for i in range(RUNS):
        for ctx, stream, t, outs, _ in lanes:
            ctx.run(t["x"], t["y"], t["layer"], t["energy"], *outs[i], stream=stream)
    for ctx, stream, t, outs, ref in lanes:
        ctx.status(stream)
        for cid, seed in outs:
            assert np.array_equal(cid.cpu().numpy(), ref["cluster_id"])
            assert np.array_equal(seed.cpu().numpy(), ref["is_seed"].astype(np.uint8))
        ctx.close()
