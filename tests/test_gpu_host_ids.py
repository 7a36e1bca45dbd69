"""The host-resident form's event ids, which the device writes from the events'
first hits where events hold 512 hits or more on average, and which are copied
otherwise: more events than one launch of that kernel takes, empty events at
both ends and in runs, chunks of one event and of many, against the oracle; and
CLUE_VALIDATE, which checks the caller's own ids."""
import os

import numpy as np
import pytest

import oracle
from oracle_cases import adversarial_event

pytestmark = pytest.mark.gpu
P = dict(dc=2.0, rho_c=5.0, delta_c=2.0, delta_o=4.0, bounds=(0, 0, 20, 20), n_layers=2)


def _batch(n_events, most=60):
    rng = np.random.default_rng(n_events)
    sizes = rng.integers(0, most, n_events)
    sizes[rng.random(n_events) < 0.4] = 0
    sizes[[0, -1]] = 0
    sizes[n_events // 2] = max(500, 2 * most)
    evs = [{k: v[:s] for k, v in adversarial_event(i, n=max(int(s), 20), n_layers=2).items()}
           for i, s in enumerate(sizes)]
    b = {k: np.concatenate([e[k] for e in evs]) for k in ("x", "y", "layer", "energy")}
    b["event"] = np.repeat(np.arange(n_events, dtype=np.int32), sizes)
    return b, sizes


@pytest.mark.parametrize("n_events", [3, 127, 128, 129, 300])
@pytest.mark.parametrize("cap_events", [1, 7, 1000])
@pytest.mark.parametrize("most", [60, 3000])
def test_ids_of_chunks(n_events, cap_events, most):
    import paper_2001_09761_amd as clue
    b, sizes = _batch(n_events, most)
    ref = oracle.run(b["x"], b["y"], b["layer"], b["energy"], dc=2.0, rho_c=5.0, delta_c=2.0, delta_o=4.0,
                     bounds=P["bounds"], n_layers=2, event=b["event"], n_events=n_events,
                     n_threads=min(16, os.cpu_count() or 1))
    for cap in (max(500, int(sizes.max())), b["x"].size):
        with clue.Context(2.0, 5.0, 2.0, 4.0, max_hits=cap, max_events=cap_events, bounds=P["bounds"],
                          n_layers=2) as ctx:
            cid, seed = ctx.run_batch_host(b["event"], n_events, b["x"], b["y"], b["layer"], b["energy"])
        assert np.array_equal(cid, ref["cluster_id"]) and np.array_equal(seed, ref["is_seed"].astype(np.uint8))


def test_validate_checks_the_callers_ids():
    import paper_2001_09761_amd as clue
    b, _ = _batch(20)
    bad = b["event"].copy()
    bad[10], bad[300] = bad[300], bad[10]  # decreasing
    with clue.Context(2.0, 5.0, 2.0, 4.0, max_hits=b["x"].size, max_events=20, bounds=P["bounds"], n_layers=2,
                      flags=clue.VALIDATE) as ctx:
        with pytest.raises(clue.ClueError) as ei:
            ctx.run_batch_host(bad, 20, b["x"], b["y"], b["layer"], b["energy"])
        assert ei.value.code == -5  # CLUE_ERR_INPUT
        ctx.run_batch_host(b["event"], 20, b["x"], b["y"], b["layer"], b["energy"])
