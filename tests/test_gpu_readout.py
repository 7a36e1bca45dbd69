"""Intermediates and follower lists copied out of a run: sizes around a
workgroup and a 16-byte word, destinations with and without 16-byte alignment,
and each destination left out in turn, against the oracle."""
import ctypes
import os

import numpy as np
import pytest

import oracle
from gpu_helpers import to_dev
from oracle_cases import adversarial_event

pytestmark = pytest.mark.gpu
KW = dict(dc=2.0, rho_c=5.0, delta_c=2.0, delta_o=4.0, bounds=(0, 0, 20, 20), n_layers=3)
GUARD = -77


@pytest.mark.parametrize("n", [20, 255, 1023, 1024, 1025, 9001])
def test_read_out(n):
    import torch
    import paper_2001_09761_amd as clue
    ev = adversarial_event(n, n=n)
    ref = oracle.run(ev["x"], ev["y"], ev["layer"], ev["energy"], n_threads=min(16, os.cpu_count() or 1), **KW)
    t = to_dev(ev, torch.device("cuda", 0))
    total = int(ref["fstart"][n])
    with clue.Context(2.0, 5.0, 2.0, 4.0, max_hits=n, bounds=KW["bounds"], n_layers=3,
                      flags=clue.KEEP_INTERMEDIATES) as ctx:
        ctx.run(t["x"], t["y"], t["layer"], t["energy"])
        L, s = ctx._L, ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
        for shift in (0, 1, 2):
            for skip in (None, 0, 1, 2):
                buf = [torch.full((n + 8,), GUARD, dtype=torch.int32, device="cuda") for _ in range(3)]
                p = [ctypes.c_void_p(0 if k == skip else b[shift:].data_ptr()) for k, b in enumerate(buf)]
                assert L.clue_get_intermediates(ctx._ctx, *p, s) == 0
                torch.cuda.synchronize()
                for k, name in enumerate(("rho", "nh", "delta2")):
                    got = buf[k].cpu().numpy()
                    want = np.full(n + 8, GUARD, np.int32)
                    if k != skip:
                        want[shift:shift + n] = ref[name].view(np.int32)
                    assert np.array_equal(got, want), (name, shift, skip)
                buf = [torch.full((n + 9,), GUARD, dtype=torch.int32, device="cuda") for _ in range(2)]
                p = [ctypes.c_void_p(0 if k == skip else b[shift:].data_ptr()) for k, b in enumerate(buf)]
                num = ctypes.c_int64(-1)
                assert L.clue_get_followers(ctx._ctx, *p, ctypes.byref(num) if skip != 2 else None, s) == 0
                torch.cuda.synchronize()
                assert num.value == (total if skip != 2 else -1)
                fs, fl = buf[0].cpu().numpy(), buf[1].cpu().numpy()
                if skip != 0:
                    assert np.array_equal(fs[shift:shift + n + 1], ref["fstart"])
                    assert np.all(fs[:shift] == GUARD) and np.all(fs[shift + n + 1:] == GUARD)
                if skip != 1:
                    assert np.array_equal(fl[shift:shift + total], ref["flist"])
                    assert np.all(fl[:shift] == GUARD) and np.all(fl[shift + n:] == GUARD)


def test_read_out_under_capture():
    """Captured once, the copy gives each later run's values when replayed."""
    import torch
    import paper_2001_09761_amd as clue
    n = 3000
    with clue.Context(2.0, 5.0, 2.0, 4.0, max_hits=n, bounds=KW["bounds"], n_layers=3,
                      flags=clue.KEEP_INTERMEDIATES) as ctx:
        buf = [torch.zeros(n, dtype=torch.int32, device="cuda") for _ in range(3)]
        graph = torch.cuda.CUDAGraph()
        for seed in range(4):
            ev = adversarial_event(seed, n=n)
            t = to_dev(ev, torch.device("cuda", 0))
            ctx.run(t["x"], t["y"], t["layer"], t["energy"])
            torch.cuda.synchronize()
            if seed == 0:
                with torch.cuda.graph(graph):
                    assert ctx._L.clue_get_intermediates(ctx._ctx, *(ctypes.c_void_p(b.data_ptr()) for b in buf),
                                                         ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)) == 0
            graph.replay()
            torch.cuda.synchronize()
            ref = oracle.run(ev["x"], ev["y"], ev["layer"], ev["energy"], **KW)
            for b, name in zip(buf, ("rho", "nh", "delta2")):
                assert np.array_equal(b.cpu().numpy(), ref[name].view(np.int32)), (seed, name)
