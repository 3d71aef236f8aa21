"""Calls that are enqueued while earlier ones still run: staged lists, blocks of freed batches, streams.
Every value must be the one that the same call gives when it is waited for."""
import numpy as np
import pytest

import mgk_workloads as W
import paper_1910_06310_amd as M

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("entry", ["pairs", "pairs_nodal"])
@pytest.mark.parametrize("streams", [1, 2])
def test_calls_in_flight_keep_their_lists_and_batches(entry, streams):
    import torch
    solver = M.Solver(0)
    resident, busy = W.config1(60), W.config1(700)
    solver.configure(resident.params)
    rng = np.random.default_rng(5)
    R, B = solver.load_batch(resident), solver.load_batch(busy)
    new = [W.molecule_like_batch(rng, 4, 10, 10 + 4 * k, resident.params) for k in range(10)]
    calls = []
    for k, wb in enumerate(new):
        n = 40 + 30 * k   # lists of unlike length
        calls.append((wb, rng.integers(0, 4, n).astype(np.int32), rng.integers(0, 60, n).astype(np.int32)))
    s = [torch.cuda.Stream() for _ in range(streams)]
    K_busy = torch.zeros((700, 700), device="cuda")

    def outputs():
        out = []
        for wb, i, j in calls:
            off = np.concatenate([[0], np.cumsum(wb.sizes()[i].astype(np.int64) * resident.sizes()[j])])
            out.append((torch.full((len(i),), float("nan"), device="cuda"),
                        torch.full((int(off[-1]),), float("nan"), device="cuda"), off[:-1]))
        torch.cuda.synchronize()
        return out

    def enqueue(call, out, stream):
        (wb, i, j), (K, x, off) = call, out
        N = solver.load_batch(wb)
        if entry == "pairs":
            solver.pairs(N, R, i, j, K, stream=stream)
        else:
            solver.pairs_nodal(N, R, i, j, K, x, off, stream=stream)
        N.free()

    alone, together = outputs(), outputs()
    for call, out in zip(calls, alone):
        enqueue(call, out, s[0])
        torch.cuda.synchronize()
    solver.gram(B, K_busy)   # builds its list
    torch.cuda.synchronize()
    for stream in s:
        solver.gram(B, K_busy, stream=stream)
    for k, (call, out) in enumerate(zip(calls, together)):
        enqueue(call, out, s[k % streams])
    torch.cuda.synchronize()
    for (K, x, _), (K1, x1, _) in zip(together, alone):
        assert np.isfinite(K1.cpu().numpy()).all()
        np.testing.assert_array_equal(K.cpu().numpy(), K1.cpu().numpy())
        np.testing.assert_array_equal(x.cpu().numpy(), x1.cpu().numpy())
    R.free()
    B.free()
