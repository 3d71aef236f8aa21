"""Whole solves on chip with the separable product: sizes at the edges of its tiles and launch shapes, every
division of the rank, rows longer than the packets read ahead, against the streaming solver node by node and the
fp64 oracle.

Values against the oracle: 1e-4, the bound of the kernel values in general.  Two solvers against each other: both
stop at a relative residual of 1e-6; 2e-5 is what the products are held to elsewhere."""
import dataclasses
import re

import numpy as np
import pytest

import mgk_workloads as W
import paper_1910_06310_amd as M
from oracle import c_oracle as C

pytestmark = pytest.mark.gpu
RTOL, RTOL_PATHS = 1e-4, 2e-5
PARAMS = W.KernelParams(q=0.05, h=0.5, length_scale=1.0)


@pytest.fixture(scope="module")
def torch():
    import torch
    return torch


@pytest.fixture(scope="module")
def solver(torch):
    return M.Solver(0)


def er(seed, sizes, density):
    rng = np.random.default_rng(seed)
    return W.concat_batches([W.erdos_renyi_batch(rng, 1, n, n, density, (0.1, 1.0), (0.0, 1.0), 4, PARAMS, w_min=1e-3)
                             for n in sizes], PARAMS, "er")


def solve(torch, solver, X, Y, wx, wy, pi, pj, path):
    solver.set_tile_path(path)
    off = np.concatenate([[0], np.cumsum(wx.sizes()[pi] * wy.sizes()[pj])]).astype(np.int64)
    K = torch.full((len(pi),), float("nan"), dtype=torch.float32, device="cuda")
    x = torch.full((int(off[-1]),), float("nan"), dtype=torch.float32, device="cuda")
    fl = torch.full((len(pi),), -1, dtype=torch.int32, device="cuda")
    solver.pairs_nodal(X, Y, pi, pj, K, x, off[:-1], None, fl)
    torch.cuda.synchronize()
    assert (fl.cpu().numpy() == 0).all()
    return K.cpu().numpy().astype(np.float64), x.cpu().numpy().astype(np.float64), solver.launch_log()


def compare(torch, solver, wx, wy, const=False, repeat=1):
    """All pairs of graphs of two batches with and without the separable product; the launches of the first."""
    pi = np.tile(np.repeat(np.arange(len(wx.sizes())), len(wy.sizes())), repeat).astype(np.int32)
    pj = np.tile(np.tile(np.arange(len(wy.sizes())), len(wx.sizes())), repeat).astype(np.int32)
    solver.configure(wx.params)
    if const:
        solver.set_edge_kernel_const(0.7)
    solver.set_solver(1e-6, 0)
    try:
        X, Y = solver.load_batch(wx), solver.load_batch(wy)
        K, x, log = solve(torch, solver, X, Y, wx, wy, pi, pj, M.TILE_AUTO)
        Kd, xd, direct = solve(torch, solver, X, Y, wx, wy, pi, pj, M.TILE_SPARSE)
        X.free()
        Y.free()
    finally:
        solver.set_tile_path(M.TILE_AUTO)
    assert "sep" not in direct
    np.testing.assert_allclose(K, Kd, rtol=RTOL_PATHS)
    assert np.linalg.norm(x - xd) <= RTOL_PATHS * np.linalg.norm(xd)
    return pi, pj, K, log


def shapes(log):
    """(features per pass, elements per thread, wavefronts, passes) of every launch."""
    return {tuple(map(int, m)) for m in re.findall(r"mgk_pcg_sep<(\d+), (\d+), (\d+)> passes=(\d+)", log)}


@pytest.mark.parametrize("length_scale,division", [(20.0, (4, 1)), (1.7, (4, 1)), (1.0, (5, 1)), (0.7, (6, 1)), (0.5, (7, 1)), (0.44, (4, 2)),
                                                   (0.33, (5, 2)), (None, (1, 1))])
def test_every_division_of_the_rank(torch, solver, length_scale, division):
    wb = er(1, (77, 90, 96), 0.2)
    wb.params = dataclasses.replace(PARAMS, length_scale=length_scale or 1.0)
    *_, log = compare(torch, solver, wb, wb, const=length_scale is None)
    assert {(rk, passes) for rk, _, _, passes in shapes(log)} == {division}


@pytest.mark.parametrize("nx,ny,density,shape", [((63, 64, 49), (17, 31, 32), 0.5, (4, 8)), ((64, 65), (63, 48), 0.4, (8, 8)),
                                                 ((72, 81), (71,), 0.3, (6, 16)), ((96, 85), (80, 85), 0.25, (8, 16)),
                                                 ((96, 97), (95, 96), 0.2, (10, 16)), ((110, 112), (109, 97), 0.12, (12, 16)),
                                                 ((119, 118), (113, 120), 0.045, (14, 16)), ((285,), (49,), 0.01, (14, 16))])
def test_edges_of_tiles_and_launch_shapes(torch, solver, nx, ny, density, shape):
    """Rows in 16s and 4s, columns in 4s and 16s, the larger graph on either side and with vertices without
    edges; every number of elements per thread."""
    lone = W.erdos_renyi_batch(np.random.default_rng(3), 1, nx[0], nx[0], density, (0.5, 1.0), (0.0, 1.0), 4, PARAMS)
    keep = (lone.src < nx[0] - 5) & (lone.dst < nx[0] - 5)   # five vertices without edges: a whole group of four
    lone.src, lone.dst, lone.weight, lone.edge_label = (a[keep] for a in (lone.src, lone.dst, lone.weight, lone.edge_label))
    lone.edge_off = np.array([0, int(keep.sum())], lone.edge_off.dtype)
    wx, wy = W.concat_batches([er(sum(nx), nx, density), lone], PARAMS, "edges"), er(sum(ny), ny, density if nx[0] < 200 else 0.22)
    for a, b in ((wx, wy), (wy, wx)):
        pi, pj, K, log = compare(torch, solver, a, b)
        assert ((5,) + shape + (1,)) in shapes(log)
    both = W.concat_batches([wy, wx], PARAMS, "both")
    once = wy.nnz()[pi].astype(np.int64) * wx.nnz()[pj] < 2e7
    np.testing.assert_allclose(K[once], C.pairs(both, pi[once], pj[once] + len(ny), tier=1), rtol=RTOL)


def test_hubs_and_the_largest_pairs(torch, solver):
    """Rows of 95 nonzeros beside rows of one (packets beyond those read ahead); pairs of more than 14336 elements stay with
    the streaming solver, in the same call as others."""
    rng = np.random.default_rng(9)
    star = W.erdos_renyi_batch(rng, 1, 96, 96, 1.0, (0.1, 1.0), (0.0, 1.0), 4, PARAMS)
    keep = (star.src < 3) | (star.dst < 3)
    star.src, star.dst, star.weight, star.edge_label = (a[keep] for a in (star.src, star.dst, star.weight, star.edge_label))
    star.edge_off = np.array([0, int(keep.sum())], star.edge_off.dtype)
    wb = W.concat_batches([star, W.barabasi_albert_batch(rng, 2, 96, 6, 4, PARAMS), er(4, (121, 128), 0.03)], PARAMS, "hubs")
    pi, pj, K, log = compare(torch, solver, wb, wb, repeat=12)
    assert shapes(log) and "mgk_pcg_small<16, 16" in log
    few = (pi <= pj) & (np.arange(len(pi)) < 25)
    np.testing.assert_allclose(K[few], C.pairs(wb, pi[few], pj[few], tier=1), rtol=RTOL)


def test_gram_with_iteration_counts_and_calls_on_two_streams(torch, solver):
    """The packets belong to the context: a call on another stream, with other labels and another length scale,
    waits for the kernels that read them.  Iterations as with the streaming solver."""
    solver.configure(PARAMS)
    solver.set_solver(1e-6, 0)
    batches, want = [], []
    for seed in (1, 2):
        B = solver.load_batch(er(seed, (80,) * 24, 0.3))
        batches.append(B)
    scales = [(1.0,), (0.6,)]
    streams = [torch.cuda.Stream() for _ in range(2)]
    out = [[torch.zeros((24, 24), dtype=torch.float32, device="cuda") for _ in range(4)] for _ in range(2)]
    its = [torch.zeros((24, 24), dtype=torch.int32, device="cuda") for _ in range(2)]
    torch.cuda.synchronize()
    for B, (ls,) in zip(batches, scales):
        solver.configure(dataclasses.replace(PARAMS, length_scale=ls))
        K = torch.zeros((24, 24), dtype=torch.float32, device="cuda")
        solver.gram(B, K, its[0])
        assert shapes(solver.launch_log())
        torch.cuda.synchronize()
        solver.set_product_cache(0)
        Kd = torch.zeros_like(K)
        solver.gram(B, Kd, its[1])
        assert not shapes(solver.launch_log())
        torch.cuda.synchronize()
        solver.set_product_cache(1)
        np.testing.assert_allclose(K.cpu().numpy(), Kd.cpu().numpy(), rtol=RTOL_PATHS)
        assert int((its[0] - its[1]).abs().max()) <= 1   # rounding of the entries next to the stop test
        want.append(K.cpu().numpy())
    for k in range(4):
        for b in range(2):
            solver.configure(dataclasses.replace(PARAMS, length_scale=scales[b][0]))
            solver.gram(batches[b], out[b][k], None, None, streams[b])
    torch.cuda.synchronize()
    for b in range(2):
        for k in range(4):
            np.testing.assert_array_equal(out[b][k].cpu().numpy(), want[b])


@pytest.mark.parametrize("length_scale,sides", [(1.0, 1), (0.44, 2), (None, 2)])
def test_without_allocation(torch, solver, length_scale, sides):
    """mgk_pairs_noalloc has its packets in a fixed array: the same kernels and bits as mgk_pairs, call after call."""
    rng = np.random.default_rng(31)
    ba = [W.concat_batches([W.barabasi_albert_batch(rng, 1, int(n), 6, 4, PARAMS) for n in rng.integers(60, 97, 24)], PARAMS, "ba") for _ in range(2)]
    solver.configure(dataclasses.replace(PARAMS, length_scale=length_scale or 1.0))
    if length_scale is None:
        solver.set_edge_kernel_const(0.7)
    solver.set_solver(1e-6, 0)
    X, Y = solver.load_batch(ba[0]), solver.load_batch(ba[1])
    if sides == 1:
        Y = X
    for n in (3000, 700):
        pi, pj = rng.integers(0, 24, n).astype(np.int32), rng.integers(0, 24, n).astype(np.int32)
        got = []
        for entry in (solver.pairs_noalloc, solver.pairs, solver.pairs_noalloc):
            K = torch.full((n,), float("nan"), dtype=torch.float32, device="cuda")
            it, fl = torch.zeros(n, dtype=torch.int32, device="cuda"), torch.full((n,), -1, dtype=torch.int32, device="cuda")
            entry(X, Y, pi, pj, K, it, fl)
            torch.cuda.synchronize()
            assert shapes(solver.launch_log())
            got.append([t.cpu().numpy() for t in (K, it, fl)])
        for k in (0, 2):
            for a, b in zip(got[1], got[k]):
                np.testing.assert_array_equal(a, b)
        assert np.isfinite(got[0][0]).all() and (got[0][2] == 0).all()


@pytest.mark.parametrize("lo,hi,weight,separable", [(0.0, 1e30, 1.0, False), (1e6, 1e6 + 1.0, 1.0, True), (-3e-30, 3e-30, 1.0, True), (5.0, 5.0, 1.0, True),
                                                    (0.0, 1.0, 1e15, True), (0.0, 1.0, 1e-15, True)])
def test_extreme_labels_and_weights(torch, solver, lo, hi, weight, separable):
    """Label ranges without a separable form, far from zero, tiny or empty, and weights near the ends of what fp32 holds of
    their products: the values of the streaming solver."""
    wb = er(6, (80, 88, 96), 0.3)
    wb.edge_label = np.float32(lo) + (wb.edge_label * np.float32(hi - lo)).astype(np.float32)
    wb.weight = (wb.weight * np.float32(weight)).astype(np.float32)
    wb.params = dataclasses.replace(PARAMS, length_scale=1.0)
    *_, log = compare(torch, solver, wb, wb, repeat=4)
    assert bool(shapes(log)) == separable
