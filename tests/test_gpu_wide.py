"""Separable product for sparse graphs of many vertices: 4 and 8 outer rows to a workgroup, at the edges of its
groups of rows and columns, against the direct product."""
import dataclasses
import re

import numpy as np
import pytest

import mgk_workloads as W
import paper_1910_06310_amd as M

pytestmark = pytest.mark.gpu
RTOL_PATHS = 2e-5   # both stop at a relative residual of 1e-6; what two products are held to elsewhere
PARAMS = W.KernelParams(q=0.05, h=0.5, length_scale=1.0)


@pytest.fixture(scope="module")
def torch():
    import torch
    return torch


@pytest.fixture(scope="module")
def solver(torch):
    return M.Solver(0)


def ring(n, k, rng, hub=0, lone=0):
    """n vertices, each joined to about the next k / 2 of a random order, a hub of `hub` neighbours, the last `lone` without edges."""
    m = n - lone
    order = rng.permutation(m)
    pairs = {(min(a, b), max(a, b)) for s in range(1, k // 2 + 1) for a, b in zip(order, np.roll(order, s)) if a != b}
    pairs |= {(0, int(b)) for b in rng.permutation(np.arange(1, m))[:hub]}
    e = np.array(sorted(pairs), np.int32)
    return n, e, rng.uniform(0.05, 1.0, len(e)), rng.uniform(0.0, 1.0, len(e)), rng.integers(0, 3, n)


def batch(graphs, length_scale=1.0):
    prm = dataclasses.replace(PARAMS, length_scale=length_scale)
    like = W.erdos_renyi_batch(np.random.default_rng(0), 1, 8, 8, 0.5, (0.1, 1.0), (0.0, 1.0), 3, prm)
    out = []
    for n, e, w, lab, v in graphs:
        out.append(dataclasses.replace(like, vtx_off=np.array([0, n], like.vtx_off.dtype), vtx_label=v.astype(like.vtx_label.dtype),
                                       edge_off=np.array([0, len(e)], like.edge_off.dtype), src=e[:, 0].astype(like.src.dtype),
                                       dst=e[:, 1].astype(like.dst.dtype), weight=w.astype(np.float32), edge_label=lab.astype(np.float32)))
    return W.concat_batches(out, prm, "ring")


def compare(torch, solver, wx, wy, pi, pj):
    pi, pj = np.array(pi, np.int32), np.array(pj, np.int32)
    solver.configure(wx.params)
    solver.set_solver(1e-6, 0)
    X = solver.load_batch(wx)
    Y = X if wy is wx else solver.load_batch(wy)
    off = np.concatenate([[0], np.cumsum(wx.sizes()[pi] * wy.sizes()[pj])]).astype(np.int64)
    got = []
    try:
        for path in (M.TILE_AUTO, M.TILE_SPARSE):
            solver.set_tile_path(path)
            K = torch.full((len(pi),), float("nan"), dtype=torch.float32, device="cuda")
            x = torch.full((int(off[-1]),), float("nan"), dtype=torch.float32, device="cuda")
            fl = torch.full((len(pi),), -1, dtype=torch.int32, device="cuda")
            solver.pairs_nodal(X, Y, pi, pj, K, x, off[:-1], None, fl)
            torch.cuda.synchronize()
            assert (fl.cpu().numpy() == 0).all()
            got.append((K.cpu().numpy().astype(np.float64), x.cpu().numpy().astype(np.float64), solver.launch_log()))
    finally:
        solver.set_tile_path(M.TILE_AUTO)
    (K, x, log), (Kd, xd, direct) = got
    assert "mgk_wide" not in direct
    np.testing.assert_allclose(K, Kd, rtol=RTOL_PATHS)
    for a, b in zip(off[:-1], off[1:]):
        assert np.linalg.norm(x[a:b] - xd[a:b]) <= RTOL_PATHS * np.linalg.norm(xd[a:b])
    return re.findall(r"mgk_wide_xmv_kernel<(\d+), (\d+), (\d+)> rank=(\d+) passes=(\d+)", log)


@pytest.mark.parametrize("n1,n2,division", [(261, 255, ("8", "9", "9", "9", "1")), (290, 284, ("8", "9", "9", "9", "1")), (286, 285, ("8", "4", "5", "9", "2")),
                                            (517, 511, ("8", "4", "5", "9", "2")), (530, 512, ("8", "4", "5", "9", "2")), (521, 513, ("4", "4", "5", "9", "2")),
                                            (1029, 1023, ("4", "4", "5", "9", "2")), (1100, 1024, ("4", "4", "5", "9", "2")),
                                            (1030, 1025, ("4", "4", "5", "9", "2")), (1700, 1637, ("4", "4", "5", "9", "2")),
                                            (2051, 2047, ("4", "4", "5", "9", "2")), (2050, 2048, ("4", "4", "5", "9", "2"))])
def test_edges_of_rows_and_columns(torch, solver, n1, n2, division):
    """Rows in 4s and 8s, columns in 8s, 16s and 64s, one pass and two, two workgroups to a compute unit and one, up to the most that
    T has room for; a hub, vertices without edges."""
    rng = np.random.default_rng(n1 + n2)
    wb = batch([ring(n1, 8, rng, hub=70, lone=3), ring(n2, 10, rng, hub=33, lone=21)], 0.42)
    forms = compare(torch, solver, wb, wb, [0, 1, 1, 1, 0, 1], [1, 0, 1, 0, 1, 1])
    assert forms == [division]


def test_graphs_larger_than_that_take_the_direct_product(torch, solver):
    rng = np.random.default_rng(1)
    wb = batch([ring(2060, 6, rng), ring(2049, 6, rng)], 0.42)
    assert compare(torch, solver, wb, wb, [0], [1]) == []


@pytest.mark.parametrize("inner", [300, 2048])
def test_outer_graphs_may_be_larger(torch, solver, inner):
    """The limit is that of an inner graph: features as an inner one are formed for no other graph, also of one batch."""
    rng = np.random.default_rng(inner)
    wb = batch([ring(2100, 6, rng), ring(3000, 8, rng, hub=40), ring(9000, 6, rng, lone=30), ring(inner, 8, rng, hub=30)], 0.42)
    assert len(compare(torch, solver, wb, wb, [0, 3, 2, 1], [3, 1, 3, 3])) == 1
    forms = compare(torch, solver, wb, batch([ring(inner, 6, rng)], 0.42), [0, 1, 2, 1], [0, 0, 0, 0])
    assert len(forms) == 1


def test_small_graphs_beside_large_ones(torch, solver):
    """The smallest inner graph that the form takes, and one smaller, in a call with larger ones."""
    rng = np.random.default_rng(2)
    wb = batch([ring(700, 8, rng, hub=40), ring(24, 6, rng), ring(23, 6, rng), ring(733, 6, rng), ring(300, 4, rng, lone=100)], 0.42)
    pi, pj = [0, 0, 3, 0, 3, 4, 0, 3] * 2, [1, 2, 1, 3, 0, 0, 0, 4] * 2
    assert {f[0] for f in compare(torch, solver, wb, wb, pi, pj)} == {"4"}


@pytest.mark.parametrize("length_scale,division", [(30.0, ("4", "4", "3", "1")), (1.9, ("5", "5", "5", "1")), (1.0, ("6", "6", "6", "1")),
                                                   (0.4, ("4", "5", "9", "2")), (0.35, ("5", "5", "10", "2")), (0.25, ("6", "6", "12", "2")),
                                                   (0.224, ("4", "5", "13", "3")), (0.2, ("5", "5", "15", "3")), (0.19, ("4", "4", "16", "4"))])
def test_every_division_of_the_rank(torch, solver, length_scale, division):
    """Features in one pass or more of four to six; graphs of two batches."""
    rng = np.random.default_rng(3)
    wx, wy = batch([ring(900, 6, rng), ring(700, 8, rng)], length_scale), batch([ring(640, 10, rng), ring(777, 6, rng)], length_scale)
    forms = compare(torch, solver, wx, wy, [0, 1, 1, 0, 1, 1, 0, 0], [0, 0, 1, 1, 0, 1, 0, 1])
    assert {f[1:] for f in forms} == {division}


@pytest.mark.parametrize("length_scale,division", [(0.6, ("8", "8", "7", "1")), (0.42, ("9", "9", "9", "1")), (0.35, ("10", "10", "10", "1"))])
def test_all_features_in_one_pass(torch, solver, length_scale, division):
    rng = np.random.default_rng(4)
    wb = batch([ring(250, 8, rng), ring(203, 12, rng, hub=50), ring(181, 6, rng)], length_scale)
    forms = compare(torch, solver, wb, wb, [0, 1, 2, 0, 0, 1] * 2, [0, 1, 2, 1, 2, 2] * 2)
    assert {f[1:] for f in forms} == {division}
