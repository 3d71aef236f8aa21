"""Off-diagonal product through a separable edge kernel (global-memory solver): sizes at the edges of
its tiles and packets, every division of the rank, against the fp64 oracle and the direct product."""
import dataclasses
import re

import numpy as np
import pytest

import mgk_workloads as W
import paper_1910_06310_amd as M
from oracle import c_oracle as C

pytestmark = pytest.mark.gpu
# Values against the oracle: the bound of the kernel values in general.  Two products against each
# other: both stop at a relative residual of 1e-6, and 2e-5 is what the tile paths are held to.
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
    """Values and node-wise solutions through the global-memory solver; the kernels that ran."""
    solver.set_tile_path(path)
    sx, sy = wx.sizes()[pi], wy.sizes()[pj]
    off = np.concatenate([[0], np.cumsum(sx * sy)]).astype(np.int64)
    K = torch.full((len(pi),), float("nan"), dtype=torch.float32, device="cuda")
    x = torch.full((int(off[-1]),), float("nan"), dtype=torch.float32, device="cuda")
    fl = torch.full((len(pi),), -1, dtype=torch.int32, device="cuda")
    solver.pairs_nodal(X, Y, pi, pj, K, x, off[:-1], None, fl)
    torch.cuda.synchronize()
    assert (fl.cpu().numpy() == 0).all()
    return K.cpu().numpy().astype(np.float64), x.cpu().numpy().astype(np.float64), solver.launch_log()


def compare(torch, solver, wx, wy, const=False, onchip=0):
    """All pairs of graphs of two batches: the chosen product against the direct one, node by node."""
    pi = np.repeat(np.arange(len(wx.sizes())), len(wy.sizes())).astype(np.int32)
    pj = np.tile(np.arange(len(wy.sizes())), len(wx.sizes())).astype(np.int32)
    solver.configure(wx.params)
    if const:
        solver.set_edge_kernel_const(0.7)
    solver.set_solver(1e-6, 0)
    solver.set_onchip_limit(onchip)
    try:
        X, Y = solver.load_batch(wx), solver.load_batch(wy)
        K, x, log = solve(torch, solver, X, Y, wx, wy, pi, pj, M.TILE_AUTO)
        Kd, xd, direct = solve(torch, solver, X, Y, wx, wy, pi, pj, M.TILE_SPARSE)
        X.free()
        Y.free()
    finally:
        solver.set_tile_path(M.TILE_AUTO)
        solver.set_onchip_limit(16384)
    assert "mgk_sep" not in direct
    np.testing.assert_allclose(K, Kd, rtol=RTOL_PATHS)
    assert np.linalg.norm(x - xd) <= RTOL_PATHS * np.linalg.norm(xd)
    return pi, pj, K, log


def forms(log):
    """Features per pass (sparse form) or tiles per wavefront (dense form; 0 on parts), rank and passes of every launch."""
    return {(k, int(a or 0), int(r), int(p or 1)) for k, a, r, p in
            re.findall(r"mgk_sep_(xmv|dense|dense_parts)_kernel(?:<(\d+)>)? rank=(\d+)(?: passes=(\d+))?", log)}


@pytest.mark.parametrize("length_scale,division", [(20.0, (4, 2, 1)), (4.0, (4, 3, 1)), (1.7, (4, 4, 1)), (1.0, (5, 5, 1)), (0.7, (6, 6, 1)),
                                                   (0.5, (7, 7, 1)), (0.44, (4, 8, 2)), (0.33, (5, 10, 2)), (0.25, (6, 12, 2)),
                                                   (0.22, (7, 13, 2)), (0.185, (5, 15, 3)), (None, (1, 1, 1))])
def test_every_division_of_the_rank(torch, solver, length_scale, division):
    """Short length scales take more features, in passes of 4 to 7; the constant kernel takes one."""
    wb = er(1, (33, 47, 64), 0.25)
    wb.params = dataclasses.replace(PARAMS, length_scale=length_scale or 1.0)
    *_, log = compare(torch, solver, wb, wb, const=length_scale is None)
    assert forms(log) == {("xmv",) + division}


@pytest.mark.parametrize("density", [0.06, 0.5, 1.0])
@pytest.mark.parametrize("sizes", [(15, 16, 17), (31, 33, 63), (64, 65, 127), (129, 130)])
def test_edges_of_tiles_against_the_oracle(torch, solver, sizes, density):
    """Rows in 16s, columns in 4s and 64s; the batch ends with vertices without edges, which have no
    packets.  At the low density the direct product is the cheaper one for the smaller of these graphs."""
    wb = er(sum(sizes), sizes, density)
    lone = W.erdos_renyi_batch(np.random.default_rng(3), 1, 21, 21, 0.5, (0.5, 1.0), (0.0, 1.0), 4, PARAMS)
    keep = (lone.src < 16) & (lone.dst < 16)   # five vertices without edges: a whole group of four
    lone.src, lone.dst, lone.weight, lone.edge_label = (a[keep] for a in (lone.src, lone.dst, lone.weight, lone.edge_label))
    lone.edge_off = np.array([0, int(keep.sum())], lone.edge_off.dtype)
    wb = W.concat_batches([wb, lone], PARAMS, "edges")
    pi, pj, K, log = compare(torch, solver, wb, wb)
    once = (pi <= pj) & (wb.nnz()[pi] * wb.nnz()[pj] < 2e7)   # the oracle evaluates every pair of nonzeros
    np.testing.assert_allclose(K[once], C.pairs(wb, pi[once], pj[once], tier=1), rtol=RTOL)
    if density >= 0.5 or max(sizes) <= 128:   # the larger sparse ones are close to either
        assert forms(log) == (set() if density < 0.5 and max(sizes) < 100 else {("xmv", 5, 5, 1)})


@pytest.mark.parametrize("sizes,const,tiles", [((145, 159, 161), False, 0), ((192, 193), False, 0), ((290,), False, 2), ((191, 225), True, 0),
                                               ((511, 449), False, 2), ((513,), False, 4), ((600, 577), True, 4)])
def test_dense_form_at_edges_of_its_tiles(torch, solver, sizes, const, tiles):
    """32 rows by 64 columns; one, two and four tiles of columns per wavefront, or on parts."""
    wb = er(sum(sizes), sizes, 1.0 if max(sizes) < 500 else 0.6)
    *_, log = compare(torch, solver, wb, wb, const=const)
    assert forms(log) == {("dense" if tiles else "dense_parts", tiles, 1 if const else 5, 1)}


@pytest.mark.parametrize("outer,inner,const", [((257, 289), (145, 159, 161), False), ((300,), (192, 193, 256), False), ((270, 261), (191, 225), True)])
def test_dense_form_with_one_tile_per_wavefront(torch, solver, outer, inner, const):
    """At most 256 columns of outer graphs that are too large for parts."""
    wx, wy = er(sum(outer), outer, 1.0), er(sum(inner), inner, 1.0)
    for a, b in ((wx, wy), (wy, wx)):
        *_, log = compare(torch, solver, a, b, const=const)
        assert forms(log) == {("dense", 1, 1 if const else 5, 1)}


@pytest.mark.parametrize("sizes,length_scale,rank", [((145, 193, 255), 1.0, 5), ((256, 160, 225), 1.0, 5), ((249, 241, 32), 0.5, 7), ((255, 254, 17), 0.185, 15),
                                                     ((257, 256), 1.0, 5)])
def test_dense_form_on_parts_at_edges_of_its_tiles(torch, solver, sizes, length_scale, rank):
    """Graphs of at most 256 vertices: columns that are no multiple of 16 or 64, rows of p at any alignment, the largest size and one
    more, many features, small graphs and vertices without edges beside them, weights over eight decades, graphs of two batches."""
    wx, wy = er(sum(sizes), sizes, 1.0), er(sum(sizes) + 1, sizes[::-1][:2], 1.0)
    lone = er(9, (40,), 1.0)
    keep = (lone.src < 9) & (lone.dst < 9)
    lone.src, lone.dst, lone.weight, lone.edge_label = (a[keep] for a in (lone.src, lone.dst, lone.weight, lone.edge_label))
    lone.edge_off = np.array([0, int(keep.sum())], lone.edge_off.dtype)
    prm = dataclasses.replace(PARAMS, length_scale=length_scale)
    wx, wy = W.concat_batches([wx, lone], prm, "x"), W.concat_batches([wy], prm, "y")
    for wb in (wx, wy):
        wb.weight = (wb.weight * 10.0 ** np.random.default_rng(7).uniform(-8, 0, len(wb.weight))).astype(np.float32)
    *_, log = compare(torch, solver, wx, wy)
    kernels = {(f[0], f[2]) for f in forms(log)}   # the small graphs beside them may take the sparse form
    assert ("dense" if max(sizes) > 256 else "dense_parts", rank) in kernels
    assert (("dense_parts" if max(sizes) > 256 else "dense"), rank) not in kernels


def test_both_dense_kernels_in_one_call(torch, solver):
    """Pairs beyond 256 vertices and enough others for launches of their own: two groups, one after the other in the same buffers."""
    wb = er(31, (290,) + (250, 241, 256, 233, 248) * 3, 1.0)
    pi, pj, K, log = compare(torch, solver, wb, wb)
    assert forms(log) == {("dense", 1, 5, 1), ("dense", 2, 5, 1), ("dense_parts", 0, 5, 1)}   # 290 vertices as inner graph once
    np.testing.assert_allclose(K.reshape(16, 16), K.reshape(16, 16).T, rtol=RTOL_PATHS)


def test_dense_form_at_its_largest_size(torch, solver):
    """1024 columns: all four tiles of every wavefront, the most LDS.  One column more has no dense form."""
    wx, wy = er(11, (1030,), 0.2), er(12, (1024, 1025), 0.2)
    *_, log = compare(torch, solver, wx, wy)
    assert forms(log) == {("dense", 4, 5, 1)} and "mgk_large_xmv_rows" in log


@pytest.mark.parametrize("sizes,length_scale,division", [((276,), 1.0, (5, 5, 1)), ((277, 300), 1.0, (4, 5, 2)), ((486, 487), 1.0, (4, 5, 2)),
                                                         ((300,), 0.25, (4, 12, 3)), ((480,), 0.185, (4, 15, 4))])
def test_sparse_form_where_few_features_fit(torch, solver, sizes, length_scale, division):
    """T of more than 276 columns leaves room for four features a pass; 487 columns are the most."""
    wb = er(sum(sizes), sizes, 0.2)
    wb.params = dataclasses.replace(PARAMS, length_scale=length_scale)
    *_, log = compare(torch, solver, wb, wb)
    assert forms(log) == {("xmv",) + division}


def test_features_of_some_graphs_of_a_batch(torch, solver):
    """Pairs of a few graphs among others, each graph in several pairs and on both sides."""
    wx, wy = er(21, (40, 70, 150, 33, 64, 129), 0.3), er(22, (48, 150, 100, 35), 0.3)
    solver.configure(PARAMS)
    solver.set_solver(1e-6, 0)
    solver.set_onchip_limit(0)
    try:
        X, Y = solver.load_batch(wx), solver.load_batch(wy)
        for pi, pj in (([4, 1, 4, 5], [3, 3, 0, 2]), ([2], [1]), ([5, 0], [0, 3])):
            pi, pj = np.array(pi, np.int32), np.array(pj, np.int32)
            K, x, log = solve(torch, solver, X, Y, wx, wy, pi, pj, M.TILE_AUTO)
            Kd, xd, _ = solve(torch, solver, X, Y, wx, wy, pi, pj, M.TILE_SPARSE)
            assert forms(log) == {("xmv", 5, 5, 1)}
            np.testing.assert_allclose(K, Kd, rtol=RTOL_PATHS)
            assert np.linalg.norm(x - xd) <= RTOL_PATHS * np.linalg.norm(xd)
        X.free()
        Y.free()
    finally:
        solver.set_tile_path(M.TILE_AUTO)
        solver.set_onchip_limit(16384)


def test_two_batches_of_unlike_sizes_and_label_ranges(torch, solver):
    """Graphs of two batches, the larger one on either side, labels of one outside the other's range."""
    wx, wy = er(5, (20, 90, 40), 0.2), er(6, (70, 33), 0.4)
    wy.edge_label = (wy.edge_label + 0.8).astype(np.float32)
    for a, b in ((wx, wy), (wy, wx)):
        *_, log = compare(torch, solver, a, b)
        assert forms(log) == {("xmv", 7, 7, 1)}


def test_calls_with_lists_of_their_own_are_refused_while_a_graph_is_recorded(torch, solver):
    """Their lists are copied from memory that later calls write again, so a replay could not be right."""
    wb = er(7, (10, 12), 0.4)
    solver.configure(PARAMS)
    solver.set_solver(1e-6, 0)
    B = solver.load_batch(wb)
    pi, pj = np.array([0, 1], np.int32), np.array([1, 1], np.int32)
    i_dev, j_dev = torch.from_numpy(pi).cuda(), torch.from_numpy(pj).cuda()
    pairs_dev = lambda X, Y, i, j, K: solver.pairs_dev(X, Y, i_dev, j_dev, K)
    K = torch.zeros(2, dtype=torch.float32, device="cuda")
    solver.pairs(B, B, pi, pj, K)
    torch.cuda.synchronize()
    before = K.cpu().numpy().copy()
    stream, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    with torch.cuda.stream(stream):
        graph.capture_begin()
        try:
            for call in (solver.pairs, solver.pairs_noalloc, pairs_dev):
                with pytest.raises(M.MgkError, match="captur"):
                    call(B, B, pi, pj, K)
            K.add_(0.0)
        finally:
            graph.capture_end()
    K.zero_()
    solver.pairs(B, B, pi, pj, K)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(K.cpu().numpy(), before)
    B.free()
