"""GPU parity of the solver of the reduced system (black vertices of the outer graph eliminated), which
calls without iteration counts take for small pairs: against the fp64 oracle at the edges of its launch
shapes, with every edge kernel, and what it shares with the solver of the full system.

Tolerance: |K - K_oracle| <= 1e-4 |K_oracle|, as for the other solvers (relative residual 1e-6, fp32)."""
import dataclasses

import numpy as np
import pytest

import mgk_workloads as W
import paper_1910_06310_amd as M
from oracle import c_oracle as C

pytestmark = pytest.mark.gpu
RTOL = 1e-4
PRM = W.KernelParams(q=0.05, h=0.3, length_scale=0.1)


@pytest.fixture(scope="module")
def torch():
    import torch
    return torch


@pytest.fixture()
def solver(torch):
    return M.Solver(0)


def graph(n, edges, rng):
    """One graph as a batch; weights and labels drawn."""
    m = len(edges)
    e = np.array(edges, np.int32).reshape(m, 2)
    return W.GraphBatch(np.array([0, n], np.int64), rng.integers(0, 3, n).astype(np.int32), np.array([0, m], np.int64),
                        e[:, 0].copy(), e[:, 1].copy(), rng.uniform(0.4, 1.6, m).astype(np.float32),
                        rng.uniform(1.0, 1.4, m).astype(np.float32), PRM)


def shapes(rng):
    """No edge, one vertex, isolated vertices beside edges, stars (a row as long as a wavefront takes, and longer),
    paths and rings of both parities, a ladder, a complete graph: few and many black vertices."""
    path = lambda n: [(i, i + 1) for i in range(n - 1)]
    ring = lambda n: path(n) + [(n - 1, 0)]
    star = lambda n: [(0, i) for i in range(1, n)]
    ladder = lambda n: path(n) + [(n + a, n + b) for a, b in path(n)] + [(i, n + i) for i in range(n)]
    full = [(i, j) for i in range(5) for j in range(i)]
    return W.concat_batches([graph(n, e, rng) for n, e in (
        (1, []), (5, []), (2, [(0, 1)]), (9, [(1, 4), (4, 7)]), (17, star(17)), (22, star(22)), (33, path(33)), (31, ring(31)),
        (40, ring(40)), (64, path(64)), (40, ladder(20)), (5, full))], PRM, "shapes")


def solve(torch, solver, X, Y, pi, pj, **kw):
    K = torch.full((len(pi),), float("nan"), dtype=torch.float32, device="cuda")
    fl = torch.full((len(pi),), -1, dtype=torch.int32, device="cuda")
    it = torch.zeros(len(pi), dtype=torch.int32, device="cuda") if kw.get("count") else None
    solver.pairs(X, Y, pi, pj, K, it, fl)
    torch.cuda.synchronize()
    return K.cpu().numpy().astype(np.float64), fl.cpu().numpy(), None if it is None else it.cpu().numpy()


def test_shapes_of_graphs(torch, solver):
    wb = shapes(np.random.default_rng(5))
    solver.configure(wb.params)
    B = solver.load_batch(wb)
    pi, pj = W.gram_pairs(wb.n_graphs)
    ref = C.pairs(wb, pi, pj, tier=0)
    K, fl, _ = solve(torch, solver, B, B, pi, pj)
    np.testing.assert_allclose(K, ref, rtol=RTOL)
    assert (fl == 0).all()
    # one at a time: no launch shape but the pair's own
    for k in range(0, len(pi), 5):
        K1, fl1, _ = solve(torch, solver, B, B, pi[k:k + 1], pj[k:k + 1])
        assert K1[0] == pytest.approx(ref[k], rel=RTOL) and fl1[0] == 0


# waves: the host gives 2 wavefronts where there are thousands of pairs, 8 where 4 do not hold the outer graph
@pytest.mark.parametrize("lo,hi,kernels", [(10, 24, "<2"), (26, 40, "<4"), (50, 58, "<8")])
def test_launch_shapes(torch, solver, lo, hi, kernels):
    rng = np.random.default_rng(lo)
    wb = W.permute_vertices(W.molecule_like_batch(rng, 12, lo, hi, PRM), rng)
    solver.configure(wb.params)
    B = solver.load_batch(wb)
    pi, pj = W.gram_pairs(12)
    many = 4096 // len(pi) + 1 if kernels == "<2" else 1
    ref = C.pairs(wb, pi, pj, tier=0)
    K, fl, _ = solve(torch, solver, B, B, np.tile(pi, many), np.tile(pj, many))
    np.testing.assert_allclose(K, np.tile(ref, many), rtol=RTOL)
    assert (fl == 0).all() and (K.reshape(many, -1) == K[:len(pi)]).all()
    assert "mgk_pcg_reduced" + kernels in solver.launch_log()


@pytest.mark.parametrize("kernel", ["const", "poly", "kron_se", "rconv_se"])
def test_edge_kernels_and_start_probabilities(torch, solver, kernel):
    rng = np.random.default_rng(11)
    wb = W.molecule_like_batch(rng, 8, 12, 36, PRM)
    wb.weight = rng.uniform(0.4, 1.6, len(wb.weight)).astype(np.float32)
    if kernel == "poly":
        wb.params = dataclasses.replace(PRM, edge_kernel="poly", poly_coef=(1.0, 0.0, -10.0, 20.0, -15.0, 4.0), poly_rho=0.25)
    elif kernel != "const":
        ls = (0.15, 0.4, 0.25) if kernel == "kron_se" else (0.3,)
        wb = W.with_label_attributes(wb, rng, 3, 0.3, dataclasses.replace(PRM, edge_kernel=kernel, label_dim=3, length_scales=ls))
    sp = rng.random(int(wb.vtx_off[-1])).astype(np.float32)
    solver.configure(wb.params)
    ref_wb = wb
    if kernel == "const":
        solver.set_edge_kernel_const(1.0)
        ref_wb = W.GraphBatch(wb.vtx_off, wb.vtx_label, wb.edge_off, wb.src, wb.dst, wb.weight, np.zeros_like(wb.edge_label), PRM)
    B = solver.load_batch(wb, start_prob=sp)
    pi, pj = W.gram_pairs(8)
    ref = C.pairs(ref_wb, pi, pj, tier=0, start_prob=sp.astype(np.float64))
    K, fl, _ = solve(torch, solver, B, B, pi, pj)
    np.testing.assert_allclose(K, ref, rtol=RTOL)
    assert (fl == 0).all() and "mgk_pcg_reduced" in solver.launch_log()


def test_two_batches_and_nodal(torch, solver):
    """Both orientations in one launch; x of black and red elements in the original numbering."""
    rng = np.random.default_rng(17)
    X, Y = W.molecule_like_batch(rng, 5, 12, 30, PRM), W.molecule_like_batch(rng, 4, 30, 50, PRM)
    X, Y = W.permute_vertices(X, rng), W.permute_vertices(Y, rng)
    solver.configure(PRM)
    BX, BY = solver.load_batch(X), solver.load_batch(Y)
    for (A, B, wa, wb) in ((BX, BY, X, Y), (BY, BX, Y, X)):
        pi = np.repeat(np.arange(wa.n_graphs), wb.n_graphs).astype(np.int32)
        pj = np.tile(np.arange(wb.n_graphs), wa.n_graphs).astype(np.int32)
        sizes = wa.sizes()[pi] * wb.sizes()[pj]
        off = np.concatenate([[0], np.cumsum(sizes)[:-1]]).astype(np.int64)
        K = torch.full((len(pi),), float("nan"), dtype=torch.float32, device="cuda")
        x = torch.full((int(sizes.sum()),), float("nan"), dtype=torch.float32, device="cuda")
        solver.pairs_nodal(A, B, pi, pj, K, x, off)
        torch.cuda.synchronize()
        xs = x.cpu().numpy().astype(np.float64)
        for k, (i, j) in enumerate(zip(pi, pj)):
            Kref, xref = C.pair_nodal(wa.graph(int(i)), wb.graph(int(j)), PRM.q, PRM.h, PRM.length_scale)
            got = xs[off[k]:off[k] + sizes[k]].reshape(xref.shape)
            np.testing.assert_allclose(got, xref, rtol=RTOL, atol=RTOL * np.abs(xref).max())
            assert float(K[k]) == pytest.approx(Kref, rel=RTOL)
        assert "mgk_pcg_reduced" in solver.launch_log()


def test_full_system_where_iterates_are_seen(torch, solver):
    """Calls with iteration counts, and with an iteration limit, are solved as before."""
    wb = W.config1(10)
    solver.configure(wb.params)
    B = solver.load_batch(wb)
    pi, pj = W.gram_pairs(10)
    K, _, _ = solve(torch, solver, B, B, pi, pj)
    assert "mgk_pcg_reduced" in solver.launch_log()
    solver.set_reduced_system(0)
    K0, fl0, it0 = solve(torch, solver, B, B, pi, pj, count=True)
    solver.set_reduced_system(1)
    K1, fl1, it1 = solve(torch, solver, B, B, pi, pj, count=True)
    assert "mgk_pcg_regs" in solver.launch_log() and (K0 == K1).all() and (it0 == it1).all()
    np.testing.assert_allclose(K, K1, rtol=2e-6)   # both stop at a relative residual of 1e-6
    solver.set_solver(1e-6, 3)
    _, fl3, _ = solve(torch, solver, B, B, pi, pj)
    assert "mgk_pcg_regs" in solver.launch_log() and (fl3 == 1).all()
    solver.set_reduced_system(2)
    _, fl4, it4 = solve(torch, solver, B, B, pi, pj, count=True)
    assert "mgk_pcg_reduced" in solver.launch_log() and (it4 == 3).all() and (fl4 == 1).all()


@pytest.mark.parametrize("first,then", [(False, True), (True, False), (False, False), (True, True)])
def test_recorded_gram_gives_what_the_eager_one_does(torch, solver, first, then):
    """Also if the list of the system it asks for has to be made meanwhile; without counts the list that is there will do."""
    wb = W.config1(12)
    solver.configure(wb.params)
    B = solver.load_batch(wb)
    K = torch.zeros((12, 12), dtype=torch.float32, device="cuda")
    it = torch.zeros((12, 12), dtype=torch.int32, device="cuda")
    solver.gram(B, K, it if first else None)
    torch.cuda.synchronize()
    ref = K.cpu().numpy()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        solver.gram(B, K, it if then else None)
    for _ in range(3):
        K.zero_()
        it.zero_()
        g.replay()
        torch.cuda.synchronize()
        if first == then or not then:
            assert (K.cpu().numpy() == ref).all()
        replayed = K.cpu().numpy(), it.cpu().numpy()
        if then:   # of Alg. 1 on the full system, as the eager call counts them
            solver.gram(B, K, it)
            torch.cuda.synchronize()
            assert (replayed[0] == K.cpu().numpy()).all() and (replayed[1] == it.cpu().numpy()).all()


def test_recorded_gram_follows_the_mode(torch, solver):
    wb = W.config1(12)
    solver.configure(wb.params)
    B = solver.load_batch(wb)
    K = torch.zeros((12, 12), dtype=torch.float32, device="cuda")
    it = torch.zeros((12, 12), dtype=torch.int32, device="cuda")
    solver.gram(B, K)
    for mode, kernel in ((0, "mgk_pcg_regs"), (2, "mgk_pcg_reduced")):
        solver.set_reduced_system(mode)
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            solver.gram(B, K, it)
        assert kernel in solver.launch_log() and solver.launch_log().count("mgk_pcg") == solver.launch_log().count(kernel)
        for _ in range(3):
            K.zero_()
            it.zero_()
            g.replay()
            torch.cuda.synchronize()
            got = K.cpu().numpy(), it.cpu().numpy()
            solver.gram(B, K, it)
            torch.cuda.synchronize()
            assert (got[0] == K.cpu().numpy()).all() and (got[1] == it.cpu().numpy()).all()


def test_pairs_that_fit_one_of_the_systems_only(torch, solver):
    """Grids and ladders: some fit the wavefronts of the solver of the full system and not those of the reduced one, in
    either orientation and beside others; two batches, few and many pairs."""
    rng = np.random.default_rng(23)
    grid = lambda a, b: (a * b, [(i * b + j, i * b + j + 1) for i in range(a) for j in range(b - 1)] +
                         [(i * b + j, (i + 1) * b + j) for i in range(a - 1) for j in range(b)])
    X = W.concat_batches([graph(*grid(a, b), rng) for a in range(4, 7) for b in range(a, 7)], PRM, "grids")
    Y = W.concat_batches([graph(*grid(2, n), rng) for n in range(8, 27, 2)], PRM, "ladders")
    both = W.concat_batches([X, Y], PRM, "both")
    solver.configure(PRM)
    BX, BY = solver.load_batch(X), solver.load_batch(Y)
    for A, B, wa, wb, oa, ob in ((BX, BX, X, X, 0, 0), (BY, BY, Y, Y, X.n_graphs, X.n_graphs), (BX, BY, X, Y, 0, X.n_graphs), (BY, BX, Y, X, X.n_graphs, 0)):
        pi = np.repeat(np.arange(wa.n_graphs), wb.n_graphs).astype(np.int32)
        pj = np.tile(np.arange(wb.n_graphs), wa.n_graphs).astype(np.int32)
        ref = C.pairs(both, pi + oa, pj + ob, tier=0)
        for many, other in ((1, "mgk_pcg_small"), (250, "mgk_pcg_regs")):   # a few join those that need the streaming solver
            K, fl, _ = solve(torch, solver, A, B, np.tile(pi, many), np.tile(pj, many))
            np.testing.assert_allclose(K, np.tile(ref, many), rtol=RTOL)
            assert (fl == 0).all() and "mgk_pcg_reduced" in solver.launch_log() and other in solver.launch_log()


def test_many_isolated_vertices(torch, solver):
    """Pairs that fit their own launch shape only, and pairs whose vertices do not fit beside the eliminated elements."""
    rng = np.random.default_rng(29)
    wb = W.concat_batches([graph(n, e, rng) for n, e in ((13, [(0, i) for i in range(1, 13)]), (1200, [(0, 1)]), (2, [(0, 1)]), (2000, [(0, 1)]),
                                                         (1, []), (9000, [(0, 1)]), (12000, [(0, 1)]))], PRM, "isolated")
    solver.configure(PRM)
    B = solver.load_batch(wb)
    for pi, pj in (([0, 2], [1, 3]), ([4, 5], [5, 4]), ([4, 6], [6, 4]), ([0, 2, 4, 4], [1, 3, 5, 6])):
        pi, pj = np.array(pi, np.int32), np.array(pj, np.int32)
        K, fl, _ = solve(torch, solver, B, B, pi, pj)
        np.testing.assert_allclose(K, C.pairs(wb, pi, pj, tier=1), rtol=RTOL)
        assert (fl == 0).all()
