"""The calls a program built on this library makes, at the sizes it makes them.

Every case goes through the public Python entry points (``Solver.load_batch``, ``gram``,
``pairs``, ``pairs_nodal``, ``normalize_gram`` ...) the way a program does that keeps one
solver and its loaded graphs and asks for kernel values again and again.  Graphs are drawn by
``mgk_workloads`` with the parameters of its own configurations; a case is a dict of plain
values:

  task     gram     all pairs of one batch (optionally normalised)
           predict  new graphs are loaded from host arrays and compared with a resident batch
           nodal    a list of pairs with the node-wise solution
           pairs    pair k = graphs (2k, 2k + 1) of one batch
  graphs   er, molecule, ba, nws, contact, geo (see ``_graphs``)
  count    graphs in the batch (predict: in the resident batch)
  lo, hi   smallest and largest number of vertices
  edge     edge base kernel: se, const, poly, kron_se, rconv_se
"""
import dataclasses
import math

import numpy as np
import torch

import mgk_workloads as W
import paper_1910_06310_amd as M

WENDLAND_C2 = (1.0, 0.0, -10.0, 20.0, -15.0, 4.0)   # (1 - r)^4 (4 r + 1)
ATTRS = 3                                            # attributes per label of the attribute kernels


def listed():
    return [
        # the smallest call: the Gram matrix of a handful of tiny graphs, where only latency counts
        {"name": "gram_er_tiny", "task": "gram", "graphs": "er", "count": 4, "lo": 6, "hi": 10,
         "density": 0.3, "edge": "se", "normalize": False},
        # a small molecular data set, one Gram per hyper-parameter setting
        {"name": "gram_molecule_100", "task": "gram", "graphs": "molecule", "count": 100, "lo": 10, "hi": 40,
         "density": 0.0, "edge": "se", "normalize": False},
        # the large molecular Gram matrix: two million pairs, pure throughput
        {"name": "gram_molecule_2000", "task": "gram", "graphs": "molecule", "count": 2000, "lo": 20, "hi": 60,
         "density": 0.0, "edge": "se", "normalize": False},
        # bonds described by several measurements, weighted edges: the Kronecker-product edge kernel
        {"name": "gram_molecule_attr", "task": "gram", "graphs": "molecule", "count": 350, "lo": 12, "hi": 55,
         "density": 0.0, "edge": "kron_se", "normalize": False},
        # prediction: a few new molecules arrive as host arrays and are compared with a resident set
        {"name": "predict_molecule", "task": "predict", "graphs": "molecule", "count": 500, "lo": 15, "hi": 55,
         "density": 0.0, "edge": "se", "queries": 8, "entry": "pairs"},
        # scale-free graphs with hubs, the second synthetic benchmark family
        {"name": "gram_ba_160", "task": "gram", "graphs": "ba", "count": 160, "lo": 96, "hi": 96,
         "density": 0.0, "edge": "se", "normalize": False},
        # node-wise similarity of small-world graphs, the first synthetic benchmark family
        {"name": "nodal_nws_256", "task": "nodal", "graphs": "nws", "count": 64, "lo": 96, "hi": 96,
         "density": 0.0, "edge": "se", "pairs": 256},
        # contact graphs as ragged as a protein data set (30 to 295 vertices), normalised similarity
        # matrix: pairs that fit on chip and pairs that do not in one call
        {"name": "gram_contact_48", "task": "gram", "graphs": "contact", "count": 48, "lo": 30, "hi": 295,
         "density": 0.0, "edge": "se", "normalize": True},
        # 256-vertex random graphs from very sparse to complete
        {"name": "pairs_er256_d001", "task": "pairs", "graphs": "er", "count": 128, "lo": 256, "hi": 256,
         "density": 0.01, "edge": "se"},
        {"name": "pairs_er256_d020", "task": "pairs", "graphs": "er", "count": 128, "lo": 256, "hi": 256,
         "density": 0.2, "edge": "se"},
        {"name": "pairs_er256_d100", "task": "pairs", "graphs": "er", "count": 128, "lo": 256, "hi": 256,
         "density": 1.0, "edge": "se"},
        # large 3-D geometric graphs that come with coordinates
        {"name": "pairs_geo_2048", "task": "pairs", "graphs": "geo", "count": 32, "lo": 2048, "hi": 2048,
         "density": 0.0, "edge": "se"},
    ]


def _log(rng, lo, hi):
    """A whole number, uniform in its logarithm."""
    return int(min(hi, max(lo, round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["tiny", "molecule", "molecule", "predict", "ba", "nws", "nodal", "contact", "er", "er", "geo"])
    if kind == "tiny":
        lo = rng.randint(4, 8)
        return {"task": "gram", "graphs": "er", "count": rng.randint(3, 12), "lo": lo, "hi": lo + rng.randint(1, 6),
                "density": round(rng.uniform(0.2, 0.6), 3), "edge": rng.choice(["se", "const"]), "normalize": rng.random() < 0.5}
    if kind == "molecule":
        lo = rng.randint(8, 24)
        return {"task": "gram", "graphs": "molecule", "count": _log(rng, 20, 1500), "lo": lo, "hi": lo + rng.randint(8, 36),
                "density": 0.0, "edge": rng.choice(["se", "se", "const", "poly", "kron_se", "rconv_se"]),
                "normalize": rng.random() < 0.5}
    if kind == "predict":
        lo = rng.randint(8, 24)
        return {"task": "predict", "graphs": "molecule", "count": _log(rng, 50, 1000), "lo": lo, "hi": lo + rng.randint(8, 36),
                "density": 0.0, "edge": rng.choice(["se", "kron_se"]), "queries": _log(rng, 1, 32),
                "entry": rng.choice(["pairs", "pairs_dev", "pairs_noalloc"])}
    if kind in ("ba", "nws"):
        lo = rng.randint(33, 96)
        return {"task": "gram", "graphs": kind, "count": _log(rng, 20, 160), "lo": lo, "hi": lo + rng.randint(0, 30),
                "density": 0.0, "edge": rng.choice(["se", "se", "const"]), "normalize": rng.random() < 0.5}
    if kind == "nodal":
        graphs = rng.choice(["nws", "molecule", "contact"])
        lo = rng.randint(20, 90)
        return {"task": "nodal", "graphs": graphs, "count": rng.randint(16, 64), "lo": lo, "hi": lo + rng.randint(0, 35),
                "density": 0.0, "edge": "se", "pairs": _log(rng, 16, 512)}
    if kind == "contact":
        lo = rng.randint(30, 60)
        return {"task": "gram", "graphs": "contact", "count": _log(rng, 12, 48), "lo": lo, "hi": rng.randint(120, 295),
                "density": 0.0, "edge": "se", "normalize": rng.random() < 0.5}
    if kind == "er":
        n = rng.randint(97, 256)
        return {"task": "pairs", "graphs": "er", "count": 2 * _log(rng, 8, 64), "lo": n - rng.randint(0, 16), "hi": n,
                "density": round(math.exp(rng.uniform(math.log(0.01), 0.0)), 4), "edge": rng.choice(["se", "se", "se", "const", "poly"])}
    n = _log(rng, 300, 2048)
    return {"task": "pairs", "graphs": "geo", "count": 2 * _log(rng, 2, 16), "lo": n, "hi": n, "density": 0.0, "edge": "se"}


# ---- graphs ---------------------------------------------------------------------------------
def _params(case):
    """Base kernels of the family, as in its configuration."""
    prm = {"molecule": W.KernelParams(q=0.05, h=0.3, length_scale=0.1),
           # unit point density: contacts within about 1.42, the cut-off over the length scale as in "geo"
           "contact": W.KernelParams(q=0.05, h=0.5, length_scale=0.65),
           "geo": W.KernelParams(q=0.05, h=0.5, length_scale=0.05)}.get(
               case["graphs"], W.KernelParams(q=0.05, h=0.5, length_scale=1.0))
    if case["edge"] == "poly":
        return dataclasses.replace(prm, edge_kernel="poly", poly_coef=WENDLAND_C2,
                                   poly_rho=0.25 if case["graphs"] == "molecule" else 1.2)
    if case["edge"] == "kron_se":
        return dataclasses.replace(prm, edge_kernel="kron_se", label_dim=ATTRS, length_scales=(0.15, 0.4, 0.25))
    if case["edge"] == "rconv_se":
        return dataclasses.replace(prm, edge_kernel="rconv_se", label_dim=ATTRS, length_scales=(0.3,))
    return prm


def _graphs(case, rng, count):
    kind, lo, hi, prm = case["graphs"], case["lo"], case["hi"], _params(case)
    if kind == "er":        # Erdos-Renyi graphs, weights and labels uniform
        if hi < 64:
            return W.erdos_renyi_batch(rng, count, lo, hi, case["density"], (0.5, 1.0), (1.0, 2.0), 3, prm)
        return W.erdos_renyi_batch(rng, count, lo, hi, case["density"], (0.0, 1.0), (0.0, 1.0), 4, prm, w_min=1e-3)
    if kind == "molecule":  # trees of maximum degree 4 with a few ring closures, bond-length labels
        wb = W.molecule_like_batch(rng, count, lo, hi, prm)
        if prm.label_dim > 1:
            wb.weight = rng.uniform(0.4, 1.6, len(wb.weight)).astype(np.float32)
            wb = W.with_label_attributes(wb, rng, prm.label_dim, 0.3, prm)
        return wb
    if kind == "geo":       # points in the unit cube, edge iff closer than a cut-off, w = exp(-d), label d
        return W.geometric_batch(rng, count, lo, 12.0, 8, prm)
    parts = []
    for _ in range(count):
        n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.49)))))
        if kind == "ba":    # preferential attachment, six edges per new vertex
            b = W.barabasi_albert_batch(rng, 1, n, 6, 4, prm)
        elif kind == "nws":  # ring lattice with shortcuts
            b = W.newman_watts_strogatz_batch(rng, 1, n, 3, 0.1, 4, prm)
        else:               # contact: points at unit density, so that the cut-off is the same for every size
            b = W.geometric_batch(rng, 1, n, 12.0, 8, prm)
            b.edge_label = (b.edge_label * n ** (1.0 / 3.0)).astype(np.float32)
            b.weight = np.exp(-b.edge_label).astype(np.float32)
        parts.append(b)
    return W.concat_batches(parts, prm, kind)


def _configure(solver, case):
    solver.configure(_params(case))
    if case["edge"] == "const":
        solver.set_edge_kernel_const(1.0)


def _load(solver, wb, case):
    if case["graphs"] == "geo":
        return solver.load_graphs_embedded(wb.vtx_off, wb.vtx_label, wb.edge_off, wb.src, wb.dst, wb.coords,
                                           wb.weight, wb.edge_label)
    return solver.load_batch(wb)


# ---- state and one pass ------------------------------------------------------------------------
def prepare(case, seed):
    rng = np.random.default_rng(seed)
    solver = M.Solver(0)
    _configure(solver, case)
    wb = _graphs(case, rng, case["count"])
    st = {"case": case, "solver": solver, "batch": _load(solver, wb, case)}
    G = case["count"]
    if case["task"] == "gram":
        shape = (G, G)
    elif case["task"] == "predict":
        Q = case["queries"]
        st["new"] = _graphs(case, rng, Q)
        st["i"] = np.repeat(np.arange(Q), G).astype(np.int32)
        st["j"] = np.tile(np.arange(G), Q).astype(np.int32)
        if case["entry"] == "pairs_dev":
            st["i"], st["j"] = torch.from_numpy(st["i"]).cuda(), torch.from_numpy(st["j"]).cuda()
        shape = (Q * G,)
    elif case["task"] == "nodal":
        shape = (case["pairs"],)
        st["i"] = rng.integers(0, G, case["pairs"]).astype(np.int32)
        st["j"] = rng.integers(0, G, case["pairs"]).astype(np.int32)
        # every pair's block padded to the largest graph, so that the offsets need no sizes
        st["off"] = np.arange(case["pairs"], dtype=np.int64) * case["hi"] ** 2
        st["x"] = torch.zeros(case["pairs"] * case["hi"] ** 2, dtype=torch.float32, device="cuda")
    else:
        shape = (G // 2,)
        st["i"] = np.arange(0, G, 2, dtype=np.int32)
        st["j"] = np.arange(1, G, 2, dtype=np.int32)
    st["K"] = torch.zeros(shape, dtype=torch.float32, device="cuda")
    st["flags"] = torch.zeros(shape, dtype=torch.int32, device="cuda")
    return st


def run(st):
    """One request: kernel values and convergence flags."""
    case, solver, batch, K, flags = st["case"], st["solver"], st["batch"], st["K"], st["flags"]
    if case["task"] == "gram":
        solver.gram(batch, K, None, flags)
        if case["normalize"]:
            solver.normalize_gram(case["count"], K)
        return {"K": K, "flags": flags}
    if case["task"] == "predict":
        new = solver.load_batch(st["new"])
        getattr(solver, case["entry"])(new, batch, st["i"], st["j"], K, None, flags)
        return {"K": K, "flags": flags}
    if case["task"] == "nodal":
        solver.pairs_nodal(batch, batch, st["i"], st["j"], K, st["x"], st["off"], None, flags)
        return {"K": K, "x": st["x"], "flags": flags}
    solver.pairs(batch, batch, st["i"], st["j"], K, None, flags)
    return {"K": K, "flags": flags}


# ---- what a pass cannot do without ----------------------------------------------------------------
def work(case):
    """Expected values over the graphs of a case.  An iteration applies the off-diagonal
    operator, which takes at least a multiply-add per entry (nnz nnz' of them) or, where the
    edge kernel splits into a product, per entry of the two one-sided products (nnz n' + n nnz'),
    and does about 16 operations per vector element."""
    n = 0.5 * (case["lo"] + case["hi"])
    if case["graphs"] in ("ba", "nws", "contact") and case["hi"] > case["lo"]:   # uniform in the logarithm
        n = (case["hi"] - case["lo"]) / math.log(case["hi"] / case["lo"])
    nnz = {"er": n * (n - 1) * case["density"], "molecule": 2 * n + 1, "ba": 12 * (n - 6), "nws": 2.2 * n}.get(
        case["graphs"], 12 * n)
    iters = {"molecule": 11, "ba": 7, "nws": 14}.get(case["graphs"], 8)   # to a relative residual of 1e-6
    G = case["count"]
    pairs = {"gram": G * (G + 1) // 2, "predict": G * case.get("queries", 0), "nodal": case.get("pairs", 0)}.get(
        case["task"], G // 2)
    labels = ATTRS if case["edge"] in ("kron_se", "rconv_se") else 1
    bytes_ = (G + case.get("queries", 0)) * (12 * n + nnz * (8 + 4 * labels))
    bytes_ += (G * G if case["task"] == "gram" else pairs) * 8
    bytes_ += 4 * n * n * pairs if case["task"] == "nodal" else 0
    return {"bytes": bytes_, "flops": pairs * iters * (2 * min(nnz * nnz, 2 * nnz * n) + 16 * n * n)}


def tolerance(case):
    """fp32 arithmetic, iteration stopped at a relative residual of 1e-6: values of two correct
    implementations agree to about 1e-5.  Flags are 0 / 1 per pair and come out the same."""
    return {"rel": 1e-5}
