"""Host path of a solve without a GPU: the library's host code on a stand-in for the HIP runtime."""
import ctypes as C
import os
import re
import shutil
import signal
import time
import types

import numpy as np
import pytest

import host_runtime
import mgk_workloads as W

pytestmark = pytest.mark.skipif(shutil.which("g++") is None or not os.path.exists("/opt/rocm/include/hip/hip_runtime_api.h"),
                                reason="needs g++ and the HIP headers")


@pytest.fixture(scope="module")
def so(tmp_path_factory):
    return host_runtime.build(tmp_path_factory.mktemp("host_runtime"))


@pytest.fixture
def host(so):
    h = host_runtime.Host(so)
    yield h
    if h.ctx is not None:
        h.destroy()


@pytest.fixture(scope="module")
def so_wide(tmp_path_factory):
    return host_runtime.build(tmp_path_factory.mktemp("host_runtime_wide"), wide=True)


@pytest.fixture
def host_wide(so_wide):
    h = host_runtime.Host(so_wide)
    yield h
    h.destroy()


def in_child(f, seconds=20):
    """Exit status of a forked child that calls f; None if it does not end."""
    pid = os.fork()
    if pid == 0:
        try:
            f()
        except BaseException:
            os._exit(1)
        os._exit(0)
    end = time.time() + seconds
    while time.time() < end:
        got, status = os.waitpid(pid, os.WNOHANG)
        if got:
            return status
        time.sleep(0.01)
    os.kill(pid, signal.SIGKILL)
    os.waitpid(pid, 0)
    return None


def test_context_survives_a_fork(so):
    """The threads of a context do not exist in a forked child: loading and destroying work there."""
    h = host_runtime.Host(so, -1)
    wb = W.config1(40)

    def child():
        h.free(h.load(wb, reorder=1))
        h.destroy()

    h.free(h.load(wb, reorder=1))   # starts the threads
    assert in_child(child) == 0
    h.free(h.load(wb, reorder=1))
    h.destroy()


def graphs(*parts):
    """A workload of (n, edges, labels) graphs with unit weights."""
    off = lambda sizes: np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    edges = [np.asarray(e, np.int32).reshape(-1, 2) for _, e, _ in parts]
    src, dst = np.concatenate(edges).T
    return types.SimpleNamespace(
        vtx_off=off([n for n, _, _ in parts]), vtx_label=np.zeros(sum(n for n, _, _ in parts), np.int32),
        edge_off=off([len(e) for e in edges]), src=src, dst=dst, weight=np.ones(len(src), np.float32),
        edge_label=np.concatenate([np.broadcast_to(np.asarray(x, np.float32), len(e)) for (_, _, x), e in zip(parts, edges)]))


def path(n, label=0.0):
    return n, np.stack([np.arange(n - 1), np.arange(1, n)], 1), label


def ring(n, k, label=0.0):
    """Every vertex joined to the k next ones."""
    i = np.repeat(np.arange(n), k)
    return n, np.stack([i, (i + 1 + np.tile(np.arange(k), n)) % n], 1), label


def launched(log, kernel):
    """Pairs of every launch of a kernel."""
    return [int(k) for k in re.findall("^%s pairs=(\\d+)" % kernel, log, re.M)]


def test_workgroups_of_a_separable_launch_stay_within_the_grid(host):
    """Pairs and blocks of rows share a grid dimension of less than 2^32 threads: many pairs beside one
    with very many rows go in several launches (the stand-in refuses a larger one, as the runtime does)."""
    B = host.load(graphs(path(16400), ring(150, 6)))
    i = np.ones(4096, np.int32)
    i[0] = 0
    assert host.pairs(B, B, i, np.ones(4096, np.int32)) == 0, host.error()
    assert sum(launched(host.log(), "init")) == 4096 and max(launched(host.log(), "sep")) > 2000
    host.free(B)


def test_batch_freed_after_its_context(so):
    """Destroying the context first was always allowed; the context's memory is not looked at again."""
    h = host_runtime.Host(so)
    before, wb = h.lib.stub_in_use(), W.config1(12)
    X, Y = h.load(wb), h.load(wb)
    assert h.pairs(X, Y, [0, 1], [2, 3]) == 0, h.error()
    h.free(Y)   # its block is kept for the next batch
    gone = h.ctx
    h.destroy()
    assert h.lib.stub_in_use() > before
    h.lib.mgk_free_batch(gone, X)
    assert h.lib.stub_in_use() == before and h.violations() == ""


@pytest.mark.parametrize("entry", ["mgk_pairs", "mgk_pairs_noalloc"])
def test_block_of_a_freed_batch_waits_for_calls_on_streams_that_are_gone(host, entry):
    """A stream may be destroyed with work under way, and its handle given to a new one, before the batch is
    freed: the block must not go to the next batch while that work reads it."""
    wb = W.config1(12)
    host.free(host.load(wb))
    for _ in range(3):
        B = host.load(wb)
        host.hold(5)
        assert host.pairs(B, B, [0, 1], [2, 3], stream=5, entry=entry) == 0, host.error()
        host.lib.stub_replace_stream(C.c_void_p(5))
        host.free(B)
        host.free(host.load(wb))
        assert host.violations() == ""


@pytest.mark.parametrize("entry", ["mgk_pairs", "mgk_pairs_noalloc"])
def test_block_of_a_freed_batch_is_used_again(host, entry):
    """Loading, comparing and freeing in turn neither allocates nor waits for the device."""
    wb = W.config1(12)
    for k in range(6):
        if k == 2:
            before = host.count("malloc"), host.count("device waits")
        B = host.load(wb)
        assert host.pairs(B, B, [0, 1], [2, 3], entry=entry) == 0, host.error()
        host.free(B)
    assert (host.count("malloc"), host.count("device waits")) == before


def test_freeing_a_batch_leaves_the_current_device(host):
    B = host.load(W.config1(12))
    assert host.pairs(B, B, [0, 1], [2, 3]) == 0, host.error()
    host.lib.stub_set_device(1)
    host.free(B)
    assert host.lib.stub_device() == 1
    host.lib.stub_set_device(0)


def test_refused_calls_leave_a_recording_as_it_was(host):
    """A call that cannot be part of a graph is refused before it records or waits for anything: lists of
    its own, and pairs of the global-memory solver."""
    host.set("onchip_limit", 400)
    small, mixed = host.load(graphs(path(10), path(12))), host.load(graphs(path(10), path(30)))
    assert host.gram(mixed) == 0 and host.gram(small) == 0
    new = host.load(graphs(path(10), path(12)))
    device = (C.c_int32 * 2)(0, 1)   # the stand-in's device memory is host memory
    calls = [lambda: host.pairs(small, small, [0, 1], [1, 1], stream=3),
             lambda: host.pairs(small, small, [0, 1], [1, 1], stream=3, entry="mgk_pairs_noalloc"),
             lambda: host.lib.mgk_pairs_dev(host.ctx, small, small, C.c_int64(2), device, device, host.out(), None, None, C.c_void_p(3)),
             lambda: host.gram(mixed, stream=3), lambda: host.gram(new, stream=3)]
    host.lib.stub_reset()
    with host.recording(3):
        for call in calls:
            assert call() == 3 and "captur" in host.error()
            assert "recorded" not in host.log() and host.count("recorded copies") == host.count("broken recordings") == 0
        assert host.gram(small, stream=3) == 0
        assert "recorded" in host.log()
    for call in calls:
        assert call() == 0, host.error()


@pytest.mark.parametrize("k,kernel", [(6, "sep"), (75, "sep dense")])
def test_features_are_formed_for_the_graphs_of_the_pairs(host, k, kernel):
    """Not for the rest of the batch, however large it is."""
    B = host.load(graphs(*[ring(151, k)] * 9))
    in_use = host.lib.stub_in_use()
    assert host.pairs(B, B, [2, 2, 7] * 20, [7, 2, 4] * 20) == 0, host.error()
    assert launched(host.log(), kernel) and launched(host.log(), kernel + " pack") == [3]
    one = 192 * 192 * 4 if kernel == "sep dense" else 151 * k * 256   # a 192 x 192 matrix; a step of 64 words to two nonzeros of four rows
    assert host.lib.stub_in_use() - in_use < 3 * one + 60 * 5 * 4 * (151 * 151 + 63) + (1 << 20)
    host.free(B)


@pytest.mark.parametrize("sizes,i,j,outer,inner", [
    ((300, 2100, 3000, 9000), (1, 2, 3, 2), (0, 0, 0, 0), 3, 1),   # larger than an inner graph may be, as outer ones
    ((2048, 2049, 24, 2047), (1, 0, 0), (0, 2, 3), 2, 3),          # the limit, both roles, the smallest
    ((700, 650, 600, 2500), (0, 0, 3), (1, 2, 1), 2, 2)])
def test_features_of_graphs_of_many_vertices_by_their_part_in_the_pairs(host_wide, sizes, i, j, outer, inner):
    """Records for the outer graphs, steps for the inner ones, which alone have a limit: of one batch and of two."""
    host = host_wide
    host.set("edge_kernel_se", 0.42)
    wb = graphs(*[ring(n, 3, np.linspace(0, 1, 3 * n)) for n in sizes])
    X, Y = host.load(wb), host.load(wb)
    for pair in ((X, X, j, i), (X, Y, i, j)):   # the larger graph second, too
        host.lib.stub_clear_log()
        assert host.pairs(*pair) == 0, host.error()
        assert launched(host.log(), "wide") and launched(host.log(), "wide outer") == [outer] and launched(host.log(), "wide inner") == [inner]
        assert host.violations() == ""


@pytest.mark.parametrize("sizes,kernel", [((256, 251), "mgk_sep_dense_parts_kernel rank="), ((257, 256), "mgk_sep_dense_kernel<1> rank="),
                                          ((513, 512), "mgk_sep_dense_kernel<2> rank=")])
def test_launch_record_names_the_dense_kernel_that_runs(host, sizes, kernel):
    host.set("edge_kernel_se", 1.0)
    B = host.load(graphs(*[ring(n, n // 2 - 1, np.linspace(0, 1, n * (n // 2 - 1))) for n in sizes]))
    assert host.pairs(B, B, [0] * 16, [1] * 16) == 0, host.error()
    assert launched(host.log(), "sep dense") and host.launch_log().startswith(kernel)


def records(log):
    """Kernel and pairs of every launch of a call that the library records."""
    return sorted((name, int(k)) for name, k in re.findall(r"^(\w+).*? pairs=(\d+)", log, re.M))


@pytest.mark.parametrize("sizes,pairs,expected", [
    ((290, 250, 240), 200, [("mgk_sep_dense_kernel", 1), ("mgk_sep_dense_parts_kernel", 200)]),   # not all with the kernel of the largest
    ((290, 250, 240), 8, [("mgk_sep_dense_kernel", 9)]),                                          # too few for launches of their own
    ((256, 250, 240), 60, [("mgk_sep_dense_parts_kernel", 61)]),
    ((256, 250, 134), 60, [("mgk_sep_dense_parts_kernel", 61)])])     # small graphs beside large ones
def test_dense_pairs_run_with_the_kernel_they_are_priced_for(host, sizes, pairs, expected):
    host.set("edge_kernel_se", 1.0)
    B = host.load(graphs(*[ring(n, n // 2 - 1, np.linspace(0, 1, n * (n // 2 - 1))) for n in sizes]))
    assert host.pairs(B, B, [0] + [1] * pairs, [0] + [2] * pairs) == 0, host.error()
    assert records(host.launch_log()) == expected


def test_pairs_are_priced_with_the_division_that_runs(host):
    """Five features in one pass up to 276 columns: a larger pair that takes another product does not count."""
    host.set("edge_kernel_se", 1.0)
    B = host.load(graphs(ring(400, 199, np.linspace(0, 1, 400 * 199)), *[ring(250, 13, np.linspace(0, 1, 250 * 13))] * 2))
    assert host.pairs(B, B, [0] + [1] * 60, [0] + [2] * 60) == 0, host.error()
    assert records(host.launch_log()) == [("mgk_sep_dense_kernel", 1), ("mgk_sep_xmv_kernel", 60)]
    assert "mgk_sep_xmv_kernel<5> rank=5 passes=1" in host.launch_log()


def test_form_of_many_vertices_has_no_fewer_terms_than_the_other(host, host_wide):
    """What it would take is first priced with the other form's rank."""
    labels = lambda n, k: ring(n, k, np.linspace(0, 1, n * k))
    A, B = host.load(graphs(labels(300, 6), labels(290, 6))), host_wide.load(graphs(labels(900, 3), labels(890, 3)))
    for length in np.geomspace(0.25, 20, 25):
        ranks = []
        for h, batch in ((host, A), (host_wide, B)):
            h.set("edge_kernel_se", float(length))
            assert h.pairs(batch, batch, [0] * 64, [1] * 64) == 0, h.error()
            ranks.append(int(re.search(r"rank=(\d+)", h.launch_log()).group(1)))
        assert "mgk_wide" in host_wide.launch_log() and ranks[0] <= ranks[1] <= ranks[0] + 1


@pytest.mark.parametrize("largest,division", [(283, "<8, 9, 9> rank=9 passes=1"), (290, "<8, 4, 5> rank=9 passes=2"), (600, "<4, 4, 5> rank=9 passes=2")])
def test_division_of_many_vertices_is_that_of_the_largest_inner_graph(host_wide, largest, division):
    host = host_wide
    host.set("edge_kernel_se", 0.42)
    B = host.load(graphs(*[ring(n, 3, np.linspace(0, 1, 3 * n)) for n in (3000, largest, 260)]))
    assert host.pairs(B, B, [0] * 20, [1] * 2 + [2] * 18) == 0, host.error()
    assert "mgk_wide_xmv_kernel" + division in host.launch_log()
    assert host.violations() == ""


@pytest.mark.parametrize("n_pairs", [1, 3, 100])
@pytest.mark.parametrize("elements", [1, 2049, 4096 * 1024 + 5, 2 ** 31 - 65, 2 ** 31 - 64 - 4 * 2 ** 20])
def test_elements_of_a_thread_of_the_vector_kernels(so, n_pairs, elements):
    """Pairs have fewer than 2^31 - 64 elements: the steps past the last one stay within 32 bits."""
    lib = C.CDLL(so)
    lib.stub_quads.restype = C.c_int64
    blocks = lib.stub_lean_blocks(C.c_int64(n_pairs), (elements + 63) & ~63)
    assert 1 <= blocks <= 1024
    for block in {0, blocks // 2, blocks - 1}:
        for thread in (0, 511):
            expected = range(block * 2048 + 4 * thread, elements, blocks * 2048)
            got = (C.c_int64 * 2)()
            assert lib.stub_quads(block, blocks, thread, elements, got) == len(expected)
            assert not expected or tuple(got) == (expected[0], expected[-1])


def test_pairs_are_solved_without_features_where_memory_is_short(host):
    """Features of the separable product are an addition to what the direct product needs: neither forming
    them nor keeping them may make a call fail that the direct product can do."""
    labels = np.linspace(0, 1, 151 * 75)
    host.set("edge_kernel_se", 0.3)   # a high rank
    X, Y = host.load(graphs(ring(151, 75, labels))), host.load(graphs(ring(140, 69, labels[:140 * 69])))
    pairs = [0] * 64
    before, small = host.lib.stub_in_use(), 64 * 5 * 4 * 151 * 140 + (2 << 20)   # the vectors, and room for the lists of the direct product
    try:
        host.lib.stub_set_limit(C.c_int64(before + small))
        assert host.pairs(X, Y, pairs, pairs) == 0, host.error()
        assert launched(host.log(), "direct dense") and not launched(host.log(), "sep dense")
        host.lib.stub_set_limit(C.c_int64(-1))
        assert host.pairs(X, Y, pairs, pairs) == 0, host.error()
        assert launched(host.log(), "sep dense") and host.lib.stub_in_use() > before + small
        # what the context keeps is given back for the lists of the direct product, and for a batch
        host.lib.stub_set_limit(C.c_int64(host.lib.stub_in_use() + 65536))
        host.set("tile_path", 1)
        assert host.pairs(X, Y, pairs, pairs) == 0, host.error()
        host.set("tile_path", 0)
        host.lib.stub_set_limit(C.c_int64(-1))
        assert host.pairs(X, Y, pairs, pairs) == 0, host.error()
        host.lib.stub_set_limit(C.c_int64(host.lib.stub_in_use() + 65536))
        host.free(host.load(graphs(ring(151, 75, labels))))
        assert host.violations() == ""
    finally:
        host.lib.stub_set_limit(C.c_int64(-1))


def test_a_freed_batch_is_no_reason_to_run_out_of_memory(so):
    """A block that is kept is given back for a batch that it is too small for."""
    one = W.config1(200)
    nine = W.concat_batches([one] * 9, one.params, "nine")
    need = []
    for wb in (one, nine):   # of a batch whose block is not kept
        h = host_runtime.Host(so)
        empty = h.lib.stub_in_use()
        B = h.load(wb)
        need.append(h.lib.stub_in_use() - empty)
        h.free(B)
        h.destroy()
    h = host_runtime.Host(so)
    h.free(h.load(one))
    try:
        h.lib.stub_set_limit(C.c_int64(empty + need[1] - need[1] // 8))   # blocks are a quarter larger than asked for
        h.free(h.load(nine))
    finally:
        h.lib.stub_set_limit(C.c_int64(-1))
        h.destroy()


def test_outputs_are_formed_twice_at_most(host):
    """Once behind the iterations foreseen, and once more if pairs still iterate then, however long."""
    B = host.load(graphs(ring(151, 6), ring(140, 6)))
    host.lib.stub_converge_after(90)   # the first call of a context foresees fewer
    for foreseen in (False, True):
        host.lib.stub_clear_log()
        assert host.pairs(B, B, [0] * 64, [1] * 64) == 0, host.error()
        assert len(launched(host.log(), "vectors")) >= 90
        assert len(launched(host.log(), "outputs")) == (2 if foreseen else 4)   # two launches each
    host.free(B)


@pytest.mark.parametrize("n,k,pairs,kernel", [(600, 30, 1, "direct dense"), (600, 30, 2, "direct dense"), (600, 30, 16, "sep dense"), (256, 26, 1, "sep"),
                                              (480, 7, 1, "direct rows"), (480, 7, 16, "sep"),
                                              (300, 6, 2, "direct rows"), (300, 6, 16, "sep")])
def test_few_pairs_take_the_product_that_fills_the_chip(host, n, k, pairs, kernel):
    """One pair of 600 vertices has 19 workgroups in the dense separable product and 600 in the row-staged one:
    5.2 ms and 2.5 ms per call; with 16 pairs 10.5 and 27 ms."""
    host.set("edge_kernel_se", 1.0)
    B = host.load(graphs(ring(n, k, np.linspace(0, 1, n * k))))
    assert host.pairs(B, B, [0] * pairs, [0] * pairs) == 0, host.error()
    assert launched(host.log(), kernel), host.log()
    host.free(B)


def test_pinned_memory_is_allocated_once(so):
    """One block by the first call that stages a list, none by the calls after it or by those that need none."""
    h = host_runtime.Host(so)
    wb = W.config1(12)
    B = h.load(wb)
    assert h.gram(B) == 0 and h.lib.stub_pinned() == 0
    for k, entry in enumerate(("mgk_pairs", "mgk_pairs", "mgk_pairs_noalloc", "mgk_pairs", "mgk_pairs_noalloc", "mgk_pairs", "mgk_pairs")):
        assert h.pairs(B, B, [0, 1, 2], [2, 3, 4], entry=entry) == 0, h.error()
        if k == 0:
            pinned = h.lib.stub_pinned()
    assert h.lib.stub_pinned() == pinned > 0
    h.free(B)
    h.destroy()
    assert h.lib.stub_pinned() == 0


class Basis(C.Structure):
    _fields_ = [("rank", C.c_int32), ("terms", C.c_int32), ("center", C.c_double), ("inv_r", C.c_double), ("coef", C.c_double * 256)]

    def features(self, x):
        s = (np.asarray(x, np.float64) - self.center) * self.inv_r
        coef = np.array(self.coef).reshape(16, 16)[:self.terms, :self.rank]
        v = np.stack([np.polyval(coef[::-1, k], s * s) for k in range(self.rank)], 1)
        v[:, 1::2] *= s[:, None]
        return v


def basis_of(host, length_scale, lo, hi):
    """The separable form of the square-exponential kernel on labels of [lo, hi]; None if it has none."""
    B = host.load(graphs(ring(151, 20, np.linspace(lo, hi, 151 * 20))))
    host.set("edge_kernel_se", float(length_scale))
    host.lib.stub_clear_log()
    assert host.pairs(B, B, [0] * 64, [0] * 64) == 0, host.error()
    packed = launched(host.log(), "sep pack") + launched(host.log(), "sep dense pack")
    host.free(B)
    host.lib.stub_basis.restype = C.POINTER(Basis)
    out = Basis()
    C.memmove(C.byref(out), host.lib.stub_basis(), C.sizeof(Basis))
    return out if packed else None


@pytest.mark.parametrize("lo,hi", [(0.0, 1.0), (-3.0, 5.0), (100.0, 100.25), (0.0, 0.0)])
def test_separable_form_of_the_kernel(host, lo, hi):
    """Its error over the label range between the points that the host looks at (MGK_SEP_TOLERANCE there), in
    double and with the features rounded to fp32, which adds at most 2^-23 in all, as sum_k phi_k^2 is 1."""
    ranks = []
    for ratio in (100.0, 10.0, 3.0, 1.5, 1.0, 0.7, 0.5, 0.33, 0.25, 0.21, 0.18):
        length = float(np.float32(ratio * ((hi - lo) or 1.0)))
        S = basis_of(host, length, lo, hi)
        x = np.linspace(lo, hi, 301)
        exact = np.exp(-0.5 * ((x[:, None] - x[None]) / length) ** 2)
        phi = S.features(x)
        low = phi.astype(np.float32).astype(np.float64)
        assert np.abs(phi @ phi.T - exact).max() <= 6.0e-8
        assert np.abs(low @ low.T - exact).max() <= 6.0e-8 + 2.0 ** -23
        ranks.append(S.rank)
    assert ranks == sorted(ranks) and (ranks[-1] >= 15 or lo == hi)
    assert lo == hi or basis_of(host, 0.12 * (hi - lo), lo, hi) is None


def test_separable_forms_of_batches_in_turn(host):
    """The forms kept for earlier label ranges and length scales are not mixed up."""
    first = [bytes(basis_of(host, l, lo, hi)) for l, lo, hi in ((1.0, 0.0, 1.0), (0.5, 0.0, 1.0), (1.0, 0.0, 2.0))]
    again = [bytes(basis_of(host, l, lo, hi)) for l, lo, hi in ((1.0, 0.0, 1.0), (0.5, 0.0, 1.0), (1.0, 0.0, 2.0))]
    assert first == again and len(set(first)) == 3


def test_label_range_at_which_the_form_is_first_looked_for(host):
    """Whether to make the separable form is decided at rank 1, which must not cost more than the rank it has:
    the first call on new labels takes the same product as later ones."""
    B = host.load(graphs(*[ring(256, 1, np.linspace(0, 1, 256))] * 2))
    paths = []
    for length in (1.0, 1.0, 0.9, 0.9):
        host.set("edge_kernel_se", length)
        assert host.pairs(B, B, [0] * 64, [1] * 64) == 0, host.error()
        paths.append(host.launch_log().split(" ")[0])
    assert paths[0] == paths[1] and paths[2] == paths[3], paths
    host.free(B)


def streaming(host, labels=(0.0, 1.0), n=90, k=8, count=24):
    """Graphs whose pairs take the separable product on chip."""
    host.set("edge_kernel_se", 1.0)
    return host.load(graphs(*[ring(n, k, np.linspace(*labels, n * k))] * count))


def test_packets_on_chip_wait_for_calls_that_read_them(host):
    """Also for those on a stream of the same handle that is gone."""
    B = streaming(host)
    assert host.gram(B) == 0   # makes the list
    for stream in (5, 5, 6):
        host.hold(stream)
        assert host.gram(B, stream) == 0 and "mgk_pcg_sep" in host.launch_log(), host.error()
        host.lib.stub_replace_stream(C.c_void_p(5))
    assert host.violations() == ""
    host.free(B)


def test_calls_on_two_streams_do_not_wait_on_the_host(host):
    """A Gram of pairs solved on chip is enqueued while another stream still solves one."""
    B = streaming(host)
    for stream in (5, 6):   # memory is allocated by the first call
        assert host.gram(B, stream) == 0
    waits = ("stream waits", "device waits", "event waits", "free")
    before = [host.count(w) for w in waits]
    for stream in (5, 6, 5, 6):
        host.hold(stream)
        assert host.gram(B, stream) == 0 and "mgk_pcg_sep" in host.launch_log(), host.error()
    assert [host.count(w) for w in waits] == before and host.violations() == ""
    host.free(B)


def test_packets_of_a_call_that_fails_have_an_end(host):
    """What it has enqueued by then writes or reads them."""
    X, Y = streaming(host), streaming(host, (0.0, 0.9), n=96)
    i = np.arange(24).repeat(12)
    assert host.gram(X, stream=6) == 0 and host.pairs(X, Y, i, i, stream=5) == 0, host.error()
    host.hold(5)
    host.lib.stub_fail(b"pcg_sep")
    assert host.pairs(X, Y, i, i, stream=5) == 3 and "mgk_pcg_sep" in host.launch_log()
    host.lib.stub_fail(b"")
    assert host.gram(X, stream=6) == 0 and "mgk_pcg_sep" in host.launch_log(), host.error()
    assert host.violations() == ""


def test_memory_of_the_packets(host):
    """Reserved when graphs are loaded that may need them, for any two batches of a call; given back where memory is short, when
    the pairs are solved without packets, by the call that may not allocate as well."""
    i = np.arange(24).repeat(12)
    both = ("mgk_pairs", "mgk_pairs_noalloc")
    separable = lambda A, B, entry: host.pairs(A, B, i, i, entry=entry) == 0 and "mgk_pcg_sep" in host.launch_log()
    before = host.lib.stub_in_use()
    host.free(host.load(W.config1(12)))   # every pair fits the registers
    assert host.lib.stub_in_use() - before < 1 << 20
    Y = streaming(host)
    X = streaming(host, n=92, count=48)   # more than twice as many nonzeros: a larger block
    assert separable(Y, Y, "mgk_pairs")   # makes the list
    before = host.count("malloc")
    for entry in both:
        for A, B in ((X, X), (X, Y), (Y, X), (Y, Y)):
            assert separable(A, B, entry), host.launch_log()
    assert host.count("malloc") == before
    try:
        host.lib.stub_set_limit(C.c_int64(host.lib.stub_in_use() + 65536))
        Z = host.load(W.config1(2000))   # needs the memory of the packets
        host.lib.stub_set_limit(C.c_int64(host.lib.stub_in_use()))
        for entry in both:
            assert not separable(Y, Y, entry) and "mgk_pcg_small" in host.launch_log()
    finally:
        host.lib.stub_set_limit(C.c_int64(-1))
    for entry in both:
        assert separable(X, Y, entry)
    assert host.violations() == ""
    host.free(Z)


def gram(host, batch, stream=0, counts=False):
    return host.lib.mgk_gram(host.ctx, batch, host.out(), host.out() if counts else None, None, C.c_void_p(stream))


@pytest.mark.parametrize("first,mode,counts,kernel", [
    (False, 1, True, "regs"), (False, 0, False, "regs"), (False, 0, True, "regs"), (False, 2, True, "reduced"),
    (True, 2, False, "reduced"), (True, 2, True, "reduced"), (True, 1, False, "regs"), (False, 1, False, "reduced")])
def test_recorded_gram_solves_the_system_it_says(host, first, mode, counts, kernel):
    """After an eager Gram with (first) or without iteration counts: whose counts are asked for, or whose mode names the
    system, gets that system, also if its list has to be made; nothing of that is recorded."""
    host.set("edge_kernel_se", 0.1)
    B = host.load(W.config1(12))
    assert gram(host, B, 3, first) == 0
    host.set("reduced_system", mode)
    host.lib.stub_clear_log()
    with host.recording(3):
        for _ in range(2):
            assert gram(host, B, 3, counts) == 0, host.error()
    assert re.findall(r"^(\w+) .* recorded$", host.log(), re.M) == [kernel] * (len(host.log().split("\n")) - 1) and kernel in host.log()
    assert host.count("recorded copies") == host.count("broken recordings") == 0 and host.violations() == ""
    host.free(B)


def test_recorded_gram_of_a_batch_with_an_older_list(host):
    """The list that is wanted was made with other settings, the other one with these; no list with these is refused."""
    host.set("edge_kernel_se", 0.1)
    B = host.load(W.config1(12))
    before = host.lib.stub_in_use()
    for k in range(3):
        host.set("schedule", k % 2)
        with host.recording(3):
            assert gram(host, B, 3, k % 2 == 0) == 3 and "captur" in host.error()
        assert gram(host, B) == 0
        with host.recording(3):
            assert gram(host, B, 3, True) == 0, host.error()
        assert gram(host, B, 0, True) == 0
        if k == 0:
            kept = host.lib.stub_in_use()
    assert host.count("recorded copies") == host.count("broken recordings") == 0 and host.violations() == ""
    assert host.lib.stub_in_use() - before <= 2 * (kept - before)
    host.free(B)


def star(n):
    return n, np.stack([np.zeros(n - 1, int), np.arange(1, n)], 1), 0.0


def grid(a, b):
    i = np.arange(a * b).reshape(a, b)
    return a * b, np.concatenate([np.stack([i[:, :-1].ravel(), i[:, 1:].ravel()], 1), np.stack([i[:-1].ravel(), i[1:].ravel()], 1)]), 0.0


def random_graph(rng, n, edges, vertices=None):
    """Any graph: isolated vertices, hubs, several parts; among the first `vertices` of n."""
    a, b = np.triu_indices(vertices or n, 1)
    pick = rng.choice(len(a), min(edges, len(a)), replace=False)
    return n, np.stack([a[pick], b[pick]], 1), 0.0


def test_schedules_of_the_reduced_solver(host):
    """As the kernel reads them (the stand-in looks them over at every launch), for graphs of all kinds: up to 160 nonzeros,
    up to 160 vertices with edges, rows longer than four, no edges; as outer graph against a small inner one."""
    rng = np.random.default_rng(8)
    parts = [path(2), path(64), path(65), path(81), star(17), star(21), ring(20, 3), ring(9, 4), (1, [], 0.0), (7, [], 0.0),
             (160, np.arange(160).reshape(-1, 2), 0.0)]
    parts += [random_graph(rng, int(n), int(e), int(v)) for n, e, v in
              zip(rng.integers(12, 150, 60), rng.integers(1, 81, 60), rng.integers(3, 13, 60))]
    parts += [random_graph(rng, int(n), int(e)) for n, e in zip(rng.integers(5, 90, 150), rng.integers(1, 81, 150))]
    host.set("reduced_system", 2)
    B, inner = host.load(graphs(*parts)), host.load(graphs(path(3), ring(6, 1), path(40)))
    i, j, log = np.arange(len(parts)).repeat(3), np.tile([0, 1, 2], len(parts)), ""
    for many in (8, 1):   # two wavefronts where there are thousands of pairs
        assert host.pairs(B, inner, np.tile(i, many), np.tile(j, many)) == 0, host.error()
        log += host.launch_log()
    assert host.violations() == "" and all("mgk_pcg_reduced<%d" % w in log for w in (2, 4, 8))
    host.free(B)
    host.free(inner)


def kinds(host):
    """Pairs by kernel of the last call."""
    got = {}
    for kernel, n in re.findall(r"mgk_pcg_(\w+)<.*> pairs=(\d+)", host.launch_log()):
        got[kernel] = got.get(kernel, 0) + int(n)
    return got


LATTICES = {"grids": [grid(a, b) for a in range(4, 7) for b in range(a, 7)], "ladders": [grid(2, n) for n in range(8, 27)]}


@pytest.mark.parametrize("name,full,streaming", [("grids", True, False), ("ladders", False, True)])
def test_pairs_that_fit_the_full_system_only_stay_register_resident(host, name, full, streaming):
    """A graph of whole rows may fit the wavefronts of the solver of the full system and not those of the reduced one.  A few of
    those go with others that need the streaming solver, if there are any."""
    got = []
    for mode in (0, 1):
        host.set("reduced_system", mode)
        B = host.load(graphs(*LATTICES[name]))
        assert host.gram(B) == 0, host.error()
        got.append(kinds(host))
        i, j = np.triu_indices(len(LATTICES[name]))
        assert host.pairs(B, B, i, j) == 0 and kinds(host) == got[-1]
        host.free(B)
    assert host.violations() == "" and got[1]["reduced"] > 0
    assert (got[1].get("regs", 0) > 0, got[1].get("small", 0) > 0) == (full, streaming)
    assert (got[0].get("small", 0) > 0) == streaming
    assert got[1].get("regs", 0) + got[1].get("small", 0) + got[1]["reduced"] == sum(got[0].values())


def test_pairs_of_the_full_system_join_launches_of_their_size_only(host):
    """Not where they would need another workgroup size, and not more than a thousand of them."""
    host.set("edge_kernel_se", 1.0)
    B = host.load(graphs(path(12), grid(6, 6), grid(2, 21), ring(24, 5)))
    stream = (1, 3)   # needs the streaming solver, four wavefronts
    for pair, count, stays in (((1, 1), 1, False), ((1, 1), 1000, False), ((0, 2), 1, True), ((1, 1), 1100, True)):   # the path: two wavefronts
        i, j = np.array([pair] * count + [stream]).T
        assert host.pairs(B, B, i, j) == 0, host.error()
        assert kinds(host) == ({"regs": count, "small": 1} if stays else {"small": count + 1}) and host.violations() == ""
    host.free(B)


@pytest.mark.parametrize("n,inner", [(9000, 1), (10300, 1), (12000, 1), (16000, 1), (1, 12000), (2, 8000)])
def test_pairs_of_many_isolated_vertices_stay_within_lds(host, n, inner):
    """The reduced solver holds the vertices of both graphs and all eliminated elements in LDS: beyond it the pair goes where it went
    without that solver."""
    B = host.load(graphs((n, [(0, 1)] if n > 1 else [], 0.0), (inner, [(0, 1)] if inner > 1 else [], 0.0)))
    kernels = []
    for mode in (0, 1):
        host.set("reduced_system", mode)
        assert host.pairs(B, B, [0, 1], [1, 0]) == 0, host.error()
        kernels.append(host.launch_log().split("<")[0])
    assert kernels[0] == kernels[1] or kernels[1] == "mgk_pcg_reduced"
    assert host.violations() == ""
    host.free(B)


def test_merged_launches_keep_the_offsets_of_the_reduced_solver(host):
    """A pair with many eliminated elements fits its own launch shape and not the larger one that few pairs are moved to."""
    edge = lambda n: (n, [(0, 1)], 0.0)
    B = host.load(graphs(star(13), edge(1200), path(2), edge(2000)))
    assert host.pairs(B, B, [0, 2], [1, 3]) == 0, host.error()
    assert "mgk_pcg_reduced<4, 8, 1> pairs=1" in host.launch_log() and host.violations() == ""
    host.free(B)


@pytest.mark.parametrize("entry", ["gram", "pairs"])
@pytest.mark.parametrize("mode", [1, 2])
def test_few_pairs_leave_the_reduced_system_only_where_nobody_asked_for_it(host, entry, mode):
    """A few tiny pairs of which one needs the streaming solver go there together, unless the mode says always reduced."""
    host.set("edge_kernel_se", 1.0)
    B = host.load(graphs(path(6), path(7), ring(9, 4), path(8)))
    i, j = np.triu_indices(4)
    assert host.gram(B) == 0   # its list is not that of mode 2
    host.set("reduced_system", mode)
    assert (host.gram(B) if entry == "gram" else host.pairs(B, B, i, j)) == 0, host.error()
    assert "mgk_pcg_small" in host.launch_log() and ("mgk_pcg_reduced" in host.launch_log()) == (mode == 2)
    host.free(B)


def test_only_kernels_with_a_separable_form_have_a_launch_for_pairs_beyond_it(host):
    """Streaming pairs of up to and of more than 14336 elements go in one launch where nothing takes the separable product, also
    if the list of the batch was made when it might; a recorded Gram takes the list that is there."""
    poly = (C.c_float * 6)(1.0, 0.0, -10.0, 20.0, -15.0, 4.0)
    B = host.load(graphs(*[ring(n, 2, np.linspace(0, 1, n * 2)) for n in (123, 122, 121, 118, 117, 116)]))
    i, j = np.triu_indices(6)
    launches = {}
    for kernel in ("poly", "se", "poly", "se"):
        if kernel == "se":
            host.set("edge_kernel_se", 1.0)
        else:
            assert host.lib.mgk_set_edge_kernel_poly(host.ctx, 6, poly, C.c_float(1.2)) == 0
        assert host.gram(B, 3) == 0, host.error()
        of_gram = host.launch_log()
        assert host.pairs(B, B, i, j) == 0, host.error()
        assert launches.setdefault(kernel, host.launch_log()) == host.launch_log() == of_gram
    assert launches["poly"].count("pairs=") == 1 and launches["se"].count("pairs=") == 2
    with host.recording(3):
        assert host.lib.mgk_set_edge_kernel_poly(host.ctx, 6, poly, C.c_float(1.2)) == 0
        assert host.gram(B, 3) == 0 and host.launch_log().count("pairs=") == 2
    host.free(B)


def test_pairs_without_allocation_take_the_same_kernels(host):
    """Also those whose packets another call would allocate; streams in turn wait as before, and nothing is allocated."""
    X, Y = streaming(host), streaming(host, (0.0, 0.9), n=96)
    i = np.arange(24).repeat(12)
    assert host.pairs(X, Y, i, i) == 0
    same = host.launch_log()
    assert "mgk_pcg_sep" in same
    before = host.count("malloc"), host.count("free"), host.lib.stub_in_use()
    for stream in (5, 6, 5):
        host.hold(stream)
        assert host.pairs(X, Y, i, i, stream=stream, entry="mgk_pairs_noalloc") == 0 and host.launch_log() == same, host.error()
    assert (host.count("malloc"), host.count("free"), host.lib.stub_in_use()) == before and host.violations() == ""
    host.free(X)
    host.free(Y)
