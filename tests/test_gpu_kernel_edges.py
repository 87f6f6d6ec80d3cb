"""Sizes at which a kernel's tiles, groups or tables end, against the oracle.
All results are whole numbers: no tolerance."""
import numpy as np
import pytest

import graphgen as gg

pytestmark = pytest.mark.gpu


def _hubs(degrees, seed=1):
    """Hubs of the given degrees over shared leaves, some leaves joined."""
    rng = np.random.default_rng(seed)
    leaves = max(degrees) + 7
    src, dst = [], []
    for h, d in enumerate(degrees):
        src += [h] * d
        dst += list(len(degrees) + rng.choice(leaves, d, replace=False))
    extra = len(degrees) + rng.integers(0, leaves, (2, 3 * leaves))
    return gg.csr_from_edges(len(degrees) + leaves, np.concatenate([src, extra[0]]),
                             np.concatenate([dst, extra[1]]), perm_seed=seed)


@pytest.mark.parametrize("degrees", [[1, 15, 16, 17], [255, 256, 257], [63, 64, 65, 600, 2, 1023]])
def test_row_walk_at_group_and_wave_sizes(citron_gpu, degrees):
    """Rows walked by 16 lanes (up to 256 entries) or by a whole wave."""
    import oracle
    g = _hubs(degrees)
    h = citron_gpu.Graph.from_csr(g.row_ptr, g.col).order()
    ptr, col = h.dag()
    want_ptr, want_col = oracle.orient(g.n, g.row_ptr, g.col)
    assert np.array_equal(ptr, want_ptr) and np.array_equal(col, want_col)
    assert h.info()["max_outdeg"] == int(np.diff(want_ptr).max())
    h.free()


@pytest.mark.parametrize("lower_row", [False, True])
def test_a_missing_mirror_entry_is_refused(citron_gpu, lower_row):
    """One entry dropped, from the row of the edge's lower endpoint (the
    mirror is searched for there) or of the higher (the counts differ); a
    second one-sided entry keeps the number of entries even."""
    g = _hubs([300, 20, 20])
    deg = np.diff(g.row_ptr)
    src = np.repeat(np.arange(g.n), deg)
    lower = (deg[src] < deg[g.col]) | ((deg[src] == deg[g.col]) & (src < g.col))
    drop = np.nonzero(lower == lower_row)[0][[3, -5]]
    assert (src[drop[0]], g.col[drop[0]]) != (g.col[drop[1]], src[drop[1]])
    keep = np.ones(g.nnz, bool)
    keep[drop] = False
    row_ptr = np.concatenate([[0], np.cumsum(np.bincount(src[keep], minlength=g.n))]).astype(np.int32)
    with pytest.raises(citron_gpu.CitronError) as e:
        citron_gpu.Graph.from_csr(row_ptr, g.col[keep])
    assert e.value.status == 1


def test_degree_ordering_after_load_with_a_core_ordered_neighbour(citron_gpu):
    """The load's out-degrees serve the degree ordering of their own graph,
    whatever another handle of the same graph does in between."""
    import oracle
    g = gg.rmat(9, 12, seed=77)
    a = citron_gpu.Graph.from_csr(g.row_ptr, g.col)
    b = citron_gpu.Graph.from_csr(g.row_ptr, g.col).order("core")
    a.order()
    want_ptr, want_col = oracle.orient(g.n, g.row_ptr, g.col)
    ptr, col = a.dag()
    assert np.array_equal(ptr, want_ptr) and np.array_equal(col, want_col)
    for k in (3, 4, 5):
        assert a.count(k) == b.count(k) == oracle.count(g, k)[0]
    a.free()
    b.free()


@pytest.mark.parametrize("n_arcs", [1, 2, 15, 16, 17, 31, 33, 4095, 4097, 70001])
@pytest.mark.parametrize("k", [4, 5])
def test_claims_at_run_shard_and_grid_sizes(citron_gpu, n_arcs, k):
    """Work items in numbers around a run, a round of the cursors, the waves
    of the grid and several runs per wave: every listed arc counted once."""
    import oracle
    g = gg.rmat(9, 20, seed=5)
    h = citron_gpu.Graph.from_csr(g.row_ptr, g.col).order()
    total, every = h.count_per_arc(k)
    assert total == oracle.count(g, k)[0] == int(every.sum())
    arcs = np.random.default_rng(n_arcs).integers(0, g.m, n_arcs).astype(np.int32)
    assert np.array_equal(h.count_arcs(k, arcs), every[arcs])
    h.free()


def test_runs_that_span_queries(citron_gpu):
    """A batch whose queries are smaller than a claimed run of items."""
    import oracle
    gs = [gg.rmat(6, 6, seed=900 + i) for i in range(40)] + [gg.rmat(11, 16, seed=950)]
    hs = [citron_gpu.Graph.from_csr(g.row_ptr, g.col).order() for g in gs]
    q = [(i, k) for k in (4, 5, 6) for i in range(len(gs))]
    got = citron_gpu.count_batch([hs[i] for i, _ in q], [k for _, k in q])
    assert got == [oracle.count(gs[i], k)[0] for i, k in q]


@pytest.mark.parametrize("n,ks", [(67, (6, 7, 8)), (98, (6, 7)), (131, (6, 7)), (195, (6,)), (259, (6,)),
                                  (323, (6,)), (388, (6,))])
def test_dense_arcs_of_complete_graphs(citron_gpu, n, ks):
    """K_n holds an arc with |C_uv| = c for every c up to n - 2, so every row
    word and tile count of the dense kernel up to that size, and every mask
    product at its largest; beyond 384 candidates the count kernel goes on."""
    from math import comb
    g = gg.complete(n)
    h = citron_gpu.Graph.from_csr(g.row_ptr, g.col).order()
    for k in ks:
        assert h.count(k) == comb(n, k)
    h.free()


@pytest.mark.parametrize("n,p,k", [(90, 0.9, 6), (90, 0.9, 7), (100, 0.75, 8), (110, 0.6, 9), (90, 0.6, 13),
                                   (150, 0.8, 6), (150, 0.5, 7), (230, 0.7, 6), (300, 0.5, 6), (420, 0.4, 6)])
def test_dense_arcs_against_the_count_kernel(citron_gpu, n, p, k):
    """Whole, per-arc, strided and batched counts of dense random graphs
    against the vertex-rooted unit and the listed arcs, which stay on the
    count kernel."""
    g = gg.erdos_renyi(n, p * (n - 1), seed=n + k)
    h = citron_gpu.Graph.from_csr(g.row_ptr, g.col).order()
    want = h.count_vertex_rooted(k)
    assert h.count(k) == want
    total, every = h.count_per_arc(k)
    assert total == want
    assert np.array_equal(every, h.count_arcs(k, np.arange(g.m)))
    parts = [h.count_part(k, i, 5) for i in range(5)]
    assert sum(c for c, _ in parts) == want and not any(o for _, o in parts)
    assert citron_gpu.count_batch([h, h, h], [6, k, 5]) == [h.count_vertex_rooted(6), want, h.count_vertex_rooted(5)]
    h.free()


@pytest.mark.parametrize("ordering", ["degree", "core"])
def test_dense_arcs_under_both_orderings(citron_gpu, ordering):
    import oracle
    g = gg.rmat(10, 32, seed=31)
    h = citron_gpu.Graph.from_csr(g.row_ptr, g.col).order(ordering)
    for k in (6, 7):
        assert h.count(k) == oracle.count(g, k)[0]
    h.free()


@pytest.mark.parametrize("k", [7, 8, 9, 10, 12, 13, 20, 32])
def test_complete_nodes_of_light_vertices(citron_gpu, k):
    """Disjoint cliques up to K_65, whose vertices are all light (out-degree
    at most 64): every probed node is complete and counted by a binomial."""
    from math import comb
    sizes = list(range(5, 66, 4)) + [64]
    g = gg.disjoint_cliques(sizes)
    h = citron_gpu.Graph.from_csr(g.row_ptr, g.col).order()
    want = sum(comb(s, k) for s in sizes)
    assert want < 2 ** 64
    assert h.count(k) == want
    assert h.count_vertex_rooted(k) == want
    total, every = h.count_per_arc(k)
    assert total == want == sum(int(x) for x in every)
    h.free()


def test_binomials_that_carry(citron_gpu):
    from math import comb
    g = gg.disjoint_cliques([65] * 6)
    h = citron_gpu.Graph.from_csr(g.row_ptr, g.col).order()
    want = 6 * comb(65, 32)
    assert want > 2 ** 64
    assert h.count_checked(32) == (want % 2 ** 64, True)
    h.free()


@pytest.mark.parametrize("n,missing,k", [(24, 1, 7), (30, 12, 7), (30, 12, 8), (28, 3, 9), (26, 40, 9), (24, 9, 10),
                                         (22, 5, 13)])
def test_nearly_complete_nodes(citron_gpu, n, missing, k):
    """A clique with a few edges taken out, beside a sparse graph: probes that
    fail at the root and hold below it."""
    import oracle
    rng = np.random.default_rng(n * 100 + k)
    i, j = np.triu_indices(n, 1)
    keep = np.ones(i.size, bool)
    keep[rng.choice(i.size, missing, replace=False)] = False
    extra = rng.integers(0, 200, (2, 900))
    g = gg.csr_from_edges(200, np.concatenate([i[keep], extra[0]]), np.concatenate([j[keep], extra[1]]), perm_seed=k)
    h = citron_gpu.Graph.from_csr(g.row_ptr, g.col).order()
    want, ovf = oracle.count(g, k)
    assert not ovf and want > 0
    assert h.count(k) == want
    assert h.count_vertex_rooted(k) == want
    total, every = h.count_per_arc(k)
    assert total == want == int(every.sum())
    assert sum(h.count_part(k, p, 7)[0] for p in range(7)) == want
    h.free()


@pytest.mark.parametrize("chains", [1, 63, 4095, 4096, 4097, 9000])
def test_peeling_at_the_sizes_where_phases_change(citron_gpu, chains):
    """Frontiers and lists of the vertices left around the sizes that one
    workgroup handles by itself (8192): chains that peel from both ends, and
    cliques whose rise of the threshold comes after them."""
    import oracle
    chain = np.arange(chains)[:, None] * 7 + np.arange(6)[None, :]
    n = chains * 7
    src, dst = [chain.ravel()], [chain.ravel() + 1]
    for size in (4, 5, 9):
        for _ in range(1 + chains // 4):
            i, j = np.triu_indices(size, 1)
            src.append(n + i)
            dst.append(n + j)
            n += size
    g = gg.csr_from_edges(n, np.concatenate(src), np.concatenate(dst), perm_seed=chains)
    h = citron_gpu.Graph.from_csr(g.row_ptr, g.col).order("core")
    key, rounds = h.order_key()
    want = oracle.peel_rounds(g.n, g.row_ptr, g.col)
    assert np.array_equal(key, want) and rounds == int(want.max()) + 1
    h.free()


@pytest.mark.parametrize("d_low,hub", [(2, 9), (3, 13), (5, 20), (5, 21), (16, 64), (16, 65), (63, 70), (64, 300),
                                       (65, 261), (127, 130), (130, 513), (200, 1000)])
def test_rows_of_short_and_long_lists(citron_gpu, d_low, hub):
    """Subgraph rows where a vertex's list is up to, and more than, four times
    shorter than its neighbours' (each side searches the other), and at sizes
    of the light and heavy builds: triangles and 4-cliques per arc against a
    direct count."""
    rng = np.random.default_rng(d_low * 1000 + hub)
    n = hub + 6
    i, j = np.triu_indices(n, 1)                       # a dense core: its out-degrees run up to n - 1
    keep = rng.random(i.size) < 0.9
    src, dst = [i[keep]], [j[keep]]
    for low in range(12):                              # short vertices over the core
        t = rng.choice(n, min(d_low, n), replace=False)
        src.append(np.full(t.size, n + low))
        dst.append(t)
    g = gg.csr_from_edges(n + 12, np.concatenate(src), np.concatenate(dst), perm_seed=hub)
    h = citron_gpu.Graph.from_csr(g.row_ptr, g.col).order()
    ptr, col = h.dag()
    a = np.zeros((g.n, g.n), bool)
    s = np.repeat(np.arange(g.n), np.diff(ptr))
    a[s, col] = True
    common = a[s] & a[col]
    tri, per3 = h.count_per_arc(3)
    assert tri == int(common.sum()) and np.array_equal(per3, common.sum(1))
    total, per4 = h.count_per_arc(4)
    f = a.astype(np.float32)
    want4 = ((common @ f) * common).sum(1).astype(np.int64)       # below 2^24: exact
    assert total == int(want4.sum()) and np.array_equal(per4, want4)
    st = h.work_stats(4)
    assert st["entries"] == int(np.diff(ptr)[col][np.diff(ptr)[s] >= 2].sum())
    h.free()


def test_blocks_reused_across_threads_and_streams(citron_gpu):
    """Graphs made, counted and freed in turn on several threads, each with a
    stream of its own: blocks of one graph serve the next, whatever they held."""
    import threading
    import oracle
    import torch
    gs = [gg.rmat(9, 20, seed=70), gg.rmat(9, 21, seed=71), gg.erdos_renyi(600, 24, seed=72),
          gg.complete(90), gg.empty(700), gg.rmat(10, 30, seed=73)]
    want = {(i, k): oracle.count(g, k)[0] if i != 3 else __import__("math").comb(90, k)
            for i, g in enumerate(gs) for k in (3, 4, 6)}
    bad = []

    def work(seed):
        rng = np.random.default_rng(seed)
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            for _ in range(25):
                i = int(rng.integers(len(gs)))
                k = int(rng.choice([3, 4, 6]))
                h = citron_gpu.Graph.from_csr(gs[i].row_ptr, gs[i].col)
                h.order("core" if rng.random() < 0.3 else "degree")
                if h.count(k) != want[(i, k)]:
                    bad.append((i, k))
                h.free()

    threads = [threading.Thread(target=work, args=(s,)) for s in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad


@pytest.mark.parametrize("n,p,k", [(66, 1.0, 4), (70, 0.6, 4), (70, 0.6, 5), (135, 0.5, 4), (200, 0.35, 5), (90, 0.3, 6)])
def test_listing_of_dense_graphs(citron_gpu, n, p, k):
    """Last levels of more than 64 candidates and of several row words, and an
    output that is not aligned to 16 bytes: against the oracle's listing."""
    import ctypes
    import oracle
    import torch
    g = gg.erdos_renyi(n, p * (n - 1), seed=n * 10 + k)
    h = citron_gpu.Graph.from_csr(g.row_ptr, g.col).order()
    got, offsets = h.list_arcs(k)
    ptr, col = h.dag()
    want, per_arc = oracle.list_arcs(g.n, ptr, col, k, np.repeat(np.arange(g.n), np.diff(ptr)).astype(np.int32), col)
    assert np.array_equal(np.diff(offsets.cpu().numpy()), per_arc.astype(np.int64))
    assert np.array_equal(got.cpu().numpy(), want)
    buf = torch.full((got.numel() + 4,), -9, dtype=torch.int32, device="cuda")
    arcs = torch.arange(g.m, dtype=torch.int32, device="cuda")
    off2 = torch.zeros(g.m + 1, dtype=torch.int64, device="cuda")
    total = ctypes.c_int64(0)
    torch.cuda.synchronize()
    st = citron_gpu.load_library().citron_list_arcs(h._handle(), k, arcs.data_ptr(), g.m, off2.data_ptr(),
                                                    buf.data_ptr() + 4, got.shape[0], ctypes.byref(total))
    assert st == 0 and total.value == got.shape[0]
    flat = buf.cpu().numpy()
    assert np.array_equal(flat[1:1 + got.numel()], got.cpu().numpy().ravel())
    assert flat[0] == -9 and (flat[1 + got.numel():] == -9).all()
    h.free()


@pytest.mark.parametrize("n", [66, 67, 98, 129, 130, 193, 258, 322, 385, 386, 400])
def test_dense_vertices_of_complete_graphs(citron_gpu, n):
    """K_n has a vertex of every out-degree up to n - 1: all the sizes of the
    dense kernel's vertices at k = 4, 5, and those above and below them."""
    from math import comb
    g = gg.complete(n)
    h = citron_gpu.Graph.from_csr(g.row_ptr, g.col).order()
    assert h.count(4) == comb(n, 4)
    assert h.count(5) == comb(n, 5)
    h.free()


@pytest.mark.parametrize("n,p,k", [(120, 0.8, 4), (120, 0.8, 5), (250, 0.5, 4), (250, 0.5, 5), (400, 0.6, 4), (400, 0.4, 5),
                                   (520, 0.9, 4), (520, 0.6, 5)])
def test_dense_vertices_against_the_count_kernel(citron_gpu, n, p, k):
    """Counts, per-arc counts, strided shares and batches of k = 4, 5 against
    the vertex-rooted unit and the listed arcs (the count kernel)."""
    g = gg.erdos_renyi(n, p * (n - 1), seed=n + k)
    h = citron_gpu.Graph.from_csr(g.row_ptr, g.col).order()
    want = h.count_vertex_rooted(k)
    assert h.count(k) == want
    total, every = h.count_per_arc(k)
    assert total == want
    assert np.array_equal(every, h.count_arcs(k, np.arange(g.m)))
    parts = [h.count_part(k, i, 6) for i in range(6)]
    assert sum(c for c, _ in parts) == want
    assert citron_gpu.count_batch([h, h], [k, 6 - k + 3]) == [want, h.count_vertex_rooted(6 - k + 3)]
    assert h.work_stats(k)["word_ops"] > 0
    h.free()


@pytest.mark.parametrize("n,k", [(67, 9), (131, 8), (195, 7), (259, 7), (323, 7), (388, 7)])
def test_dense_items_of_more_masks_than_one_sum_holds(citron_gpu, n, k):
    """Items whose masks are summed several times, for every number of row
    words: a wave adds up at most 2^20 / (64 words) masks at once."""
    from math import comb
    g = gg.complete(n)
    h = citron_gpu.Graph.from_csr(g.row_ptr, g.col).order()
    assert h.count(k) == comb(n, k)
    h.free()


@pytest.mark.parametrize("n,p,k", [(150, 0.8, 8), (230, 0.6, 7), (300, 0.5, 7), (400, 0.4, 7)])
def test_deep_dense_arcs_against_the_count_kernel(citron_gpu, n, p, k):
    """Searches above the masks' nodes in subgraphs of several row words."""
    g = gg.erdos_renyi(n, p * (n - 1), seed=n + k)
    h = citron_gpu.Graph.from_csr(g.row_ptr, g.col).order()
    want = h.count_vertex_rooted(k)
    assert h.count(k) == want
    assert h.count_per_arc(k)[0] == want
    h.free()


@pytest.mark.parametrize("n,p", [(440, 0.97), (620, 0.75)])
def test_arcs_of_vertices_too_large_for_a_dense_item_at_k_5(citron_gpu, n, p):
    """k = 5 with out-degrees on both sides of 384: whole vertices below, arcs
    above, in the same dense classes."""
    g = gg.erdos_renyi(n, p * (n - 1), seed=n)
    h = citron_gpu.Graph.from_csr(g.row_ptr, g.col).order()
    assert h.info()["max_outdeg"] > 384
    want = h.count_vertex_rooted(5)
    assert h.count(5) == want
    total, every = h.count_per_arc(5)
    assert total == want
    assert np.array_equal(every, h.count_arcs(5, np.arange(g.m)))
    parts = [h.count_part(5, i, 4) for i in range(4)]
    assert sum(c for c, _ in parts) == want
    assert citron_gpu.count_batch([h, h], [5, 4]) == [want, h.count_vertex_rooted(4)]
    h.free()


@pytest.mark.parametrize("n,p", [(90, 0.7), (300, 0.5), (440, 0.9)])
def test_per_arc_counts_of_k_5_keep_a_schedule_of_their_own(citron_gpu, n, p):
    """Per-arc counts of k = 5 take arcs where whole counts take vertices: both
    from one handle in turn, also after a change of split."""
    import oracle
    g = gg.erdos_renyi(n, p * (n - 1), seed=n)
    h = citron_gpu.Graph.from_csr(g.row_ptr, g.col).order()
    want = h.count_vertex_rooted(5)
    every = h.count_arcs(5, np.arange(g.m))
    assert int(every.sum()) == want
    if n < 400:
        ptr, col = h.dag()
        src = np.repeat(np.arange(g.n), np.diff(ptr)).astype(np.int32)
        assert np.array_equal(every, oracle.count_arcs(g.n, ptr, col, 5, src, col)[0])
    for split in (100, 50, 100):
        h.set_tuning(split_pct=split)
        for _ in range(2):
            assert h.count(5) == want
            total, per = h.count_per_arc(5)
            assert total == want and np.array_equal(per, every)
    assert h.count_per_arc(4)[0] == h.count(4)
    assert citron_gpu.count_batch([h], [5]) == [want]
    h.free()


@pytest.mark.parametrize("k", [8, 9, 11])
def test_light_vertices_of_deep_and_shallow_subgraphs(citron_gpu, k):
    """k >= 9 splits light vertices further from the triangles of K_24 on: out-
    degrees around 24 and 64, complete subgraphs beside sparse ones of the same
    out-degree, in whole counts, shares, batches and per arc."""
    from math import comb
    sizes = [23, 24, 25, 26, 40, 64, 65, 66]
    cl = gg.disjoint_cliques(sizes)
    er = gg.erdos_renyi(400, 90, seed=k)
    ptr = np.concatenate([cl.row_ptr, cl.row_ptr[-1] + er.row_ptr[1:]]).astype(np.int32)
    g = gg.CSR(cl.n + er.n, ptr, np.concatenate([cl.col, er.col + cl.n]).astype(np.int32), "mixed")
    h = citron_gpu.Graph.from_csr(g.row_ptr, g.col).order()
    sparse = citron_gpu.Graph.from_csr(er.row_ptr, er.col).order()
    want = sum(comb(s, k) for s in sizes) + sparse.count_vertex_rooted(k)
    assert h.count(k) == want
    assert h.count_vertex_rooted(k) == want
    assert sum(h.count_part(k, i, 5)[0] for i in range(5)) == want
    total, per = h.count_per_arc(k)
    assert total == want and int(per.sum()) == want
    assert citron_gpu.count_batch([h, sparse, h], [k, k, 9]) == [want, sparse.count(k), h.count(9)]
    assert sparse.count(k) == sparse.count_vertex_rooted(k)
    for x in (h, sparse):
        x.free()


@pytest.mark.parametrize("k", [6, 7, 8, 9, 10])
def test_heavy_arcs_of_every_density_class(citron_gpu, k):
    """One graph of heavy vertices of four densities: from k = 7 on the dense
    kernel takes the arcs of the denser ones only, the count kernel the rest."""
    sizes = ((620, 0.2), (260, 0.55), (180, 0.8)) if k < 9 else ((620, 0.2), (220, 0.5), (110, 0.8))
    parts = [gg.erdos_renyi(n, p * (n - 1), seed=n) for n, p in sizes] + [gg.complete(84 if k < 9 else 70)]
    n = 0
    ptr, col = [np.zeros(1, np.int64)], []
    for g in parts:
        ptr.append(g.row_ptr[1:] + ptr[-1][-1])
        col.append(g.col + n)
        n += g.n
    g = gg.CSR(n, np.concatenate(ptr).astype(np.int32), np.concatenate(col).astype(np.int32), "classes")
    h = citron_gpu.Graph.from_csr(g.row_ptr, g.col).order()
    want = 0
    for p in parts:
        one = citron_gpu.Graph.from_csr(p.row_ptr, p.col).order()
        want += one.count_vertex_rooted(k)
        one.free()
    assert h.count(k) == want
    assert sum(h.count_part(k, i, 3)[0] for i in range(3)) == want
    total, per = h.count_per_arc(k)
    assert total == want and int(per.sum()) == want
    some = np.random.default_rng(k).choice(g.m, 300, replace=False)
    assert np.array_equal(h.count_arcs(k, some), per[some])
    assert citron_gpu.count_batch([h, h], [k, 5]) == [want, h.count(5)]
    h.free()


def test_released_memory_returns_to_the_device(citron_gpu):
    """What freed graphs leave in the pool is the program's again on request,
    and graphs in use stay as they are."""
    import torch
    keep = citron_gpu.Graph.from_csr(*(lambda g: (g.row_ptr, g.col))(gg.rmat(9, 16, seed=5))).order()
    want = keep.count(5)
    citron_gpu.release_memory()
    before = torch.cuda.mem_get_info()[0]
    g = gg.rmat(16, 16, seed=6)
    h = citron_gpu.Graph.from_csr(g.row_ptr, g.col).order()
    h.count(4)
    h.free()
    held = before - torch.cuda.mem_get_info()[0]
    citron_gpu.release_memory()
    left = before - torch.cuda.mem_get_info()[0]
    assert held > 16 << 20 and left < held // 4
    assert keep.count(5) == want and keep.count(6) == keep.count_vertex_rooted(6)
    keep.free()


def test_memory_that_only_scheduled_counts_need_is_theirs(citron_gpu):
    """Triangle counts, vertex-rooted counts and listing hold the subgraph rows
    once; a scheduled count brings the heavy vertices' sorted rows, once."""
    g = gg.rmat(13, 24, seed=13)
    h = citron_gpu.Graph.from_csr(g.row_ptr, g.col).order()
    tri = h.count(3)
    built = h.info()["device_bytes"]
    assert int(h.count_per_arc(3)[1].sum()) == tri and h.count_vertex_rooted(3) == tri
    some = np.arange(0, g.m, 97)
    assert h.list_arcs(3, some)[0].shape[0] == int(h.count_arcs(3, some).sum())
    assert h.info()["device_bytes"] - built < 16 << 20          # stacks and tables
    four = h.count_vertex_rooted(4)
    every = h.count_arcs(4, np.arange(g.m))
    assert int(every.sum()) == four
    before = h.info()["device_bytes"]
    assert h.count(4) == four
    sorted_rows = h.info()["device_bytes"] - before
    assert sorted_rows > 8 * g.m                                  # rows, positions, arcs by size
    assert h.count(5) == h.count_vertex_rooted(5) and h.count(4) == four
    assert h.info()["device_bytes"] - before - sorted_rows < 16 << 20
    assert np.array_equal(h.count_per_arc(4)[1], every)
    h.free()


def test_threads_and_streams_all_finish_with_the_oracles_results(citron_gpu):
    """As test_blocks_reused_across_threads_and_streams, with every thread's
    errors reported, its passes counted, and order keys and DAGs compared: a
    block handed on too early shows as any of these."""
    from concurrent.futures import ThreadPoolExecutor
    from math import comb
    import oracle
    import torch
    gs = [gg.rmat(9, 20, seed=80), gg.rmat(10, 14, seed=81), gg.erdos_renyi(700, 26, seed=82), gg.complete(80), gg.empty(500)]
    want = {(i, k): comb(80, k) if i == 3 else oracle.count(g, k)[0] for i, g in enumerate(gs) for k in (3, 4, 6)}
    dags = {(i, o): (oracle.orient(g.n, g.row_ptr, g.col) if o == "degree" else oracle.orient_peel(g))
            for i, g in enumerate(gs) for o in ("degree", "core")}

    def work(seed):
        rng = np.random.default_rng(seed)
        with torch.cuda.stream(torch.cuda.Stream()):
            for done in range(25):
                i, k = int(rng.integers(len(gs))), int(rng.choice([3, 4, 6]))
                ordering = "core" if rng.random() < 0.3 else "degree"
                h = citron_gpu.Graph.from_csr(gs[i].row_ptr, gs[i].col).order(ordering)
                ptr, col = h.dag()
                assert np.array_equal(ptr, dags[(i, ordering)][0]) and np.array_equal(col, dags[(i, ordering)][1])
                assert h.count(k) == want[(i, k)], (i, k, ordering)
                if rng.random() < 0.3:
                    assert citron_gpu.count_batch([h, h], [4, k]) == [want[(i, 4)], want[(i, k)]]
                h.free()
        return done + 1

    with ThreadPoolExecutor(4) as pool:
        assert list(pool.map(work, range(4))) == [25] * 4
