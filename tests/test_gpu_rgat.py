"""GPU parity of the attention aggregation (R-GAT) against the fp64 oracle of oracle/rgat.py.

Tolerances: `max_j |got_ij - ref_ij| <= tol * max(1, max_j |ref_ij|)` per row, tol = 1e-4 wherever both
sides read identical inputs (fp32 accumulation of fp32 or bf16-exact values), 2e-2 for the bf16-storage
layer.  In that mode Z_r = H0_s W_r is stored as bf16 for the weighted sums, but the attention logits are
taken from the input tables (el = <H0_s, W_r a_r> in fp32), so a sharp softmax does not amplify the storage
rounding; embeddings and every gradient are compared with the plain fp64 oracle.  The largest observed scaled
error is printed per family.  The ReLU decision is kept away from its kink as in
the other layer tests: the upstream gradient is zeroed where the oracle's embedding is within the forward
tolerance of zero.
"""
import numpy as np
import pytest
import torch

import paper_2408_09697_amd as heta
from gen import rng, workloads
from gen.graphs import HetGraph, NodeType, power_law_relation, reverse_relation, uniform_relation
from oracle import rgat
from tests.harness import assert_rows_close, dev_table, kink_guard, make_graph, row_err

pytestmark = pytest.mark.gpu


def up(x):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32)).cuda()


def host(x):
    return x.float().cpu().numpy()


# ---- scores -------------------------------------------------------------------------------------------

@pytest.mark.parametrize("n,d,heads,pad", [(1000, 256, 4, 4), (333, 64, 1, 4), (50, 30, 3, 1), (100, 1024, 8, 4),
                                           (77, 7, 1, 1), (0, 64, 2, 4), (4100, 128, 16, 4)])
@pytest.mark.parametrize("per_head", [True, False])
@pytest.mark.parametrize("storage", ["f32", "bf16"])
def test_attn_score_and_its_backward(n, d, heads, pad, per_head, storage):
    g = rng.stream("tests", f"score{n}x{d}x{heads}{per_head}")
    x = g.standard_normal((n, d)).astype(np.float32)
    if storage == "bf16":
        x = rng.round_to_bf16(x)
    F = d // heads
    vec = g.standard_normal((heads, F if per_head else d)).astype(np.float32)
    xd = dev_table(x, storage, (8 if storage == "bf16" else 4) if pad > 1 else 1)
    score = torch.empty((n, heads), dtype=torch.float32, device="cuda")
    heta.heta_attn_score(xd, up(vec), per_head, score)
    x64 = x.astype(np.float64)
    if per_head:
        ref = np.einsum("nkf,kf->nk", x64.reshape(n, heads, F), vec.astype(np.float64))
    else:
        ref = x64 @ vec.astype(np.float64).T
    assert_rows_close(host(score), ref, 1e-4, "score")
    # backward
    ds = g.standard_normal((n, heads)).astype(np.float32)
    dx0 = g.standard_normal((n, d)).astype(np.float32)
    graph = heta.heta_graph_create([(4, 4, 0)], [(0, 0, np.zeros(5, dtype=np.int64), np.zeros(0, dtype=np.int32))])
    for beta in (0.0, 1.0):
        dx = dev_table(dx0, "f32", 4 if pad > 1 else 1)
        dvec = torch.full(vec.shape, 7.0, dtype=torch.float32, device="cuda")
        heta.heta_attn_score_bwd(graph, xd, up(vec), per_head, up(ds), dx=dx, beta=beta, dvec=dvec)
        if per_head:
            rdx = (ds.astype(np.float64)[:, :, None] * vec.astype(np.float64)[None]).reshape(n, d)
            rdv = np.einsum("nk,nkf->kf", ds.astype(np.float64), x64.reshape(n, heads, F))
        else:
            rdx = ds.astype(np.float64) @ vec.astype(np.float64)
            rdv = ds.astype(np.float64).T @ x64
        assert_rows_close(host(dx), rdx + beta * dx0, 1e-4, "dx")
        assert_rows_close(host(dvec), rdv, 1e-4, "dvec")
    graph.destroy()


def test_attn_score_of_more_rows_than_a_grid_has_wavefronts():
    """Six columns go row by row, a wavefront each: 2^26 rows and some are more than 2^32 threads."""
    n = 67_200_000
    x, vec = torch.randn((n, 6), device="cuda"), torch.randn((1, 6), device="cuda")
    score = torch.full((n, 1), float("nan"), device="cuda")
    heta.heta_attn_score(x, vec, False, score)
    ref = (x * vec).sum(1, keepdim=True)
    assert bool(((score - ref).abs() <= 1e-5 * (x * vec).abs().sum(1, keepdim=True)).all())


@pytest.mark.parametrize("n,d,heads,n_sets", [(49_153, 128, 4, 4), (200_007, 128, 16, 5), (60_001, 100, 15, 8), (150_000, 36, 8, 7),
                                             (131_075, 20, 3, 1)])
@pytest.mark.parametrize("storage", ["f32", "bf16"])
def test_scores_of_more_rows_than_one_round_of_tiles(n, d, heads, n_sets, storage):
    """Several tiles of rows per wavefront, one or two groups of vectors, NaN in the columns past the table's width."""
    gen = torch.Generator(device="cuda").manual_seed(n + d)
    dt = torch.float32 if storage == "f32" else torch.bfloat16
    wide = torch.full((n, d + 8 if d % 8 == 0 else (d + 7) // 8 * 8), float("nan"), dtype=dt, device="cuda")
    x = wide[:, :d]
    x.copy_(torch.randn((n, d), generator=gen, device="cuda"))
    vecs = [torch.randn((heads, d), generator=gen, device="cuda") for _ in range(n_sets)]
    scores = [torch.full((n, heads), float("nan"), device="cuda") for _ in range(n_sets)]
    heta.heta_attn_score_multi(x, vecs, scores)
    # a score passes through at most 16 roundings (products and sums of eight, pairwise sums), each off by at most 2^-23
    x64 = x.double()
    for v, sc in zip(vecs, scores):
        bound = 16 * 2.0 ** -23 * (x64.abs() @ v.double().abs().T)
        assert bool(((sc.double() - x64 @ v.double().T).abs() <= bound).all())


@pytest.mark.parametrize("n,d,heads,n_sets,pad", [(3000, 128, 4, 6, 4), (1001, 128, 4, 8, 4), (700, 64, 1, 3, 4), (513, 100, 3, 5, 4),
                                                  (40, 128, 16, 2, 4), (1, 8, 2, 1, 4),
                                                  (150, 128, 8, 6, 4),
                                                  # shapes served set by set: wide table, unaligned rows, too many vectors
                                                  (300, 256, 4, 3, 4), (200, 30, 3, 2, 1), (150, 128, 16, 8, 4)])
@pytest.mark.parametrize("storage", ["f32", "bf16"])
def test_scores_of_several_vector_sets_in_one_pass(n, d, heads, n_sets, pad, storage):
    g = rng.stream("tests", f"multi_score{n}x{d}x{heads}x{n_sets}")
    x = g.standard_normal((n, d)).astype(np.float32)
    if storage == "bf16":
        x = rng.round_to_bf16(x)
    x64 = x.astype(np.float64)
    vecs = [g.standard_normal((heads, d)).astype(np.float32) for _ in range(n_sets)]
    xd = dev_table(x, storage, (8 if storage == "bf16" else 4) if pad > 1 else 1)
    scores = [torch.full((n, heads), float("nan"), dtype=torch.float32, device="cuda") for _ in range(n_sets)]
    heta.heta_attn_score_multi(xd, [up(v) for v in vecs], scores)
    for v, sc in zip(vecs, scores):
        assert_rows_close(host(sc), x64 @ v.astype(np.float64).T, 1e-4, "score")
    ds = [g.standard_normal((n, heads)).astype(np.float32) for _ in range(n_sets)]
    dx0 = g.standard_normal((n, d)).astype(np.float32)
    graph = heta.heta_graph_create([(4, 4, 0)], [(0, 0, np.zeros(5, dtype=np.int64), np.zeros(0, dtype=np.int32))])
    try:
        rdx = sum(a.astype(np.float64) @ v.astype(np.float64) for a, v in zip(ds, vecs))
        for beta in (0.0, 1.0):
            dx = dev_table(dx0, "f32", 4 if pad > 1 else 1)
            dvecs = [torch.full(v.shape, 7.0, dtype=torch.float32, device="cuda") for v in vecs]
            dvecs[-1] = None if n_sets > 1 else dvecs[-1]  # a set whose vector gradient is not wanted
            heta.heta_attn_score_bwd_multi(graph, xd, [up(v) for v in vecs], [up(a) for a in ds], dx=dx, beta=beta, dvecs=dvecs)
            assert_rows_close(host(dx), rdx + beta * dx0, 1e-4, "dx")
            for a, dv in zip(ds, dvecs):
                if dv is not None:
                    assert_rows_close(host(dv), a.astype(np.float64).T @ x64, 1e-4, "dvec")
        # run to run the same bits (slab partials are added in a fixed order)
        again = [torch.empty_like(v) if v is not None else None for v in dvecs]
        heta.heta_attn_score_bwd_multi(graph, xd, [up(v) for v in vecs], [up(a) for a in ds], dvecs=again)
        for u, w in zip(dvecs, again):
            if u is not None:
                assert torch.equal(u.view(torch.int32), w.view(torch.int32))
    finally:
        graph.destroy()


@pytest.mark.parametrize("n,d,heads,n_sets", [(33, 128, 8, 7), (129, 96, 5, 7), (4097, 128, 15, 8), (66000, 32, 2, 5), (127, 4, 1, 8),
                                              (63, 64, 1, 1), (66, 68, 1, 1), (1, 64, 2, 1), (257, 60, 16, 1), (321, 64, 9, 2), (193, 68, 9, 2),
                                              (65, 128, 16, 8),  # 128 vectors: set by set
                                              (131_143, 128, 4, 6), (131_143, 128, 8, 6)])
@pytest.mark.parametrize("storage", ["f32", "bf16"])
def test_scores_of_vector_sets_at_tile_edges(n, d, heads, n_sets, storage):
    """Row tiles of 16 and 32, vector tiles of 16 and 32, column chunks of 64 and slabs of 128 rows: remainders of each.  131,143 rows are the launches
    of large tables: slabs of 192 rows, a ragged last one, and more rows than one pass of the capped grids of the scores
    (32,768 rows with more than 16 vectors) and of the input gradient (98,304) takes."""
    test_scores_of_several_vector_sets_in_one_pass(n, d, heads, n_sets, 4, storage)


def test_vector_gradient_of_a_bf16_table_takes_no_longer_than_of_an_fp32_one():
    """Half of the bytes and the same products; with every load waited for before the next it took 146 us, fp32 116."""
    n, d, best = 700_000, 128, {}
    vec, ds, dv = (torch.randn(s, device="cuda") for s in ((1, d), (n, 1), (1, d)))
    graph = heta.heta_graph_create([(4, 4, 0)], [(0, 0, np.zeros(5, dtype=np.int64), np.zeros(0, dtype=np.int32))])
    for dtype in (torch.float32, torch.bfloat16):
        x = torch.randn((n, d), device="cuda").to(dtype)
        start, end, times = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True), []
        for _ in range(8):
            start.record()
            for _ in range(10):
                heta.heta_attn_score_bwd_multi(graph, x, [vec], [ds], dvecs=[dv])
            end.record()
            torch.cuda.synchronize()
            times.append(start.elapsed_time(end))
        best[dtype] = min(times)
    graph.destroy()
    assert best[torch.bfloat16] <= 1.1 * best[torch.float32]


# ---- one relation ---------------------------------------------------------------------------------------

def _relation_case(kind, n_src, n_dst, n_edges):
    nts = [NodeType("s", n_src, 4, False), NodeType("t", n_dst, 4, False)]
    G = HetGraph(nts)
    wl = f"tests/attn/{kind}/{n_src}/{n_dst}/{n_edges}"
    if kind == "uniform":
        G.relations.append(uniform_relation("r", 0, 1, n_src, n_dst, n_edges, wl))
    elif kind == "skew_dst":   # hubs among the destinations: the forward's long rows
        G.relations.append(power_law_relation("r", 0, 1, n_src, n_dst, n_edges, 1.5, wl))
    else:                      # hubs among the sources: the backward's long rows
        base = power_law_relation("b", 1, 0, n_dst, n_src, n_edges, 1.5, wl)
        G.relations.append(reverse_relation("r", base, n_dst))
    return G


@pytest.mark.parametrize("kind,n_src,n_dst,n_edges", [("uniform", 700, 900, 6000), ("skew_dst", 2000, 3000, 60000),
                                                       ("skew_src", 2500, 1800, 50000), ("uniform", 5, 6, 0)])
@pytest.mark.parametrize("d,heads", [(64, 4), (256, 1), (24, 4), (520, 2), (128, 16), (48, 3)])
@pytest.mark.parametrize("storage", ["f32", "bf16"])
@pytest.mark.parametrize("saved_pos", [True, False])
def test_rel_attn_forward_and_backward(kind, n_src, n_dst, n_edges, d, heads, storage, saved_pos):
    G = _relation_case(kind, n_src, n_dst, n_edges)
    r = G.relations[0]
    src, dst = r.edge_list()
    if kind != "uniform":
        deg_d = np.bincount(dst, minlength=n_dst)
        deg_s = np.bincount(src, minlength=n_src)
        assert max(deg_d.max(), deg_s.max()) >= 512, "the case is meant to contain a hub row"
    g = rng.stream("tests", f"attn{kind}{d}x{heads}")
    z = g.standard_normal((n_src, d)).astype(np.float32)
    if storage == "bf16":
        z = rng.round_to_bf16(z)
    el = (2.0 * g.standard_normal((n_src, heads))).astype(np.float32)
    er = (2.0 * g.standard_normal((n_dst, heads))).astype(np.float32)
    go = g.standard_normal((n_dst, d)).astype(np.float32)
    slope = 0.2
    graph = heta.heta_graph_create([(n_src, 4, 0), (n_dst, 4, 0)], [(0, 1, r.rowptr, r.col)])
    pad = 8 if storage == "bf16" else 4
    zd = dev_table(z, storage, pad if d % 4 == 0 else 1)
    out = dev_table(np.full((n_dst, d), 3.0, dtype=np.float32), "f32", 4 if d % 4 == 0 else 1)
    smax = torch.empty((n_dst, heads), dtype=torch.float32, device="cuda")
    sinv = torch.empty_like(smax)
    # out_pos: the sum over the edges with a positive logit, which lets the backward skip one gather
    out_pos = dev_table(np.full((n_dst, d), 3.0, dtype=np.float32), "f32", 4 if d % 4 == 0 else 1) if saved_pos else None
    heta.heta_rel_attn_fwd(graph, 0, zd, up(el), up(er), slope, out, beta=0.0, smax=smax, sinv=sinv, out_pos=out_pos)
    ref_o, alpha = rgat.gat_aggregate_fwd(src, dst, n_dst, z, el, er, slope)
    assert_rows_close(host(out), ref_o, 1e-4, "out")
    if saved_pos:
        pos = (el.astype(np.float32)[src] + er.astype(np.float32)[dst]) > 0
        ref_pos = np.zeros((n_dst, heads, d // heads))
        np.add.at(ref_pos, dst, (alpha * pos)[:, :, None] * z.astype(np.float64)[src].reshape(-1, heads, d // heads))
        assert_rows_close(host(out_pos), ref_pos.reshape(n_dst, d), 1e-4, "out_pos")
    # accumulate on top (beta = 1) without the saved statistics
    out2 = out.clone()
    heta.heta_rel_attn_fwd(graph, 0, zd, up(el), up(er), slope, out2, beta=1.0)
    assert_rows_close(host(out2), 2.0 * ref_o, 1e-4, "out, beta = 1")
    dz = dev_table(np.full((n_src, d), 5.0, dtype=np.float32), "f32", 4 if d % 4 == 0 else 1)
    d_el = torch.full((n_src, heads), 5.0, dtype=torch.float32, device="cuda")
    d_er = torch.full((n_dst, heads), 5.0, dtype=torch.float32, device="cuda")
    heta.heta_rel_attn_bwd(graph, 0, zd, up(el), up(er), slope, smax, sinv, out, up(go), dz, d_el, d_er, o_pos=out_pos)
    torch.cuda.synchronize()
    rdz, rdel, rder = rgat.gat_aggregate_bwd(src, dst, n_src, n_dst, z, el, er, alpha, go, slope)
    assert_rows_close(host(dz), rdz, 1e-4, "dz")
    assert_rows_close(host(d_el), rdel, 1e-4, "del")
    assert_rows_close(host(d_er), rder, 1e-4, "der")
    graph.destroy()


ROW_CLASS_DEGREES = [0, 1, 3, 4, 5, 8, 9, 31, 32, 33, 64, 65, 511, 512, 513, 768, 769, 1100] + [4, 5, 0, 31, 32] * 9


@pytest.mark.parametrize("heads", [1, 2, 3, 4, 8, 16])
@pytest.mark.parametrize("side", ["dst", "src"])
def test_sweeps_at_the_edges_of_the_row_classes(heads, side):
    """Rows of 4 / 5, 31 / 32 and 511 / 512 edges change the kernel that sweeps them, 256 the hub chunk; the
    forward sweeps the destinations' rows, the backward also the sources'."""
    deg = np.array(ROW_CLASS_DEGREES)
    n_many, n_other = deg.size, 300
    g = rng.stream("tests", f"row_classes{heads}{side}")
    many = np.repeat(np.arange(n_many), deg)
    other = g.integers(0, n_other, many.size)
    dst, src = (many, other) if side == "dst" else (other, many)
    n_dst, n_src = (n_many, n_other) if side == "dst" else (n_other, n_many)
    order = np.argsort(dst, kind="stable")
    src, dst = src[order], dst[order]
    rowptr = np.concatenate([[0], np.cumsum(np.bincount(dst, minlength=n_dst))]).astype(np.int64)
    d = 8 * heads
    z, go = g.standard_normal((n_src, d)).astype(np.float32), g.standard_normal((n_dst, d)).astype(np.float32)
    el, er = (2.0 * g.standard_normal((n_src, heads))).astype(np.float32), (2.0 * g.standard_normal((n_dst, heads))).astype(np.float32)
    graph = heta.heta_graph_create([(n_src, 4, 0), (n_dst, 4, 0)], [(0, 1, rowptr, src.astype(np.int32))])
    try:
        out, pos = (torch.full((n_dst, d), 3.0, device="cuda") for _ in range(2))
        smax, sinv, d_er = (torch.full((n_dst, heads), 5.0, device="cuda") for _ in range(3))
        dz, d_el = torch.full((n_src, d), 5.0, device="cuda"), torch.full((n_src, heads), 5.0, device="cuda")
        heta.heta_rel_attn_fwd(graph, 0, up(z), up(el), up(er), 0.2, out, smax=smax, sinv=sinv, out_pos=pos)
        heta.heta_rel_attn_bwd(graph, 0, up(z), up(el), up(er), 0.2, smax, sinv, out, up(go), dz, d_el, d_er, o_pos=pos)
        ref_o, alpha = rgat.gat_aggregate_fwd(src, dst, n_dst, z, el, er, 0.2)
        rdz, rdel, rder = rgat.gat_aggregate_bwd(src, dst, n_src, n_dst, z, el, er, alpha, go, 0.2)
        for got, ref, what in ((out, ref_o, "out"), (dz, rdz, "dz"), (d_el, rdel, "del"), (d_er, rder, "der")):
            assert_rows_close(host(got), ref, 1e-4, what)
        # the form without a sweep over the destinations' edges
        apos, pack = torch.full((n_dst, heads), 5.0, device="cuda"), torch.full((n_dst, 4 * heads), 5.0, device="cuda")
        heta.heta_rel_attn_fwd_train(graph, 0, up(z), up(el), up(er), 0.2, out, smax=smax, sinv=sinv, out_pos=pos, apos=apos)
        ref_apos = np.zeros((n_dst, heads))
        np.add.at(ref_apos, dst, alpha * ((el[src] + er[dst]) > 0))
        assert_rows_close(host(apos), ref_apos, 1e-4, "apos")
        for t in (d_er, dz, d_el):
            t.fill_(5.0)
        heta.heta_attn_bwd_dst(graph, 1, [0], 0.2, heta.HETA_ACT_NONE, None, up(go), None, [out], [pos], [up(er)], [smax], [sinv], [apos],
                               [d_er], [pack])
        heta.heta_rel_attn_bwd_src(graph, 0, up(z), up(el), 0.2, pack, up(go), dz, d_el)
        for got, ref, what in ((dz, rdz, "dz"), (d_el, rdel, "del"), (d_er, rder, "der")):
            assert_rows_close(host(got), ref, 1e-4, what)
    finally:
        graph.destroy()


@pytest.mark.parametrize("heads", [1, 2, 4, 8, 16])
@pytest.mark.parametrize("degrees", [[63, 64, 65, 127, 128, 129, 255, 256, 257, 510], [1] * 200 + [0] * 100, [2, 1] * 150])
def test_forward_at_the_edges_of_the_slots_per_lane(heads, degrees):
    """Rows of one wavefront take 1, 2, 4 or 8 slots per lane, wavefronts of single rows per thread 1 or 4."""
    deg = np.array(degrees)
    n_dst, n_src, d = deg.size, 300, 8 * heads
    g = rng.stream("tests", f"slots{heads}x{deg.max()}")
    dst, src = np.repeat(np.arange(n_dst), deg), g.integers(0, n_src, deg.sum())
    z = g.standard_normal((n_src, d)).astype(np.float32)
    el, er = ((2.0 * g.standard_normal((n, heads))).astype(np.float32) for n in (n_src, n_dst))
    graph = heta.heta_graph_create([(n_src, 4, 0), (n_dst, 4, 0)], [(0, 1, np.concatenate([[0], np.cumsum(deg)]).astype(np.int64), src.astype(np.int32))])
    try:
        out, pos = (torch.full((n_dst, d), 3.0, device="cuda") for _ in range(2))
        smax, sinv, apos = (torch.full((n_dst, heads), 5.0, device="cuda") for _ in range(3))
        heta.heta_rel_attn_fwd_train(graph, 0, up(z), up(el), up(er), 0.2, out, smax=smax, sinv=sinv, out_pos=pos, apos=apos)
        ref_o, alpha = rgat.gat_aggregate_fwd(src, dst, n_dst, z, el, er, 0.2)
        gate = alpha * ((el[src] + er[dst]) > 0)
        ref_apos, ref_pos = np.zeros((n_dst, heads)), np.zeros((n_dst, heads, 8))
        np.add.at(ref_apos, dst, gate)
        np.add.at(ref_pos, dst, gate[:, :, None] * z.astype(np.float64)[src].reshape(-1, heads, 8))
        for got, ref, what in ((out, ref_o, "out"), (pos, ref_pos.reshape(n_dst, d), "out_pos"), (apos, ref_apos, "apos")):
            assert_rows_close(host(got), ref, 1e-4, what)
    finally:
        graph.destroy()


def test_forward_of_short_wavefront_rows_costs_about_what_its_edges_do():
    """Rows of 40 edges do not pay for the slots of rows of 511: 1.9 times the time of as many edges in rows of 300 when
    they did, 1.3 times without."""
    heads, d, best = 8, 64, {}
    z, el = torch.randn((50_000, d), device="cuda"), torch.randn((50_000, heads), device="cuda")
    for rows, degree in ((20_000, 40), (2_667, 300)):
        col = rng.stream("tests", f"short_rows{degree}").integers(0, 50_000, rows * degree).astype(np.int32)
        graph = heta.heta_graph_create([(50_000, 4, 0), (rows, 4, 0)], [(0, 1, np.arange(rows + 1, dtype=np.int64) * degree, col)])
        er, out = torch.randn((rows, heads), device="cuda"), torch.empty((rows, d), device="cuda")
        start, end, times = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True), []
        for _ in range(8):
            start.record()
            for _ in range(20):
                heta.heta_rel_attn_fwd(graph, 0, z, el, er, 0.2, out)
            end.record()
            torch.cuda.synchronize()
            times.append(start.elapsed_time(end))
        best[degree] = min(times)
        graph.destroy()
    assert best[40] <= 1.6 * best[300]


@pytest.mark.parametrize("heads", [1, 2, 4, 8])
@pytest.mark.parametrize("slope", [-0.5, 0.0, 1.0])
def test_positive_logits_are_those_before_the_activation(heads, slope):
    """With a slope that is not positive the activated logit does not carry the sign any more: out_pos, apos and der of
    every row class, hub rows included, by the logit itself."""
    deg = np.array(ROW_CLASS_DEGREES)
    n_dst, n_src, d = deg.size, 300, 8 * heads
    g = rng.stream("tests", f"logit_sign{heads}{slope}")
    dst, src = np.repeat(np.arange(n_dst), deg), g.integers(0, n_src, deg.sum())
    src[np.unique(dst, return_index=True)[1]] = 0  # every row with edges has one of source 0
    z, go = g.standard_normal((n_src, d)).astype(np.float32), g.standard_normal((n_dst, d)).astype(np.float32)
    el, er = (g.standard_normal((n, heads)).astype(np.float32) for n in (n_src, n_dst))
    graph = heta.heta_graph_create([(n_src, 4, 0), (n_dst, 4, 0)], [(0, 1, np.concatenate([[0], np.cumsum(deg)]).astype(np.int64), src.astype(np.int32))])
    try:
        out, pos = (torch.full((n_dst, d), 3.0, device="cuda") for _ in range(2))
        smax, sinv, apos, d_er = (torch.full((n_dst, heads), 5.0, device="cuda") for _ in range(4))
        dz, d_el, pack = torch.empty((n_src, d), device="cuda"), torch.empty((n_src, heads), device="cuda"), torch.empty((n_dst, 4 * heads), device="cuda")
        heta.heta_rel_attn_fwd_train(graph, 0, up(z), up(el), up(er), slope, out, smax=smax, sinv=sinv, out_pos=pos, apos=apos)
        heta.heta_attn_bwd_dst(graph, 1, [0], slope, heta.HETA_ACT_NONE, None, up(go), None, [out], [pos], [up(er)], [smax], [sinv], [apos],
                               [d_er], [pack])
        heta.heta_rel_attn_bwd_src(graph, 0, up(z), up(el), slope, pack, up(go), dz, d_el)
        ref_o, alpha = rgat.gat_aggregate_fwd(src, dst, n_dst, z, el, er, slope)
        rdz, rdel, rder = rgat.gat_aggregate_bwd(src, dst, n_src, n_dst, z, el, er, alpha, go, slope)
        gate = alpha * ((el[src] + er[dst]) > 0)
        ref_apos, ref_pos = np.zeros((n_dst, heads)), np.zeros((n_dst, heads, d // heads))
        np.add.at(ref_apos, dst, gate)
        np.add.at(ref_pos, dst, gate[:, :, None] * z.astype(np.float64)[src].reshape(-1, heads, d // heads))
        for got, ref, what in ((out, ref_o, "out"), (pos, ref_pos.reshape(n_dst, d), "out_pos"), (apos, ref_apos, "apos"), (dz, rdz, "dz"),
                               (d_el, rdel, "del"), (d_er, rder, "der")):
            assert_rows_close(host(got), ref, 1e-4, what)
        # an infinite positive logit makes the row's weights NaN, those of its positive logits too
        el[0] = np.inf
        heta.heta_rel_attn_fwd_train(graph, 0, up(z), up(el), up(er), slope, out, smax=smax, sinv=sinv, out_pos=pos, apos=apos)
        for t in (out, pos, apos):
            assert np.isnan(host(t)[deg > 0]).all()
    finally:
        graph.destroy()


@pytest.mark.parametrize("n,d,heads,n_rels,pad", [(1000, 256, 4, 3, 4), (257, 64, 8, 1, 4), (130, 60, 3, 2, 4), (67, 100, 5, 8, 4), (5, 4, 1, 2, 4),
                                                  # two rows per lane group (from n x lanes = 2^20 on), the last workgroup not full
                                                  (16389, 256, 4, 2, 4), (16389, 512, 8, 1, 4),
                                                  # two and four chunks per lane: heads inside a step of 64 chunks, of one and of several steps
                                                  (33, 320, 5, 1, 4), (50, 512, 8, 2, 4), (33, 512, 1, 2, 4), (21, 768, 12, 1, 4), (21, 1024, 4, 3, 4),
                                                  (18, 1024, 2, 1, 4), (9, 1024, 1, 1, 4),
                                                  # served row by row, 16 bytes a load: long rows with heads of 20, 25, 65 and 96 chunks, more than 256 chunks
                                                  (33, 320, 4, 2, 4), (50, 600, 6, 2, 4), (19, 260, 1, 1, 4), (19, 768, 2, 1, 4), (7, 2048, 16, 1, 4),
                                                  # row by row, element by element: heads of 6 and 15 columns, unaligned rows
                                                  (50, 18, 3, 2, 4), (40, 30, 2, 1, 1), (40, 512, 4, 1, 1)])
@pytest.mark.parametrize("relu", [True, False])
def test_destination_side_of_the_backward(n, d, heads, n_rels, pad, relu):
    g = rng.stream("tests", f"dst_side{n}x{d}x{heads}x{n_rels}")
    go, h = (g.standard_normal((n, d)).astype(np.float32) for _ in range(2))
    o, u = ([g.standard_normal((n, d)).astype(np.float32) for _ in range(n_rels)] for _ in range(2))
    er, smax, sinv, apos = ([g.standard_normal((n, heads)).astype(np.float32) for _ in range(n_rels)] for _ in range(4))
    graph = heta.heta_graph_create([(3, 4, 0), (n, 4, 0)], [(0, 1, np.zeros(n + 1, dtype=np.int64), np.zeros(0, dtype=np.int32))] * n_rels)
    try:
        tab = lambda x: dev_table(x, "f32", pad) if pad > 1 else dev_table(np.pad(x, ((0, 0), (0, 1))), "f32", 1)[:, :d]  # noqa: E731
        god, gi = tab(go), tab(np.full((n, d), 7.0, dtype=np.float32))
        der, pack = [torch.full((n, heads), 5.0, device="cuda") for _ in o], [torch.full((n, 4 * heads), 5.0, device="cuda") for _ in o]
        got = heta.heta_attn_bwd_dst(graph, 1, list(range(n_rels)), 0.2, heta.HETA_ACT_RELU if relu else heta.HETA_ACT_NONE, tab(h) if relu else None,
                                     god, gi if relu else None, [tab(x) for x in o], [tab(x) for x in u], [up(x) for x in er],
                                     [up(x) for x in smax], [up(x) for x in sinv], [up(x) for x in apos], der, pack)
        ref = np.where(h > 0, go, 0.0).astype(np.float32) if relu else go
        assert got is (gi if relu else god) and np.array_equal(host(got), ref)
        dots = lambda x: (ref.astype(np.float64) * x).reshape(n, heads, -1).sum(2)  # noqa: E731
        for j in range(n_rels):
            dot = dots(o[j])
            assert_rows_close(host(der[j]), 0.8 * (dots(u[j]) - apos[j] * dot), 1e-4, "der")
            assert_rows_close(host(pack[j]), np.stack([er[j], smax[j], sinv[j], dot], axis=2).reshape(n, 4 * heads), 1e-4, "pack")
    finally:
        graph.destroy()


@pytest.mark.parametrize("d,heads", [(64, 8), (256, 4), (30, 3), (256, 1)])
@pytest.mark.parametrize("storage", ["f32", "bf16"])
def test_attention_of_several_relations_in_one_call(d, heads, storage):
    """Ten relations (more than a sweep launch or a gather launch takes), one of them empty, with hub, long and short rows:
    bitwise what one call per relation gives, forward and source side of the backward."""
    gen = torch.Generator().manual_seed(d + heads)
    n_src, n_dst, graph_rels = 300, 400, []
    for r in range(10):
        deg = torch.randint(0, 6, (n_dst,), generator=gen)
        if r % 3 == 0:
            deg[7], deg[8], deg[9] = 1300, 512, 40
        if r == 4:
            deg.zero_()
        rowptr = torch.cat([deg.new_zeros(1), torch.cumsum(deg, 0)])
        graph_rels.append((0, 1, rowptr.numpy(), torch.randint(0, n_src, (int(rowptr[-1]),), generator=gen, dtype=torch.int32).numpy()))
    hg = heta.heta_graph_create([(n_src, 4, 0), (n_dst, 4, 0)], graph_rels)
    dt = torch.float32 if storage == "f32" else torch.bfloat16
    rels = list(range(10))

    def rand(n, w, dtype=torch.float32):
        return [torch.randn((n, w), generator=gen).to(dtype).cuda() for _ in rels]

    def buffers(n, w):
        return [[torch.full((n, w), 7.0, device="cuda") for _ in rels] for _ in range(2)]

    try:
        z, el, er, grad = rand(n_src, d, dt), rand(n_src, heads), rand(n_dst, heads), rand(n_dst, d)
        out, pos, smax, sinv, apos = (buffers(n_dst, w) for w in (d, d, heads, heads, heads))
        dz, del_ = buffers(n_src, d), buffers(n_src, heads)
        for r in rels:
            heta.heta_rel_attn_fwd_train(hg, r, z[r], el[r], er[r], 0.2, out[0][r], smax=smax[0][r], sinv=sinv[0][r], out_pos=pos[0][r], apos=apos[0][r])
        heta.heta_rel_attn_fwd_train_multi(hg, rels, z, el, er, 0.2, out[1], smax[1], sinv[1], pos[1], apos[1])
        pack = [torch.stack([er[r], smax[0][r], sinv[0][r], torch.randn((n_dst, heads), generator=gen).cuda()], 2).reshape(n_dst, 4 * heads).contiguous()
                for r in rels]
        for r in rels:
            heta.heta_rel_attn_bwd_src(hg, r, z[r], el[r], 0.2, pack[r], grad[r], dz[0][r], del_[0][r])
        heta.heta_rel_attn_bwd_src_multi(hg, rels, z, el, 0.2, pack, grad, dz[1], del_[1])
        torch.cuda.synchronize()
        for one, all_ in (out, pos, smax, sinv, apos, dz, del_):
            for r in rels:
                assert torch.equal(one[r].view(torch.int32), all_[r].view(torch.int32)), r
        with pytest.raises(heta.HetaError, match="overlap"):
            heta.heta_rel_attn_bwd_src_multi(hg, [0, 1], z[:2], el[:2], 0.2, pack[:2], grad[:2], [dz[0][0], dz[0][0]], del_[0][:2])
        with pytest.raises(heta.HetaError, match="overlap"):
            heta.heta_rel_attn_fwd_train_multi(hg, [0, 1], z[:2], el[:2], er[:2], 0.2, out[0][:2], smax[0][:2], sinv[0][:2],
                                               [pos[0][0], out[0][0]], apos[0][:2])
    finally:
        hg.destroy()


@pytest.mark.parametrize("d,storage,train", [(256, "f32", False), (256, "f32", True), (200, "f32", True), (512, "bf16", False), (512, "bf16", True),
                                             (384, "f32", False), (384, "f32", True), (768, "bf16", True)])
def test_edges_of_a_long_row_are_added_in_order(d, storage, train):
    """Long rows have one lane group of up to 64 lanes: 64 edges of one weight (2^-6 exactly, since all scores are equal) are
    added one after the other, whether one sum or two are taken."""
    gen = torch.Generator().manual_seed(d)
    n_src, n_dst, heads = 300, 5, 4
    col = torch.randint(0, n_src, (64 * n_dst,), generator=gen, dtype=torch.int32)
    hg = heta.heta_graph_create([(n_src, 4, 0), (n_dst, 4, 0)], [(0, 1, np.arange(n_dst + 1, dtype=np.int64) * 64, col.numpy())])
    try:
        z = torch.randn((n_src, d), generator=gen).to(torch.float32 if storage == "f32" else torch.bfloat16)
        el, er = torch.ones((n_src, heads), device="cuda"), torch.ones((n_dst, heads), device="cuda")
        out, pos = torch.full((n_dst, d), 7.0, device="cuda"), torch.full((n_dst, d), 7.0, device="cuda")
        heta.heta_rel_attn_fwd(hg, 0, z.cuda(), el, er, 0.2, out, out_pos=pos if train else None)
        want = torch.zeros((n_dst, d))
        for e in range(64):
            want += z.float()[col.view(n_dst, 64)[:, e].long()] * 2.0 ** -6
        assert torch.equal(out.cpu(), want)
        assert not train or torch.equal(pos.cpu(), want)  # every logit is positive
    finally:
        hg.destroy()


@pytest.mark.parametrize("d_in,heads,F", [(128, 4, 64), (70, 3, 20), (1, 1, 5), (33, 2, 16), (768, 8, 33)])
@pytest.mark.parametrize("storage", ["f32", "bf16"])
def test_folded_score_vector_is_summed_in_order(d_in, heads, F, storage):
    """wa[k, j] = sum_f W[j, k F + f] a[k, f], f = 0, 1, ...: factors of 12 bits make the products exact, and every sum of two
    fp32 values of these sizes is exact in 64 bits, so each step rounds once, as the fused multiply-add does."""
    gen = torch.Generator().manual_seed(F)

    def factors(shape, bits):
        return torch.randint(1 << (bits - 1), 1 << bits, shape, generator=gen) * torch.randint(0, 2, shape, generator=gen).mul(2).sub(1) / float(1 << bits)

    W, a = factors((d_in, heads * F), 12 if storage == "f32" else 8), factors((heads, F), 12)
    W = W.to(torch.float32 if storage == "f32" else torch.bfloat16)
    wa = torch.full((heads, d_in), 7.0, device="cuda")
    heta.heta_attn_fold(W.cuda(), a.float().cuda(), wa)
    want = torch.zeros((heads, d_in), dtype=torch.float64)
    for f in range(F):
        want = (want + W.double().view(d_in, heads, F)[:, :, f].T * a.double()[:, f:f + 1]).float().double()
    assert torch.equal(wa.cpu(), want.float())


@pytest.mark.parametrize("heads,pad", [(4, 4), (3, 4), (2, 1)])
@pytest.mark.parametrize("storage", ["f32", "bf16"])
def test_calls_over_several_types_equal_their_single_calls(heads, pad, storage):
    """Workgroups laid end to end: rows at the edges of a workgroup's share and of a launch's number of types, 1 to 8 sets,
    tables of every kernel (and of none); every output has the bits of the call of its own."""
    g = rng.stream("tests", f"types{heads}x{pad}{storage}")
    rows = [1, 129, 4097, 31, 0, 700, 64, 257, 2, 65]
    cols = [128, 64, 32, 100, 128, 30, 128, 60, 768, 16]
    sets = [7, 1, 3, 2, 2, 1, 5, 8, 1, 4]
    graph = heta.heta_graph_create([(n, 4, 0) for n in rows], [(t, t, np.zeros(n + 1, dtype=np.int64), np.zeros(0, dtype=np.int32))
                                                               for t, n in enumerate(rows)])
    rand = lambda *shape: g.standard_normal(shape).astype(np.float32)  # noqa: E731
    new = lambda *shape: torch.full(shape, 7.0, dtype=torch.float32, device="cuda")  # noqa: E731
    mats = lambda n, d: dev_table(rand(n, d), "f32", pad)  # noqa: E731
    x = [dev_table(rng.round_to_bf16(rand(n, d)), storage, 2 * pad if storage == "bf16" and pad > 1 else pad) for n, d in zip(rows, cols)]
    vecs = [[up(rand(heads, d)) for _ in range(k)] for d, k in zip(cols, sets)]
    scores = [[[new(n, heads) for _ in range(k)] for n, k in zip(rows, sets)] for _ in range(2)]
    heta.heta_attn_score_tables(list(zip(x, vecs, scores[0])))
    for t in range(len(rows)):
        heta.heta_attn_score_multi(x[t], vecs[t], scores[1][t])
    dx0 = [rand(n, d) for n, d in zip(rows, cols)]
    dx = [[dev_table(a, "f32", pad) for a in dx0] for _ in range(2)]
    dvecs = [[[new(heads, d) for _ in range(k)] for d, k in zip(cols, sets)] for _ in range(2)]
    betas = [float(t % 2) for t in range(len(rows))]
    heta.heta_attn_score_bwd_tables(graph, [(x[t], vecs[t], scores[0][t], dx[0][t], betas[t], dvecs[0][t]) for t in range(len(rows))])
    for t in range(len(rows)):
        heta.heta_attn_score_bwd_multi(graph, x[t], vecs[t], scores[0][t], dx=dx[1][t], beta=betas[t], dvecs=dvecs[1][t])

    F, items = 20, ([], [])
    for t in range(30):  # more than one launch takes
        W = dev_table(rng.round_to_bf16(rand(1 + 7 * t, heads * F)), storage, 8 if storage == "bf16" else 4)
        a, dwa, dW0 = up(rand(heads, F)), up(rand(heads, W.shape[0])), rand(*W.shape)
        for out in items:
            out.append((W, a, new(heads, W.shape[0]), dwa, up(dW0), new(heads, F)))
    heta.heta_attn_fold_multi([it[:3] for it in items[0]])
    heta.heta_attn_fold_bwd_multi([(W, a, dwa, dW, da) for W, a, _, dwa, dW, da in items[0]], beta=1.0)
    for W, a, wa, dwa, dW, da in items[1]:
        heta.heta_attn_fold(W, a, wa)
        heta.heta_attn_fold_bwd(W, a, dwa, dW=dW, beta=1.0, da=da)

    d = 12 * heads
    parts = [[mats(n, d) for _ in range(k)] for n, k in zip(rows, sets)]
    live = [t for t, n in enumerate(rows) if n]
    sums = [[new(n, d) for n in rows] for _ in range(2)]
    heta.heta_cross_rel_reduce_multi(graph, [(t, parts[t], sums[0][t]) for t in live], heta.HETA_ACT_RELU)
    for t in live:
        heta.heta_cross_rel_reduce(graph, t, parts[t], sums[1][t], heta.HETA_ACT_RELU)
    cols_of = lambda t, w: [up(rand(rows[t], w)) for _ in range(2)]  # noqa: E731
    ins = [(t, [t, t], mats(rows[t], d), mats(rows[t], d), [mats(rows[t], d) for _ in range(2)], [mats(rows[t], d) for _ in range(2)],
            *[cols_of(t, heads) for _ in range(4)]) for t in live]
    dst = [[(new(rows[t], d), [new(rows[t], heads) for _ in range(2)], [new(rows[t], 4 * heads) for _ in range(2)]) for t in live] for _ in range(2)]
    heta.heta_attn_bwd_dst_multi(graph, [(t, rs, h, go, gi, *rest, d_er, pack) for (t, rs, h, go, *rest), (gi, d_er, pack) in zip(ins, dst[0])], 0.2,
                                 heta.HETA_ACT_RELU)
    for (t, rs, h, go, *rest), (gi, d_er, pack) in zip(ins, dst[1]):
        heta.heta_attn_bwd_dst(graph, t, rs, 0.2, heta.HETA_ACT_RELU, h, go, gi, *rest, d_er, pack)

    def flat(v):
        return [v] if isinstance(v, torch.Tensor) else [y for w in v for y in flat(w)]

    for one, two in [scores, dx, dvecs, items, sums, dst]:
        for p, q in zip(flat(one), flat(two)):
            assert torch.equal(p, q)
    with pytest.raises(heta.HetaError, match="overlap"):
        heta.heta_cross_rel_reduce_multi(graph, [(0, parts[0], sums[0][0]), (0, parts[0], sums[0][0])])
    with pytest.raises(heta.HetaError, match="overlap"):
        heta.heta_attn_score_bwd_tables(graph, [(x[0], vecs[0], scores[0][0], dx[0][0], 0.0, dvecs[0][0]), (x[0], vecs[0], scores[0][0], dx[0][0], 0.0, dvecs[1][0])])


def test_attention_argument_checks():
    graph = heta.heta_graph_create([(4, 4, 0)], [(0, 0, np.array([0, 1, 2, 2, 2], dtype=np.int64), np.array([1, 0], dtype=np.int32))])
    z = torch.zeros((4, 12), device="cuda")
    el = torch.zeros((4, 5), device="cuda")
    with pytest.raises(heta.HetaError, match="heads"):   # 5 heads do not divide 12 columns
        heta.heta_rel_attn_fwd(graph, 0, z, el, el, 0.2, torch.zeros((4, 12), device="cuda"))
    el = torch.zeros((4, 3), device="cuda")
    with pytest.raises(heta.HetaError, match="beta"):
        heta.heta_rel_attn_fwd(graph, 0, z, el, el, 0.2, torch.zeros((4, 12), device="cuda"), beta=0.5)
    with pytest.raises(heta.HetaError, match="smax and sinv"):
        heta.heta_rel_attn_fwd(graph, 0, z, el, el, 0.2, torch.zeros((4, 12), device="cuda"), smax=torch.zeros((4, 3), device="cuda"))
    graph.destroy()


# ---- the whole layer ---------------------------------------------------------------------------------

def _run_layer(p, ap, tol):
    a64 = [np.asarray(x, np.float64) for x in ap.a]
    q64 = [np.asarray(x, np.float64) for x in ap.q]
    fwd = rgat.rgat_forward(p, a64, q64, ap.slope)
    # keep the ReLU decision away from its kink (both sides get the same, guarded, upstream gradient)
    G = {t: np.where(kink_guard(fwd.H[t], tol), p.G[t], 0.0).astype(np.float32) for t in p.G}
    ref = rgat.rgat_backward(p, a64, q64, fwd, G, ap.slope)
    graph = make_graph(p)
    pad = 8 if p.storage == "bf16" else 4
    tables = [dev_table(t, p.storage, pad) for t in p.tables]
    W = [dev_table(w, p.storage, pad) for w in p.W]
    layer = heta.RgatLayer(graph, tables, W, [up(x) for x in ap.a], [up(np.ascontiguousarray(x.T)) for x in ap.q],
                           p.d_out, ap.heads, ap.slope, relu=p.relu)
    H = layer.forward()
    dW, da, dq, dH0 = layer.backward({t: up(g) for t, g in G.items()})
    torch.cuda.synchronize()
    worst = {}

    def check(got, want, what, family):
        assert_rows_close(got, want, tol, what)
        worst[family] = max(worst.get(family, 0.0), row_err(got, want))

    for t, h in fwd.H.items():
        check(host(H[t]), h, f"H[{t}]", "H")
    rdW, rda, rdq, rdH0 = ref
    for i in range(len(p.W)):
        check(host(dW[i]), rdW[i], f"dW[{i}]", "dW")
        check(host(da[i]), rda[i], f"da[{i}]", "da")
        check(host(dq[i]), rdq[i].T, f"dq[{i}]", "dq")
    assert set(dH0) == set(rdH0)
    for t, x in rdH0.items():
        check(host(dH0[t]), x, f"dH0[{t}]", "dH0")
    graph.destroy()
    print(f"\n[observed] rgat {p.name} {p.storage}: " + " ".join(f"{k}={v:.2e}" for k, v in worst.items()))
    return worst


@pytest.mark.parametrize("storage,tol", [("f32", 1e-4), ("bf16", 2e-2)])
@pytest.mark.parametrize("heads", [1, 4])
def test_rgat_layer_tiny(storage, tol, heads):
    p = workloads.rgat_tiny(storage)
    worst = _run_layer(p, workloads.attention_params(p, heads, gain=2.0), tol)
    # the observed error stays well inside the contractual tolerance (a regression guard, not the contract)
    assert max(worst.values()) <= (1.2e-2 if storage == "bf16" else 1e-5)


def test_rgat_layer_with_more_relations_into_a_type_than_one_destination_pass_takes():
    """Ten relations into one type: the destination side runs in two passes, the activation's backward in the first."""
    nts = [NodeType("A", 700, 24, False), NodeType("B", 300, 16, False)]
    G = HetGraph(nts)
    for i in range(10):
        G.relations.append(uniform_relation(f"r{i}", i % 2, 0, nts[i % 2].num_nodes, 700, 2000 + 100 * i, f"tests/rgat/many/{i}"))
    tabs = [rng.normal_table(t.num_nodes, t.feat_dim, "tests/rgat/many", t.name) for t in nts]
    W = [workloads.glorot(nts[r.src_type].feat_dim, 32, "tests/rgat/many", f"W/{r.name}") for r in G.relations]
    p = workloads.LayerProblem("rgat-many", G, "sum", "f32", tabs, W, 32, {0: rng.normal_table(700, 32, "tests/rgat/many", "G")}, relu=True)
    assert max(_run_layer(p, workloads.attention_params(p, 4, gain=1.5), 1e-4).values()) <= 1e-5


@pytest.mark.parametrize("storage,tol", [("f32", 1e-4), ("bf16", 2e-2)])
def test_rgat_layer_config3_scaled(storage, tol):
    p = workloads.config3(storage, scale=0.02)
    p.relu = True
    worst = _run_layer(p, workloads.attention_params(p, 4, gain=1.0), tol)
    assert max(worst.values()) <= (1.2e-2 if storage == "bf16" else 1e-5)


def test_rgat_layer_on_a_sampled_block():
    """R-GAT over a mini-batch block: the block's node types are the base types twice (source role k,
    destination role T + k); both roles read compact tables gathered by the block's id lists
    (heta_feature_gather), and the gradients come back per role."""
    mb = workloads.config2(scale=0.02)
    b = mb.blocks[0]
    T = b.n_base_types
    g = b.graph
    tabs_host, tabs_dev = [], []
    for k in range(2 * T):
        base_t = k % T
        ids = b.src_gid[k] if k < T else b.dst_gid[k]
        ids = np.zeros(0, dtype=np.int64) if ids is None else ids
        full = dev_table(mb.tables[base_t], "f32", 4)
        out = dev_table(np.zeros((max(1, ids.size), full.shape[1]), dtype=np.float32), "f32", 4)[:ids.size]
        if ids.size:
            heta.heta_feature_gather(full, torch.from_numpy(ids).cuda(), out)
        tabs_dev.append(out if ids.size else dev_table(np.zeros((1, full.shape[1]), dtype=np.float32), "f32", 4)[:0])
        tabs_host.append(mb.tables[base_t][ids])
    rels = [i for i, r in enumerate(g.relations) if g.ntypes[r.dst_type].num_nodes > 0 and g.ntypes[r.src_type].num_nodes > 0]
    W = [workloads.glorot(g.ntypes[r.src_type].feat_dim, 64, "tests/rgat/block", f"W/{r.name}") for r in g.relations]
    Gup = {t: rng.normal_table(g.ntypes[t].num_nodes, 64, "tests/rgat/block", f"G/{t}")
           for t in {g.relations[i].dst_type for i in rels}}
    p = workloads.LayerProblem("rgat-block", g, "sum", "f32", tabs_host, W, 64, Gup, relu=True)
    ap = workloads.attention_params(p, 4, gain=1.5)
    a64, q64 = [np.asarray(x, np.float64) for x in ap.a], [np.asarray(x, np.float64) for x in ap.q]
    fwd = rgat.rgat_forward(p, a64, q64, ap.slope, rels=rels)
    G = {t: np.where(kink_guard(fwd.H[t], 1e-4), p.G[t], 0.0).astype(np.float32) for t in fwd.H}
    rdW, rda, rdq, rdH0 = rgat.rgat_backward(p, a64, q64, fwd, G, ap.slope, rels=rels)
    hg = make_graph(p)
    layer = heta.RgatLayer(hg, tabs_dev, [dev_table(w, "f32", 4) for w in W], [up(x) for x in ap.a],
                           [up(np.ascontiguousarray(x.T)) for x in ap.q], 64, 4, ap.slope, relu=True, rels=rels)
    H = layer.forward()
    dW, da, dq, dH0 = layer.backward({t: up(x) for t, x in G.items()})
    torch.cuda.synchronize()
    for t, h in fwd.H.items():
        assert_rows_close(host(H[t]), h, 1e-4, f"H[{t}]")
    for i in rels:
        assert_rows_close(host(dW[i]), rdW[i], 1e-4, f"dW[{i}]")
        assert_rows_close(host(da[i]), rda[i], 1e-4, f"da[{i}]")
        assert_rows_close(host(dq[i]), rdq[i].T, 1e-4, f"dq[{i}]")
    for t, x in rdH0.items():
        if x.shape[0]:
            assert_rows_close(host(dH0[t]), x, 1e-4, f"dH0[{t}]")
    hg.destroy()


def test_attention_is_bitwise_reproducible_run_to_run():
    """No atomics anywhere: two runs on a relation with hub rows give identical bits, forward and backward."""
    G = _relation_case("skew_dst", 2000, 3000, 60000)
    r = G.relations[0]
    g = rng.stream("tests", "attn/repro")
    d, heads = 128, 4
    z = up(g.standard_normal((2000, d)))
    el, er = up(2.0 * g.standard_normal((2000, heads))), up(2.0 * g.standard_normal((3000, heads)))
    go = up(g.standard_normal((3000, d)))
    graph = heta.heta_graph_create([(2000, 4, 0), (3000, 4, 0)], [(0, 1, r.rowptr, r.col)])
    runs = []
    for _ in range(2):
        out, pos = torch.empty((3000, d), device="cuda"), torch.empty((3000, d), device="cuda")
        smax, sinv = torch.empty((3000, heads), device="cuda"), torch.empty((3000, heads), device="cuda")
        dz, d_el, d_er = torch.empty((2000, d), device="cuda"), torch.empty((2000, heads), device="cuda"), torch.empty((3000, heads), device="cuda")
        heta.heta_rel_attn_fwd(graph, 0, z, el, er, 0.2, out, smax=smax, sinv=sinv, out_pos=pos)
        heta.heta_rel_attn_bwd(graph, 0, z, el, er, 0.2, smax, sinv, out, go, dz, d_el, d_er, o_pos=pos)
        torch.cuda.synchronize()
        # the form that RgatLayer runs
        apos, pack = torch.empty((3000, heads), device="cuda"), torch.empty((3000, 4 * heads), device="cuda")
        dz2, d_el2, d_er2 = torch.empty_like(dz), torch.empty_like(d_el), torch.empty_like(d_er)
        heta.heta_rel_attn_fwd_train(graph, 0, z, el, er, 0.2, out, smax=smax, sinv=sinv, out_pos=pos, apos=apos)
        heta.heta_attn_bwd_dst(graph, 1, [0], 0.2, heta.HETA_ACT_NONE, None, go, None, [out], [pos], [er], [smax], [sinv], [apos], [d_er2], [pack])
        heta.heta_rel_attn_bwd_src(graph, 0, z, el, 0.2, pack, go, dz2, d_el2)
        torch.cuda.synchronize()
        runs.append((out, pos, smax, sinv, dz, d_el, d_er, apos, pack, dz2, d_el2, d_er2))
    for a, b in zip(*runs):
        assert torch.equal(a, b)
    graph.destroy()


def test_fold_of_more_than_2_32_elements():
    """Five relations of 2^30 elements each: more threads than one launch has."""
    heads, d_in = 16, 1 << 26
    W = torch.randn((d_in, heads), device="cuda", dtype=torch.bfloat16)
    a = [torch.full((heads, 1), 0.5 * (i + 1), device="cuda") for i in range(5)]
    wa = [torch.empty((heads, d_in), device="cuda") for _ in a]
    heta.heta_attn_fold_multi([(W, x, out) for x, out in zip(a, wa)])
    for x, out in zip(a, wa):  # d_out / heads is 1: each element is one product
        for j in range(0, d_in, 1 << 24):
            assert torch.equal(out[:, j:j + (1 << 24)], (W[j:j + (1 << 24)].float() * x.view(1, -1)).t())
    del W, wa, out
    torch.cuda.empty_cache()
