"""GPU parity: every C-ABI entry point against the CPU oracle on the same seeded inputs.

Index work (CSC, degrees, gathers, integer-valued sums) must match bit for bit; floating point
must satisfy  max_j |got_ij - ref_ij| <= tol * max(1, max_j |ref_ij|)  for every row i, with
tol = 1e-4 for fp32 storage and 2e-2 for bf16 storage (fp32 accumulation in both).
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2408_09697_amd as heta
from gen import rng, workloads
from gen.graphs import HetGraph, NodeType, Relation, power_law_degrees
from tests.harness import (WEIGHT_PATTERNS, assert_product, assert_rows_close, compare_layer, dev_table, make_graph, make_layer,
                           patterned_weights, run_layer_on_gpu)

pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-4, "bf16": 2e-2}


def skewed_relation(n_src=3000, n_dst=2000, n_edges=60000, name="skew"):
    """Power-law in-degrees plus hand-placed rows around every scheduling threshold: empty rows,
    rows of 1, 7, 8, 9, 127, 128, 129, 511, 512, 513 edges, and one 3000-edge hub."""
    g = rng.stream("tests", name)
    deg = power_law_degrees(n_dst, n_edges, 2.0, g)
    for row, k in zip(range(3, 40, 3), [0, 1, 7, 8, 9, 127, 128, 129, 511, 512, 513, 3000, 0]):
        deg[row] = k
    rowptr = np.zeros(n_dst + 1, dtype=np.int64)
    np.cumsum(deg, out=rowptr[1:])
    col = g.integers(0, n_src, size=int(rowptr[-1]), dtype=np.int32)
    col[:50] = 0                       # a popular source as well: a hub column for the backward
    return Relation(name, 0, 1, rowptr, col)


def one_relation_graph(rel, n_src, n_dst):
    g = HetGraph([NodeType("s", n_src, 8, False), NodeType("t", n_dst, 8, False)], [rel])
    nts = [(n_src, 8, 0), (n_dst, 8, 0)]
    return g, heta.heta_graph_create(nts, [(0, 1, rel.rowptr, rel.col)])


INGEST_MODE = {"host_ingest": 1, "device_ingest": 2, "block_ingest": 3}


@pytest.fixture(scope="module", params=["host_ingest", "device_ingest", "block_ingest"])
def skew(request):
    """The skewed relation, ingested by the host path (what a relation of this size gets by default), by the
    per-relation device kernels (what relations of 2^18+ edges and rows get) and by the whole-block device
    ingest (what the relations of a sampled block of 2^16+ edges and rows get together)."""
    rel = skewed_relation()
    heta.heta_ingest_force(INGEST_MODE[request.param])
    g, hg = one_relation_graph(rel, 3000, 2000)
    heta.heta_ingest_force(0)
    yield rel, hg
    hg.destroy()


# ---- a1: ingest ---------------------------------------------------------------------------------

def test_ingest_csc_and_degrees_bit_exact(skew):
    rel, hg = skew
    src, dst = rel.edge_list()
    colptr, row = heta.heta_graph_get_csc(hg, 0)
    ref_colptr, ref_row = oracle.csc(src, dst, 3000)
    assert np.array_equal(colptr, ref_colptr) and np.array_equal(row, ref_row)
    assert np.array_equal(heta.heta_graph_get_degrees(hg, 0), oracle.in_degree(src, dst, 2000))


@pytest.mark.parametrize("n_src,mode", [(100_000, 2), (100_000, 3), (200_000, 3), (40_000_000, 2)])
def test_ingest_transpose_at_key_widths_that_take_nine_bit_passes(n_src, mode):
    """Source counts of 17, 18 and 26 bits: the radix sort behind the transpose takes 9 bits per pass there (two
    passes instead of three, three instead of four).  CSC and degrees against the definition, bit for bit."""
    g = rng.stream("tests", f"ingest-bits/{n_src}")
    n_dst, n_e = 5000, 60_000
    dst = np.sort(g.integers(0, n_dst, size=n_e)).astype(np.int64)
    src = g.integers(0, n_src, size=n_e, dtype=np.int64).astype(np.int32)
    src[:2000] = n_src - 1                                   # a column of many edges at the top of the key range
    rowptr = np.zeros(n_dst + 1, dtype=np.int64)
    np.add.at(rowptr, dst + 1, 1)
    rowptr = np.cumsum(rowptr)
    heta.heta_ingest_force(mode)
    try:
        hg = heta.heta_graph_create([(n_src, 8, 0), (n_dst, 8, 0)], [(0, 1, rowptr, src)])
    finally:
        heta.heta_ingest_force(0)
    colptr, row = heta.heta_graph_get_csc(hg, 0)
    ref_colptr, ref_row = oracle.csc(src, dst.astype(np.int32), n_src)
    assert np.array_equal(colptr, ref_colptr) and np.array_equal(row, ref_row)
    assert np.array_equal(heta.heta_graph_get_degrees(hg, 0), np.diff(rowptr))
    hg.destroy()


@pytest.mark.parametrize("mode", [2, 3], ids=["device_ingest", "block_ingest"])
@pytest.mark.parametrize("n", [2046, 2047, 2048, 8191, 8192, 16383, 16384, 24577, 32767, 32768])
def test_ingest_at_the_edges_of_the_one_workgroup_scan(n, mode):
    """The scans over rows and digit counts run in one workgroup up to 32,768 elements, rounds of 8,192; a scan has one
    element more than there are rows.  CSC and degrees bit for bit; the schedule through sums of whole numbers, exact."""
    g = rng.stream("tests", f"ingest-scan/{n}")
    dst, src = np.sort(g.integers(0, n, size=3 * n)).astype(np.int32), g.integers(0, n, size=3 * n).astype(np.int32)
    rowptr = np.concatenate([[0], np.cumsum(np.bincount(dst, minlength=n))]).astype(np.int64)
    heta.heta_ingest_force(mode)
    try:
        hg = heta.heta_graph_create([(n, 4, 0), (n, 4, 0)], [(0, 1, rowptr, src)])
    finally:
        heta.heta_ingest_force(0)
    colptr, row = heta.heta_graph_get_csc(hg, 0)
    ref_colptr, ref_row = oracle.csc(src, dst, n)
    assert np.array_equal(colptr, ref_colptr) and np.array_equal(row, ref_row)
    assert np.array_equal(heta.heta_graph_get_degrees(hg, 0), np.diff(rowptr))
    x = g.integers(-50, 50, size=(n, 4)).astype(np.float32)
    ref = np.zeros((n, 4), dtype=np.float32)
    np.add.at(ref, dst, x[src])
    out = torch.full((n, 4), 3.0, device="cuda")
    heta.heta_rel_aggregate_fwd(hg, 0, heta.HETA_SUM, torch.from_numpy(x).cuda(), out)
    assert np.array_equal(out.cpu().numpy(), ref)
    hg.destroy()


@pytest.mark.parametrize("mode", [1, 2, 3])
def test_ingest_config1_and_device_pointers(mode):
    p = workloads.config1()
    nts = [(t.num_nodes, t.feat_dim, int(t.learnable)) for t in p.graph.ntypes]
    rels = [(r.src_type, r.dst_type, torch.from_numpy(r.rowptr).cuda(), torch.from_numpy(r.col).cuda())
            for r in p.graph.relations]
    heta.heta_ingest_force(mode)
    try:
        hg = heta.heta_graph_create(nts, rels, flags=heta.HETA_PTRS_ON_DEVICE)
    finally:
        heta.heta_ingest_force(0)
    for i, r in enumerate(p.graph.relations):
        src, dst = r.edge_list()
        n_s, n_t = p.graph.ntypes[r.src_type].num_nodes, p.graph.ntypes[r.dst_type].num_nodes
        colptr, row = heta.heta_graph_get_csc(hg, i)
        rc, rr = oracle.csc(src, dst, n_s)
        assert np.array_equal(colptr, rc) and np.array_equal(row, rr)
        assert np.array_equal(heta.heta_graph_get_degrees(hg, i), oracle.in_degree(src, dst, n_t))
    hg.destroy()
    # a bad CSR that lives on the device is rejected by the validation kernels, with the host validator's wording
    z = torch.zeros(1, dtype=torch.int32).cuda()
    for rowptr, col, needle in [([0, 2, 1] + [1] * 1998, z, "decreases at row 1"), ([1] * 2001, z, "rowptr[0]"),
                                ([0] * 2000 + [2], z, "num_edges"),
                                ([0] * 2000 + [1], torch.full((1,), 2000, dtype=torch.int32).cuda(), "col[0]"),
                                ([0] * 2000 + [1], torch.full((1,), -1, dtype=torch.int32).cuda(), "col[0]")]:
        bad = [(0, 0, torch.tensor(rowptr, dtype=torch.int64).cuda(), col)]
        for bad_mode in (0, 3):   # by size (this one goes to the host), and through the whole-block device ingest
            heta.heta_ingest_force(bad_mode)
            try:
                with pytest.raises(heta.HetaError) as ei:
                    heta.heta_graph_create(nts, bad, flags=heta.HETA_PTRS_ON_DEVICE)
            finally:
                heta.heta_ingest_force(0)
            assert ei.value.status == heta.HETA_ERR_BAD_CSR and needle in ei.value.message, ei.value.message


@pytest.mark.parametrize("mode", [2, 3], ids=["device_ingest", "block_ingest"])
def test_device_ingest_edge_cases(mode):
    """Device-built index arrays on shapes that stress the sort and the scans: no edges, one row, one
    column holding every edge, a ragged last sort tile, more tiles than one scan tile of tile counts."""
    heta.heta_ingest_force(mode)
    try:
        g = rng.stream("tests", "ingest-edge")
        cases = [(5, 7, 0), (1, 1, 1), (1, 9, 4097), (3, 1, 5000), (40000, 70000, 300001)]
        for n_src, n_dst, n_e in cases:
            dst = np.sort(g.integers(0, n_dst, size=n_e)).astype(np.int64)
            src = g.integers(0, n_src, size=n_e, dtype=np.int32)
            if n_e > 1000:
                src[: n_e // 3] = n_src - 1                      # a hub column
            rowptr = np.zeros(n_dst + 1, dtype=np.int64)
            np.add.at(rowptr, dst + 1, 1)
            rowptr = np.cumsum(rowptr)
            hg = heta.heta_graph_create([(n_src, 8, 0), (n_dst, 8, 0)], [(0, 1, rowptr, src)])
            colptr, row = heta.heta_graph_get_csc(hg, 0)
            rc, rr = oracle.csc(src, dst.astype(np.int32), n_src)
            assert np.array_equal(colptr, rc) and np.array_equal(row, rr), (n_src, n_dst, n_e)
            assert np.array_equal(heta.heta_graph_get_degrees(hg, 0), np.diff(rowptr)), (n_src, n_dst, n_e)
            # the schedule-ordered adjacency, through an exact integer aggregation in both directions
            x = torch.arange(n_src, dtype=torch.float32, device="cuda").remainder(5).sub(2).reshape(-1, 1).repeat(1, 4).contiguous()
            out = torch.full((n_dst, 4), float("nan"), dtype=torch.float32, device="cuda")
            heta.heta_rel_aggregate_fwd(hg, 0, heta.HETA_SUM, x, out)
            ref = np.zeros(n_dst)
            np.add.at(ref, dst, (src % 5 - 2).astype(np.float64))
            assert np.array_equal(out[:, 0].cpu().numpy().astype(np.float64), ref), (n_src, n_dst, n_e)
            y = torch.arange(n_dst, dtype=torch.float32, device="cuda").remainder(3).sub(1).reshape(-1, 1).repeat(1, 4).contiguous()
            back = torch.full((n_src, 4), float("nan"), dtype=torch.float32, device="cuda")
            heta.heta_rel_aggregate_bwd(hg, 0, heta.HETA_SUM, y, back)
            refb = np.zeros(n_src)
            np.add.at(refb, src, (dst % 3 - 1).astype(np.float64))
            assert np.array_equal(back[:, 0].cpu().numpy().astype(np.float64), refb), (n_src, n_dst, n_e)
            hg.destroy()
    finally:
        heta.heta_ingest_force(0)


@pytest.mark.parametrize("n_src,n_dst,n_e,hubs", [
    (1, 1, 1, 0), (3, 5, 0, 0), (0, 4, 0, 0), (4, 0, 0, 0), (1, 700, 5000, 0), (700, 1, 5000, 0), (63, 64, 65, 0), (1023, 255, 1023, 0),
    (1024, 256, 1024, 0), (1025, 257, 1025, 2), (2049, 513, 4097, 3), (9000, 40, 40000, 5), (31, 15000, 33333, 2), (65536, 16384, 65536, 4),
    (65537, 16385, 65537, 1), (130000, 132000, 143, 0), (2000, 200000, 60000, 9), (200000, 2000, 60143, 9), (1, 1, 262141, 0)])
def test_block_ingest_at_the_edges_of_its_workgroups(n_src, n_dst, n_e, hubs):
    """The whole-block build at the edges of its workgroups' shares (256 rows, 1,024 edges, 1,024 or 2,048 sources; 64 or 128
    workgroups), with no, some and only hub rows, up to just below 2^18 edges + rows: CSC, degrees and both schedules
    (through exact integer sums) of three relations built together, from host and device arrays."""
    g = rng.stream("tests", f"ingest-one/{n_src}/{n_dst}/{n_e}")
    made = []
    for k in range(3):
        dst = np.sort(g.integers(0, max(n_dst, 1), size=n_e)).astype(np.int32)
        src = g.integers(0, max(n_src, 1), size=n_e).astype(np.int32)
        for h in range(hubs):  # hub rows of 512, 513, ... edges and a hub column
            at = np.arange(h * (512 + h), min(n_e, (h + 1) * (512 + h)))
            dst[at] = min(n_dst - 1, 7 * h)
            src[at[::2]] = n_src - 1
        dst = np.sort(dst)
        if k == 2:
            dst, src = dst[:n_e // 2], src[:n_e // 2]
        made.append((dst, src, np.concatenate([[0], np.cumsum(np.bincount(dst, minlength=n_dst))]).astype(np.int64)))
    for device in (False, True):
        rels = [(0, 1, torch.from_numpy(p).cuda(), torch.from_numpy(s).cuda()) if device else (0, 1, p, s) for _, s, p in made]
        heta.heta_ingest_force(3)
        try:
            hg = heta.heta_graph_create([(n_src, 4, 0), (n_dst, 4, 0)], rels, flags=heta.HETA_PTRS_ON_DEVICE if device else 0)
        finally:
            heta.heta_ingest_force(0)
        for r, (dst, src, rowptr) in enumerate(made):
            colptr, row = heta.heta_graph_get_csc(hg, r)
            ref_colptr, ref_row = oracle.csc(src, dst, n_src)
            assert np.array_equal(colptr, ref_colptr) and np.array_equal(row, ref_row)
            assert np.array_equal(heta.heta_graph_get_degrees(hg, r), np.diff(rowptr))
            if n_src == 0 or n_dst == 0:
                continue
            x, y = (g.integers(-50, 50, size=(n, 4)).astype(np.float32) for n in (n_src, n_dst))
            fwd, bwd = np.zeros((n_dst, 4), dtype=np.float32), np.zeros((n_src, 4), dtype=np.float32)
            np.add.at(fwd, dst, x[src])
            np.add.at(bwd, src, y[dst])
            out, back = torch.full((n_dst, 4), 3.0, device="cuda"), torch.full((n_src, 4), 3.0, device="cuda")
            heta.heta_rel_aggregate_fwd(hg, r, heta.HETA_SUM, torch.from_numpy(x).cuda(), out)
            heta.heta_rel_aggregate_bwd(hg, r, heta.HETA_SUM, torch.from_numpy(y).cuda(), back)
            assert np.array_equal(out.cpu().numpy(), fwd) and np.array_equal(back.cpu().numpy(), bwd)
        hg.destroy()


# ---- a2: heterogeneous gather ----------------------------------------------------------------------

@pytest.mark.parametrize("d,storage,pad", [(128, "f32", 4), (7, "bf16", 8), (7, "bf16", 1), (300, "f32", 1), (789, "bf16", 8)])
def test_feature_gather_bit_exact(d, storage, pad):
    x = rng.normal_table(5000, d, "tests", f"gather{d}")
    tab = dev_table(x, storage, pad)
    gid = rng.stream("tests", "gid").integers(0, 5000, size=1234)
    out = torch.zeros((1234, d), dtype=tab.dtype, device="cuda")
    heta.heta_feature_gather(tab, torch.from_numpy(gid).cuda(), out)
    heta.heta_check_ids(torch.from_numpy(gid).cuda(), 5000)
    ref = (rng.round_to_bf16(x) if storage == "bf16" else x)[gid]
    assert np.array_equal(out.float().cpu().numpy(), ref)
    with pytest.raises(heta.HetaError):
        heta.heta_check_ids(torch.tensor([0, 5000], dtype=torch.int64).cuda(), 5000)


# ---- a3: forward aggregation -----------------------------------------------------------------------

@pytest.mark.parametrize("op", ["sum", "mean"])
@pytest.mark.parametrize("d,storage,pad", [
    (1, "f32", 4), (4, "f32", 4), (7, "f32", 4), (32, "f32", 4), (100, "f32", 4), (128, "f32", 4), (300, "f32", 4),
    (520, "f32", 4), (1024, "f32", 4),
    (7, "bf16", 8), (24, "bf16", 8), (64, "bf16", 8), (128, "bf16", 8), (300, "bf16", 8), (512, "bf16", 8),
    (768, "bf16", 8), (789, "bf16", 8), (1100, "bf16", 8),
    (7, "f32", 1), (789, "bf16", 1), (33, "bf16", 1),       # unpadded rows: element-wise kernels
])
def test_aggregate_fwd(skew, op, d, storage, pad):
    rel, hg = skew
    src, dst = rel.edge_list()
    x = rng.normal_table(3000, d, "tests", f"x{d}")
    if storage == "bf16":
        x = rng.round_to_bf16(x)
    tab = dev_table(x, storage, pad)
    out = torch.full((2000, d), float("nan"), dtype=torch.float32, device="cuda")
    heta.heta_rel_aggregate_fwd(hg, 0, heta.HETA_MEAN if op == "mean" else heta.HETA_SUM, tab, out)
    ref = oracle.aggregate_fwd(src, dst, 2000, x, op)
    assert_rows_close(out.cpu().numpy(), ref, 1e-4, f"M d={d} {storage}")
    deg = np.diff(rel.rowptr)
    assert not out.cpu().numpy()[deg == 0].any()           # empty rows are exactly zero


@pytest.mark.parametrize("storage", ["f32", "bf16"])
def test_aggregate_fwd_with_gid_and_bf16_output(skew, storage):
    rel, hg = skew
    src, dst = rel.edge_list()
    d = 128
    x = rng.normal_table(10000, d, "tests", "bigtable")
    if storage == "bf16":
        x = rng.round_to_bf16(x)
    gid = rng.stream("tests", "gid2").permutation(10000)[:3000].astype(np.int64)
    tab = dev_table(x, storage, 8)
    ref = oracle.aggregate_fwd(src, dst, 2000, x, "mean", gid=gid)
    out = torch.zeros((2000, d), dtype=torch.float32, device="cuda")
    heta.heta_rel_aggregate_fwd(hg, 0, heta.HETA_MEAN, tab, out, src_gid=torch.from_numpy(gid).cuda())
    assert_rows_close(out.cpu().numpy(), ref, 1e-4, "gid fp32 out")
    # strided bf16 output (a column slice of a wider buffer), as used to feed the bf16 projection
    wide = torch.zeros((2000, 3 * d), dtype=torch.bfloat16, device="cuda")
    heta.heta_rel_aggregate_fwd(hg, 0, heta.HETA_MEAN, tab, wide[:, d:2 * d], src_gid=torch.from_numpy(gid).cuda())
    w = wide.float().cpu().numpy()
    assert_rows_close(w[:, d:2 * d], ref, 2e-2, "gid bf16 out")
    assert not w[:, :d].any() and not w[:, 2 * d:].any()


def test_aggregate_integer_inputs_bit_exact(skew):
    """Small-integer features: every partial sum is exact in fp32, so any summation order must
    reproduce the oracle's bits (pins binning, hub splitting and the index paths)."""
    rel, hg = skew
    src, dst = rel.edge_list()
    for d, storage in [(128, "f32"), (128, "bf16"), (7, "bf16"), (768, "bf16"), (300, "f32")]:
        x = rng.small_int_table(3000, d, -2, 2, "tests", f"int{d}")
        tab = dev_table(x, storage, 8)
        out = torch.zeros((2000, d), dtype=torch.float32, device="cuda")
        heta.heta_rel_aggregate_fwd(hg, 0, heta.HETA_SUM, tab, out)
        assert np.array_equal(out.cpu().numpy().astype(np.float64), oracle.aggregate_fwd(src, dst, 2000, x, "sum"))
        g = rng.small_int_table(2000, d, -2, 2, "tests", f"intg{d}")
        gs = torch.zeros((3000, d), dtype=torch.float32, device="cuda")
        heta.heta_rel_aggregate_bwd(hg, 0, heta.HETA_SUM, dev_table(g, "f32", 4), gs)
        assert np.array_equal(gs.cpu().numpy().astype(np.float64),
                              oracle.aggregate_bwd(src, dst, 3000, 2000, g.astype(np.float64), "sum"))
    # one-hot rows count every gathered index
    d = 16
    e = np.zeros((3000, d), dtype=np.float32)
    e[np.arange(3000), np.arange(3000) % d] = 1.0
    out = torch.zeros((2000, d), dtype=torch.float32, device="cuda")
    heta.heta_rel_aggregate_fwd(hg, 0, heta.HETA_SUM, dev_table(e, "f32", 4), out)
    cnt = np.zeros((2000, d))
    np.add.at(cnt, (dst, src % d), 1.0)
    assert np.array_equal(out.cpu().numpy(), cnt)


# ---- a7: backward aggregation over the CSC -----------------------------------------------------------

@pytest.mark.parametrize("op", ["sum", "mean"])
@pytest.mark.parametrize("d,pad,storage", [(1, 4, "f32"), (7, 4, "f32"), (32, 4, "f32"), (128, 4, "f32"), (300, 4, "f32"),
                                           (768, 4, "f32"), (1024, 4, "f32"), (33, 1, "f32"),
                                           (7, 8, "bf16"), (64, 8, "bf16"), (128, 8, "bf16"), (300, 8, "bf16"),
                                           (789, 8, "bf16"), (33, 1, "bf16")])
def test_aggregate_bwd(skew, op, d, pad, storage):
    """fp32 gradient rows, and rows kept in bf16 (a dM_r stored in the storage type): the oracle
    reads the same rounded values, so only the fp32 accumulation order differs."""
    rel, hg = skew
    src, dst = rel.edge_list()
    gm = rng.normal_table(2000, d, "tests", f"gm{d}")
    seen = rng.round_to_bf16(gm) if storage == "bf16" else gm
    ref = oracle.aggregate_bwd(src, dst, 3000, 2000, seen.astype(np.float64), op)
    out = torch.full((3000, d), float("nan"), dtype=torch.float32, device="cuda")
    hop = heta.HETA_MEAN if op == "mean" else heta.HETA_SUM
    heta.heta_rel_aggregate_bwd(hg, 0, hop, dev_table(gm, storage, pad), out, beta=0.0)
    assert_rows_close(out.cpu().numpy(), ref, 1e-4, f"dH0 d={d}")
    # beta = 1 accumulates on top
    heta.heta_rel_aggregate_bwd(hg, 0, hop, dev_table(gm, storage, pad), out, beta=1.0)
    assert_rows_close(out.cpu().numpy(), 2 * ref, 1e-4, f"dH0 accumulate d={d}")


def test_adjoint_identity_on_gpu_outputs(skew):
    rel, hg = skew
    d = 64
    x = rng.normal_table(3000, d, "tests", "adjx")
    gm = rng.normal_table(2000, d, "tests", "adjg")
    for hop in (heta.HETA_SUM, heta.HETA_MEAN):
        fwd = torch.zeros((2000, d), dtype=torch.float32, device="cuda")
        bwd = torch.zeros((3000, d), dtype=torch.float32, device="cuda")
        heta.heta_rel_aggregate_fwd(hg, 0, hop, dev_table(x, "f32", 4), fwd)
        heta.heta_rel_aggregate_bwd(hg, 0, hop, dev_table(gm, "f32", 4), bwd)
        lhs = np.vdot(gm.astype(np.float64), fwd.cpu().numpy().astype(np.float64))
        rhs = np.vdot(x.astype(np.float64), bwd.cpu().numpy().astype(np.float64))
        assert abs(lhs - rhs) <= 1e-5 * max(1.0, abs(lhs))


def test_million_edge_hub_row_and_empty_relation():
    n_src, n_dst = 5000, 70
    deg = np.zeros(n_dst, dtype=np.int64)
    deg[5] = 1 << 20
    deg[6] = 3
    rowptr = np.zeros(n_dst + 1, dtype=np.int64)
    np.cumsum(deg, out=rowptr[1:])
    col = rng.stream("tests", "hub").integers(0, n_src, size=int(rowptr[-1]), dtype=np.int32)
    rel = Relation("hub", 0, 1, rowptr, col)
    empty = Relation("empty", 0, 1, np.zeros(n_dst + 1, dtype=np.int64), np.zeros(0, dtype=np.int32))
    hg = heta.heta_graph_create([(n_src, 8, 0), (n_dst, 8, 0)],
                                [(0, 1, rel.rowptr, rel.col), (0, 1, empty.rowptr, empty.col)])
    src, dst = rel.edge_list()
    d = 24
    x = rng.small_int_table(n_src, d, -2, 2, "tests", "hubx")
    out = torch.full((n_dst, d), float("nan"), dtype=torch.float32, device="cuda")
    heta.heta_rel_aggregate_fwd(hg, 0, heta.HETA_SUM, dev_table(x, "bf16", 8), out)
    assert np.array_equal(out.cpu().numpy().astype(np.float64), oracle.aggregate_fwd(src, dst, n_dst, x, "sum"))
    g = rng.normal_table(n_dst, d, "tests", "hubg")
    gs = torch.zeros((n_src, d), dtype=torch.float32, device="cuda")
    heta.heta_rel_aggregate_bwd(hg, 0, heta.HETA_MEAN, dev_table(g, "f32", 4), gs)
    assert_rows_close(gs.cpu().numpy(), oracle.aggregate_bwd(src, dst, n_src, n_dst, g.astype(np.float64), "mean"), 1e-4)
    # the empty relation: forward gives zeros, backward with beta = 1 leaves the buffer alone
    heta.heta_rel_aggregate_fwd(hg, 1, heta.HETA_MEAN, dev_table(x, "bf16", 8), out)
    assert not out.cpu().numpy().any()
    before = gs.clone()
    heta.heta_rel_aggregate_bwd(hg, 1, heta.HETA_MEAN, dev_table(g, "f32", 4), gs, beta=1.0)
    assert torch.equal(before, gs)
    heta.heta_rel_aggregate_bwd(hg, 1, heta.HETA_MEAN, dev_table(g, "f32", 4), gs, beta=0.0)
    assert not gs.cpu().numpy().any()
    hg.destroy()


def test_zero_destination_relation_is_a_noop():
    hg = heta.heta_graph_create([(10, 8, 0), (0, 8, 0)], [(0, 1, np.zeros(1, dtype=np.int64), np.zeros(0, dtype=np.int32))])
    x = dev_table(np.ones((10, 8), dtype=np.float32), "f32", 4)
    out = torch.zeros((1, 8), dtype=torch.float32, device="cuda")
    heta.heta_rel_aggregate_fwd(hg, 0, heta.HETA_MEAN, x, out)
    gs = torch.ones((10, 8), dtype=torch.float32, device="cuda")
    heta.heta_rel_aggregate_bwd(hg, 0, heta.HETA_MEAN, out, gs, beta=0.0)
    assert not gs.cpu().numpy().any()
    hg.destroy()


def test_run_to_run_bitwise_determinism(skew):
    rel, hg = skew
    x = dev_table(rng.normal_table(3000, 128, "tests", "detx"), "f32", 4)
    outs = []
    for _ in range(3):
        o = torch.zeros((2000, 128), dtype=torch.float32, device="cuda")
        heta.heta_rel_aggregate_fwd(hg, 0, heta.HETA_MEAN, x, o)
        outs.append(o)
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])


def test_edge_order_and_node_labels_do_not_matter():
    """Scheduling independence: the neighbours of every row listed in another order, and the source and
    destination nodes relabelled, give the same rows (permuted accordingly): within 1e-4 for random
    inputs, bit for bit for small-integer inputs, forward and backward."""
    rel = skewed_relation(name="perm")
    n_src, n_dst = 3000, 2000
    g = rng.stream("tests", "perm/how")
    deg = np.diff(rel.rowptr)
    # 1. another order inside every row
    col2 = rel.col.copy()
    for v in range(n_dst):
        a, b = rel.rowptr[v], rel.rowptr[v + 1]
        col2[a:b] = g.permutation(col2[a:b])
    # 2. relabelled nodes: source u -> ps[u], destination v -> pd[v]
    ps, pd = g.permutation(n_src), g.permutation(n_dst)
    inv_pd = np.argsort(pd)
    deg3 = deg[inv_pd]
    rowptr3 = np.zeros(n_dst + 1, dtype=np.int64)
    np.cumsum(deg3, out=rowptr3[1:])
    col3 = np.concatenate([ps[rel.col[rel.rowptr[v]:rel.rowptr[v + 1]]] for v in inv_pd]).astype(np.int32)
    graphs = [one_relation_graph(r, n_src, n_dst)[1] for r in (rel, Relation("p2", 0, 1, rel.rowptr, col2),
                                                                Relation("p3", 0, 1, rowptr3, col3))]
    for kind in ("normal", "int"):
        X = (rng.normal_table(n_src, 128, "tests", "perm/x") if kind == "normal"
             else rng.small_int_table(n_src, 128, -2, 2, "tests", "perm/xi"))
        Gm = (rng.normal_table(n_dst, 128, "tests", "perm/g") if kind == "normal"
              else rng.small_int_table(n_dst, 128, -2, 2, "tests", "perm/gi"))
        X3 = np.empty_like(X)
        X3[ps] = X
        G3 = np.empty_like(Gm)
        G3[pd] = Gm
        op = heta.HETA_MEAN if kind == "normal" else heta.HETA_SUM
        fwd, bwd = [], []
        for hg, x, gm in zip(graphs, (X, X, X3), (Gm, Gm, G3)):
            o = torch.empty((n_dst, 128), dtype=torch.float32, device="cuda")
            heta.heta_rel_aggregate_fwd(hg, 0, op, dev_table(x, "f32", 4), o)
            b = torch.empty((n_src, 128), dtype=torch.float32, device="cuda")
            heta.heta_rel_aggregate_bwd(hg, 0, op, dev_table(gm, "f32", 4), b)
            fwd.append(o.cpu().numpy())
            bwd.append(b.cpu().numpy())
        same = np.array_equal if kind == "int" else (lambda a, b: (assert_rows_close(a, b.astype(np.float64), 1e-4, "perm"), True)[1])
        assert same(fwd[1], fwd[0]) and same(bwd[1], bwd[0])
        assert same(fwd[2][pd], fwd[0]) and same(bwd[2][ps], bwd[0])
    for hg in graphs:
        hg.destroy()


# ---- a4 / a6: projection ------------------------------------------------------------------------------

@pytest.fixture(params=["direct", "staged"])
def gemm_path(request):
    """Both projection kernels: the direct-to-LDS pipeline (default wherever operand rows are 16-byte
    aligned) and the register-staged kernel (forced here, otherwise the fallback)."""
    heta.heta_projection_force_staged(request.param == "staged")
    yield request.param
    heta.heta_projection_force_staged(False)


PROJ_SHAPES = [(1000, 32, 32), (777, 128, 256), (300, 7, 256), (513, 24, 256), (400, 300, 256),
               (260, 789, 256), (129, 768, 1024), (64, 1024, 1024), (1, 5, 3), (2000, 64, 40),
               # more than 96 tiles of 128 x 128: the full-size tiles (the shapes above take the 64 x 64 ones)
               (20000, 128, 256), (13001, 256, 100)]


@pytest.mark.parametrize("n,d_in,d_out", PROJ_SHAPES)
@pytest.mark.parametrize("in_s,w_s", [("f32", "f32"), ("bf16", "bf16"), ("f32", "bf16")])
@pytest.mark.parametrize("trans", [False, True])
def test_project(n, d_in, d_out, in_s, w_s, trans, gemm_path):
    x = rng.normal_table(n, d_in, "tests", f"px{n}")
    w = rng.normal_table(d_out, d_in, "tests", f"pw{n}") if trans else rng.normal_table(d_in, d_out, "tests", f"pw{n}")
    w = w * np.float32(1.0 / np.sqrt(d_in))
    xr = rng.round_to_bf16(x) if in_s == "bf16" else x
    wr = rng.round_to_bf16(w) if w_s == "bf16" else w
    ref = xr.astype(np.float64) @ (wr.astype(np.float64).T if trans else wr.astype(np.float64))
    out = torch.full((n, d_out), float("nan"), dtype=torch.float32, device="cuda")
    heta.heta_project(dev_table(x, in_s, 8), dev_table(w, w_s, 8), out, trans_w=trans)
    tol = 1e-4 if (in_s, w_s) == ("f32", "f32") else 2e-2
    assert_rows_close(out.cpu().numpy(), ref, tol, f"project {n}x{d_in}x{d_out}")


@pytest.mark.parametrize("pad", [1, 4])
def test_project_row_scale_beta_and_odd_strides(pad, gemm_path):
    n, d_in, d_out = 333, 37, 45
    x = rng.normal_table(n, d_in, "tests", "rsx")
    w = rng.normal_table(d_in, d_out, "tests", "rsw")
    s = rng.uniform_table(n, 1, 0.5, 2.0, "tests", "rss")[:, 0].copy()
    prev = rng.normal_table(n, d_out, "tests", "rsp")
    out = dev_table(prev, "f32", pad)
    heta.heta_project(dev_table(x, "f32", pad), dev_table(w, "f32", pad), out,
                      row_scale=torch.from_numpy(s).cuda(), beta=1.0)
    ref = prev.astype(np.float64) + s[:, None].astype(np.float64) * (x.astype(np.float64) @ w.astype(np.float64))
    assert_rows_close(out.cpu().numpy(), ref, 1e-4, "row_scale+beta")


@pytest.mark.parametrize("n,d_in,d_out", [(2000, 32, 32), (5000, 128, 256), (3000, 7, 256), (1500, 300, 256),
                                          (700, 789, 256), (40, 16, 8), (5000, 768, 1024),
                                          # splits summed by four wavefronts and by one: 196,400 and 196,608 elements, one split
                                          (500, 491, 400), (500, 768, 256), (100, 1000, 333)])
@pytest.mark.parametrize("in_s", ["f32", "bf16"])
def test_project_wgrad(n, d_in, d_out, in_s, gemm_path):
    rel = Relation("w", 0, 1, np.zeros(n + 1, dtype=np.int64), np.zeros(0, dtype=np.int32))
    hg = heta.heta_graph_create([(4, 8, 0), (n, 8, 0)], [(0, 1, rel.rowptr, rel.col)])
    m = rng.normal_table(n, d_in, "tests", f"wgm{n}")
    g = rng.normal_table(n, d_out, "tests", f"wgg{n}")
    mr = rng.round_to_bf16(m) if in_s == "bf16" else m
    ref = mr.astype(np.float64).T @ g.astype(np.float64)
    dW = torch.full((d_in, d_out), float("nan"), dtype=torch.float32, device="cuda")
    heta.heta_rel_project_wgrad(hg, 0, dev_table(m, in_s, 8), dev_table(g, "f32", 4), dW)
    tol = 1e-4 if in_s == "f32" else 2e-2
    # the contraction runs over n rows: scale the bound by the row norm of the reference
    assert_rows_close(dW.cpu().numpy(), ref, tol, f"wgrad {n}x{d_in}x{d_out}")
    heta.heta_rel_project_wgrad(hg, 0, dev_table(m, in_s, 8), dev_table(g, "f32", 4), dW, beta=1.0)
    assert_rows_close(dW.cpu().numpy(), 2 * ref, tol, "wgrad accumulate")
    hg.destroy()


def test_project_wgrad_of_more_elements_than_a_grid_has_threads():
    """Four wavefronts add the splits of 64 elements: from 2^30 elements on, those are 2^32 threads and more."""
    n, d_in, d_out = 20, 32800, 32768
    assert d_in * d_out * 4 > 1 << 32
    hg = heta.heta_graph_create([(n, 8, 0)], [])
    x, g = torch.randn((n, d_in), device="cuda"), torch.randn((n, d_out), device="cuda")
    dW = torch.full((d_in, d_out), float("nan"), device="cuda")
    heta.heta_project_wgrad_batch(hg, [x], [g], [dW])
    bound = 1e-5 * float(x.abs().sum(0).max() * g.abs().max())
    for i in range(0, d_in, 1025):
        ref = x[:, i:i + 1025].double().T @ g.double()
        assert bool((dW[i:i + 1025] - ref).abs().max() <= bound), f"rows {i} ff."
    hg.destroy()
    del dW
    torch.cuda.empty_cache()


# ---- a5: cross-relation sum ---------------------------------------------------------------------------

def test_elementwise_calls_of_more_elements_than_a_grid_has_threads():
    """One element per thread (odd width), 2^32 elements and some: the rows past the bound are computed like the others."""
    n, d = 1_048_000, 4099
    assert n * d > 1 << 32
    hg = heta.heta_graph_create([(n, 8, 0)], [])
    x = torch.empty((n, d), device="cuda")
    for i in range(0, n, 65_500):
        x[i:i + 65_500] = torch.randn((min(65_500, n - i), d), device="cuda")
    out = torch.full((n, d), float("nan"), device="cuda")
    for call in (lambda: heta.heta_act_bwd(heta.HETA_ACT_RELU, x, x, out),
                 lambda: heta.heta_cross_rel_reduce(hg, 0, [x], out, act=heta.HETA_ACT_RELU)):
        out.fill_(float("nan"))
        call()
        for i in range(0, n, 65_500):
            assert torch.equal(out[i:i + 65_500], x[i:i + 65_500].clamp(min=0.0)), f"rows {i} ff."
    hg.destroy()
    del x, out
    torch.cuda.empty_cache()


@pytest.mark.parametrize("d,k,relu", [(256, 3, False), (256, 1, True), (33, 5, True), (32, 16, False)])
def test_cross_rel_reduce_and_act_bwd(d, k, relu):
    n = 1237
    hg = heta.heta_graph_create([(n, 8, 0)], [])
    parts = [rng.normal_table(n, d, "tests", f"part{i}") for i in range(k)]
    ref = oracle.cross_rel_sum(parts, relu=relu)
    out = torch.zeros((n, d), dtype=torch.float32, device="cuda")
    heta.heta_cross_rel_reduce(hg, 0, [dev_table(q, "f32", 1) for q in parts], out,
                               act=heta.HETA_ACT_RELU if relu else heta.HETA_ACT_NONE)
    assert_rows_close(out.cpu().numpy(), ref, 1e-6, "cross-relation sum")
    g = rng.normal_table(n, d, "tests", "actg")
    gi = torch.zeros((n, d), dtype=torch.float32, device="cuda")
    heta.heta_act_bwd(heta.HETA_ACT_RELU if relu else heta.HETA_ACT_NONE, out, dev_table(g, "f32", 1), gi)
    expect = g * (out.cpu().numpy() > 0) if relu else g
    assert np.array_equal(gi.cpu().numpy(), expect.astype(np.float32))
    hg.destroy()


# ---- whole layers ---------------------------------------------------------------------------------------

@pytest.mark.parametrize("mode", ["fused", "per_relation", "unfused"])
def test_layer_config1(mode, gemm_path):
    p = workloads.config1()
    got = run_layer_on_gpu(p, mode=mode)
    ref_f = oracle.layer_forward(p)
    ref_b = oracle.layer_backward(p, ref_f, p.G)
    compare_layer(p, got, ref_f, ref_b, tol=1e-4)


def test_layer_config1_relation_split_equals_whole():
    """Proposition 1 on the GPU path: partial aggregations of two relation subsets, summed by
    heta_cross_rel_reduce, equal the layer over all relations."""
    p = workloads.config1()
    hg = make_graph(p)
    whole = make_layer(p, hg)
    H = whole.forward()
    a = make_layer(p, hg, rels=[0, 2])
    b = make_layer(p, hg, rels=[1, 3])
    Ha, Hb = a.forward(), b.forward()
    tot = torch.zeros_like(H[0])
    heta.heta_cross_rel_reduce(hg, 0, [Ha[0], Hb[0]], tot)
    ref = oracle.layer_forward(p)
    assert_rows_close(tot.cpu().numpy(), ref.H[0], 1e-4, "split sum")
    assert_rows_close(H[0].cpu().numpy(), ref.H[0], 1e-4, "whole")
    assert_rows_close(Ha[1].cpu().numpy() if 1 in Ha else Hb[1].cpu().numpy(), ref.H[1], 1e-4, "type B")
    hg.destroy()


def test_no_pass_of_a_layer_over_some_relations_allocates():
    """A worker's share of a full graph has its backward's buffers from the start; a sampled block's layer makes them when asked."""
    p = workloads.config1()
    hg = make_graph(p)
    G = {t: torch.from_numpy(np.ascontiguousarray(g, dtype=np.float32)).cuda() for t, g in p.G.items()}
    for sampled in (False, True):
        hg.sampled = sampled
        layer = make_layer(p, hg, rels=[0, 2])
        layer.forward()
        before = torch.cuda.memory_allocated()
        layer.backward(G)
        assert (torch.cuda.memory_allocated() > before) == sampled
    hg.destroy()


def test_layer_config1_meta_partitions_sum_to_the_whole():
    """The relation sets that the library's meta-partitioning deals to two partitions (Section 5), each run
    as its own layer: the partial aggregations of the target type add up to the whole layer's
    embeddings, each weight gradient is computed by exactly one partition, the table gradients add up."""
    p = workloads.config1()
    hg = make_graph(p)
    mp = hg.meta_partition(root=0, k=1, p=2)
    sets = [[i for i, m in enumerate(mask) if m] for mask in mp["rel_mask"]]
    into_root = [i for i, (s, t, _) in enumerate(hg.rels) if t == 0]
    assert sorted(sets[0] + sets[1]) == into_root and sets[0] and sets[1]
    ref_f = oracle.layer_forward(p, rels=into_root)
    ref_dW, ref_dH0, _ = oracle.layer_backward(p, ref_f, p.G, rels=into_root)
    layers = [make_layer(p, hg, rels=s) for s in sets]
    parts = [l.forward()[0] for l in layers]
    tot = torch.zeros_like(parts[0])
    heta.heta_cross_rel_reduce(hg, 0, parts, tot)
    assert_rows_close(tot.cpu().numpy(), ref_f.H[0], 1e-4, "sum of the partitions' partial aggregations")
    G = {0: torch.from_numpy(np.ascontiguousarray(p.G[0], dtype=np.float32)).cuda()}
    dH0 = {}
    for l, s in zip(layers, sets):
        dW, dh, _ = l.backward(G)
        for r in s:
            assert_rows_close(dW[r].cpu().numpy(), ref_dW[r], 1e-4, f"dW[{r}]")
        for t, g in dh.items():
            dH0[t] = g.cpu().numpy().astype(np.float64) + dH0.get(t, 0.0)
    assert sorted(dH0) == sorted(ref_dH0)
    for t in dH0:
        assert_rows_close(dH0[t], ref_dH0[t], 1e-4, f"dH0[{t}]")
    hg.destroy()


@pytest.mark.parametrize("mode", ["fused", "per_relation"])
@pytest.mark.parametrize("storage", ["f32", "bf16"])
def test_layer_config3_scaled(storage, mode, gemm_path):
    p = workloads.config3(storage, scale=0.02)
    got = run_layer_on_gpu(p, mode=mode)
    ref_f = oracle.layer_forward(p)
    ref_b = oracle.layer_backward(p, ref_f, p.G)
    # contract: 1e-4 / 2e-2.  Observed on this data: ~1e-6 for fp32; for bf16 storage 3.9e-3 on M_r (one
    # rounding of a stored value in [1, 2): 2^-8 absolute) and 6.1e-3 on dH0 (a few such terms per row).
    # Guarded at 1e-5 / 1e-2.
    compare_layer(p, got, ref_f, ref_b, tol=TOL[storage], observed_max=1e-2 if storage == "bf16" else 1e-5)


@pytest.mark.parametrize("storage", ["f32", "bf16"])
def test_layer_config3_scaled_device_ingest(storage):
    heta.heta_ingest_force(2)
    try:
        p = workloads.config3(storage, scale=0.02)
        got = run_layer_on_gpu(p)
    finally:
        heta.heta_ingest_force(0)
    ref_f = oracle.layer_forward(p)
    ref_b = oracle.layer_backward(p, ref_f, p.G)
    compare_layer(p, got, ref_f, ref_b, tol=TOL[storage])


@pytest.mark.parametrize("project_first", [None, False])
def test_layer_config4_scaled(gemm_path, project_first):
    """Default: relations wider than the output (300, 512, 789 -> 256) are projected first and aggregated
    at the output width; False: every relation aggregates first.  Same embeddings and gradients."""
    p = workloads.config4(scale=0.01)
    got = run_layer_on_gpu(p, project_first=project_first)
    assert (len(got["M"]) < len(p.graph.relations)) == (project_first is None)
    ref_f = oracle.layer_forward(p)
    ref_b = oracle.layer_backward(p, ref_f, p.G)
    compare_layer(p, got, ref_f, ref_b, tol=2e-2, observed_max=1e-2)


def test_explicit_project_first_is_rejected_with_a_row_map_or_a_fixed_map():
    """Project-first runs over whole source tables; with src_gid or a fixed per-type map in front it would
    project the wrong rows, so an explicit request is an error (the automatic choice never makes it)."""
    from tests.test_oracle_pins import tiny_problem
    p = tiny_problem(0, "mean", relu=False, with_gid=True)
    with pytest.raises(heta.HetaError, match="whole-table"):
        make_layer(p, project_first=[0])
    with pytest.raises(heta.HetaError, match="whole-table"):
        make_layer(workloads.config1(), project_first=[0])


def test_layer_with_relu_and_gid():
    from tests.test_oracle_pins import tiny_problem
    for seed in range(3):
        p = tiny_problem(seed, "mean", relu=True, with_gid=True)
        got = run_layer_on_gpu(p)
        ref_f = oracle.layer_forward(p)
        ref_b = oracle.layer_backward(p, ref_f, p.G)
        compare_layer(p, got, ref_f, ref_b, tol=1e-4)


@pytest.mark.parametrize("in_s,w_s", [("f32", "f32"), ("bf16", "bf16")])
@pytest.mark.parametrize("d_out,relu", [(256, False), (40, True)])
@pytest.mark.parametrize("n", [1500, 7000])   # 7000 rows: enough 128 x 128 tiles for the full-size kernels (fp32: packed weights)
def test_cross_rel_project_family(n, in_s, w_s, d_out, relu, gemm_path):
    """Fused projection + cross-relation sum over relations of different widths, and its backward."""
    widths = [7, 24, 64, 128, 300, 37]
    hg = heta.heta_graph_create([(n, 8, 0)], [])
    tol = 1e-4 if in_s == "f32" else 2e-2
    xs = [rng.normal_table(n, d, "tests", f"crx{d}") for d in widths]
    ws = [rng.normal_table(d, d_out, "tests", f"crw{d}") * np.float32(1 / np.sqrt(d)) for d in widths]
    xr = [rng.round_to_bf16(x) if in_s == "bf16" else x for x in xs]
    wr = [rng.round_to_bf16(w) if w_s == "bf16" else w for w in ws]
    ref = sum(x.astype(np.float64) @ w.astype(np.float64) for x, w in zip(xr, wr))
    dx = [dev_table(x, in_s, 8) for x in xs]
    dw = [dev_table(w, w_s, 8) for w in ws]
    out = torch.full((n, d_out), float("nan"), dtype=torch.float32, device="cuda")
    heta.heta_cross_rel_project(hg, 0, dx, dw, out, act=heta.HETA_ACT_RELU if relu else heta.HETA_ACT_NONE)
    assert_rows_close(out.cpu().numpy(), np.maximum(ref, 0) if relu else ref, tol, "fused forward")
    # beta = 1 on a split of the relation set (Proposition 1 through the fused call)
    out2 = torch.zeros((n, d_out), dtype=torch.float32, device="cuda")
    heta.heta_cross_rel_project(hg, 0, dx[:2], dw[:2], out2)
    heta.heta_cross_rel_project(hg, 0, dx[2:], dw[2:], out2, beta=1.0)
    assert_rows_close(out2.cpu().numpy(), ref, tol, "fused forward in two parts")
    g = rng.normal_table(n, d_out, "tests", "crg")
    dg = dev_table(g, "f32", 4)
    dMs = [torch.full((n, d), float("nan"), dtype=torch.float32, device="cuda") for d in widths]
    heta.heta_cross_rel_project_bwd(hg, 0, dg, dw, dMs)
    for m, w in zip(dMs, wr):
        assert_rows_close(m.cpu().numpy(), g.astype(np.float64) @ w.astype(np.float64).T, tol, "fused dM")
    if in_s == "bf16":  # dM_r kept in the storage type: one rounding of the fp32 accumulator on the way out
        hMs = [dev_table(np.full((n, d), np.nan, dtype=np.float32), "bf16", 8) for d in widths]
        heta.heta_cross_rel_project_bwd(hg, 0, dg, dw, hMs)
        for m, w in zip(hMs, wr):
            assert_rows_close(m.float().cpu().numpy(), g.astype(np.float64) @ w.astype(np.float64).T, tol, "fused dM (bf16)")
    dWs = [torch.full((d, d_out), float("nan"), dtype=torch.float32, device="cuda") for d in widths]
    heta.heta_cross_rel_project_wgrad(hg, 0, dx, dg, dWs)
    for w, x in zip(dWs, xr):
        assert_rows_close(w.cpu().numpy(), x.astype(np.float64).T @ g.astype(np.float64), tol, "fused dW")
    hg.destroy()


@pytest.mark.parametrize("in_s,w_s", [("f32", "f32"), ("bf16", "bf16")])
@pytest.mark.parametrize("n,with_handle", [(1100, False), (5000, True), (5000, False)])   # 5000 rows: full-size tiles
def test_project_batch_sum_and_wgrad_batch(n, with_handle, in_s, w_s, gemm_path):
    """The batched projection calls used when relations are projected before they are aggregated:
    independent products sharing an input, a k-concatenated sum with transposed weights, and weight
    gradients with one gradient operand each (also fed as two bf16 terms)."""
    d_in, d_out = 300, 256
    tol = 1e-4 if in_s == "f32" else 2e-2
    hg = heta.heta_graph_create([(n, 8, 0)], [])
    owner = hg if with_handle else None   # a handle lends the two handle-less calls its packing buffer
    x = rng.normal_table(n, d_in, "tests", "pbx")
    ws = [rng.normal_table(d_in, d_out, "tests", f"pbw{i}") * np.float32(1 / np.sqrt(d_in)) for i in range(3)]
    xr = rng.round_to_bf16(x) if in_s == "bf16" else x
    wr = [rng.round_to_bf16(w) if w_s == "bf16" else w for w in ws]
    dx, dw = dev_table(x, in_s, 8), [dev_table(w, w_s, 8) for w in ws]
    for out_s in (["f32", "bf16"] if in_s == "bf16" else ["f32"]):
        outs = [dev_table(np.full((n, d_out), np.nan, dtype=np.float32), out_s, 8) for _ in ws]
        heta.heta_project_batch([dx] * 3, dw, outs, graph=owner)
        for o, w in zip(outs, wr):
            assert_rows_close(o.float().cpu().numpy(), xr.astype(np.float64) @ w.astype(np.float64), tol, f"batch -> {out_s}")
    gs = [rng.normal_table(n, d_out, "tests", f"pbg{i}") * np.float32(30.0) for i in range(3)]   # "summed over edges": large
    dg = [dev_table(g, "f32", 4) for g in gs]
    prev = rng.normal_table(n, d_in, "tests", "pbprev")
    acc = dev_table(prev, "f32", 4)
    heta.heta_project_sum(dg, dw, acc, trans_w=True, beta=1.0, graph=owner)
    ref = prev.astype(np.float64) + sum(g.astype(np.float64) @ w.astype(np.float64).T for g, w in zip(gs, wr))
    assert_rows_close(acc.cpu().numpy(), ref, tol, "k-concatenated sum with W^T")
    for two in (False, True):
        dWs = [torch.full((d_in, d_out), float("nan"), dtype=torch.float32, device="cuda") for _ in ws]
        heta.heta_project_wgrad_batch(hg, [dx] * 3, dg, dWs, gout_two_terms=two)
        for w, g in zip(dWs, gs):
            refw = xr.astype(np.float64).T @ g.astype(np.float64)
            assert_rows_close(w.cpu().numpy(), refw, tol, f"wgrad batch two_terms={two}")
            if two and in_s == "bf16":   # 16 significant bits of the gradient operand: far inside the storage tolerance
                assert_rows_close(w.cpu().numpy(), refw, 2e-4, "wgrad batch, two-term gradient")
    hg.destroy()


# ---- determinism of a whole layer step ---------------------------------------------------------------

@pytest.mark.parametrize("storage", ["f32", "bf16"])
def test_whole_layer_is_bitwise_reproducible_run_to_run(storage):
    """No floating-point atomics anywhere on the path: two forward + backward passes of the whole layer
    over the same buffers give identical bits - embeddings (k-concatenated projection), every weight
    gradient (row range split over workgroups, partials added in split order) and every input gradient -
    with relations of both orders in the layer.  A second layer object on a second handle, fed the same
    inputs, must agree with the first as well."""
    p = workloads.config3(storage, scale=0.02)
    G = {t: torch.from_numpy(np.ascontiguousarray(g, dtype=np.float32)).cuda() for t, g in p.G.items()}
    runs = []
    layers = [make_layer(p, project_first=[p.graph.rel_index("rev_affiliated"), p.graph.rel_index("rev_has_topic")]) for _ in range(2)]
    for layer in (layers[0], layers[0], layers[1]):
        H = layer.forward()
        dW, dH0, _ = layer.backward(G)
        torch.cuda.synchronize()
        runs.append(([H[t].clone() for t in sorted(H)], [dW[r].clone() for r in sorted(dW)], [dH0[s].clone() for s in sorted(dH0)]))
    for other in runs[1:]:
        for fam_a, fam_b in zip(runs[0], other):
            for a, b in zip(fam_a, fam_b):
                assert torch.equal(a, b)
    for layer in layers:
        layer.g.destroy()


def test_one_full_size_relation_weight_gradient_and_projection_are_reproducible():
    """The same at the size the benchmark runs: one relation of 700 k destination rows (the split weight
    gradient with its ordered combine, the projection and its backward), twice."""
    n, d_in, d_out = 700_000, 128, 256
    hg = heta.heta_graph_create([(n, 8, 0)], [(0, 0, np.zeros(n + 1, dtype=np.int64), np.zeros(0, dtype=np.int32))])
    gen_dev = torch.Generator(device="cuda")
    gen_dev.manual_seed(5)
    for dt in (torch.float32, torch.bfloat16):
        M = torch.randn((n, d_in), generator=gen_dev, device="cuda").to(dt)
        W = (torch.randn((d_in, d_out), generator=gen_dev, device="cuda") / 11).to(dt)
        Gd = torch.randn((n, d_out), generator=gen_dev, device="cuda")
        outs = []
        for _ in range(2):
            Z = torch.empty((n, d_out), device="cuda")
            dW = torch.empty((d_in, d_out), device="cuda")
            dM = torch.empty((n, d_in), device="cuda")
            heta.heta_rel_project(hg, 0, M, W, Z)
            heta.heta_rel_project_wgrad(hg, 0, M, Gd, dW)
            heta.heta_rel_project(hg, 0, Gd, W, dM, trans_w=True)
            torch.cuda.synchronize()
            outs.append((Z, dW, dM))
        for a, b in zip(*outs):
            assert torch.equal(a, b)
    hg.destroy()


# ---- the boundary's CSC and reverse_of fields -----------------------------------------------------------

def _reverse_pair_graph(mode):
    """config 3 at a small scale with the three relations the generator built as exact transposes, ingested
    by the host path or by the device kernels."""
    from paper_2408_09697_amd.problems import relation_tuples
    p = workloads.config3("f32", scale=0.02, exact=True)
    nts = [(t.num_nodes, t.feat_dim, int(t.learnable)) for t in p.graph.ntypes]
    heta.heta_ingest_force(mode)
    try:
        declared = heta.heta_graph_create(nts, relation_tuples(p.graph, True))
        plain = heta.heta_graph_create(nts, relation_tuples(p.graph, False))
    finally:
        heta.heta_ingest_force(0)
    return p, declared, plain


@pytest.mark.parametrize("mode", [1, 2, 3], ids=["host_ingest", "device_ingest", "block_ingest"])
def test_declared_reverse_relations_share_arrays_and_give_the_same_results(mode):
    """A relation declared as the reverse of an earlier one is checked against that relation's transposed
    adjacency and (device-built) shares its arrays.  Index data read back is the oracle's for every relation;
    with integer inputs forward and backward aggregations equal those of the undeclared graph bit for bit;
    and for sum aggregation the backward of a relation is the forward of its reverse (both on the GPU)."""
    p, declared, plain = _reverse_pair_graph(mode)
    g = p.graph
    pairs = [(g.rel_index(r.reverse_of), i) for i, r in enumerate(g.relations) if r.reverse_of]
    assert len(pairs) == 3
    if mode == 2:   # device-built: the reverses hold no adjacency of their own
        assert heta.heta_graph_index_bytes(declared) < 0.75 * heta.heta_graph_index_bytes(plain)
    else:
        assert heta.heta_graph_index_bytes(declared) == heta.heta_graph_index_bytes(plain)
    d = 24
    for i, r in enumerate(g.relations):
        src, dst = r.edge_list()
        n_s, n_t = g.ntypes[r.src_type].num_nodes, g.ntypes[r.dst_type].num_nodes
        colptr, row = heta.heta_graph_get_csc(declared, i)
        rc, rr = oracle.csc(src, dst, n_s)
        assert np.array_equal(colptr, rc) and np.array_equal(row, rr), r.name
        assert np.array_equal(heta.heta_graph_get_degrees(declared, i), oracle.in_degree(src, dst, n_t)), r.name
        x = rng.small_int_table(n_s, d, -2, 2, "tests", f"rev/x/{r.name}")
        gx = rng.small_int_table(n_t, d, -2, 2, "tests", f"rev/g/{r.name}")
        outs = []
        for hg in (declared, plain):
            f = torch.empty((n_t, d), device="cuda")
            b = torch.empty((n_s, d), device="cuda")
            heta.heta_rel_aggregate_fwd(hg, i, heta.HETA_MEAN, dev_table(x, "f32", 4), f)
            heta.heta_rel_aggregate_bwd(hg, i, heta.HETA_SUM, dev_table(gx, "f32", 4), b)
            outs.append((f, b))
        assert torch.equal(outs[0][0], outs[1][0]) and torch.equal(outs[0][1], outs[1][1]), r.name
        assert_rows_close(outs[0][0].cpu().numpy(), oracle.aggregate_fwd(src, dst, n_t, x, "mean"), 1e-4, r.name)
        assert np.array_equal(outs[0][1].cpu().numpy().astype(np.float64), oracle.aggregate_bwd(src, dst, n_s, n_t, gx.astype(np.float64), "sum"))
    for j, i in pairs:   # backward of the base (sum) == forward of its reverse (sum), floating-point inputs
        n_s, n_t = g.ntypes[g.relations[j].src_type].num_nodes, g.ntypes[g.relations[j].dst_type].num_nodes
        gm = dev_table(rng.normal_table(n_t, d, "tests", f"rev/p9/{j}"), "f32", 4)
        b = torch.empty((n_s, d), device="cuda")
        f = torch.empty((n_s, d), device="cuda")
        heta.heta_rel_aggregate_bwd(declared, j, heta.HETA_SUM, gm, b)
        heta.heta_rel_aggregate_fwd(declared, i, heta.HETA_SUM, gm, f)
        assert_rows_close(f.cpu().numpy(), b.cpu().numpy().astype(np.float64), 1e-5, "bwd(base) vs fwd(reverse)")
    declared.destroy()
    plain.destroy()


@pytest.mark.parametrize("mode", [1, 2, 3], ids=["host_ingest", "device_ingest", "block_ingest"])
def test_supplied_csc_and_reverse_declarations_are_validated(mode):
    rel = skewed_relation()
    src, dst = rel.edge_list()
    colptr, row = oracle.csc(src, dst, 3000)
    nts = [(3000, 8, 0), (2000, 8, 0)]
    heta.heta_ingest_force(mode)
    try:
        hg = heta.heta_graph_create(nts, [(0, 1, rel.rowptr, rel.col, {"csc": (colptr, row)})])   # the right one is accepted
        got = heta.heta_graph_get_csc(hg, 0)
        assert np.array_equal(got[0], colptr) and np.array_equal(got[1], row)
        hg.destroy()
        # the same through device pointers
        dev = lambda a: torch.from_numpy(a).cuda()
        hg = heta.heta_graph_create(nts, [(0, 1, dev(rel.rowptr), dev(rel.col), {"csc": (dev(colptr), dev(row))})],
                                    flags=heta.HETA_PTRS_ON_DEVICE)
        hg.destroy()
        u = int(np.argmax(np.diff(colptr) >= 2))            # a column with two edges
        bad_row = row.copy()
        a = int(colptr[u])
        if bad_row[a] == bad_row[a + 1]:
            bad_row[a + 1] = (bad_row[a + 1] + 1) % 2000     # another destination
        else:
            bad_row[a], bad_row[a + 1] = bad_row[a + 1], bad_row[a]   # same edges, wrong order within the column
        bad_ptr = colptr.copy()
        bad_ptr[5] += 1
        for csc in ((colptr, bad_row), (bad_ptr, row)):
            with pytest.raises(heta.HetaError) as ei:
                heta.heta_graph_create(nts, [(0, 1, rel.rowptr, rel.col, {"csc": csc})])
            assert ei.value.status == heta.HETA_ERR_BAD_CSR and "supplied CSC" in ei.value.message
        # a declared reverse that is the transpose of something else
        other = Relation("other", 0, 1, rel.rowptr, rng.stream("tests", "revbad").permutation(rel.col))   # same degrees, other sources
        osrc, odst = other.edge_list()
        ocp, orow = oracle.csc(osrc, odst, 3000)
        with pytest.raises(heta.HetaError) as ei:
            heta.heta_graph_create(nts, [(0, 1, rel.rowptr, rel.col), (1, 0, ocp, orow, {"reverse_of": 0})])
        assert ei.value.status == heta.HETA_ERR_BAD_CSR and "transposed adjacency of relation 0" in ei.value.message
        hg = heta.heta_graph_create(nts, [(0, 1, rel.rowptr, rel.col), (1, 0, colptr, row, {"reverse_of": 0})])
        assert np.array_equal(heta.heta_graph_get_degrees(hg, 1), np.diff(colptr))
        hg.destroy()
    finally:
        heta.heta_ingest_force(0)


BLOCK_SHAPES = {
    # 12 relations over 5 node types: empty relations, relations without rows, multi-edges, a hub column of more
    # than 512 edges, a hub row
    "mixed": ([3000, 1, 0, 700, 5000],
              [(0, 3, 9000), (3, 0, 20000), (0, 0, 0), (1, 0, 2500), (0, 1, 1200), (2, 0, 0), (0, 2, 0), (4, 4, 30000), (4, 0, 7),
               (3, 4, 4000), (0, 4, 15000), (3, 3, 1)]),
    # 14 relations of 40 ... 180 rows: 1,024 consecutive rows of the block span up to ten schedules (the row kernel
    # keeps four per workgroup in LDS and sends the rest straight to the global counters); one hub row and column
    "narrow": ([90, 40, 180, 120, 60, 150],
               [(0, 1, 700), (1, 2, 9000), (2, 3, 1500), (3, 4, 400), (4, 5, 2500), (5, 0, 900), (0, 2, 1300), (2, 0, 60), (1, 1, 300),
                (3, 3, 800), (4, 0, 0), (5, 5, 2000), (0, 4, 450), (2, 5, 1100)]),
}


@pytest.mark.parametrize("shape", sorted(BLOCK_SHAPES))
def test_block_ingest_of_many_relations_matches_the_host_path_bit_for_bit(shape):
    """Blocks of 12 to 14 relations: every index array the whole-block device ingest produces is
    the host path's, read back through the public calls and through exact integer aggregations."""
    g = rng.stream("tests", "block-ingest" if shape == "mixed" else f"block-ingest/{shape}")
    n_nodes, specs = BLOCK_SHAPES[shape]
    nts = [(n, 8, 0) for n in n_nodes]
    rels, lists = [], []
    for k, (s, t, n_e) in enumerate(specs):
        n_s, n_t = n_nodes[s], n_nodes[t]
        dst = np.sort(g.integers(0, max(n_t, 1), size=n_e)).astype(np.int64)
        src = g.integers(0, max(n_s, 1), size=n_e, dtype=np.int32)
        if n_e >= 9000:
            src[: n_e // 10] = n_s // 2                       # a hub column
            dst[: 600] = 0                                     # a hub row (stays sorted: the smallest id)
        rowptr = np.zeros(n_t + 1, dtype=np.int64)
        np.add.at(rowptr, dst + 1, 1)
        rowptr = np.cumsum(rowptr)
        rels.append((s, t, rowptr, src))
        lists.append((src, dst.astype(np.int32), n_s, n_t))
    graphs = []
    for mode in (1, 3):
        heta.heta_ingest_force(mode)
        try:
            graphs.append(heta.heta_graph_create(nts, rels))
        finally:
            heta.heta_ingest_force(0)
    host, block = graphs
    for i, (src, dst, n_s, n_t) in enumerate(lists):
        a, b = heta.heta_graph_get_csc(host, i), heta.heta_graph_get_csc(block, i)
        assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1]), i
        rc, rr = oracle.csc(src, dst, n_s)
        assert np.array_equal(b[0], rc) and np.array_equal(b[1], rr), i
        assert np.array_equal(heta.heta_graph_get_degrees(block, i), oracle.in_degree(src, dst, n_t)), i
        if n_s == 0 or n_t == 0:
            continue
        x = rng.small_int_table(n_s, 12, -2, 2, "tests", f"blk/x/{i}")
        gx = rng.small_int_table(n_t, 12, -2, 2, "tests", f"blk/g/{i}")
        for hg in (host, block):
            f = torch.full((n_t, 12), float("nan"), device="cuda")
            bk = torch.full((n_s, 12), float("nan"), device="cuda")
            heta.heta_rel_aggregate_fwd(hg, i, heta.HETA_SUM, dev_table(x, "f32", 4), f)
            heta.heta_rel_aggregate_bwd(hg, i, heta.HETA_MEAN, dev_table(gx, "f32", 4), bk)
            assert np.array_equal(f.cpu().numpy().astype(np.float64), oracle.aggregate_fwd(src, dst, n_t, x, "sum")), i
            assert_rows_close(bk.cpu().numpy(), oracle.aggregate_bwd(src, dst, n_s, n_t, gx.astype(np.float64), "mean"), 1e-4, f"bwd {i}")
    assert heta.heta_graph_index_bytes(host) == heta.heta_graph_index_bytes(block)
    host.destroy()
    block.destroy()


# ---- several relations per launch ------------------------------------------------------------------
def _multi_relation_graph():
    """Seven relations over three node types: five of one shape class (so that one group spills into a second
    launch), one with hub rows, one empty; sources shared between relations for the backward rounds."""
    g = rng.stream("tests", "multi")
    n = [1500, 900, 1100]
    rels = []
    for i, (s, t, e) in enumerate([(0, 1, 9000), (1, 0, 7000), (2, 1, 4000), (0, 2, 12000), (1, 2, 3000), (2, 0, 0)]):
        deg = power_law_degrees(n[t], e, 1.5, g) if e else np.zeros(n[t], dtype=np.int64)
        rowptr = np.zeros(n[t] + 1, dtype=np.int64)
        np.cumsum(deg, out=rowptr[1:])
        rels.append(Relation(f"m{i}", s, t, rowptr, g.integers(0, n[s], size=int(rowptr[-1]), dtype=np.int32)))
    hub = skewed_relation(n_src=n[0], n_dst=n[1], n_edges=20000, name="multi_hub")
    rels.append(Relation("hub", 0, 1, hub.rowptr, hub.col))
    hg = heta.heta_graph_create([(k, 8, 0) for k in n], [(r.src_type, r.dst_type, r.rowptr, r.col) for r in rels])
    return n, rels, hg


@pytest.mark.parametrize("storage", ["f32", "bf16"])
@pytest.mark.parametrize("op", ["sum", "mean"])
def test_multi_relation_aggregation_equals_the_single_calls_bit_for_bit(storage, op):
    n, rels, hg = _multi_relation_graph()
    hop = heta.HETA_SUM if op == "sum" else heta.HETA_MEAN
    dt = torch.float32 if storage == "f32" else torch.bfloat16
    gen = torch.Generator(device="cpu").manual_seed(5)
    try:
        for widths in ([128] * 7, [128, 64, 128, 300, 7, 128, 128]):
            tabs = {(t, d): torch.randn((n[t], d), generator=gen).to(dt).cuda() for t in range(3) for d in set(widths)}
            idx = list(range(len(rels)))
            srcs = [tabs[(rels[i].src_type, widths[i])] for i in idx]
            single = [torch.full((n[rels[i].dst_type], widths[i]), 7.0, dtype=dt, device="cuda") for i in idx]
            multi = [t.clone() for t in single]
            for i in idx:
                heta.heta_rel_aggregate_fwd(hg, i, hop, srcs[i], single[i])
            heta.heta_rel_aggregate_fwd_multi(hg, idx, hop, srcs, multi)
            torch.cuda.synchronize()
            for i in idx:
                assert torch.equal(single[i].view(torch.int16 if storage == "bf16" else torch.int32),
                                   multi[i].view(torch.int16 if storage == "bf16" else torch.int32)), (widths, i)
            # forward against the oracle as well (one relation per shape class is enough: the rest are bitwise equal)
            e_src, e_dst = rels[6].edge_list()
            ref = oracle.aggregate_fwd(e_src, e_dst, n[1], srcs[6].float().cpu().numpy().astype(np.float64), op)
            assert_rows_close(multi[6].float().cpu().numpy(), ref, TOL[storage])
            # backward: relation i's gradient rows gathered into a buffer per relation, beta = 1 on top of ones
            gouts = [tabs[(rels[i].dst_type, widths[i])] for i in idx]
            gs_single = [torch.ones((n[rels[i].src_type], widths[i]), dtype=torch.float32, device="cuda") for i in idx]
            gs_multi = [t.clone() for t in gs_single]
            for i in idx:
                heta.heta_rel_aggregate_bwd(hg, i, hop, gouts[i], gs_single[i], beta=1.0)
            heta.heta_rel_aggregate_bwd_multi(hg, idx, hop, gouts, gs_multi, betas=[1.0] * len(idx))
            torch.cuda.synchronize()
            for i in idx:
                assert torch.equal(gs_single[i].view(torch.int32), gs_multi[i].view(torch.int32)), (widths, i)
        # items that write the same rows are refused before anything runs
        shared = torch.zeros((n[1], 128), dtype=dt, device="cuda")
        with pytest.raises(heta.HetaError) as ei:
            heta.heta_rel_aggregate_fwd_multi(hg, [0, 6], hop, [srcs[0], srcs[6]], [shared, shared[:, :128]])
        assert ei.value.status == heta.HETA_ERR_INVALID_ARG and "overlap" in str(ei.value)
        torch.cuda.synchronize()
        assert float(shared.float().abs().max()) == 0.0
        with pytest.raises(heta.HetaError):
            heta.heta_rel_aggregate_bwd_multi(hg, [0, 3], hop, [gouts[0], gouts[3]], [gs_multi[0], gs_multi[0]])
        heta.heta_rel_aggregate_fwd_multi(hg, [], hop, [], [])
    finally:
        hg.destroy()


@pytest.mark.parametrize("dtype,widths", [
    (torch.float32, [128, 100, 97, 128, 65]),    # one lane class, different widths: one launch of four relations and one of one
    (torch.float32, [129, 200, 256, 260, 384]),  # more than 32 chunks: column tiles, the last one ragged
    (torch.bfloat16, [256, 130, 200, 136, 256]),
    (torch.bfloat16, [264, 512, 520, 768, 257]),
    (torch.float32, [3, 4, 8, 5, 12]),
])
def test_rows_of_all_classes_share_a_launch(dtype, widths):
    """Hub, long, short and empty rows of several relations in one grid, few and many long rows (four wavefronts per
    row, or one), against sums in 64 bits: n fp32 additions in any order are off by at most n 2^-24 of the sum of
    magnitudes, one more for the mean."""
    gen = torch.Generator().manual_seed(11)
    n_src, shapes = 700, [(40, 0), (3000, 2600), (500, 3), (1, 1), (64, 0)]  # (rows, long rows)
    types, rels, lists = [(n_src, 4, 0)], [], []
    for t, (rows, long_rows) in enumerate(shapes):
        deg = torch.randint(0, 32, (rows,), generator=gen)
        deg[:long_rows] = torch.randint(32, 60, (long_rows,), generator=gen)
        if rows > 1:
            deg[-1], deg[-2], deg[-3] = 1500, 512, 0
        rowptr = torch.cat([deg.new_zeros(1), torch.cumsum(deg, 0)])
        col = torch.randint(0, n_src, (int(rowptr[-1]),), generator=gen, dtype=torch.int32)
        types.append((rows, 4, 0))
        rels.append((0, t + 1, rowptr.cuda(), col.cuda()))
        lists.append((torch.repeat_interleave(torch.arange(rows), deg), col.long(), deg))
    hg = heta.heta_graph_create(types, rels, heta.HETA_PTRS_ON_DEVICE)
    try:
        q = 16 // dtype.itemsize
        tabs = []
        for d in widths:
            x = torch.zeros((n_src, (d + q - 1) // q * q), dtype=dtype)[:, :d]
            x.copy_(torch.randn((n_src, d), generator=gen))
            tabs.append(x)
        dev = [torch.zeros((n_src, (d + q - 1) // q * q), dtype=dtype, device="cuda")[:, :d].copy_(x) for d, x in zip(widths, tabs)]
        outs = [torch.full((rows, d), 7.0, device="cuda") for (rows, _), d in zip(shapes, widths)]
        for op in (heta.HETA_SUM, heta.HETA_MEAN):
            heta.heta_rel_aggregate_fwd_multi(hg, list(range(5)), op, dev, outs)
            torch.cuda.synchronize()
            for x, out, (dst, src, deg) in zip(tabs, outs, lists):
                rows = x.double()[src]
                ref = torch.zeros((deg.numel(), x.shape[1]), dtype=torch.float64).index_add_(0, dst, rows)
                mag = torch.zeros_like(ref).index_add_(0, dst, rows.abs())
                n = deg.double().unsqueeze(1)
                bound = (n + 1) * 2.0 ** -24 * mag
                if op == heta.HETA_MEAN:
                    ref, bound = ref / n.clamp_min(1), bound / n.clamp_min(1) * (1 + 1 / n.clamp_min(1)) + 2.0 ** -23 * (ref / n.clamp_min(1)).abs()
                assert ((out.cpu().double() - ref).abs() <= bound).all(), (op, x.shape)
        # behind the accumulation, an activation on every second relation: the rows are bitwise those of the two steps
        for beta in (0.0, 1.0):
            start = [torch.randn(o.shape, generator=gen).cuda() for o in outs]
            plain, act = [x.clone() for x in start], [x.clone() for x in start]
            heta.heta_rel_aggregate_fwd_multi(hg, list(range(5)), heta.HETA_SUM, dev, plain, betas=[beta] * 5)
            heta.heta_rel_aggregate_fwd_multi_act(hg, list(range(5)), [heta.HETA_ACT_RELU if i % 2 == 0 else heta.HETA_ACT_NONE for i in range(5)],
                                                  heta.HETA_SUM, dev, act, betas=[beta] * 5)
            torch.cuda.synchronize()
            for i in range(5):
                assert torch.equal(act[i], plain[i].relu() if i % 2 == 0 else plain[i]), (beta, i)
        with pytest.raises(heta.HetaError):
            heta.heta_rel_aggregate_fwd_multi_act(hg, [0], [7], heta.HETA_SUM, dev[:1], outs[:1])
    finally:
        hg.destroy()


def test_calibration_mfma_runs_and_reports_its_flops():
    sink = torch.full((2048,), 3.0, dtype=torch.float32, device="cuda")
    assert heta.heta_calibration_mfma(heta.HETA_F32, 10, sink) == 2.0 * 32 * 32 * 2 * 16 * 10 * 4 * 512
    assert heta.heta_calibration_mfma(heta.HETA_BF16, 10, sink) == 2.0 * 32 * 32 * 16 * 16 * 10 * 4 * 512
    torch.cuda.synchronize()
    assert float(sink.abs().max()) == 0.0  # one operand is zero: the accumulators stay zero
    for dt in (heta.HETA_F32, heta.HETA_BF16):   # varying operands: the same work, finite non-zero sums
        sink.zero_()
        assert heta.heta_calibration_mfma(dt, 10, sink, varying=True) == heta.heta_calibration_mfma(dt, 10, sink)
        heta.heta_calibration_mfma(dt, 10, sink, varying=True)
        torch.cuda.synchronize()
        assert torch.isfinite(sink[:2048]).all() and (sink[:2048] != 0).any()
    with pytest.raises(heta.HetaError):
        heta.heta_calibration_mfma(heta.HETA_F32, 10, sink[:100])
    with pytest.raises(heta.HetaError):
        heta.heta_calibration_mfma(heta.HETA_F32, 0, sink)


@pytest.mark.parametrize("n,d_in,d_out,trans", [(7000, 384, 256, False), (13000, 256, 128, True), (20000, 128, 256, False),
                                                (777, 300, 40, False)])
def test_f32_products_as_six_bf16_terms_are_as_accurate_as_the_fp32_mfma(n, d_in, d_out, trans):
    """fp32 projections split every operand into three bf16 terms and feed six MFMA terms per product.  The
    claim is fp32 accuracy, so the measure is the fp32 MFMA itself (the test switch): both paths against the
    fp64 oracle on operands spread over twelve binades, entries of mixed sign."""
    g = rng.stream("tests", f"x3_{n}_{d_in}")
    x = (g.standard_normal((n, d_in)) * np.exp2(g.integers(-6, 6, size=(n, d_in)))).astype(np.float32)
    w_shape = (d_out, d_in) if trans else (d_in, d_out)
    w = (g.standard_normal(w_shape) * np.exp2(g.integers(-6, 6, size=w_shape)) / np.sqrt(d_in)).astype(np.float32)
    ref = x.astype(np.float64) @ (w.astype(np.float64).T if trans else w.astype(np.float64))
    scale = np.maximum(1.0, np.abs(ref).max(axis=1, keepdims=True))
    err = {}
    try:
        for native in (False, True):
            heta.heta_projection_f32_native(native)
            out = torch.full((n, d_out), float("nan"), dtype=torch.float32, device="cuda")
            heta.heta_project(dev_table(x, "f32", 4), dev_table(w, "f32", 4), out, trans_w=trans)
            err[native] = float((np.abs(out.cpu().numpy().astype(np.float64) - ref) / scale).max())
    finally:
        heta.heta_projection_f32_native(False)
    assert err[True] <= 1e-5 and err[False] <= 1e-5, err
    # no worse than the fp32 MFMA beyond the noise of the summation order
    assert err[False] <= 2.0 * err[True] + 1e-7, err
    hg = heta.heta_graph_create([(n, 8, 0)], [])
    # with a graph handle and enough rows for full-size tiles the weights are split once into a packing buffer and
    # the kernel splits only the features: the same bound
    if n * ((d_out + 127) // 128) > 96 * 128:
        out = torch.full((n, d_out), float("nan"), dtype=torch.float32, device="cuda")
        heta.heta_project_sum([dev_table(x, "f32", 4)], [dev_table(w, "f32", 4)], out, trans_w=trans, graph=hg)
        err_packed = float((np.abs(out.cpu().numpy().astype(np.float64) - ref) / scale).max())
        assert err_packed <= 1e-5 and err_packed <= 2.0 * err[True] + 1e-7, (err_packed, err)
    # the weight gradient takes the same path with both operands row-major over the contraction index
    try:
        gout = (g.standard_normal((n, d_out)) * np.exp2(g.integers(-6, 6, size=(n, d_out)))).astype(np.float32)
        ref_w = x.astype(np.float64).T @ gout.astype(np.float64)
        errw = {}
        for native in (False, True):
            heta.heta_projection_f32_native(native)
            dw = torch.full((d_in, d_out), float("nan"), dtype=torch.float32, device="cuda")
            heta.heta_project_wgrad_batch(hg, [dev_table(x, "f32", 4)], [dev_table(gout, "f32", 4)], [dw], n_rows=n)
            errw[native] = float(np.abs(dw.cpu().numpy().astype(np.float64) - ref_w).max() / np.abs(ref_w).max())
    finally:
        heta.heta_projection_f32_native(False)
        hg.destroy()
    assert errw[True] <= 1e-5 and errw[False] <= 2.0 * errw[True] + 1e-7, errw


@pytest.mark.parametrize("n,d_in,d_out,trans", [(12545, 128, 64, False), (13001, 100, 63, True), (30000, 17, 33, False), (12800, 300, 65, False),
                                                (16385, 64, 4, True)])
def test_f32_products_of_narrow_outputs(n, d_in, d_out, trans):
    """Up to 64 output columns take tiles of their own (256 x 64, weight gradients 128 x 64); 65 is the first width that
    does not.  The row counts leave ragged tiles and more than, and fewer than, 128 splits of the contraction."""
    test_f32_products_as_six_bf16_terms_are_as_accurate_as_the_fp32_mfma(n, d_in, d_out, trans)


@pytest.mark.parametrize("on_device", [False, True])
@pytest.mark.parametrize("mode", [0, 1, 3], ids=["by_size", "host_ingest", "block_ingest"])
def test_graphs_created_in_one_batch_equal_graphs_created_one_by_one(mode, on_device):
    """heta_graph_create_batch: three graphs of different type counts and sizes (one with a declared reverse and a
    supplied CSC, one with an empty relation), every derived array compared with the single creation bit for bit,
    the handles destroyed in an order that releases the shared memory last from the middle one."""
    g = rng.stream("tests", "create_batch")

    def relation(n_src, n_dst, e):
        deg = power_law_degrees(n_dst, e, 1.8, g) if e else np.zeros(n_dst, dtype=np.int64)
        rowptr = np.zeros(n_dst + 1, dtype=np.int64)
        np.cumsum(deg, out=rowptr[1:])
        return rowptr, g.integers(0, max(n_src, 1), size=int(rowptr[-1]), dtype=np.int32)

    sizes = [[900, 1400, 300], [5000, 2500], [64, 64, 64, 10]]
    layouts = [[(0, 1, 20000), (1, 2, 6000), (2, 0, 900)], [(0, 1, 70000), (1, 0, 0)], [(0, 1, 200), (1, 2, 300), (3, 0, 50)]]
    specs = []
    for n, rels in zip(sizes, layouts):
        specs.append(([(k, 8, 0) for k in n], [(s, t) + relation(n[s], n[t], e) for s, t, e in rels]))
    # graph 0 gets the exact transpose of its first relation, declared and with its CSC supplied
    nts0, rels0 = specs[0]
    src0, dst0 = np.repeat(np.arange(sizes[0][1]), np.diff(rels0[0][2])), rels0[0][3].astype(np.int64)
    order = np.lexsort((np.arange(len(dst0)), dst0))           # stable by source id = the unique CSC order
    colptr = np.zeros(sizes[0][0] + 1, dtype=np.int64)
    np.cumsum(np.bincount(dst0, minlength=sizes[0][0]), out=colptr[1:])
    # its own CSC is relation 0's CSR with every row's sources in ascending order (the order is part of the contract)
    row_sorted = rels0[0][3][np.lexsort((rels0[0][3], src0))]
    rels0.append((1, 0, colptr, src0[order].astype(np.int32), {"reverse_of": 0, "csc": (rels0[0][2], row_sorted)}))

    def up(spec):
        if not on_device:
            return spec, 0
        nts, rels = spec
        out = []
        for r in rels:
            ex = dict(r[4]) if len(r) > 4 else {}
            if "csc" in ex:
                ex["csc"] = (torch.from_numpy(ex["csc"][0]).cuda(), torch.from_numpy(ex["csc"][1]).cuda())
            out.append((r[0], r[1], torch.from_numpy(r[2]).cuda(), torch.from_numpy(r[3]).cuda(), ex))
        return (nts, out), heta.HETA_PTRS_ON_DEVICE

    heta.heta_ingest_force(mode)
    try:
        flags = up(specs[0])[1]
        together = heta.heta_graph_create_batch([up(s)[0] for s in specs], flags=flags)
        singles = [heta.heta_graph_create(*up(s)[0], flags=flags) for s in specs]
    finally:
        heta.heta_ingest_force(0)
    try:
        for a, b, (nts, rels) in zip(together, singles, specs):
            for i in range(len(rels)):
                ca, cb = heta.heta_graph_get_csc(a, i), heta.heta_graph_get_csc(b, i)
                assert np.array_equal(ca[0], cb[0]) and np.array_equal(ca[1], cb[1])
                assert np.array_equal(heta.heta_graph_get_degrees(a, i), heta.heta_graph_get_degrees(b, i))
                e_dst = np.repeat(np.arange(nts[rels[i][1]][0]), np.diff(rels[i][2]))
                ref_ptr, ref_row = oracle.csc(rels[i][3], e_dst, nts[rels[i][0]][0])
                assert np.array_equal(ca[0], ref_ptr) and np.array_equal(ca[1], ref_row)
                # the schedules through an integer aggregation in both directions
                d = 8
                x = torch.from_numpy(g.integers(-3, 4, size=(nts[rels[i][0]][0], d)).astype(np.float32)).cuda()
                go = torch.from_numpy(g.integers(-3, 4, size=(nts[rels[i][1]][0], d)).astype(np.float32)).cuda()
                outs = []
                for h in (a, b):
                    o = torch.zeros((nts[rels[i][1]][0], d), device="cuda")
                    gs = torch.zeros((nts[rels[i][0]][0], d), device="cuda")
                    heta.heta_rel_aggregate_fwd(h, i, heta.HETA_SUM, x, o)
                    heta.heta_rel_aggregate_bwd(h, i, heta.HETA_SUM, go, gs)
                    outs.append((o, gs))
                assert torch.equal(outs[0][0], outs[1][0]) and torch.equal(outs[0][1], outs[1][1])
        # the first and the last handle go; the middle one still works on the memory the three share
        together[0].destroy()
        together[2].destroy()
        nts, rels = specs[1]
        x = torch.ones((nts[0][0], 4), device="cuda")
        o = torch.zeros((nts[1][0], 4), device="cuda")
        heta.heta_rel_aggregate_fwd(together[1], 0, heta.HETA_SUM, x, o)
        torch.cuda.synchronize()
        assert np.array_equal(o[:, 0].cpu().numpy().astype(np.int64), np.diff(rels[0][2]))
    finally:
        for h in together + singles:
            h.destroy()
    # a bad relation anywhere fails the whole call and leaves no handle
    bad_ptr = rels0[1][2].copy()
    bad_ptr[3] = bad_ptr[4] + 1
    bad = (specs[1][0], [(0, 1, specs[1][1][0][2], specs[1][1][0][3])]), (nts0, [(rels0[1][0], rels0[1][1], bad_ptr, rels0[1][3])])
    with pytest.raises(heta.HetaError) as ei:
        heta.heta_graph_create_batch(list(bad))
    assert ei.value.status == heta.HETA_ERR_BAD_CSR
    assert heta.heta_graph_create_batch([]) == []


@pytest.mark.parametrize("kind", ["growing", "late", "compensated", "specials"])
@pytest.mark.parametrize("n,k,d_out,trans,segments", [(300, 70, 40, False, 1), (33001, 129, 256, True, 1), (120001, 100, 64, True, 2), (70001, 72, 130, False, 3), (50001, 129, 256, True, 1),
                                                      (200003, 20, 100, False, 2)])
def test_f32_products_over_a_wide_range(n, k, d_out, trans, segments, kind):
    """Every element of an fp32 operand keeps its own 24 bits, whatever stands beside it.  growing: every 16 columns (and
    every 16 rows, for the weight gradient) 2^6 larger than those before; late: rows that start with zeros; compensated:
    features spread over 2^40 whose weights make up for it; specials: rows with an infinity or a NaN, which stay alone, and
    so do the columns of the weight gradient that belong to them.  Launches of small and of packed tiles of 64 and 128
    columns, sums and independent products."""
    g = rng.stream("tests", f"range_{kind}_{n}_{k}")
    xs = [g.standard_normal((n, k)).astype(np.float32) for _ in range(segments)]
    ws = [g.standard_normal((k, d_out)).astype(np.float32) for _ in range(segments)]
    gout = g.standard_normal((n, d_out)).astype(np.float32)
    bad, bad_col = np.array([5, n // 2, n - 1]), [0, k // 2, k - 1]
    for x, w in zip(xs, ws):
        if kind == "growing":
            x *= np.exp2(6.0 * (np.arange(k) // 16) + np.arange(n)[:, None] // 16 % 13 * 6.0 - 60.0).astype(np.float32)
        if kind == "late":
            x[:, : k // 2] *= (np.arange(n)[:, None] % 3 == 0)
            x[n // 3: n // 2] = 0.0
        if kind == "compensated":
            r = np.exp2(np.linspace(-20.0, 20.0, k)[g.permutation(k)]).astype(np.float32)
            x *= r
            w /= r[:, None]
            w[k // 2] = 0.0
        if kind == "specials":
            x[bad, bad_col] = [np.inf, np.nan, -np.inf]
    specials = kind == "specials"
    good = np.setdiff1d(np.arange(n), bad) if specials else np.arange(n)
    good_col = np.setdiff1d(np.arange(k), bad_col) if specials else np.arange(k)
    up = [dev_table(x, "f32", 4) for x in xs]
    wd = [dev_table(w.T.copy() if trans else w, "f32", 4) for w in ws]
    hg = heta.heta_graph_create([(n, 8, 0)], [])
    try:
        out = torch.full((n, d_out), float("nan"), dtype=torch.float32, device="cuda")
        heta.heta_project_sum(up, wd, out, trans_w=trans, graph=hg)
        out = out.cpu().numpy()
        assert_product(out[good], [x[good] for x in xs], ws, "sum")
        assert not specials or not np.isfinite(out[bad]).any()
        outs = [torch.full((n, d_out), float("nan"), dtype=torch.float32, device="cuda") for _ in xs]
        heta.heta_project_batch(up, wd, outs, trans_w=trans, graph=hg)
        for o, x, w in zip(outs, xs, ws):
            assert_product(o.cpu().numpy()[good], [x[good]], [w], "batch")
        dws = [torch.full((k, d_out), float("nan"), dtype=torch.float32, device="cuda") for _ in xs]
        heta.heta_project_wgrad_batch(hg, up, [dev_table(gout, "f32", 4) for _ in xs], dws, n_rows=n)
        for o, x in zip(dws, xs):
            o = o.cpu().numpy()
            assert_product(o[good_col], [x.T[good_col]], [gout], "weight gradient")
            assert not specials or not np.isfinite(o[bad_col]).any()
    finally:
        hg.destroy()


@pytest.mark.parametrize("pattern", WEIGHT_PATTERNS)
@pytest.mark.parametrize("n,k,d_out,segments", [(500, 128, 128, 1), (60001, 128, 256, 1), (70001, 128, 64, 3), (40001, 256, 128, 2)])
@pytest.mark.parametrize("trans", [False, True])
def test_f32_products_with_weights_of_any_pattern(n, k, d_out, segments, trans, pattern):
    """Diagonal, block-diagonal, pruned and partly decayed weights: every output column by itself, small launches and packed
    weights, sums and independent products; the other segments' weights are ordinary."""
    g = rng.stream("tests", f"pattern_{pattern}_{n}_{d_out}")
    xs = [g.standard_normal((n, k)).astype(np.float32) for _ in range(segments)]
    ws = [patterned_weights(pattern if s == 0 else "", k, d_out, g) for s in range(segments)]
    up = [dev_table(x, "f32", 4) for x in xs]
    wd = [dev_table(w.T.copy() if trans else w, "f32", 4) for w in ws]
    hg = heta.heta_graph_create([(n, 8, 0)], [])
    try:
        out = torch.full((n, d_out), float("nan"), dtype=torch.float32, device="cuda")
        heta.heta_project_sum(up, wd, out, trans_w=trans, graph=hg)
        assert_product(out.cpu().numpy(), xs, ws, "sum")
        outs = [torch.full((n, d_out), float("nan"), dtype=torch.float32, device="cuda") for _ in xs]
        heta.heta_project_batch(up, wd, outs, trans_w=trans, graph=hg)
        for o, x, w in zip(outs, xs, ws):
            assert_product(o.cpu().numpy(), [x], [w], "batch")
    finally:
        hg.destroy()


@pytest.mark.parametrize("n", [500, 60001])
@pytest.mark.parametrize("trans", [False, True])
@pytest.mark.parametrize("value", [np.inf, np.nan])
def test_an_infinite_weight_stays_in_its_column(n, trans, value):
    k, d_out = 128, 256
    g = rng.stream("tests", f"infinite_{n}")
    x, w = g.standard_normal((n, k)).astype(np.float32), g.standard_normal((k, d_out)).astype(np.float32)
    bad = [0, 101]  # the first and an odd column
    w[[17, 90], bad] = value
    good = np.setdiff1d(np.arange(d_out), bad)
    hg = heta.heta_graph_create([(n, 8, 0)], [])
    try:
        out = torch.full((n, d_out), 7.0, dtype=torch.float32, device="cuda")
        heta.heta_project_sum([dev_table(x, "f32", 4)], [dev_table(w.T.copy() if trans else w, "f32", 4)], out, trans_w=trans, graph=hg)
        out = out.cpu().numpy()
        assert not np.isfinite(out[:, bad]).any()
        assert_product(out[:, good], [x], [w[:, good]])
    finally:
        hg.destroy()


@pytest.mark.parametrize("n", [3000, 40001])
@pytest.mark.parametrize("power", [20, 40, 100])
def test_f32_weight_gradients_beside_rows_without_gradient(n, power):
    """Rows 2^power larger than the others whose gradient is zero (a masked hub of a sum) leave nothing behind, and neither
    does a gradient 2^power larger than the others where the features are zero; the products of both are exact zeros."""
    k, d_out = 128, 64
    g = rng.stream("tests", f"masked_{n}_{power}")
    x, go = np.abs(g.standard_normal((n, k))).astype(np.float32), g.standard_normal((n, d_out)).astype(np.float32)
    hubs, masked = [3, n // 2], [n // 3, n - 2]
    x[hubs], go[hubs] = x[hubs] * np.float32(2.0 ** power), 0.0
    go[masked], x[masked] = go[masked] * np.float32(2.0 ** power), 0.0
    hg = heta.heta_graph_create([(n, 8, 0)], [])
    try:
        dw = torch.full((k, d_out), float("nan"), dtype=torch.float32, device="cuda")
        heta.heta_project_wgrad_batch(hg, [dev_table(x, "f32", 4)], [dev_table(go, "f32", 4)], [dw], n_rows=n)
        assert_product(dw.cpu().numpy(), [x.T], [go])
    finally:
        hg.destroy()


@pytest.mark.parametrize("d_in,d_out", [(128, 256), (64, 128), (100, 40)])
def test_errors_of_f32_gradients_do_not_lean_to_one_side(d_in, d_out):
    """Gradients are summed on, over splits or over the rows that a hub gathers: an error that leans to one side adds up there.
    Independent errors have a mean of 1 / sqrt(number) of their size: 0.0006 here for input gradients, at most 0.02 for weight
    gradients; an accumulator that loses more downwards shows 0.02 to 0.06 and about 0.5.  Zero rows stay positive zeros."""
    n = 65_536
    gen = torch.Generator(device="cuda").manual_seed(d_in)
    x, go, w = (torch.randn(shape, generator=gen, device="cuda") for shape in ((n, d_in), (n, d_out), (d_in, d_out)))
    go[128:400] = 0.0
    hg = heta.heta_graph_create([(n, 8, 0)], [])
    try:
        out, dw = torch.full((n, d_in), 7.0, device="cuda"), torch.full((d_in, d_out), 7.0, device="cuda")
        heta.heta_project_batch([go], [w], [out], trans_w=True, graph=hg)
        heta.heta_project_wgrad_batch(hg, [x], [go], [dw], n_rows=n)
        assert not out[128:400].view(torch.int32).any()
        for got, ref, most in ((out, go.double() @ w.double().t().contiguous(), 0.005), (dw, x.double().t().contiguous() @ go.double(), 0.1)):
            err = got.double() - ref
            assert abs(float(err.mean() / err.square().mean().sqrt())) <= most, (d_in, d_out, most)
    finally:
        hg.destroy()


@pytest.mark.parametrize("n,k,d_out", [(12801, 128, 128), (60000, 128, 64), (33001, 100, 40), (13000, 300, 65)])
def test_f32_products_of_any_launch_size_have_the_same_bits(n, k, d_out):
    """Launches of moderate size split both operands, larger ones pack the weights: a row's product is the same in both."""
    gen = torch.Generator(device="cuda").manual_seed(n)
    x = torch.randn((n, (k + 3) // 4 * 4), generator=gen, device="cuda")[:, :k]
    w = torch.randn((k, (d_out + 3) // 4 * 4), generator=gen, device="cuda")[:, :d_out]
    steps = -(-n // 64) * -(-d_out // 64) * -(-k // 16)
    assert -(-n // 128) * -(-d_out // 128) > 96 and steps <= 16384 < 8 * steps  # alone: moderate; eight times: packed
    hg = heta.heta_graph_create([(n, 8, 0)], [])
    try:
        one, many = torch.full((n, d_out), 7.0, device="cuda"), [torch.full((n, d_out), 8.0, device="cuda") for _ in range(8)]
        heta.heta_project_batch([x], [w], [one], graph=hg)
        heta.heta_project_batch([x] * 8, [w] * 8, many, graph=hg)
        for o in many:
            assert torch.equal(o, one)
    finally:
        hg.destroy()


@pytest.mark.parametrize("k", [8192, 8193, 9000])
@pytest.mark.parametrize("n", [200, 12700])
def test_f32_products_with_many_rows_of_weights(n, k):
    """More rows of weights, spread over 2^40, than a workgroup has threads for by far; small tiles and packed weights."""
    d_out = 16
    g = rng.stream("tests", f"tall_{k}")
    w = (g.standard_normal((k, d_out)) * np.exp2(np.linspace(-20.0, 20.0, k))[g.permutation(k), None]).astype(np.float32)
    x = torch.randn((n, (k + 3) // 4 * 4), generator=torch.Generator(device="cuda").manual_seed(k), device="cuda")[:, :k]
    hg = heta.heta_graph_create([(n, 8, 0)], [])
    try:
        out = torch.full((n, d_out), float("nan"), dtype=torch.float32, device="cuda")
        heta.heta_project_batch([x], [dev_table(w, "f32", 4)], [out], graph=hg)
        rows = torch.arange(0, n, max(1, n // 150))
        assert_product(out[rows.cuda()].cpu().numpy(), [x[rows.cuda()].cpu().numpy()], [w])
    finally:
        hg.destroy()


@pytest.mark.parametrize("d,storage", [(40, "f32"), (200, "f32"), (257, "f32"), (256, "bf16")])
def test_hub_rows_are_summed_in_sixteen_chains(d, storage):
    """The order of a hub row's sum does not depend on its tiling: partials of 256 edges, the q-th of sixteen chains takes
    every 16th from q on, the chains are added in order.  Whole numbers make the partials exact, so only that order rounds."""
    g = rng.stream("tests", f"hub_{d}")
    degs, n_src = [25_700, 513, 8192, 9000 + d], 500
    table = g.integers(1 << 14, 1 << 15, size=(n_src, d)) * 2 + 1
    if storage == "bf16":
        table = g.integers(128, 256, size=(n_src, d)) << g.integers(0, 9, size=(n_src, d))
    table = table.astype(np.float32)
    rowptr = np.concatenate([[0], np.cumsum(degs)]).astype(np.int64)
    col = g.integers(0, n_src, size=int(rowptr[-1]), dtype=np.int32)
    hg = heta.heta_graph_create([(n_src, 8, 0), (len(degs), 8, 0)], [(0, 1, rowptr, col)])
    try:
        out = torch.full((len(degs), d), 7.0, device="cuda")
        heta.heta_rel_aggregate_fwd(hg, 0, heta.HETA_SUM, dev_table(table, storage, 8), out)
        for row, (e0, e1) in enumerate(zip(rowptr[:-1], rowptr[1:])):
            chains = np.zeros((16, d), dtype=np.float32)
            for i, e in enumerate(range(e0, e1, 256)):
                partial = table[col[e:min(e + 256, e1)]].astype(np.float64).sum(0)
                assert partial.max() < 2.0 ** 24
                chains[i % 16] += partial.astype(np.float32)
            want = np.zeros(d, dtype=np.float32)
            for c in chains:
                want += c
            assert np.array_equal(out[row].cpu().numpy(), want), (row, d)
    finally:
        hg.destroy()


@pytest.mark.parametrize("d,storage", [(132, "f32"), (256, "f32"), (260, "f32"), (392, "f32"), (520, "f32"), (264, "bf16"), (512, "bf16"), (520, "bf16"), (1032, "bf16")])
def test_edges_of_a_long_row_of_many_chunks_are_added_in_order(d, storage):
    """More than 32 chunks: short rows are walked in tiles of 32 chunks, long rows in tiles of 64, so that their edges are added
    one after the other.  Rows of 1 to 64 edges, the first and last chunk of every tile."""
    gen = torch.Generator().manual_seed(d)
    n_src, degs = 300, [64, 33, 32, 31, 5, 1, 0, 64, 50]
    rowptr = np.concatenate([[0], np.cumsum(degs)]).astype(np.int64)
    col = torch.randint(0, n_src, (int(rowptr[-1]),), generator=gen, dtype=torch.int32)
    dt = torch.float32 if storage == "f32" else torch.bfloat16
    x = torch.randn((n_src, d), generator=gen).to(dt)
    hg = heta.heta_graph_create([(n_src, 4, 0), (len(degs), 4, 0)], [(0, 1, rowptr, col.numpy())])
    try:
        out = torch.full((len(degs), d), 7.0, device="cuda")
        heta.heta_rel_aggregate_fwd(hg, 0, heta.HETA_SUM, x.cuda(), out)
        for row, (e0, e1) in enumerate(zip(rowptr[:-1], rowptr[1:])):
            want = torch.zeros(d)
            for e in range(e0, e1):
                want += x[int(col[e])].float()
            assert torch.equal(out[row].cpu(), want), (row, d)
    finally:
        hg.destroy()


# ---- the products of several node types in one call ----------------------------------------------------------

def _padded_rand(g, n, d, dtype):
    q = 16 // torch.empty(0, dtype=dtype).element_size()
    x = torch.zeros((max(n, 1), (d + q - 1) // q * q), dtype=dtype, device="cuda")[:, :d]  # an address also without rows
    x.copy_(torch.from_numpy(g.standard_normal((max(n, 1), d)).astype(np.float32)))
    return x


def _close(got, ref, bound=None):
    """fp32 results of exact operands: what the accumulation leaves; bf16 results are rounded once, by half a unit in the last of
    eight bits (2^-8 of a value just above a power of two).  Relative to the largest value."""
    bound = bound or (1e-5 if got.dtype == torch.float32 else 2.0 ** -8 + 1e-5)
    scale = max(1.0, float(ref.abs().max())) if ref.numel() else 1.0
    err = float((got.double() - ref).abs().max()) / scale if ref.numel() else 0.0
    assert err <= bound, err


@pytest.mark.parametrize("storage", ["f32", "bf16"])
@pytest.mark.parametrize("rows", [[0, 1, 63, 64], [65, 129, 1000, 4097], [300_000, 9000, 0, 257], [40, 50, 60, 70, 80, 90, 100, 110, 120]])
def test_project_multi_against_fp64(rows, storage):
    """Sums, independent products of several widths and transposed weights, for items that share a launch (by rows, widths and
    their number: 8 calls and 16 products at most), items too large to, and items without rows."""
    g = rng.stream("tests", f"project-multi/{storage}/{rows[0]}")
    hg = heta.heta_graph_create([(1, 1, 0)], [(0, 0, np.zeros(2, dtype=np.int64), np.zeros(0, dtype=np.int32))])
    dt = torch.float32 if storage == "f32" else torch.bfloat16
    widths, depths = [7, 64, 65, 128, 200, 256, 300], [16, 24, 100, 128]
    for trans in (False, True):
        sums, singles, ref_sums, ref_singles = [], [], [], []
        for i, n in enumerate(rows):
            d_out, k = widths[i % len(widths)], 1 + i % 3
            ins = [_padded_rand(g, n, depths[(i + p) % 4], dt if not trans else torch.float32) for p in range(k)]
            Ws = [_padded_rand(g, *((d_out, x.shape[1]) if trans else (x.shape[1], d_out)), dt) for x in ins]
            out = _padded_rand(g, n, d_out, torch.float32)
            wide = [w.double().t() if trans else w.double() for w in Ws]
            # the bf16 product rounds its fp32 operand
            xs = [x.to(torch.bfloat16).double() if storage == "bf16" else x.double() for x in ins]
            relu, beta = i % 2, float(i % 3 == 1)
            total = beta * out.double() + sum(x @ w for x, w in zip(xs, wide))
            ref_sums.append(total.relu() if relu else total)
            sums.append((n, ins, Ws, out, heta.HETA_ACT_RELU if relu else heta.HETA_ACT_NONE, beta))
            many = [_padded_rand(g, *((d, depths[0]) if trans else (depths[0], d)), dt) for d in (widths[i % 7], widths[(i + 1) % 7])]
            x = _padded_rand(g, n, depths[0], dt if not trans else torch.float32)
            outs = [_padded_rand(g, n, w.shape[0 if trans else 1], dt) for w in many]
            x64 = x.to(torch.bfloat16).double() if storage == "bf16" else x.double()
            ref_singles.append([x64 @ (w.double().t() if trans else w.double()) for w in many])
            singles.append((n, [x, x], many, outs))
        heta.heta_project_multi(hg, sums, trans_w=trans, sum=True)
        heta.heta_project_multi(hg, singles, trans_w=trans)
        for item, ref in zip(sums, ref_sums):
            _close(item[3][:item[0]], ref[:item[0]])
        for item, refs in zip(singles, ref_singles):
            for o, ref in zip(item[3], refs):
                _close(o[:item[0]], ref[:item[0]])
    o = torch.zeros((64, 64), device="cuda")
    w, x = torch.zeros((64, 64), device="cuda"), torch.zeros((64, 64), device="cuda")
    with pytest.raises(heta.HetaError) as e:
        heta.heta_project_multi(hg, [(64, [x], [w], [o]), (64, [x], [w], [o])])
    assert e.value.status == heta.HETA_ERR_INVALID_ARG
    hg.destroy()


@pytest.mark.parametrize("n,k,d_out,n_seg", [(70_001, 1000, 33, 1), (70_001, 520, 100, 1), (130_000, 264, 65, 2), (530_000, 104, 72, 1), (70_001, 520, 200, 1),
                                             (270_000, 72, 300, 1), (70_001, 272, 257, 3), (70_001, 200, 321, 2), (1000, 40, 100, 2)])
def test_packed_bf16_weights_against_fp64(n, k, d_out, n_seg):
    """bf16 weights rewritten as octets: every tile that takes them, ragged rows, columns and k-values, forward and (heta_project_multi,
    from 48 k steps of 64 x 64 x 16 on) transposed, sums and products sharing their input.  Operands exact in bf16: what remains is the
    fp32 accumulation."""
    g = torch.Generator(device="cuda").manual_seed(n + k)
    hg = heta.heta_graph_create([(1, 1, 0)], [(0, 0, np.zeros(2, dtype=np.int64), np.zeros(0, dtype=np.int32))])
    rand = lambda *shape: torch.randn(shape, generator=g, device="cuda").to(torch.bfloat16)  # noqa: E731
    for trans in (False, True):
        Ws = [rand(d_out, k) if trans else rand(k, d_out if n_seg == 1 else (d_out + 7) // 8 * 8)[:, :d_out] for _ in range(n_seg)]
        wide = [(w.t() if trans else w).double() for w in Ws]
        xs = [rand(n, k) for _ in range(n_seg)]
        if trans:
            xs = [x.float() for x in xs]
        out = torch.full((n, d_out), 2.0, device="cuda")
        heta.heta_project_sum(xs, Ws, out, trans_w=trans, beta=1.0, graph=hg)
        _close(out, 2.0 + sum(x.double() @ w for x, w in zip(xs, wide)))
        outs = [torch.full((n, d_out), float("nan"), device="cuda") for _ in Ws]
        heta.heta_project_batch([xs[0]] * n_seg, Ws, outs, trans_w=trans, graph=hg)
        for o, w in zip(outs, wide):
            _close(o, xs[0].double() @ w)
        if trans:  # the single calls leave transposed weights as they are
            out.fill_(2.0)
            heta.heta_project_multi(hg, [(n, xs, Ws, out, heta.HETA_ACT_NONE, 1.0)], trans_w=True, sum=True)
            _close(out, 2.0 + sum(x.double() @ w for x, w in zip(xs, wide)))
            outs = [o.fill_(float("nan")) for o in outs]
            heta.heta_project_multi(hg, [(n, [xs[0]] * n_seg, Ws, outs)], trans_w=True)
            for o, w in zip(outs, wide):
                _close(o, xs[0].double() @ w)
    hg.destroy()


def test_transposed_bf16_products_take_no_buffer_of_the_handle():
    """A first call can be captured: it allocates nothing.  Replays against the eager result."""
    g = torch.Generator(device="cuda").manual_seed(9)
    hg = heta.heta_graph_create([(1, 1, 0)], [(0, 0, np.zeros(2, dtype=np.int64), np.zeros(0, dtype=np.int32))])
    n, k, d = 100_000, 128, 256  # 50,016 steps of 64 x 64 x 16
    x = torch.randn((n, k), generator=g, device="cuda")
    w = torch.randn((d, k), generator=g, device="cuda").to(torch.bfloat16)
    total, each = torch.empty((n, d), device="cuda"), torch.empty((n, d), device="cuda")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        heta.heta_project_sum([x], [w], total, trans_w=True, graph=hg)
        heta.heta_project_batch([x], [w], [each], trans_w=True, graph=hg)
    eager = torch.empty_like(total)
    for turn in range(3):
        x.mul_(0.5)
        total.zero_(), each.zero_()
        graph.replay()
        heta.heta_project_sum([x], [w], eager, trans_w=True, graph=hg)
        torch.cuda.synchronize()
        assert torch.equal(total, eager) and torch.equal(each, eager), turn
    hg.destroy()


@pytest.mark.parametrize("storage", ["f32", "bf16"])
@pytest.mark.parametrize("rows", [[1, 0, 31, 33], [127, 1000, 4097, 20_000], [200_000, 129, 64, 5000]])
def test_wgrad_multi_against_fp64(rows, storage):
    """Weight gradients of several node types: calls of one kind share a launch, of few and many rows, wide and narrow inputs
    and outputs; a call without rows leaves zeros."""
    g = rng.stream("tests", f"wgrad-multi/{storage}/{rows[0]}")
    hg = heta.heta_graph_create([(1, 1, 0)], [(0, 0, np.zeros(2, dtype=np.int64), np.zeros(0, dtype=np.int32))])
    dt = torch.float32 if storage == "f32" else torch.bfloat16
    for d_out in (40, 64, 128, 256):
        items, refs = [], []
        for i, n in enumerate(rows):
            d_ins = [[16], [128, 24], [300, 128], [64, 64, 100]][i % 4]
            ins, go = [_padded_rand(g, n, d, dt) for d in d_ins], [_padded_rand(g, n, d_out, torch.float32) for _ in d_ins]
            items.append((n, ins, go, [torch.full((d, d_out), 7.0, device="cuda") for d in d_ins]))
            refs.append([x[:n].double().t() @ y[:n].double() for x, y in zip(ins, go)])
        heta.heta_project_wgrad_multi(hg, items, gout_two_terms=True)
        for item, ref in zip(items, refs):
            for w, r in zip(item[3], ref):
                # bf16 inputs are exact; the gradient as two bf16 terms is off by 2^-16 of itself, as one by 2^-8
                _close(w, r, None if storage == "f32" else 2.0 ** -15)
        if storage == "bf16":  # one term: the gradient rounded once
            heta.heta_project_wgrad_multi(hg, items)
            for n, ins, go, dW in items:
                for w, x, y in zip(dW, ins, go):
                    _close(w, x[:n].double().t() @ y[:n].to(torch.bfloat16).double())
    hg.destroy()


@pytest.mark.parametrize("in_dt,w_dt", [(torch.bfloat16, torch.float32), (torch.float32, torch.bfloat16), (torch.bfloat16, torch.bfloat16)])
@pytest.mark.parametrize("pad", [0, 1])
def test_project_multi_of_mixed_types_against_fp64(in_dt, w_dt, pad):
    """Every pair of element types, whichever kernel takes it (pad: rows that no 16-byte load takes), items of unequal rows: sums
    with beta and ReLU, and independent products.  The product rounds both operands to bf16; what remains is the accumulation."""
    g = torch.Generator(device="cuda").manual_seed(11 + pad)
    hg = heta.heta_graph_create([(1, 1, 0)], [(0, 0, np.zeros(2, dtype=np.int64), np.zeros(0, dtype=np.int32))])
    rand = lambda n, d, dt: torch.randn((n, d + 7 & ~7 if not pad else d + 1), generator=g, device="cuda").to(dt)[:, :d]  # noqa: E731
    wide = lambda x: x.to(torch.bfloat16).double()  # noqa: E731
    for trans in (False, True):
        for d_out in (40, 128, 264):
            sums, batch, refs = [], [], []
            for i, (n, k) in enumerate(((1000, 64), (3, 128), (70, 100), (517, 64))):
                ins = [rand(n, k, in_dt) for _ in range(1 + i % 2)]
                Ws = [rand(d_out, k, w_dt) if trans else rand(k, d_out, w_dt) for _ in ins]
                each = [wide(x) @ (wide(w).t() if trans else wide(w)) for x, w in zip(ins, Ws)]
                out = rand(n, d_out, torch.float32)
                total = sum(each) + (out.double() if i == 2 else 0.0)
                refs.append((each, total.relu() if i == 1 else total))
                sums.append((n, ins, Ws, out, heta.HETA_ACT_RELU if i == 1 else heta.HETA_ACT_NONE, float(i == 2)))
                batch.append((n, ins, Ws, [torch.full((n, d_out), 7.0, device="cuda") for _ in ins]))
            heta.heta_project_multi(hg, sums, trans_w=trans, sum=True)
            heta.heta_project_multi(hg, batch, trans_w=trans)
            for one, many, (each, total) in zip(sums, batch, refs):
                _close(one[3], total)
                for o, r in zip(many[3], each):
                    _close(o, r)
    hg.destroy()


@pytest.mark.parametrize("storage", ["f32", "bf16"])
def test_wgrad_multi_of_rows_far_apart(storage):
    """Rows 8 MB apart (columns of a very wide matrix), which the direct pipeline does not take, beside ordinary ones of other
    split counts: each the bits of its own call."""
    g = torch.Generator(device="cuda").manual_seed(5)
    hg = heta.heta_graph_create([(1, 1, 0)], [(0, 0, np.zeros(2, dtype=np.int64), np.zeros(0, dtype=np.int32))])
    dt = torch.float32 if storage == "f32" else torch.bfloat16
    far = torch.empty((140, 1 << 21), device="cuda")
    rand = lambda n, d, dtype=torch.float32: torch.randn((n, d), generator=g, device="cuda").to(dtype)  # noqa: E731
    items = []
    for n, wide in ((2000, False), (140, True), (300, False), (33, True)):
        go = rand(n, 128)
        if wide:
            at = 256 * len(items)
            far[:n, at:at + 128] = go
            go = far[:n, at:at + 128]
        items.append((n, [rand(n, 64, dt)], [go], [torch.full((64, 128), 7.0, device="cuda")]))
    heta.heta_project_wgrad_multi(hg, items, gout_two_terms=True)
    for n, ins, gouts, dW in items:
        one = [torch.empty_like(dW[0])]
        heta.heta_project_wgrad_batch(hg, ins, gouts, one, gout_two_terms=True)
        assert torch.equal(one[0], dW[0]), n
        ref = ins[0].double().t() @ gouts[0].double()
        assert float((dW[0].double() - ref).abs().max()) <= 1e-4 * float(ref.abs().max())  # two bf16 terms: 2^-16 of every product
    hg.destroy()


@pytest.mark.parametrize("storage", ["f32", "bf16"])
@pytest.mark.parametrize("widths", [(64, 40), (100, 128), (200, 256)])
def test_products_do_not_depend_on_what_shares_their_launch(widths, storage):
    """Items of every form (small, moderate, with packed weights) together, and each by itself, bit for bit."""
    g = torch.Generator(device="cuda").manual_seed(widths[0])
    hg = heta.heta_graph_create([(1, 1, 0)], [(0, 0, np.zeros(2, dtype=np.int64), np.zeros(0, dtype=np.int32))])
    dt = torch.float32 if storage == "f32" else torch.bfloat16
    rand = lambda *shape, dtype=torch.float32: torch.randn(shape, generator=g, device="cuda").to(dtype)  # noqa: E731
    for trans in (False, True):
        a_dt = torch.float32 if trans else dt
        for total in (True, False):
            items = []
            for i, n in enumerate([300, 9000, 50_000, 20_000, 100_000, 77]):
                ins = [rand(n, 128, dtype=a_dt) for _ in range(1 + i % 2)]
                Ws = [rand(*((widths[i % 2], 128) if trans else (128, (widths[i % 2] + 7) // 8 * 8)), dtype=dt)[:, :128 if trans else widths[i % 2]] for _ in ins]
                outs = rand(n, widths[i % 2]) if total else [rand(n, widths[i % 2]) for _ in ins]
                items.append((n, ins, Ws, outs, i % 2, float(i % 3 == 0)) if total else (n, ins, Ws, outs))
            alone = [it[:3] + (it[3].clone() if total else [o.clone() for o in it[3]],) + it[4:] for it in items]
            heta.heta_project_multi(hg, items, trans_w=trans, sum=total)
            for it, one in zip(items, alone):
                heta.heta_project_multi(hg, [one], trans_w=trans, sum=total)
                for a, b in zip([it[3]] if total else it[3], [one[3]] if total else one[3]):
                    assert torch.equal(a, b), (trans, total, it[0])
    items = []
    for n, d_in in ((90, 128), (3000, 128), (16_000, 100), (40_000, 24), (120_000, 128)):
        items.append((n, [rand(n, d_in, dtype=dt) if dt == torch.float32 else _padded_rand(rng.stream("tests", f"share/{n}"), n, d_in, dt)],
                      [rand(n, widths[0])], [torch.empty((d_in, widths[0]), device="cuda")]))
    heta.heta_project_wgrad_multi(hg, items, gout_two_terms=True)
    for n, ins, gouts, dW in items:
        one = [torch.empty_like(w) for w in dW]
        heta.heta_project_wgrad_batch(hg, ins, gouts, one, gout_two_terms=True)
        assert all(torch.equal(a, b) for a, b in zip(dW, one)), n
    hg.destroy()


def test_packed_input_gradients_of_narrow_outputs_change_sign_every_256_rows():
    """The row blocks that form the negative product are 256 rows high whatever the tile: one row repeated gives one result per
    block, and the two kinds of block differ in the last bits."""
    g = torch.Generator(device="cuda").manual_seed(3)
    hg = heta.heta_graph_create([(1, 1, 0)], [(0, 0, np.zeros(2, dtype=np.int64), np.zeros(0, dtype=np.int32))])
    n = 160_000  # 2,500 x 8 steps of 64 x 64 x 16: packed
    x = torch.randn((1, 128), generator=g, device="cuda").expand(n, 128).contiguous()
    w = torch.randn((64, 128), generator=g, device="cuda")
    out = torch.empty((n, 64), device="cuda")
    heta.heta_project_sum([x], [w], out, trans_w=True, graph=hg)
    blocks = out.view(-1, 256, 64)
    assert torch.equal(blocks, blocks[:, :1].expand_as(blocks))
    assert torch.equal(blocks[2:], blocks[:-2]) and not torch.equal(blocks[0], blocks[1])
    hg.destroy()


@pytest.mark.parametrize("mode", [0, 1, 3])
def test_offsets_of_a_relation_without_destinations_are_checked(mode):
    heta.heta_ingest_force(mode)
    try:
        rels = lambda at: [(0, 1, torch.tensor([0, 1, 2], device="cuda"), torch.tensor([0, 1], dtype=torch.int32, device="cuda")),  # noqa: E731
                           (0, 2, torch.tensor([at], device="cuda"), torch.zeros(0, dtype=torch.int32, device="cuda"))]
        heta.heta_graph_create([(2, 4, 0), (2, 4, 0), (0, 4, 0)], rels(0), heta.HETA_PTRS_ON_DEVICE).destroy()
        with pytest.raises(heta.HetaError) as e:
            heta.heta_graph_create([(2, 4, 0), (2, 4, 0), (0, 4, 0)], rels(5), heta.HETA_PTRS_ON_DEVICE)
        assert e.value.status == heta.HETA_ERR_BAD_CSR
    finally:
        heta.heta_ingest_force(0)


def test_items_that_meet_in_memory_are_refused_and_column_slices_accepted():
    g = torch.Generator(device="cuda").manual_seed(2)
    n = 96
    hg = heta.heta_graph_create([(n, 1, 0)] * 2, [(0, 0, np.zeros(n + 1, dtype=np.int64), np.zeros(0, dtype=np.int32))])
    rand = lambda *shape: torch.randn(shape, generator=g, device="cuda")  # noqa: E731
    x, w, wide = [rand(n, 64) for _ in range(2)], [rand(64, 64) for _ in range(2)], torch.full((n, 160), 7.0, device="cuda")
    part = [wide[:, :64], wide[:, 96:]]
    other = [rand(n, 64) for _ in range(2)]
    refused = [
        lambda: heta.heta_project_multi(hg, [(n, [x[0]], [w[0]], [other[0]]), (n, [other[0]], [w[1]], [other[1]])]),
        lambda: heta.heta_project_multi(hg, [(n, [x[0]], [w[0]], [other[0]]), (n, [x[1]], [other[0][:64]], [other[1]])]),
        lambda: heta.heta_project_multi(hg, [(n, [x[0]], [w[0]], wide[:, :64]), (n, [x[1]], [w[1]], wide[:, 63:127])], sum=True),
        lambda: heta.heta_project_multi(hg, [(n - 1, [x[0]], [w[0]], wide[1:, 96:]), (n, [x[1]], [w[1]], wide[:, 60:124])], sum=True),
        lambda: heta.heta_project_wgrad_multi(hg, [(n, [x[0]], [x[1]], [other[0][:64]]), (n, [x[0]], [other[0]], [other[1][:64]])]),
        lambda: heta.heta_cross_rel_reduce_multi(hg, [(0, [x[0], x[1]], other[0]), (1, [x[0], other[0]], other[1])]),
    ]
    for call in refused:
        with pytest.raises(heta.HetaError) as e:
            call()
        assert e.value.status == heta.HETA_ERR_INVALID_ARG
    heta.heta_project_multi(hg, [(n, [a], [b], o) for a, b, o in zip(x, w, part)], sum=True)
    for a, b, o in zip(x, w, part):
        _close(o, a.double() @ b.double())
    heta.heta_cross_rel_reduce_multi(hg, [(t, [x[t], w[0].new_zeros((n, 64))], part[t]) for t in range(2)])
    assert all(torch.equal(o, a) for o, a in zip(part, x)) and bool((wide[:, 64:96] == 7.0).all())
    hg.destroy()


def test_scratch_release_gives_recycled_blocks_back():
    """Workspaces of destroyed handles stay with the library for the next one, until they are asked back."""
    x, go = torch.randn((60_000, 768), device="cuda"), torch.randn((60_000, 1024), device="cuda")
    dW = torch.empty((768, 1024), device="cuda")

    def handles(n):
        hgs = []
        for _ in range(n):
            hgs.append(heta.heta_graph_create([(1, 1, 0)], [(0, 0, np.zeros(2, dtype=np.int64), np.zeros(0, dtype=np.int32))]))
            heta.heta_project_wgrad_batch(hgs[-1], [x], [go], [dW])
        free = torch.cuda.mem_get_info()[0]
        for hg in hgs:
            hg.destroy()
        return free

    handles(1)  # what the first call loads stays
    heta.heta_scratch_release()
    before = torch.cuda.mem_get_info()[0]
    assert before - handles(3) >= 3 * dW.numel() * 4  # one partial sum each at least
    heta.heta_scratch_release()
    assert before - torch.cuda.mem_get_info()[0] <= 4 << 20  # what the runtime keeps for itself


@pytest.mark.parametrize("d,n_items", [(64, 4), (7, 3), (100, 17)])
def test_act_bwd_multi(d, n_items):
    """Gradients of several node types behind a ReLU, vectorised or not, in one launch or (more than 16) one by one."""
    g = rng.stream("tests", f"act-multi/{d}")
    rows = [1 + (97 * i * i) % 1000 for i in range(n_items)]
    h, go = ([torch.from_numpy(g.standard_normal((n, d)).astype(np.float32)).cuda() for n in rows] for _ in range(2))
    gi = [torch.full_like(x, 5.0) for x in go]
    if n_items == 4:  # one of them at an odd address
        go[1] = torch.cat([go[1].new_zeros(1), go[1].flatten()])[1:].view(rows[1], d)
    heta.heta_act_bwd_multi(heta.HETA_ACT_RELU, h, go, gi)
    for a, b, c in zip(h, go, gi):
        assert torch.equal(c, torch.where(a > 0, b, torch.zeros_like(b)))
