"""GPU parity of the device neighbour sampler against oracle/sampler.py: index work, so every array is
compared bit for bit (block row offsets, sampled global source ids in order, ascending unique source
sets, local ids), and the blocks the sequencer builds are checked against the oracle's blocks and then
run through a layer."""
import ctypes

import numpy as np
import pytest
import torch

import paper_2408_09697_amd as heta
from gen import rng, workloads
from gen.graphs import HetGraph, NodeType, power_law_relation, uniform_relation
from oracle import sampler as osampler
from tests.harness import make_graph

pytestmark = pytest.mark.gpu


def _graph(kind):
    wl = f"tests/sampler/{kind}"
    nts = [NodeType("s", 3000, 4, False), NodeType("t", 2500, 4, False)]
    G = HetGraph(nts)
    if kind == "uniform":
        G.relations.append(uniform_relation("r", 0, 1, 3000, 2500, 20000, wl))
    else:
        G.relations.append(power_law_relation("r", 0, 1, 3000, 2500, 80000, 1.6, wl))
    return G


@pytest.mark.parametrize("kind", ["uniform", "skew"])
@pytest.mark.parametrize("fanout", [1, 5, 25, 64])
def test_sample_neighbors_bit_exact(kind, fanout):
    G = _graph(kind)
    r = G.relations[0]
    hg = heta.heta_graph_create([(3000, 4, 0), (2500, 4, 0)], [(0, 1, r.rowptr, r.col)])
    g = rng.stream("tests", f"sampler/{kind}/{fanout}")
    deg = np.diff(r.rowptr)
    ids = np.concatenate([g.permutation(2500)[:700], [int(np.argmax(deg))] * 2, np.flatnonzero(deg == 0)[:3]]).astype(np.int64)
    for seed in (0, 0xDEADBEEFCAFEF00D):
        rowptr, src = heta.heta_sample_neighbors(hg, 0, torch.from_numpy(ids).cuda(), fanout, seed)
        ref_ptr, ref_src = osampler.sample_neighbors(r.rowptr, r.col, ids, fanout, seed)
        assert np.array_equal(rowptr.cpu().numpy(), ref_ptr)
        assert np.array_equal(src.cpu().numpy(), ref_src)
    # empty frontier, and ids out of range are refused
    rowptr, src = heta.heta_sample_neighbors(hg, 0, torch.zeros(0, dtype=torch.int64, device="cuda"), fanout, 1)
    assert rowptr.cpu().tolist() == [0] and src.numel() == 0
    with pytest.raises(heta.HetaError, match="outside"):
        heta.heta_sample_neighbors(hg, 0, torch.tensor([3, 2500], dtype=torch.int64, device="cuda"), fanout, 1)
    with pytest.raises(heta.HetaError, match="fanout"):
        heta.heta_sample_neighbors(hg, 0, torch.tensor([3], dtype=torch.int64, device="cuda"), 65, 1)
    hg.destroy()


@pytest.mark.parametrize("limits", [[1, 64, 65], [16383, 16384, 16385, 5], [3_000_000, 40], [67_000_000], [80_000_000, 100_000_000]],
                         ids=["words", "tiles", "many_tiles", "largest_bitmap", "sorted"])
@pytest.mark.parametrize("n", [1, 777, 70_000])
def test_unique_relabel_over_id_ranges(limits, n):
    """Ranges at the edges of a 64-bit word and of a tile of 16,384 ids, an empty set between two others, the largest
    ranges that go by bitmap and the first that are sorted; skewed ids (one of them half of all) and both range ends."""
    g = np.random.default_rng(n + len(limits))
    groups = []
    for lim in limits:
        ids = g.integers(0, lim, n)
        ids[g.random(n) < 0.5] = lim // 3
        groups.append([np.concatenate([ids, [lim - 1, 0]]), g.integers(0, min(lim, 100), n // 2)])
    groups.insert(1, [np.zeros(0, dtype=np.int64)])
    bounds = [limits[0], 7] + limits[1:]
    out = heta.heta_unique_relabel_batch([[torch.from_numpy(x.astype(np.int64)).cuda() for x in grp] for grp in groups], bounds)
    for grp, (u, ls) in zip(groups, out):
        ref_u, ref_l = osampler.unique_relabel(grp)
        assert np.array_equal(u.cpu().numpy(), ref_u)
        for a, b in zip(ls, ref_l):
            assert np.array_equal(a.cpu().numpy(), b)
    with pytest.raises(heta.HetaError, match="outside"):
        heta.heta_unique_relabel_batch([[torch.tensor([0, limits[0]], device="cuda")]], [limits[0]])


@pytest.mark.parametrize("n", [1, 511, 513, 4096, 4097, 16_383, 16_384, 70_000])
def test_unique_relabel_of_ids_that_share_words(n):
    """Up to 4,096 ids are marked one by one, more through a copy of a small set (ranges of at most 262,144 ids, four ids
    and more per 64 of them) or 512 at a time through a table of 1,024 words: one id, one word, a word per id (some find
    no slot in their probes), a hub between others, and an id outside the range among the others."""
    g = np.random.default_rng(n)
    spread = np.arange(n) * 64 % 700_000
    hub = np.where(g.random(n) < 0.5, 4711, g.integers(0, 700_000, n))
    for ids, limit in ((np.full(n, 63), 64), (g.integers(0, 64, n), 64), (g.integers(0, 1000, n), 1000), (g.integers(0, 262_144, n), 262_144),
                       (g.integers(0, 262_145, n), 262_145), (spread, 700_000), (hub, 700_000)):
        (u, (l,)), = heta.heta_unique_relabel_batch([[torch.from_numpy(ids.astype(np.int64)).cuda()]], [limit])
        ref_u, (ref_l,) = osampler.unique_relabel([ids])
        assert np.array_equal(u.cpu().numpy(), ref_u) and np.array_equal(l.cpu().numpy(), ref_l)
        bad = ids.astype(np.int64)
        bad[n // 2] = limit
        with pytest.raises(heta.HetaError, match="outside"):
            heta.heta_unique_relabel_batch([[torch.from_numpy(bad).cuda()]], [limit])


@pytest.mark.parametrize("limit,share", [(1_100_000, 0.5), (64, 0.0)])
def test_unique_relabel_of_a_hub_takes_no_longer_than_of_spread_ids(limit, share):
    """Every sampled copy of an id marks the same word.  Updated one by one they took 2.6 and 3.0 ms, some 15 and 18 times
    as long as a million ids spread over 1.1 M."""
    n = 1_000_000
    spread = torch.randint(1_100_000, (n,), device="cuda")
    ids = torch.randint(limit, (n,), device="cuda")
    ids[torch.rand(n, device="cuda") < share] = limit // 3

    def best(x, lim):
        start, end, times = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True), []
        for _ in range(8):
            start.record()
            heta.heta_unique_relabel_batch([[x]], [lim])
            end.record()
            torch.cuda.synchronize()
            times.append(start.elapsed_time(end))
        return min(times)

    assert best(ids, limit) <= 3.0 * best(spread, 1_100_000)


@pytest.mark.parametrize("n", [5, 4000])
@pytest.mark.parametrize("where", ["unique", "unique_of_another_set", "local"])
def test_unique_relabel_into_the_memory_of_its_lists(where, n):
    """The C call may write the unique ids, or the local ids, over the id lists that it was given."""
    g = np.random.default_rng(n)
    lists = [g.integers(0, 3000, n), g.integers(500, 3500, n)]
    buf = torch.from_numpy(np.concatenate(lists).astype(np.int64)).cuda()   # set 0's list, then set 1's
    src = [buf.data_ptr(), buf.data_ptr() + 8 * n]
    spare = torch.empty(4 * n, dtype=torch.int64, device="cuda")
    uniq = [spare.data_ptr(), spare.data_ptr() + 8 * n]
    local = [spare.data_ptr() + 16 * n, spare.data_ptr() + 24 * n]
    if where == "local":
        local = src
    else:
        uniq = src if where == "unique" else src[::-1]
    arr = lambda kind, x: (kind * len(x))(*x)  # noqa: E731
    count = (ctypes.c_int64 * 2)()
    lib = heta.binding.load_library()
    lib.heta_unique_relabel_batch.argtypes = [ctypes.c_int32] + [ctypes.c_void_p] * 8
    torch.cuda.synchronize()
    status = lib.heta_unique_relabel_batch(2, arr(ctypes.c_int32, [0, 1, 2]), arr(ctypes.c_void_p, src), arr(ctypes.c_int64, [n, n]),
                                           arr(ctypes.c_int64, [3500, 3500]), arr(ctypes.c_void_p, uniq), count, arr(ctypes.c_void_p, local), None)
    assert status == 0
    both = [buf.cpu().numpy(), spare.cpu().numpy()]

    def at(ptr, dtype, k):
        of = 0 if buf.data_ptr() <= ptr < buf.data_ptr() + 16 * n else 1
        off = ptr - (buf, spare)[of].data_ptr()
        return both[of].view(np.uint8)[off:off + k * np.dtype(dtype).itemsize].view(dtype)

    for j in range(2):
        ref_u, (ref_l,) = osampler.unique_relabel([lists[j]])
        assert count[j] == ref_u.size
        assert np.array_equal(at(uniq[j], np.int64, count[j]), ref_u)
        assert np.array_equal(at(local[j], np.int32, n), ref_l)


def test_unique_relabel_bit_exact():
    g = rng.stream("tests", "sampler/unique")
    lists = [g.integers(0, 50000, 30000), np.zeros(0, dtype=np.int64), g.integers(0, 50000, 7), g.integers(49990, 50000, 5000)]
    uniq, local = heta.heta_unique_relabel([torch.from_numpy(l.astype(np.int64)).cuda() for l in lists], 50000)
    ref_u, ref_l = osampler.unique_relabel(lists)
    assert np.array_equal(uniq.cpu().numpy(), ref_u)
    for a, b in zip(local, ref_l):
        assert np.array_equal(a.cpu().numpy(), b)
    uniq, local = heta.heta_unique_relabel([torch.zeros(0, dtype=torch.int64, device="cuda")], 10)
    assert uniq.numel() == 0 and local[0].numel() == 0
    with pytest.raises(heta.HetaError, match="outside"):
        heta.heta_unique_relabel([torch.tensor([1, 10], dtype=torch.int64, device="cuda")], 10)


def test_sampled_blocks_match_the_oracle_and_run_a_layer():
    base = workloads.academic_graph(scale=0.02, workload="tests/sampler/blocks")
    T = len(base.ntypes)
    rels = [(r.src_type, r.dst_type, r.rowptr, r.col) for r in base.relations]
    hg = heta.heta_graph_create([(t.num_nodes, t.feat_dim, int(t.learnable)) for t in base.ntypes], rels)
    seeds = np.sort(rng.stream("tests", "sampler/seeds").choice(base.ntypes[0].num_nodes, 256, replace=False)).astype(np.int64)
    fanouts, seed = [25, 20], 20240809
    blocks = heta.sampler.sample_blocks(hg, 0, torch.from_numpy(seeds).cuda(), fanouts, seed)
    ref = osampler.sample_blocks(T, rels, 0, seeds, fanouts, seed)
    assert len(blocks) == len(ref) == 2
    for b, rb in zip(blocks, ref):
        for t in range(T):
            assert np.array_equal(b.src_ids[t].cpu().numpy(), rb["src_ids"][t])
            if rb["dst_ids"][t] is None:
                assert b.dst_ids[t] is None
            else:
                assert np.array_equal(b.dst_ids[t].cpu().numpy(), rb["dst_ids"][t])
        for i, (ptr, loc) in enumerate(rb["rels"]):
            assert np.array_equal(b.rowptr[i].cpu().numpy(), ptr)
            assert np.array_equal(b.col[i].cpu().numpy(), loc)
    # the outermost block drives one aggregation through its local -> global maps: sums of a table of
    # ones count the sampled in-edges of every destination
    b = blocks[0]
    for i, (s, t, _) in enumerate(hg.rels):
        n_dst = b.graph.n_dst(i)
        if n_dst == 0:
            continue
        table = torch.ones((hg.ntypes[s][0], 8), dtype=torch.float32, device="cuda")
        out = torch.empty((n_dst, 8), dtype=torch.float32, device="cuda")
        heta.heta_rel_aggregate_fwd(b.graph, i, heta.HETA_SUM, table, out, src_gid=b.src_ids[s])
        want = np.diff(ref[0]["rels"][i][0]).astype(np.float32)
        assert np.array_equal(out.cpu().numpy(), np.repeat(want[:, None], 8, axis=1))
    for b in blocks:
        b.graph.destroy()
    hg.destroy()


def test_batched_sampling_and_relabelling_match_the_oracle():
    """Several relations (and several id sets) in one call: item by item the results of the oracle, with an
    empty frontier, a repeated relation and different seeds in the batch; an id out of range in any item
    fails the call and names the relation."""
    wl = "tests/sampler/batch"
    nts = [NodeType("a", 3000, 4, False), NodeType("b", 2500, 4, False), NodeType("c", 40, 4, False)]
    G = HetGraph(nts)
    G.relations.append(uniform_relation("ab", 0, 1, 3000, 2500, 20000, wl))
    G.relations.append(power_law_relation("ba", 1, 0, 2500, 3000, 60000, 1.7, wl))
    G.relations.append(power_law_relation("ca", 2, 0, 40, 3000, 9000, 1.5, wl))
    hg = make_graph(type("P", (), {"graph": G})())
    g = rng.stream("tests", "sampler/batch")
    fr = [g.permutation(nts[t].num_nodes)[:k].astype(np.int64) for t, k in ((1, 600), (0, 900), (0, 0), (1, 37))]
    rels, seeds = [0, 1, 2, 0], [11, 0xFEEDFACE12345678, 13, 14]
    for fanout in (3, 20):
        got = heta.heta_sample_neighbors_batch(hg, rels, [torch.from_numpy(f).cuda() for f in fr], fanout, seeds)
        srcs = []
        for (rp, src), i, f, sd in zip(got, rels, fr, seeds):
            r = G.relations[i]
            ref_ptr, ref_src = osampler.sample_neighbors(r.rowptr, r.col, f, fanout, sd)
            assert np.array_equal(rp.cpu().numpy(), ref_ptr) and np.array_equal(src.cpu().numpy(), ref_src)
            srcs.append(src)
        # source sets per source type: relations 0 and 3 leave type a, 1 leaves b, 2 leaves c; plus an empty group
        groups = [[srcs[0], srcs[3]], [srcs[1]], [srcs[2]], []]
        out = heta.heta_unique_relabel_batch(groups, [3000, 2500, 40, 10])
        for grp, (uniq, local) in zip(groups, out):
            ref_u, ref_l = osampler.unique_relabel([x.cpu().numpy() for x in grp])
            assert np.array_equal(uniq.cpu().numpy(), ref_u)
            assert len(local) == len(ref_l)
            for a, b in zip(local, ref_l):
                assert np.array_equal(a.cpu().numpy(), b)
    bad = [torch.from_numpy(f).cuda() for f in fr]
    bad[1] = torch.tensor([5, 3000], dtype=torch.int64, device="cuda")      # relation 1's destinations are type a: 3000 is out
    with pytest.raises(heta.HetaError, match="relation 1"):
        heta.heta_sample_neighbors_batch(hg, rels, bad, 3, seeds)
    with pytest.raises(heta.HetaError, match="outside"):
        heta.heta_unique_relabel_batch([[srcs[0]], [srcs[1]]], [3000, 5])
    assert heta.heta_sample_neighbors_batch(hg, [], [], 3, []) == [] and heta.heta_unique_relabel_batch([], []) == []
    hg.destroy()


def test_batches_beyond_the_fused_limits_take_the_per_item_path():
    """More than 32 items in one sampling call, and id sets whose set index does not fit above the ids in a
    32-bit key (three sets with 2^31 possible ids each): same results, item by item."""
    wl = "tests/sampler/batch"
    nts = [NodeType("a", 3000, 4, False), NodeType("b", 2500, 4, False)]
    G = HetGraph(nts)
    G.relations.append(uniform_relation("ab", 0, 1, 3000, 2500, 20000, wl))
    G.relations.append(power_law_relation("ba", 1, 0, 2500, 3000, 60000, 1.7, wl))
    hg = make_graph(type("P", (), {"graph": G})())
    g = rng.stream("tests", "sampler/fallback")
    rels = [i % 2 for i in range(35)]
    fr = [g.permutation(nts[1 - r].num_nodes)[:(0 if i == 7 else 40 + 3 * i)].astype(np.int64) for i, r in enumerate(rels)]
    seeds = [1000 + i for i in range(35)]
    got = heta.heta_sample_neighbors_batch(hg, rels, [torch.from_numpy(f).cuda() for f in fr], 6, seeds)
    for (rp, src), i, f, sd in zip(got, rels, fr, seeds):
        ref_ptr, ref_src = osampler.sample_neighbors(G.relations[i].rowptr, G.relations[i].col, f, 6, sd)
        assert np.array_equal(rp.cpu().numpy(), ref_ptr) and np.array_equal(src.cpu().numpy(), ref_src)
    big = [np.array([2**31 - 1, 5, 5, 2**30, 0], dtype=np.int64), np.array([7, 7, 7], dtype=np.int64), np.array([2**31 - 2], dtype=np.int64)]
    out = heta.heta_unique_relabel_batch([[torch.from_numpy(x).cuda()] for x in big], [2**31] * 3)
    for x, (uniq, local) in zip(big, out):
        ref_u, ref_l = osampler.unique_relabel([x])
        assert np.array_equal(uniq.cpu().numpy(), ref_u) and np.array_equal(local[0].cpu().numpy(), ref_l[0])
    hg.destroy()


@pytest.mark.parametrize("n_types,rels,n_nodes,n_dst,fanout", [
    (3, [(0, 1), (1, 0), (2, 0), (0, 2), (2, 2)], [3000, 2500, 40], [700, 255, 16], 5),      # a hop of a small graph
    (2, [(0, 1), (1, 1), (0, 0)], [5_000_000, 70_000], [1, 257], 64),                            # more than 256 tiles of ids: counted in a launch
    (2, [(0, 1), (1, 0)], [1_100_000, 1_100_000], [1_050_000, 0], 2),                            # more than 4,096 chunks of destinations; an item without any
    (1, [(0, 0)] * 33, [900], [300], 3),                                                          # more items than one launch takes
    (2, [(0, 1)], [70_000_000, 50], [0, 50], 7)])                                                # id ranges past the bitmap
def test_sample_hop_equals_its_two_calls(n_types, rels, n_nodes, n_dst, fanout):
    """A hop in one call against the batched sampling and the batched unique / relabel, bit for bit, and against the oracle
    where it is quick; out-of-range destinations are refused alike."""
    g = rng.stream("tests", f"hop/{n_types}/{len(rels)}/{n_nodes[0]}")
    made = []
    for s, t in rels:
        deg = np.minimum(g.zipf(1.6, size=n_nodes[t]), 300) * (g.random(n_nodes[t]) < 0.7)
        rowptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int64)
        made.append((s, t, rowptr, g.integers(0, n_nodes[s], size=int(rowptr[-1]), dtype=np.int32)))
    hg = heta.heta_graph_create([(n, 4, 0) for n in n_nodes], made)
    fr = [np.sort(g.choice(n_nodes[t], size=n_dst[t], replace=False)).astype(np.int64) for t in range(n_types)]
    dst = [torch.from_numpy(fr[t]).cuda() for _, t in rels]
    seeds = [77 + 13 * i for i in range(len(rels))]
    sampled = heta.heta_sample_neighbors_batch(hg, list(range(len(rels))), dst, fanout, seeds)
    by_type = [[i for i, (s, _) in enumerate(rels) if s == k] for k in range(n_types)]
    relabelled = heta.heta_unique_relabel_batch([[sampled[i][1] for i in rs] for rs in by_type], n_nodes)
    for _ in range(2):
        rowptr, local, uniq = heta.heta_sample_hop(hg, list(range(len(rels))), dst, fanout, seeds)
        for k, rs in enumerate(by_type):
            assert torch.equal(uniq[k], relabelled[k][0])
            for i, l in zip(rs, relabelled[k][1]):
                assert torch.equal(rowptr[i], sampled[i][0]) and torch.equal(local[i], l)
    if sum(n_dst) < 2000:
        for i, (_, t, ptr, col) in enumerate(made):
            ref_ptr, ref_src = osampler.sample_neighbors(ptr, col, fr[t], fanout, seeds[i])
            assert np.array_equal(rowptr[i].cpu().numpy(), ref_ptr)
            assert np.array_equal(uniq[rels[i][0]].cpu().numpy()[local[i].cpu().numpy()], ref_src)
    bad = [d.clone() for d in dst]
    k = max(range(len(rels)), key=lambda i: bad[i].numel())
    bad[k][-1] = n_nodes[rels[k][1]]
    with pytest.raises(heta.HetaError) as e:
        heta.heta_sample_hop(hg, list(range(len(rels))), bad, fanout, seeds)
    assert e.value.status == heta.HETA_ERR_INVALID_ARG
    hg.destroy()


@pytest.mark.parametrize("n_dst,fanout", [(300_000, 64), (200_000, 40)])
def test_memory_of_a_large_hop(n_dst, fanout):
    """Few edges below a large fan-out: what is kept is of the sampled size, and of more than 64 MB of local ids none is taken
    by capacity (8 bytes of global source ids per destination and fan-out are)."""
    g = rng.stream("tests", f"hop-memory/{n_dst}")
    n_src = 9_000_000
    deg = g.integers(0, 4, size=n_dst)
    rowptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int64)
    hg = heta.heta_graph_create([(n_src, 4, 0), (n_dst, 4, 0)], [(0, 1, rowptr, g.integers(0, n_src, size=int(rowptr[-1]), dtype=np.int32))])
    dst = torch.arange(n_dst, device="cuda")
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    torch.cuda.reset_peak_memory_stats()
    before = torch.cuda.memory_allocated()
    kept = heta.heta_sample_hop(hg, [0], [dst], fanout, [3])
    capacity, edges = n_dst * fanout, int(rowptr[-1])
    if capacity > 1 << 24:
        assert torch.cuda.max_memory_allocated() - before <= 8 * capacity + 8 * (n_dst + 1) + 12 * edges + (8 << 20)
    assert torch.cuda.memory_allocated() - before <= 8 * (n_dst + 1) + 12 * edges + (16 << 20)
    assert kept[0][0].numel() == n_dst + 1 and int(kept[0][0][-1]) == edges == kept[1][0].numel()
    hg.destroy()
