"""GPU parity of the query launches where a call takes one path or another: boxes shared by several
workgroups (calls with and without a planning launch), boxes whose node tables overflow and are
redone in parts or in classes of nodes, against the CPU oracle.

Bounds as in test_gpu.py (fractions: relative error below 1e-5, exact zeros) and test_gpu_quant.py
(uncertainties: 2e-4 relative, plus 1e-6 of the largest). A shared box adds one fp32 addition with
its compensation per part and source, the terms of one more node: inside the same bounds.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import footprint as ofp
from oracle import quant, scan
from paper_2009_02702_amd import Graph, MGError, _lib, synth

from test_gpu import _compare, _dev, _graph, _sparse_to_dense
from test_gpu_quant import _compare as _compare_quant
from test_gpu_quant import _compare_err

pytestmark = pytest.mark.gpu

DIMS = (160, 150, 140)


def _boxes(n, large):
    """n boxes: `large` ones of most of the volume (odd corners: up to 150,000 cubes), then an empty
    one, one outside, then small ones of odd sizes."""
    rng = np.random.default_rng(n)
    b = np.concatenate([rng.integers(0, 130, size=(n, 3)), rng.integers(1, 24, size=(n, 3))], axis=1)
    k = min(n, large)
    b[:k, :3] = rng.integers(0, 3, size=(k, 3)) * 2 + 1
    b[:k, 3:] = np.asarray(DIMS) - rng.integers(6, 13, size=(k, 3))
    if n > k + 2:
        b[k] = [5, 5, 5, 0, 4, 4]
        b[k + 1] = [DIMS[0], 0, 0, 3, 3, 3]
    return b[rng.permutation(n)].astype(np.uint32)


@pytest.mark.parametrize("n,large", [(1, 1), (3, 2), (255, 5), (1024, 3), (1025, 3), (1500, 40)])
def test_boxes_shared_by_several_workgroups(n, large):
    """Calls of up to 1,024 boxes (one launch) and of more (planned): large boxes are shared by
    several workgroups, the others are not; with tiny tables parts overflow and are redone, in LDS
    or in global memory. Twice each: the call leaves its workspace as it found it."""
    w = synth.workload(2, dims=DIMS, segments=300, n_boxes=1)
    vol = synth.make_volume(w)
    g = _graph("paths", vol)
    boxes = _boxes(n, large)
    ids, vol_c = scan.compact(vol)
    _, ref = scan.box_counts(vol_c, len(ids), boxes)
    db = _dev(boxes)
    ws = g.workspace(n)
    try:
        for tables in ((0, 0, 0), (64, 64, 1024), (64, 64, 64)):
            g.set_launch_config(table_big=tables[0], table_small=tables[1], table_retry=tables[2])
            for again in range(2):
                got = g.query(db, workspace=ws).cpu().numpy()
                _compare(got, ref, None, "%d boxes, tables %s, call %d" % (n, tables, again))
    finally:
        g.set_launch_config(table_big=0, table_small=0, table_retry=0)


_QUANT = []


def _quantized():
    """A quantized graph, boxes of 1 to 27,000 cubes, and the oracle's fractions and uncertainties."""
    if not _QUANT:
        dims = (72, 70, 66)
        g = Graph.build(synth.make_volume(synth.workload(2, dims=dims, segments=150, n_boxes=1)))
        S = g.info()["nseg"]
        d = g.export_dag()
        rep, nodes, _, _ = quant.quantize_dag(S, d["child_a"][S:], d["child_b"][S:],
                                              d["wnum"][S:] / d["wden"][S:], 9)
        mu, dmu = quant.propagate(S, nodes)
        maps = [g.export_map(l) for l in range(g.info()["n_levels"])]
        boxes = np.array([[1, 1, 1, 70, 67, 64], [1, 3, 1, 68, 63, 64], [3, 1, 1, 66, 69, 62], [0, 0, 0, 72, 70, 66],
                          [5, 9, 7, 20, 31, 6], [7, 7, 7, 1, 1, 1], [9, 9, 9, 4, 0, 4]], dtype=np.uint32)
        f, u = np.zeros((len(boxes), S)), np.zeros((len(boxes), S))
        cubes, l0 = np.zeros(len(boxes), dtype=np.int64), np.zeros(len(boxes), dtype=bool)
        for i, bx in enumerate(boxes.astype(np.int64)):
            counts, levels = {}, set()
            for lev, c in ofp.assembly(bx[:3], bx[3:], dims):
                node = rep[int(maps[lev][c[2], c[1], c[0]])]
                counts[node] = counts.get(node, 0) + 8 ** lev
                levels.add(lev)
                cubes[i] += 1
            if counts:
                f[i], u[i] = quant.box_histogram(counts, mu, dmu, float(np.prod(bx[3:])))
                l0[i] = levels == {0}
        q = g.quantize(9).upload(0)
        q.lut_build()
        _QUANT.append((q, boxes, f, u, l0, cubes))
    return _QUANT[0]


@pytest.mark.parametrize("n", [7, 1024, 1025])
def test_uncertainty_boxes_redone_by_classes_of_nodes(n):
    """Large boxes (from 2^14 cubes) of an uncertainty query whose table overflows are redone by
    workgroups that each take one class of the nodes: every node's count still meets its row whole.
    More such boxes than can be shared in one call are redone whole."""
    q, boxes, f, u, l0, cubes = _quantized()
    assert (cubes[:3] >= 1 << 14).all()
    pick = np.arange(n) % len(boxes)
    db = _dev(boxes[pick])
    ws = q.workspace(n)
    try:
        for tables in ((0, 0, 0), (64, 64, 1024), (64, 64, 64)):
            q.set_launch_config(table_big=tables[0], table_small=tables[1], table_retry=tables[2])
            for again in range(2):
                out, err = q.query_err(db, workspace=ws)
                tag = "%d boxes, tables %s, call %d" % (n, tables, again)
                _compare_quant(out.cpu().numpy(), f[pick], l0[pick], tag)
                _compare_err(err.cpu().numpy(), u[pick], tag)
    finally:
        q.set_launch_config(table_big=0, table_small=0, table_retry=0)


_SMALL_CELLS = []


def _small_cells():
    """A graph of more sources than the per-source LDS arrays hold, cells of about 50 voxels: most
    cubes above level 0 are on nodes of rank >= 3, whose expansion meets new sources. 1,500 boxes of
    a few to 8,000 voxels, and the oracle's fractions."""
    if not _SMALL_CELLS:
        dims = (62, 59, 61)
        vol = synth.make_volume(synth.workload(2, dims=dims, segments=4000, n_boxes=1))
        g = Graph.build(vol).upload(0)
        rng = np.random.default_rng(5)
        b = np.concatenate([rng.integers(0, 50, size=(1500, 3)), rng.integers(1, 21, size=(1500, 3))], axis=1)
        b[:3] = [[4, 4, 4, 16, 16, 16], [7, 7, 7, 0, 3, 3], [61, 58, 60, 9, 9, 9]]
        ids, vol_c = scan.compact(vol)
        _, ref = scan.box_counts(vol_c, len(ids), b.astype(np.uint32))
        assert g.info()["nseg"] == len(ids) > 2048
        _SMALL_CELLS.append((g, b.astype(np.uint32), ref))
    return _SMALL_CELLS[0]


@pytest.mark.parametrize("variant", ["batched", "plain", "sparse"])
def test_expansion_that_inserts_sources_into_the_node_table(variant):
    """Sources as entries of the node table, inserted while its nodes are expanded: every node's
    count meets its row exactly once, in each of several calls."""
    g, boxes, ref = _small_cells()
    db = _dev(boxes)
    nnz = int((ref > 0).sum())
    for call in range(4):
        if variant == "sparse":
            index, seg, val, total = g.query_sparse(db, capacity=nnz)
            assert int(total.item()) == nnz
            got = _sparse_to_dense(index.cpu().numpy(), seg.cpu().numpy(), val.cpu().numpy(), *ref.shape)
        else:
            got = g.query(db, variant=variant).cpu().numpy()
        _compare(got, ref, None, "%s, call %d" % (variant, call))


def test_a_failed_call_leaves_its_workspace_clean():
    """A retry table that no workgroup's LDS holds refuses a call with MG_ELIMIT, and a call that
    finds an earlier error of its thread fails after its launches: the next call on the same
    workspace (or on the library's scratch) answers every box."""
    vol = synth.make_volume(synth.workload(2, dims=(62, 59, 61), segments=5000, n_boxes=1))
    g = Graph.build(vol).upload(0)
    rng = np.random.default_rng(6)
    boxes = np.concatenate([rng.integers(0, 40, size=(1300, 3)), rng.integers(1, 33, size=(1300, 3))],
                           axis=1).astype(np.uint32)
    boxes[:2] = [[0, 0, 0, 62, 59, 61], [1, 3, 1, 60, 55, 57]]
    ids, vol_c = scan.compact(vol)
    _, ref = scan.box_counts(vol_c, len(ids), boxes)
    assert len(ids) > 4500
    ws = g.workspace(len(boxes))
    db = _dev(boxes)
    out = torch.empty(ref.shape, dtype=torch.float32, device="cuda")
    index = torch.empty((len(boxes), 2), dtype=torch.int32, device="cuda")
    one = [torch.empty(1, dtype=t, device="cuda") for t in (torch.int32, torch.float32, torch.int32)]
    calls = {"sparse": lambda k: g.query_sparse(db[:k], capacity=1, workspace=ws, bufs=(index[:k], *one)),
             "batched": lambda k: g.query(db[:k], out=out[:k], workspace=ws),
             "plain": lambda k: g.query(db[:k], out=out[:k], variant="plain", workspace=ws),
             "noalloc": lambda k: g.query_noalloc(db[:k], out=out[:k])}
    for n in (1300, 900):  # with and without planning launches
        for name, call in calls.items():
            g.set_launch_config(table_retry=8192)
            with pytest.raises(MGError) as e:
                call(n)
            assert e.value.code == -8
            g.set_launch_config(table_retry=0)
            try:
                _lib.load().hipSetDevice(1 << 20)  # an error that may wait for the next hipGetLastError
                call(n)
            except MGError as e:
                assert e.code != -8
            for again in range(2):
                tag = "%s, %d boxes, call %d" % (name, n, again)
                _compare(g.query(db[:n], workspace=ws).cpu().numpy(), ref[:n], None, tag)
                _compare(g.query_noalloc(db[:n]).cpu().numpy(), ref[:n], None, tag + ", noalloc")
    g.close()


def test_captured_noalloc_calls_replayed_among_other_graphs_calls():
    """Captured calls on the library's scratch, replayed after calls of a graph with another layout
    of it (which the capture could not know of), with shared boxes and with boxes that overflow
    into the scratch's global tables: every replay and every call between them answers every box."""
    cases = []
    for dims, segments in (((160, 150, 140), 300), ((96, 80, 72), 900)):
        vol = synth.make_volume(synth.workload(2, dims=dims, segments=segments, n_boxes=1))
        g = Graph.build(vol).upload(0)
        b = np.minimum(_boxes(40, 4), np.asarray(dims + dims)).astype(np.uint32)
        ids, vol_c = scan.compact(vol)
        _, ref = scan.box_counts(vol_c, len(ids), b)
        out = torch.empty(ref.shape, dtype=torch.float32, device="cuda")
        cases.append((g, _dev(b), ref, out))
    try:
        for tables in ((0, 0, 0), (64, 64, 64)):
            graphs = []
            for g, db, ref, out in cases:
                g.set_launch_config(table_big=tables[0], table_small=tables[1], table_retry=tables[2])
                _compare(g.query_noalloc(db, out=out).cpu().numpy(), ref, None, "before capture")
                graph = torch.cuda.CUDAGraph()
                with torch.cuda.graph(graph):
                    g.query_noalloc(db, out=out)
                graphs.append(graph)
            # (replay or call, graph): each graph's after the other's, in both forms
            for step, (replay, k) in enumerate([(1, 0), (0, 1), (1, 0), (1, 1), (1, 0), (0, 0), (1, 1), (0, 1), (0, 0),
                                                (1, 1), (1, 1), (0, 1)]):
                g, db, ref, out = cases[k]
                out.fill_(-1.0)
                if replay:
                    graphs[k].replay()
                else:
                    g.query_noalloc(db, out=out)
                torch.cuda.synchronize()
                _compare(out.cpu().numpy(), ref, None, "tables %s, step %d" % (tables, step))
            del graphs
    finally:
        for g, _, _, _ in cases:
            g.close()


def test_graph_too_large_for_mixture_rows():
    """Noise of 2,000 sources, whose nodes of rank >= 3 would need more than 2^25 row entries: the
    batched calls push mass rank by rank, in the tiers and in the global tables their overflows end
    in, and the lookup table is read where it is named; large boxes shared by several workgroups
    among them. All against the oracle."""
    dims = (149, 151, 147)
    vol = np.random.default_rng(3).integers(1, 2001, size=dims[::-1]).astype(np.uint32)
    g = Graph.build(vol).upload(0)
    g.lut_build()
    ptr, _, _ = g.export_lut()
    rank_ptr = g.export_dag()["rank_ptr"]
    assert int(ptr[-1] - ptr[rank_ptr[3]]) > 1 << 25
    rng = np.random.default_rng(4)
    boxes = np.concatenate([rng.integers(0, 130, size=(1106, 3)), rng.integers(1, 9, size=(1106, 3))], axis=1)
    boxes[:40, 3:] = rng.integers(9, 40, size=(40, 3))
    boxes[1100:] = _boxes(6, 6)
    boxes = boxes.astype(np.uint32)
    ids, vol_c = scan.compact(vol)
    _, ref = scan.box_counts(vol_c, len(ids), boxes)
    db = _dev(boxes)
    ws = g.workspace(len(boxes))
    for variant, lo, hi in (("batched", 0, 300), ("batched", 0, 1106), ("batched", 1000, 1106),
                            ("batched", 1100, 1101), ("plain", 0, 300), ("lut", 0, 1106),
                            ("lut", 1000, 1106), ("lut", 1100, 1101)):
        for tables in ((0, 0, 0), (64, 64, 64)):
            g.set_launch_config(table_big=tables[0], table_small=tables[1], table_retry=tables[2])
            for again in range(2):
                got = g.query(db[lo:hi], variant=variant, workspace=ws).cpu().numpy()
                _compare(got, ref[lo:hi], None, "%s, boxes %d..%d, tables %s, call %d" % (variant, lo, hi, tables, again))
    g.close()


@pytest.mark.parametrize("segments", [1500, 12000])
def test_shared_boxes_with_sparse_output_and_sources_as_entries(segments):
    """Boxes shared by several workgroups whose sums are read out as sparse entries: from per-source
    arrays (1,500 sources), and where sources are entries of every table (12,000), which the box's
    last part reads from the shared sums. With and without planning launches; with tiny tables the
    parts overflow and are redone."""
    vol = synth.make_volume(synth.workload(2, dims=DIMS, segments=segments, n_boxes=1))
    g = Graph.build(vol).upload(0)
    boxes = _boxes(1100, 12)
    boxes[0] = [1, 3, 1, DIMS[0] - 7, DIMS[1] - 9, DIMS[2] - 11]
    ids, vol_c = scan.compact(vol)
    _, ref = scan.box_counts(vol_c, len(ids), boxes)
    nnz = (ref > 0).sum(axis=1)
    db = _dev(boxes)
    ws = g.workspace(len(boxes))
    for n in (1, 400, 1100):
        cap = int(nnz[:n].sum())
        for tables in ((0, 0, 0), (64, 64, 1024), (64, 64, 64)):
            g.set_launch_config(table_big=tables[0], table_small=tables[1], table_retry=tables[2])
            for again in range(2):
                tag = "%d sources, %d boxes, tables %s, call %d" % (len(ids), n, tables, again)
                index, seg, val, total = g.query_sparse(db[:n], capacity=cap, workspace=ws)
                assert int(total.item()) == cap, tag
                assert np.array_equal(index[:, 1].cpu().numpy(), nnz[:n]), tag
                got = _sparse_to_dense(index.cpu().numpy(), seg.cpu().numpy(), val.cpu().numpy(), n, len(ids))
                _compare(got, ref[:n], None, tag)
                _compare(g.query(db[:n], workspace=ws).cpu().numpy(), ref[:n], None, tag + ", dense rows")
    g.close()


def test_autotune_on_few_boxes_leaves_what_such_calls_do_not_read():
    """Calls of at most 1,024 boxes take one launch that reads none of the tiers' settings: tuning on
    such a call keeps them as they were set for larger ones."""
    vol = synth.make_volume(synth.workload(2, dims=(64, 64, 64), segments=40, n_boxes=1))
    g = Graph.build(vol).upload(0)
    boxes = synth.make_boxes(synth.workload(2, dims=(64, 64, 64), segments=40, n_boxes=1025))
    kept = dict(unroll_big=4, unroll_small=16, table_small=512, block_small=256, block_big=512, chunk_small=3)
    for n in (1, 1024):
        g.set_launch_config(**kept)
        cfg = g.autotune(_dev(boxes[:n]), reps=1)
        assert {k: cfg[k] for k in kept} == kept and g.launch_config() == cfg
        assert cfg["run_min_row"] in (0, 8, 32, 64)
    cfg = g.autotune(_dev(boxes), reps=1)
    assert g.launch_config() == cfg
    ids, vol_c = scan.compact(vol)
    _, ref = scan.box_counts(vol_c, len(ids), boxes)
    _compare(g.query(_dev(boxes)).cpu().numpy(), ref, None, "after autotune")
    g.close()


def test_largest_set_tables_of_the_push():
    """Calls that push (16 bytes per table slot) with tables set to 8,192 slots and 1,800 sources,
    which fit the LDS but for the kernels' fixed arrays: answered, in calls with and without planning
    launches (half the size is used)."""
    vol = synth.make_volume(synth.workload(2, dims=(62, 59, 61), segments=1800, n_boxes=1))
    g = Graph.build(vol).upload(0)
    rng = np.random.default_rng(8)
    boxes = np.concatenate([rng.integers(0, 40, size=(1100, 3)), rng.integers(1, 33, size=(1100, 3))],
                           axis=1).astype(np.uint32)
    ids, vol_c = scan.compact(vol)
    _, ref = scan.box_counts(vol_c, len(ids), boxes)
    assert 1750 < len(ids) < 1900
    for n in (1100, 500):
        for tables in ((8192, 64), (64, 8192), (8192, 8192)):
            g.set_launch_config(table_big=tables[0], table_retry=tables[1])
            out, _ = g.query_stats(_dev(boxes[:n]))
            _compare(out.cpu().numpy(), ref[:n], None, "tables %s, %d boxes" % (tables, n))
    g.close()
