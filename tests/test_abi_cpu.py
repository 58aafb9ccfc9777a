"""CPU checks of the C ABI library: it loads, exports every symbol the header
declares, builds graph indexes on the host bit-exactly (host-only graphs need
no GPU), and turns bad inputs into the documented status codes."""
import ctypes
import os
import re

import numpy as np
import pytest

import oracle
import workloads

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _rgnn():
    from paper_2301_06284_amd import rgnn
    return rgnn


def test_header_symbols_exported():
    rgnn = _rgnn()
    hdr = open(os.path.join(ROOT, "include", "rgnn.h")).read()
    hdr = re.sub(r"/\*.*?\*/", "", hdr, flags=re.S)
    declared = set(re.findall(r"\b(?:rgnn_status|const char\s*\*)\s*(\w+)\s*\(", hdr))
    assert declared, "no declarations found"
    lib = ctypes.CDLL(rgnn.LIB_PATH)
    for name in sorted(declared):
        assert hasattr(lib, name), f"{name} declared in rgnn.h but not exported"
    assert declared <= set(rgnn.EXPORTED) | {"rgnn_graph_t"}


@pytest.mark.parametrize("kind", ["random", "hub", "srchub", "dups", "isolated", "empty", "complete"])
@pytest.mark.parametrize("seed", [0, 1])
def test_host_graph_index_bit_exact(kind, seed):
    rgnn = _rgnn()
    g = workloads.tiny_graph(seed, N=90, E=700, R=5, T=3, kind=kind)
    G = rgnn.Graph.from_dict(g, host_only=True)
    ix = oracle.graph_index(g)
    for k in rgnn.INDEX_KINDS:
        np.testing.assert_array_equal(G.export(k), ix[k], err_msg=k)
    inf = G.info()
    assert inf["num_src_pairs"] == ix["U_src"] and inf["num_dst_segments"] == ix["U_dst"]
    G.close()


def test_host_graph_index_workload1():
    rgnn = _rgnn()
    g = workloads.make_graph(1)
    G = rgnn.Graph.from_dict(g, host_only=True)
    ix = oracle.graph_index(g)
    for k in rgnn.INDEX_KINDS:
        np.testing.assert_array_equal(G.export(k), ix[k], err_msg=k)


def test_csr_equals_coo():
    rgnn = _rgnn()
    g = workloads.tiny_graph(4, N=50, E=400, R=4, T=2, kind="hub")
    order = np.argsort(g["dst"], kind="stable")
    rowptr = np.zeros(g["N"] + 1, np.int64)
    np.cumsum(np.bincount(g["dst"], minlength=g["N"]), out=rowptr[1:])
    Gc = rgnn.Graph.from_csr(g["N"], g["T"], g["R"], rowptr, g["src"][order], g["rel"][order],
                             g["ntype"], host_only=True)
    g2 = dict(g, src=g["src"][order], dst=g["dst"][order], rel=g["rel"][order])
    ix = oracle.graph_index(g2)
    for k in rgnn.INDEX_KINDS:
        np.testing.assert_array_equal(Gc.export(k), ix[k], err_msg=k)


def test_error_codes():
    rgnn = _rgnn()
    g = workloads.tiny_graph(1, N=10, E=30, R=3, T=2)
    bad = dict(g, src=g["src"].copy()); bad["src"][3] = 10
    with pytest.raises(rgnn.RgnnError) as e:
        rgnn.Graph.from_dict(bad, host_only=True)
    assert e.value.status == rgnn.ERANGE
    bad = dict(g, rel=g["rel"].copy()); bad["rel"][0] = -1
    with pytest.raises(rgnn.RgnnError) as e:
        rgnn.Graph.from_dict(bad, host_only=True)
    assert e.value.status == rgnn.ERANGE
    bad = dict(g, ntype=g["ntype"].copy()); bad["ntype"][2] = 2
    with pytest.raises(rgnn.RgnnError) as e:
        rgnn.Graph.from_dict(bad, host_only=True)
    assert e.value.status == rgnn.ERANGE
    with pytest.raises(rgnn.RgnnError) as e:
        rgnn.Graph.from_coo(10, 0, 3, g["src"], g["dst"], g["rel"], host_only=True)
    assert e.value.status == rgnn.EINVAL
    rowptr = np.array([0, 2, 1, 3], np.int64)
    with pytest.raises(rgnn.RgnnError) as e:
        rgnn.Graph.from_csr(3, 1, 1, rowptr, np.zeros(3, np.int32), np.zeros(3, np.int32), host_only=True)
    assert e.value.status == rgnn.EINVAL
    # a host-only graph cannot run layers
    G = rgnn.Graph.from_dict(g, host_only=True)
    lib = rgnn.lib()
    st = lib.rgcn_forward(G.handle, None, None, None, 64, 64, 0, 0, None, None, 0, None)
    assert st == rgnn.EINVAL and b"host-only" in lib.rgnn_last_error()
    # export buffer too small
    buf = np.zeros(2, np.int32)
    st = lib.rgnn_graph_export(G.handle, 1, buf.ctypes.data_as(ctypes.c_void_p), buf.nbytes)
    assert st == rgnn.EINVAL


def test_workspace_and_plan_model():
    rgnn = _rgnn()
    g = workloads.make_graph(1)
    G = rgnn.Graph.from_dict(g, host_only=True)
    for layer, heads in [(rgnn.LAYER_RGCN, 1), (rgnn.LAYER_RGAT, 1), (rgnn.LAYER_RGAT, 4),
                         (rgnn.LAYER_HGT, 4), (rgnn.LAYER_RGAT_BACKWARD, 1), (rgnn.LAYER_RGAT_BACKWARD, 4)]:
        for plan in (1, 2):
            assert rgnn.workspace_size(G, layer, 64, 64, heads, plan) > 0
    # the attention+message rows are wider than the message rows
    assert (rgnn.workspace_size(G, rgnn.LAYER_RGAT, 64, 64, 1, rgnn.PLAN_TRANSFORM_FIRST_ATTMSG) >
            rgnn.workspace_size(G, rgnn.LAYER_RGAT, 64, 64, 1, rgnn.PLAN_TRANSFORM_FIRST))
    with pytest.raises(rgnn.RgnnError):
        rgnn.workspace_size(G, rgnn.LAYER_RGCN, 64, 64, 1, rgnn.PLAN_TRANSFORM_FIRST_ATTMSG)
    with pytest.raises(rgnn.RgnnError):
        rgnn.workspace_size(G, rgnn.LAYER_RGAT, 64, 64, 1, 5)
    plan, tf, af = rgnn.select_plan(G, rgnn.LAYER_RGAT, 64, 64, 1)
    assert plan == (2 if af < tf else 1) and tf > 0 and af > 0
    # multi-head RGAT always resolves to transform-first
    assert rgnn.select_plan(G, rgnn.LAYER_RGAT, 64, 64, 4)[0] == 1


def test_product_does_not_import_oracle():
    """The GPU package never reaches the oracle (no CPU fallback)."""
    import ast
    pkg = os.path.join(ROOT, "paper_2301_06284_amd")
    for fn in os.listdir(pkg):
        if fn.endswith(".py"):
            tree = ast.parse(open(os.path.join(pkg, fn)).read())
            for node in ast.walk(tree):
                if isinstance(node, ast.Import):
                    assert all(not a.name.startswith("oracle") for a in node.names), fn
                if isinstance(node, ast.ImportFrom):
                    assert not (node.module or "").startswith("oracle"), fn


def test_graph_without_compaction_host_only():
    """RGNN_GRAPH_NO_COMPACT: one materialized row per edge, in (rel, src,
    edge id) order; everything else as with compaction."""
    rgnn = _rgnn()
    g = workloads.tiny_graph(39, N=50, E=400, R=4, kind="dups")
    a = rgnn.Graph.from_dict(g, host_only=True)
    b = rgnn.Graph.from_dict(g, host_only=True, compact=False)
    ia, ib = a.info(), b.info()
    assert ib["num_src_pairs"] == g["E"] < ia["num_src_pairs"] + g["E"]
    assert ia["num_src_pairs"] < g["E"]   # the dups graph has repeated (src, rel) pairs
    order = np.lexsort((np.arange(g["E"]), g["src"], g["rel"]))
    np.testing.assert_array_equal(b.export("uniq_src"), g["src"][order])
    e2u = b.export("edge2uniq")
    inv = np.empty(g["E"], np.int64); inv[order] = np.arange(g["E"])
    np.testing.assert_array_equal(e2u, inv[b.export("in_eid")])
    for k in ("dst_rowptr", "in_src", "in_rel", "in_eid", "seg_ptr", "out_pos"):
        np.testing.assert_array_equal(a.export(k), b.export(k), err_msg=k)
    a.close(); b.close()


@pytest.mark.parametrize("T", [1, 96])
def test_segment_gemm_workspace_grows_with_rows(T):
    """A workspace sized for the most rows serves every smaller call: the size
    never falls as the rows grow, also where the tiles' rows step up."""
    rgnn = _rgnn()
    rows = [0, 1, 63, 64, 65, 1000]
    for k in range(1, 10):   # the steps lie at multiples of 64 * 768 rows
        rows += [k * 49152 - 1, k * 49152, k * 49152 + 1, k * 49152 + 20000]
    sizes = [rgnn.segment_gemm_workspace_size(m, T) for m in rows + [1000003, 10000000]]
    assert sizes == sorted(sizes)


@pytest.mark.parametrize("d,heads", [(32, 2), (64, 4), (128, 1)])
def test_hgt_backward_folds_by_size(d, heads):
    """One-type graphs with few relations keep no queries, output gradients or
    query gradients per node (three [N, d] arrays less); with relations that
    outweigh the nodes they take the general path's workspace, as mixed
    destination types do."""
    rgnn = _rgnn()
    rng = np.random.default_rng(d)
    N, E = 2000, 6000
    ends = [rng.integers(0, N, E, dtype=np.int32) for _ in range(2)]
    for R, folded in ((5, True), (600, False)):
        rel = rng.integers(0, R, E, dtype=np.int32)
        sizes = []
        for T, ntype in ((1, np.zeros(N, np.int32)), (2, rng.integers(0, 2, N, dtype=np.int32))):
            g = rgnn.Graph.from_coo(N, T, R, ends[0], ends[1], rel, ntype, host_only=True)
            sizes.append(rgnn.workspace_size(g, rgnn.LAYER_HGT_BACKWARD, d, d, heads) - (T * d * 3 * d * 4 if d <= 64 else 0))
            g.close()
        chunks = 2 * 2 * d * d * 4 * 32 + 4096   # at most one chunk more per node type, and padding
        if folded:
            assert sizes[1] - sizes[0] > 2 * N * d * 4
        else:
            assert abs(sizes[1] - sizes[0]) <= chunks


@pytest.mark.parametrize("N,E", [(500000, 1000), (500000, 200000), (1000000, 40000), (3000, 50), (100000, 900000)])
def test_work_items_of_sparse_graphs(N, E):
    """Work items follow the edges and the nodes: a graph with far fewer edges than
    nodes has full bundles of 32 destinations once those make 12 288 items, small
    graphs finer ones."""
    rgnn = _rgnn()
    rng = np.random.default_rng(N + E)
    src, dst = (rng.integers(0, N, E, dtype=np.int32) for _ in range(2))
    g = rgnn.Graph.from_coo(N, 1, 2, src, dst, rng.integers(0, 2, E, dtype=np.int32), host_only=True)
    items = g.info()["num_items"]
    g.close()
    per = 8 * max(1, -(-(E // 12288) // 8))      # edges of a bundle, at least 16 and at most 64
    per = min(64, max(16, per))
    nodes = min(32, max(per // 2, N // 12288))   # and destinations
    assert items <= N / nodes + 2 * E / per + 1
    assert items >= N / 32


@pytest.mark.parametrize("d,heads,kept", [(32, 2, 1), (64, 4, 1), (128, 2, 0)])
def test_hgt_backward_workspace_of_typed_relations(d, heads, kept):
    """Folded weights need no query weights of their own, and the node weights side by
    side ([T, d, 3 d]) only at d <= 64: the workspace grows with R and T by the
    arrays that are used."""
    rgnn = _rgnn()

    def size(R, T):
        N = 100
        g = rgnn.Graph.from_coo(N, T, R, [0] * 4, [1] * 4, [0] * 4, np.zeros(N, np.int32), host_only=True)
        n = rgnn.workspace_size(g, rgnn.LAYER_HGT_BACKWARD, d, d, heads)
        g.close()
        return n
    mat = d * d * 4
    heads_part = -(-(heads * (d // heads) ** 2) // 256) * 4   # shares of dmu per relation
    per_rel = 5 * mat + heads_part                            # Wmt, OT, M2, Wf, Wg
    assert abs(size(32, 1) - size(16, 1) - 16 * per_rel) <= 512
    assert size(32, 65) - size(32, 1) == kept * 64 * 3 * mat
