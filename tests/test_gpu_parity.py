"""GPU parity on small graphs: every layer and plan through the C ABI against
the fp64 oracle, element by element, on graphs that still span many work
items, split hub destinations, empty destinations, duplicate edges and
ragged GEMM tiles.  Index arrays are compared bit for bit."""
import numpy as np
import pytest

import oracle
import workloads
from helpers import TOL, Runner, rgat_backward_ref, row_err

pytestmark = pytest.mark.gpu

KINDS = ["random", "hub", "srchub", "dups", "isolated", "empty"]


@pytest.fixture(scope="module", autouse=True)
def gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2301_06284_amd import rgnn  # noqa: F401  (fails loudly if not built)
    torch.cuda.set_device(0)


def graph(kind, seed=5, N=300, E=4000, R=6, T=3):
    return workloads.tiny_graph(seed, N=N, E=E, R=R, T=T, kind=kind)


@pytest.mark.parametrize("kind", KINDS + ["complete"])
def test_device_graph_index_bit_exact(kind):
    from paper_2301_06284_amd import rgnn
    g = graph(kind, N=120 if kind == "complete" else 300)
    print(f"graph index {kind}", flush=True)
    G = rgnn.Graph.from_dict(g)
    ix = oracle.graph_index(g)
    for k in rgnn.INDEX_KINDS:
        np.testing.assert_array_equal(G.export(k), ix[k], err_msg=k)
    G.close()


@pytest.mark.parametrize("K,Nc", [(32, 32), (64, 64), (128, 128), (64, 128), (128, 64)])
def test_segment_gemm(K, Nc):
    import torch
    from paper_2301_06284_amd import rgnn
    rng = np.random.default_rng(K + Nc)
    type_ptr = np.array([0, 5, 5, 200, 201, 777, 1000], np.int64)   # empty and 1-row types
    M, T = int(type_ptr[-1]), len(type_ptr) - 1
    X = rng.standard_normal((1500, K)).astype(np.float32)
    W = rng.standard_normal((T, K, Nc)).astype(np.float32)
    gather = rng.integers(0, 1500, M).astype(np.int32)
    scatter = rng.permutation(1200)[:M].astype(np.int32)
    print(f"segment_gemm {K}x{Nc}", flush=True)
    dev = torch.device("cuda:0")
    Xd, Wd = torch.from_numpy(X).to(dev), torch.from_numpy(W).to(dev)
    gd, sd = torch.from_numpy(gather).to(dev), torch.from_numpy(scatter).to(dev)
    Y = torch.zeros(1200, Nc, device=dev)
    ws = torch.empty(rgnn.segment_gemm_workspace_size(M, T), dtype=torch.uint8, device=dev)
    rgnn.segment_gemm(Xd, gd, type_ptr, Wd, Y, sd, ws, K, Nc)
    torch.cuda.synchronize()
    ref = np.zeros((1200, Nc))
    for t in range(T):
        rows = np.arange(type_ptr[t], type_ptr[t + 1])
        ref[scatter[rows]] = X[gather[rows]].astype(np.float64) @ W[t].astype(np.float64)
    assert row_err(Y.cpu().numpy(), ref) <= TOL


@pytest.mark.parametrize("K,Nc", [(32, 32), (64, 64), (128, 128), (64, 128), (128, 64)])
def test_segment_gemm_fp32_grade(K, Nc):
    """Every output entry within a few fp32 unit roundoffs of the exact product,
    relative to sum_k |x_k w_k| (a sequential fp32 dot product is bounded by K of
    them): the 64-deep shapes, whose products run on split bf16 pieces, must be
    as accurate as the fp32 MFMA ones.  Rows span twelve decades of scale, and
    a plain bf16 (or two-piece bf16) product would miss the bound by far."""
    import torch
    from paper_2301_06284_amd import rgnn
    rng = np.random.default_rng(1000 + K + Nc)
    type_ptr = np.array([0, 700, 701, 1500, 2048], np.int64)
    M, T = int(type_ptr[-1]), len(type_ptr) - 1
    X = (rng.standard_normal((M, K)) * 10.0 ** rng.uniform(-6, 6, (M, 1))).astype(np.float32)
    W = (rng.standard_normal((T, K, Nc)) * 10.0 ** rng.uniform(-3, 3, (T, 1, Nc))).astype(np.float32)
    gather = np.arange(M, dtype=np.int32)
    scatter = rng.permutation(M).astype(np.int32)
    print(f"segment_gemm fp32 grade {K}x{Nc}", flush=True)
    dev = torch.device("cuda:0")
    Y = torch.zeros(M, Nc, device=dev)
    ws = torch.empty(rgnn.segment_gemm_workspace_size(M, T), dtype=torch.uint8, device=dev)
    rgnn.segment_gemm(torch.from_numpy(X).to(dev), torch.from_numpy(gather).to(dev), type_ptr,
                      torch.from_numpy(W).to(dev), Y, torch.from_numpy(scatter).to(dev), ws, K, Nc)
    torch.cuda.synchronize()
    got = Y.cpu().numpy().astype(np.float64)
    u = 2.0 ** -24
    worst = 0.0
    for t in range(T):
        rows = np.arange(type_ptr[t], type_ptr[t + 1])
        x, w = X[rows].astype(np.float64), W[t].astype(np.float64)
        exact = x @ w
        scale = np.abs(x) @ np.abs(w)
        worst = max(worst, float((np.abs(got[scatter[rows]] - exact) / (u * scale)).max()))
    print(f"  max error / (u sum |x w|) = {worst:.2f}", flush=True)
    assert worst <= 8.0


@pytest.mark.parametrize("d,heads", [(128, 1), (128, 2), (64, 1)])
def test_rgat_many_relations(d, heads):
    """More relations than the segment-term kernel can stage in LDS (their
    reordered w_dst vectors: 700 x d floats per head): the vectors are read
    with the rows instead.  Forward (both plans) and backward."""
    g = graph("random", seed=9, N=600, E=6000, R=700, T=2)
    t = workloads.tiny_tensors(9, g, d, d, heads=heads, att_var=1.0)
    print(f"rgat many relations d={d} heads={heads}", flush=True)
    run = Runner(g, t)
    ref = oracle.rgat_forward(g, t["h"], t["W"], t["w_src"], t["w_dst"], heads=heads)
    for plan in (1, 2) if heads == 1 else (1,):
        assert row_err(run.rgat(heads=heads, plan=plan), ref) <= TOL
    gh, gW, gs, gt = run.rgat_backward(heads=heads)
    run.close()
    dh, dW, dws, dwt = rgat_backward_ref(g, t, heads=heads)
    isolated = (np.bincount(g["src"], minlength=g["N"]) + np.bincount(g["dst"], minlength=g["N"])) == 0
    assert row_err(gh, dh, structural_zero=isolated, cancel_floor=1e-6) <= TOL
    assert row_err(gW.reshape(-1, d), dW.reshape(-1, d), cancel_floor=1e-6) <= TOL
    assert row_err(gs, dws, cancel_floor=1e-6) <= TOL
    assert row_err(gt, dwt, cancel_floor=1e-6) <= TOL


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("plan", [1, 2])
@pytest.mark.parametrize("W0,relu", [(True, False), (False, False), (True, True), (False, True)])
def test_rgcn_small(kind, plan, W0, relu):
    g = graph(kind)
    t = workloads.tiny_tensors(1, g, 64, 64)
    print(f"rgcn {kind} plan={plan} W0={W0} relu={relu}", flush=True)
    run = Runner(g, t)
    got = run.rgcn(W0=W0, relu=relu, plan=plan)
    ref = oracle.rgcn_forward(g, t["h"], t["W"], t["W0"] if W0 else None, relu=relu)
    run.close()
    assert row_err(got, ref) <= TOL


@pytest.mark.parametrize("d_in,d_out", [(128, 128), (64, 128), (128, 64)])
@pytest.mark.parametrize("plan", [1, 2])
def test_rgcn_dims(d_in, d_out, plan):
    g = graph("hub", seed=9)
    t = workloads.tiny_tensors(9, g, d_in, d_out)
    print(f"rgcn dims {d_in}->{d_out} plan={plan}", flush=True)
    run = Runner(g, t)
    got = run.rgcn(plan=plan)
    ref = oracle.rgcn_forward(g, t["h"], t["W"], t["W0"])
    run.close()
    assert row_err(got, ref) <= TOL


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("plan,heads", [(1, 1), (2, 1), (1, 2), (1, 4), (2, 2), (2, 4), (4, 1), (4, 2), (4, 4)])
def test_rgat_small(kind, plan, heads):
    """Plans 1 (transform-first), 2 (aggregate-first; several heads as one
    masked pass per head) and 4 (transform-first with attention+message
    rows), 1 to 4 heads: output and saved statistics against the oracle."""
    g = graph(kind)
    t = workloads.tiny_tensors(2, g, 64, 64, heads=heads, att_var=1.0)
    print(f"rgat {kind} plan={plan} heads={heads}", flush=True)
    run = Runner(g, t)
    got, saved = run.rgat(heads=heads, plan=plan, want_saved=True)
    ref, mx, sm = oracle.rgat_forward(g, t["h"], t["W"], t["w_src"], t["w_dst"], heads=heads,
                                      want_stats=True)
    run.close()
    assert row_err(got, ref) <= TOL
    sv = saved.cpu().numpy()
    np.testing.assert_allclose(sv[..., 0], mx, rtol=1e-4, atol=1e-4)
    np.testing.assert_allclose(sv[..., 1], sm, rtol=1e-4, atol=1e-5)


@pytest.mark.parametrize("plan,heads", [(1, 1), (2, 1), (1, 8), (2, 8), (4, 8), (4, 1)])
def test_rgat_d128(plan, heads):
    g = graph("hub", seed=4)
    t = workloads.tiny_tensors(4, g, 128, 128, heads=heads, att_var=1.0)
    print(f"rgat d128 plan={plan} heads={heads}", flush=True)
    run = Runner(g, t)
    got = run.rgat(heads=heads, plan=plan)
    ref = oracle.rgat_forward(g, t["h"], t["W"], t["w_src"], t["w_dst"], heads=heads)
    run.close()
    assert row_err(got, ref) <= TOL


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("plan", [1, 2])
@pytest.mark.parametrize("W0,relu", [(True, True), (False, False)])
def test_rgcn_d32(kind, plan, W0, relu):
    """Hidden size 32 (the narrow end of the hidden-size sweep)."""
    g = graph(kind, seed=41)
    t = workloads.tiny_tensors(41, g, 32, 32)
    print(f"rgcn d32 {kind} plan={plan} W0={W0} relu={relu}", flush=True)
    run = Runner(g, t)
    got = run.rgcn(W0=W0, relu=relu, plan=plan)
    ref = oracle.rgcn_forward(g, t["h"], t["W"], t["W0"] if W0 else None, relu=relu)
    run.close()
    assert row_err(got, ref) <= TOL


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("plan,heads", [(1, 1), (2, 1), (3, 1), (1, 2)])
def test_rgat_d32(kind, plan, heads):
    g = graph(kind, seed=42)
    t = workloads.tiny_tensors(42, g, 32, 32, heads=heads, att_var=1.0)
    print(f"rgat d32 {kind} plan={plan} heads={heads}", flush=True)
    run = Runner(g, t)
    got, saved = run.rgat(heads=heads, plan=plan, want_saved=True)
    ref, mx, sm = oracle.rgat_forward(g, t["h"], t["W"], t["w_src"], t["w_dst"], heads=heads,
                                      want_stats=True)
    run.close()
    assert row_err(got, ref) <= TOL
    sv = saved.cpu().numpy()
    np.testing.assert_allclose(sv[..., 0], mx, rtol=1e-4, atol=1e-4)
    np.testing.assert_allclose(sv[..., 1], sm, rtol=1e-4, atol=1e-5)


def test_d32_huge_hub():
    """d = 32 through the 256- and 1024-thread reductions and the split
    destination merges (a hub with thousands of in-edges)."""
    g = graph("hub", seed=43, N=200, E=70000, R=3)
    t = workloads.tiny_tensors(43, g, 32, 32, att_var=1.0)
    print("d32 huge hub", flush=True)
    run = Runner(g, t)
    ref_gcn = oracle.rgcn_forward(g, t["h"], t["W"], t["W0"])
    ref_gat = oracle.rgat_forward(g, t["h"], t["W"], t["w_src"], t["w_dst"])
    for plan in (1, 2):
        assert row_err(run.rgcn(plan=plan), ref_gcn) <= TOL
        assert row_err(run.rgat(plan=plan), ref_gat) <= TOL
    ref_rel = oracle.rgat_forward(g, t["h"], t["W"], t["w_src"], t["w_dst"], scope=1)
    assert row_err(run.rgat(scope=1), ref_rel) <= TOL
    run.close()


def test_d32_rejects_mixed_widths():
    import torch
    from paper_2301_06284_amd import rgnn
    g = graph("random", seed=44)
    t = workloads.tiny_tensors(44, g, 32, 64)
    print("d32 mixed widths rejected", flush=True)
    run = Runner(g, t)
    T = run.T
    out = torch.empty(g["N"], 64, device="cuda:0")
    ws = run.ws(0, 32, 64, 1, 1)
    with pytest.raises(rgnn.RgnnError) as e:
        rgnn.rgcn_forward(run.G, T["h"], T["W"], None, out, ws, 32, 64, plan=rgnn.PLAN_TRANSFORM_FIRST)
    assert e.value.status == rgnn.EUNSUPPORTED
    run.close()


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("d", [32, 64, 128])
def test_rgat_per_relation_softmax(kind, d):
    """Softmax over the in-edges of one (destination, relation) segment."""
    g = graph(kind)
    t = workloads.tiny_tensors(21, g, d, d, att_var=1.0)
    print(f"rgat per-relation softmax {kind} d={d}", flush=True)
    run = Runner(g, t)
    got = run.rgat(plan=0, scope=1)
    again = run.rgat(plan=2, scope=1)
    run.close()
    ref = oracle.rgat_forward(g, t["h"], t["W"], t["w_src"], t["w_dst"], scope=1)
    assert row_err(got, ref) <= TOL
    assert np.array_equal(got, again)


def test_rgat_per_relation_softmax_big_segment():
    """One (destination, relation) segment cut into more pieces than one
    thread reduces (the workgroup-per-segment statistics path)."""
    g = graph("hub", seed=22, N=200, E=6000, R=1)
    t = workloads.tiny_tensors(22, g, 64, 64, att_var=1.0)
    print("rgat per-relation softmax big segment", flush=True)
    run = Runner(g, t)
    got = run.rgat(scope=1)
    run.close()
    ref = oracle.rgat_forward(g, t["h"], t["W"], t["w_src"], t["w_dst"], scope=1)
    assert row_err(got, ref) <= TOL


@pytest.mark.parametrize("R", [1, 3])
def test_huge_hub(R):
    """Destinations with hundreds to thousands of virtual segments (the
    workgroup-per-destination reductions at the front of the reduction grid)
    beside ordinary ones, through every plan of RGCN and RGAT."""
    g = graph("hub", seed=24, N=200, E=70000, R=R)
    t = workloads.tiny_tensors(24, g, 64, 64, att_var=1.0)
    print(f"huge hub R={R}", flush=True)
    run = Runner(g, t)
    ref_gcn = oracle.rgcn_forward(g, t["h"], t["W"], t["W0"])
    ref_gat = oracle.rgat_forward(g, t["h"], t["W"], t["w_src"], t["w_dst"])
    for plan in (1, 2):
        assert row_err(run.rgcn(plan=plan), ref_gcn) <= TOL
        assert row_err(run.rgat(plan=plan), ref_gat) <= TOL
    ref_rel = oracle.rgat_forward(g, t["h"], t["W"], t["w_src"], t["w_dst"], scope=1)
    assert row_err(run.rgat(scope=1), ref_rel) <= TOL
    run.close()


def test_rgat_per_relation_softmax_rejects():
    import torch
    from paper_2301_06284_amd import rgnn
    g = graph("random", seed=23)
    t = workloads.tiny_tensors(23, g, 64, 64)
    print("rgat per-relation softmax argument checks", flush=True)
    run = Runner(g, t)
    T = run.T
    out = torch.empty(g["N"], 64, device="cuda:0")
    saved = torch.empty(g["N"], 1, 2, device="cuda:0")
    ws = run.ws(1, 64, 64, 1, 2)
    with pytest.raises(rgnn.RgnnError, match="aggregate-first"):
        rgnn.rgat_forward(run.G, T["h"], T["W"], T["w_src"], T["w_dst"], out, None, ws, 64, 64,
                          softmax_scope=rgnn.SOFTMAX_PER_DST_REL, plan=rgnn.PLAN_TRANSFORM_FIRST)
    run.close()


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("heads", [1, 2, 4])
def test_hgt_small(kind, heads):
    g = graph(kind, T=4, R=7)
    t = workloads.tiny_tensors(3, g, 64, 64, heads=heads)
    scale = 1.0 / np.sqrt(64 // heads)
    print(f"hgt {kind} heads={heads}", flush=True)
    run = Runner(g, t)
    got = run.hgt(heads, scale)
    ref = oracle.hgt_forward(g, t["h"], t["Wk"], t["Wq"], t["Wv"], t["Wa"], t["Watt"], t["Wmsg"],
                             t["mu"], heads=heads, att_scale=scale)
    run.close()
    assert row_err(got, ref) <= TOL


@pytest.mark.parametrize("kind", ["random", "hub", "dups", "empty"])
@pytest.mark.parametrize("d,heads", [(32, 1), (32, 2), (128, 1), (128, 2), (128, 4), (128, 8)])
def test_hgt_hidden_sizes(kind, d, heads):
    """HGT at d = 32 and 128 (the hidden-size sweep), every head count with
    d_k >= 16; R = 7 keeps W_msg in LDS except at d = 128 with one or two
    heads (global reads)."""
    g = graph(kind, T=4, R=7)
    t = workloads.tiny_tensors(49, g, d, d, heads=heads)
    scale = 1.0 / np.sqrt(d // heads)
    print(f"hgt d={d} {kind} heads={heads}", flush=True)
    run = Runner(g, t)
    got = run.hgt(heads, scale)
    ref = oracle.hgt_forward(g, t["h"], t["Wk"], t["Wq"], t["Wv"], t["Wa"], t["Watt"], t["Wmsg"],
                             t["mu"], heads=heads, att_scale=scale)
    run.close()
    assert row_err(got, ref) <= TOL


@pytest.mark.parametrize("kind", ["typed", "typedhub"])
@pytest.mark.parametrize("d,heads", [(32, 1), (32, 2), (64, 1), (64, 2), (64, 4), (128, 2), (128, 8)])
def test_hgt_typed_relations(kind, d, heads):
    """Relations that each join one source type to one destination type: the
    forward folds the query projection into the segment-query weights (all
    widths where the traversal does not form the queries itself)."""
    g = graph(kind, T=4, R=7)
    t = workloads.tiny_tensors(51, g, d, d, heads=heads)
    t["mu"] = (1.0 + 0.25 * np.arange(7)).astype(np.float32)
    scale = 1.0 / np.sqrt(d // heads)
    print(f"hgt typed d={d} {kind} heads={heads}", flush=True)
    run = Runner(g, t)
    got = run.hgt(heads, scale)
    ref = oracle.hgt_forward(g, t["h"], t["Wk"], t["Wq"], t["Wv"], t["Wa"], t["Watt"], t["Wmsg"],
                             t["mu"], heads=heads, att_scale=scale)
    run.close()
    assert row_err(got, ref) <= TOL


@pytest.mark.parametrize("heads,R", [(2, 12), (4, 24)])
def test_hgt_many_relations(heads, R):
    """Enough relations that the per-relation message matrices no longer fit
    in LDS beside the staged items (the traversal reads them from memory)."""
    g = graph("random", T=3, R=R, E=5000)
    t = workloads.tiny_tensors(4, g, 64, 64, heads=heads)
    scale = 1.0 / np.sqrt(64 // heads)
    print(f"hgt heads={heads} R={R}", flush=True)
    run = Runner(g, t)
    got = run.hgt(heads, scale)
    ref = oracle.hgt_forward(g, t["h"], t["Wk"], t["Wq"], t["Wv"], t["Wa"], t["Watt"], t["Wmsg"],
                             t["mu"], heads=heads, att_scale=scale)
    run.close()
    assert row_err(got, ref) <= TOL


@pytest.mark.parametrize("flags", [0, 2, 4])
def test_hgt_flags(flags):
    g = graph("hub", T=2, R=3)
    t = workloads.tiny_tensors(6, g, 64, 64, heads=4)
    print(f"hgt flags={flags}", flush=True)
    run = Runner(g, t)
    got = run.hgt(4, 0.3, flags=flags)
    ref = oracle.hgt_forward(g, t["h"], t["Wk"], t["Wq"], t["Wv"], t["Wa"], t["Watt"], t["Wmsg"],
                             t["mu"], heads=4, att_scale=0.3, residual=bool(flags & 2),
                             a_linear=bool(flags & 4))
    run.close()
    assert row_err(got, ref) <= TOL


@pytest.mark.parametrize("kind", KINDS)
def test_rgat_backward_small(kind):
    g = graph(kind, E=3000)
    t = workloads.tiny_tensors(8, g, 64, 64, att_var=1.0)
    print(f"rgat backward {kind}", flush=True)
    run = Runner(g, t)
    gh, gW, gs, gt = run.rgat_backward()
    run.close()
    dh, dW, dws, dwt = rgat_backward_ref(g, t)
    isolated = (np.bincount(g["src"], minlength=g["N"]) + np.bincount(g["dst"], minlength=g["N"])) == 0
    assert row_err(gh, dh, structural_zero=isolated, cancel_floor=1e-6) <= TOL
    assert row_err(gW.reshape(-1, 64), dW.reshape(-1, 64)) <= TOL
    assert row_err(gs, dws) <= TOL
    assert row_err(gt, dwt) <= TOL


@pytest.mark.parametrize("kind", KINDS)
def test_rgat_backward_per_relation_softmax(kind):
    """Softmax per (dst, rel) segment: the forward's per-segment (max, sum)
    feed the backward; s is summed per segment."""
    g = graph(kind, E=3000)
    t = workloads.tiny_tensors(47, g, 64, 64, att_var=1.0)
    print(f"rgat backward per-relation softmax {kind}", flush=True)
    run = Runner(g, t)
    gh, gW, gs, gt = run.rgat_backward(scope=1)
    run.close()
    dh, dW, dws, dwt = rgat_backward_ref(g, t, scope=1)
    isolated = (np.bincount(g["src"], minlength=g["N"]) + np.bincount(g["dst"], minlength=g["N"])) == 0
    assert row_err(gh, dh, structural_zero=isolated, cancel_floor=1e-6) <= TOL
    # a relation whose segments each repeat one (src, rel) pair has uniform
    # attention, Y = 0 on all its edges and zero w_dst / w_src gradients by
    # cancellation (fp64 ~1e-17, fp32 ~1e-8)
    assert row_err(gW.reshape(-1, 64), dW.reshape(-1, 64), cancel_floor=1e-6) <= TOL
    assert row_err(gs, dws, cancel_floor=1e-6) <= TOL
    assert row_err(gt, dwt, cancel_floor=1e-6) <= TOL


@pytest.mark.parametrize("kind", ["random", "hub", "dups", "empty"])
@pytest.mark.parametrize("heads", [2, 4])
def test_rgat_per_relation_softmax_multihead(kind, heads):
    """Softmax per (dst, rel) segment with several heads: the forward as one
    masked one-head pass per head, the backward in one pass over all heads,
    against the oracle."""
    g = graph(kind, E=3000)
    t = workloads.tiny_tensors(50, g, 64, 64, heads=heads, att_var=1.0)
    print(f"rgat per-relation softmax {kind} heads={heads}", flush=True)
    run = Runner(g, t)
    got, saved = run.rgat(heads=heads, scope=1, want_saved=True)
    ref = oracle.rgat_forward(g, t["h"], t["W"], t["w_src"], t["w_dst"], heads=heads, scope=1)
    assert row_err(got, ref) <= TOL
    sv = saved.cpu().numpy()
    if len(sv):
        assert np.isfinite(sv).all() and (sv[..., 1] >= 1 - 1e-5).all()
    gh, gW, gs, gt = run.rgat_backward(heads=heads, scope=1)
    run.close()
    dh, dW, dws, dwt = rgat_backward_ref(g, t, heads=heads, scope=1)
    isolated = (np.bincount(g["src"], minlength=g["N"]) + np.bincount(g["dst"], minlength=g["N"])) == 0
    assert row_err(gh, dh, structural_zero=isolated, cancel_floor=1e-6) <= TOL
    assert row_err(gW.reshape(-1, 64), dW.reshape(-1, 64), cancel_floor=1e-6) <= TOL
    assert row_err(gs, dws, cancel_floor=1e-6) <= TOL
    assert row_err(gt, dwt, cancel_floor=1e-6) <= TOL


def test_rgat_backward_per_relation_softmax_hub_segments():
    """Segments cut into many pieces (one relation, a 5000-edge hub: more
    than 32 pieces in one segment) and destinations split over work items."""
    g = graph("hub", seed=48, N=400, E=12000, R=1)
    t = workloads.tiny_tensors(48, g, 64, 64, att_var=1.0)
    print("rgat backward per-relation softmax hub segments", flush=True)
    run = Runner(g, t)
    _, saved = run.rgat(scope=1, want_saved=True)
    sv = saved.cpu().numpy()
    assert np.isfinite(sv).all() and (sv[..., 1] >= 1 - 1e-5).all()
    gh, gW, gs, gt = run.rgat_backward(scope=1)
    run.close()
    dh, dW, dws, dwt = rgat_backward_ref(g, t, scope=1)
    isolated = (np.bincount(g["src"], minlength=g["N"]) + np.bincount(g["dst"], minlength=g["N"])) == 0
    assert row_err(gh, dh, structural_zero=isolated, cancel_floor=1e-6) <= TOL
    # a relation whose segments each repeat one (src, rel) pair has uniform
    # attention, Y = 0 on all its edges and zero w_dst / w_src gradients by
    # cancellation (fp64 ~1e-17, fp32 ~1e-8)
    assert row_err(gW.reshape(-1, 64), dW.reshape(-1, 64), cancel_floor=1e-6) <= TOL
    assert row_err(gs, dws, cancel_floor=1e-6) <= TOL
    assert row_err(gt, dwt, cancel_floor=1e-6) <= TOL


@pytest.mark.parametrize("kind", ["random", "hub", "srchub", "dups", "empty"])
@pytest.mark.parametrize("d,heads,scope", [(32, 1, 0), (32, 2, 0), (32, 2, 1), (32, 1, 1), (64, 2, 1), (64, 4, 1),
                                           (128, 1, 0), (128, 2, 0), (128, 4, 1), (128, 8, 0), (128, 8, 1),
                                           (128, 1, 1)])
def test_rgat_backward_hidden_sizes(kind, d, heads, scope):
    """RGAT backward at d = 32, 64 and 128, one to eight heads, both softmax
    scopes (the outer products as 64 x 64 tiles: one zero-padded tile at 32,
    four at 128)."""
    g = graph(kind, E=3000)
    t = workloads.tiny_tensors(51, g, d, d, heads=heads, att_var=1.0)
    print(f"rgat backward d={d} heads={heads} scope={scope} {kind}", flush=True)
    run = Runner(g, t)
    gh, gW, gs, gt = run.rgat_backward(heads=heads, scope=scope)
    run.close()
    dh, dW, dws, dwt = rgat_backward_ref(g, t, heads=heads, scope=scope)
    isolated = (np.bincount(g["src"], minlength=g["N"]) + np.bincount(g["dst"], minlength=g["N"])) == 0
    assert row_err(gh, dh, structural_zero=isolated, cancel_floor=1e-6) <= TOL
    assert row_err(gW.reshape(-1, d), dW.reshape(-1, d), cancel_floor=1e-6) <= TOL
    assert row_err(gs, dws, cancel_floor=1e-6) <= TOL
    assert row_err(gt, dwt, cancel_floor=1e-6) <= TOL


@pytest.mark.parametrize("kind", ["random", "hub", "srchub", "dups", "empty"])
@pytest.mark.parametrize("d", [32, 128])
@pytest.mark.parametrize("W0,relu", [(True, True), (False, False)])
def test_rgcn_backward_hidden_sizes(kind, d, W0, relu):
    g = graph(kind, seed=52)
    t = workloads.tiny_tensors(52, g, d, d)
    print(f"rgcn backward d={d} {kind} W0={W0} relu={relu}", flush=True)
    run = Runner(g, t)
    out = oracle.rgcn_forward(g, t["h"], t["W"], t["W0"] if W0 else None, relu=True) if relu else None
    gh, gW, gW0 = run.rgcn_backward(W0=W0, relu=relu, out=out)
    run.close()
    dh, dW, dW0 = oracle.rgcn_backward(g, t["h"], t["W"], t["W0"] if W0 else None, t["grad_out"], relu=relu)
    isolated = (np.bincount(g["src"], minlength=g["N"]) + np.bincount(g["dst"], minlength=g["N"])) == 0
    assert row_err(gh, dh, structural_zero=None if W0 else isolated, cancel_floor=1e-6) <= TOL
    assert row_err(gW.reshape(-1, d), dW.reshape(-1, d), cancel_floor=1e-6) <= TOL
    if W0:
        assert row_err(gW0, dW0) <= TOL


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("heads", [2, 4])
def test_rgat_backward_multihead(kind, heads):
    """Several heads in one backward pass (gradients in the message space)."""
    g = graph(kind, E=3000)
    t = workloads.tiny_tensors(45, g, 64, 64, heads=heads, att_var=1.0)
    print(f"rgat backward {kind} heads={heads}", flush=True)
    run = Runner(g, t)
    gh, gW, gs, gt = run.rgat_backward(heads=heads)
    run.close()
    dh, dW, dws, dwt = rgat_backward_ref(g, t, heads=heads)
    isolated = (np.bincount(g["src"], minlength=g["N"]) + np.bincount(g["dst"], minlength=g["N"])) == 0
    assert row_err(gh, dh, structural_zero=isolated, cancel_floor=1e-6) <= TOL
    assert row_err(gW.reshape(-1, 64), dW.reshape(-1, 64)) <= TOL
    assert row_err(gs, dws) <= TOL
    assert row_err(gt, dwt) <= TOL


@pytest.mark.parametrize("d,heads,kind", [(64, 2, "hub"), (64, 4, "hub"), (128, 8, "hub"), (64, 4, "srchub"),
                                         (32, 2, "srchub"), (128, 4, "srchub")])
def test_rgat_backward_multihead_mid_size(d, heads, kind):
    """Several heads on a 200k-edge graph with hubs (split destinations and
    sources with many out-edges), every gradient in full, at the standard
    cancellation floor.

    The multi-head forward (transform-first) forms its logits from the message
    rows, the backward from h . (W_r w_src): the two round differently.  The
    backward sums its own softmax denominator, so its alpha sums to one in its
    own arithmetic.  This graph has sources whose only out-edges enter the
    10^5-edge hub (dh norm ~1e-5 of the median) and whose one in-edge forms a
    one-edge softmax, whose Jacobian is exactly zero: with alpha normalised by
    the forward's denominator instead, that zero came out as ~1e-7 |dalpha|,
    a 3e-4 row error.
    With a source hub (half the edges leave node 0: pairs of ~8 000 out-edges,
    cut into 64-edge pieces over several workgroup chunks at d <= 64, and a
    source split over ~1 500 out-edge items) the same checks hold."""
    g = workloads.tiny_graph(46, N=20000, E=200000, R=12, T=2, kind=kind)
    t = workloads.tiny_tensors(46, g, d, d, heads=heads, att_var=1.0)
    print(f"rgat backward d={d} heads={heads} {kind} mid size", flush=True)
    run = Runner(g, t)
    gh, gW, gs, gt = run.rgat_backward(heads=heads)
    run.close()
    dh, dW, dws, dwt = rgat_backward_ref(g, t, heads=heads)
    isolated = (np.bincount(g["src"], minlength=g["N"]) + np.bincount(g["dst"], minlength=g["N"])) == 0
    assert row_err(gh, dh, structural_zero=isolated, cancel_floor=1e-6) <= TOL
    assert row_err(gW.reshape(-1, d), dW.reshape(-1, d)) <= TOL
    assert row_err(gs, dws) <= TOL
    assert row_err(gt, dwt) <= TOL


@pytest.mark.parametrize("plan", [1, 2])
def test_rgat_backward_mid_size_one_head(plan):
    """The graph above with one head, from the saved statistics of either
    forward plan (transform-first forms the source logit from the message
    row, aggregate-first from h . (W_r w_src)), standard cancellation floor."""
    g = workloads.tiny_graph(46, N=20000, E=200000, R=12, T=2, kind="hub")
    t = workloads.tiny_tensors(46, g, 64, 64, heads=1, att_var=1.0)
    print(f"rgat backward heads=1 mid size forward plan={plan}", flush=True)
    run = Runner(g, t)
    gh, gW, gs, gt = run.rgat_backward(heads=1, plan=plan)
    run.close()
    dh, dW, dws, dwt = rgat_backward_ref(g, t)
    isolated = (np.bincount(g["src"], minlength=g["N"]) + np.bincount(g["dst"], minlength=g["N"])) == 0
    assert row_err(gh, dh, structural_zero=isolated, cancel_floor=1e-6) <= TOL
    assert row_err(gW.reshape(-1, 64), dW.reshape(-1, 64)) <= TOL
    assert row_err(gs, dws) <= TOL
    assert row_err(gt, dwt) <= TOL


@pytest.mark.parametrize("d", [64, 128])
def test_backward_mid_size_source_hub(d):
    """One-head RGAT and RGCN backward on a 200k-edge graph whose node 0 sends
    half the edges: its out-edges span ~1 500 work items, whose sums are added
    to its row in slot order."""
    g = workloads.tiny_graph(47, N=20000, E=200000, R=12, T=2, kind="srchub")
    t = workloads.tiny_tensors(47, g, d, d, heads=1, att_var=1.0)
    print(f"rgat/rgcn backward d={d} source hub mid size", flush=True)
    run = Runner(g, t)
    gh, gW, gs, gt = run.rgat_backward(heads=1)
    rh, rW, rW0 = run.rgcn_backward(W0=True, relu=False)
    run.close()
    dh, dW, dws, dwt = rgat_backward_ref(g, t)
    isolated = (np.bincount(g["src"], minlength=g["N"]) + np.bincount(g["dst"], minlength=g["N"])) == 0
    assert row_err(gh, dh, structural_zero=isolated, cancel_floor=1e-6) <= TOL
    assert row_err(gW.reshape(-1, d), dW.reshape(-1, d)) <= TOL
    assert row_err(gs, dws) <= TOL
    assert row_err(gt, dwt) <= TOL
    eh, eW, eW0 = oracle.rgcn_backward(g, t["h"], t["W"], t["W0"], t["grad_out"], relu=False)
    assert row_err(rh, eh) <= TOL
    assert row_err(rW.reshape(-1, d), eW.reshape(-1, d)) <= TOL
    assert row_err(rW0, eW0) <= TOL


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("W0,relu", [(True, False), (False, False), (True, True), (False, True)])
def test_rgcn_backward_small(kind, W0, relu):
    g = graph(kind, E=3000)
    t = workloads.tiny_tensors(31, g, 64, 64)
    w0 = t["W0"] if W0 else None
    print(f"rgcn backward {kind} W0={W0} relu={relu}", flush=True)
    # the ReLU derivative is read from the oracle's forward output, so both
    # sides take the same mask
    out = oracle.rgcn_forward(g, t["h"], t["W"], w0, relu=True) if relu else None
    run = Runner(g, t)
    gh, gW, gW0 = run.rgcn_backward(W0=W0, relu=relu, out=out)
    run.close()
    dh, dW, dW0 = oracle.rgcn_backward(g, t["h"], t["W"], w0, t["grad_out"], relu=relu)
    assert row_err(gh, dh) <= TOL
    assert row_err(gW.reshape(-1, 64), dW.reshape(-1, 64)) <= TOL
    if W0:
        assert row_err(gW0, dW0) <= TOL


def test_rgcn_backward_after_forward():
    """Forward then backward through this library (the mask from its own output)."""
    g = graph("hub", seed=32, E=3000)
    t = workloads.tiny_tensors(32, g, 64, 64)
    print("rgcn forward + backward", flush=True)
    run = Runner(g, t)
    gh, gW, gW0 = run.rgcn_backward(W0=True, relu=True)
    run.close()
    dh, dW, dW0 = oracle.rgcn_backward(g, t["h"], t["W"], t["W0"], t["grad_out"], relu=True)
    assert row_err(gh, dh) <= TOL
    assert row_err(gW.reshape(-1, 64), dW.reshape(-1, 64)) <= TOL
    assert row_err(gW0, dW0) <= TOL


def check_hgt_grads(got, ref, heads, d=64):
    dk = d // heads
    assert row_err(got["dh"], ref["dh"]) <= TOL
    for k in ("dWk", "dWq", "dWv", "dWa"):
        if ref[k] is None:
            continue
        assert row_err(got[k].reshape(-1, d), ref[k].reshape(-1, d)) <= TOL, k
    for k in ("dWatt", "dWmsg"):
        assert row_err(got[k].reshape(-1, dk), ref[k].reshape(-1, dk)) <= TOL, k
    assert row_err(got["dmu"].reshape(1, -1), ref["dmu"].reshape(1, -1)) <= TOL


def hgt_case(kind, heads, seed, flags=None, R=7, T=4, E=4000, scale=None):
    g = graph(kind, seed=seed, T=T, R=R, E=E)
    t = workloads.tiny_tensors(seed, g, 64, 64, heads=heads)
    t["mu"] = (1.0 + 0.25 * np.arange(R)).astype(np.float32)   # distinct priors
    scale = 1.0 / np.sqrt(64 // heads) if scale is None else scale
    return g, t, scale


@pytest.mark.parametrize("use_saved", [False, True])
@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("heads", [1, 2, 4])
def test_hgt_backward_small(kind, heads, use_saved):
    g, t, scale = hgt_case(kind, heads, 33)
    print(f"hgt backward {kind} heads={heads} saved={use_saved}", flush=True)
    run = Runner(g, t)
    got = run.hgt_backward(heads, scale, use_saved=use_saved)
    run.close()
    ref = oracle.hgt_backward(g, t["h"], t["Wk"], t["Wq"], t["Wv"], t["Wa"], t["Watt"], t["Wmsg"],
                              t["mu"], t["grad_out"], heads=heads, att_scale=scale)
    check_hgt_grads(got, ref, heads)


@pytest.mark.parametrize("use_saved", [False, True])
@pytest.mark.parametrize("kind", ["random", "hub", "dups", "empty"])
@pytest.mark.parametrize("d,heads", [(32, 1), (32, 2), (128, 2), (128, 8)])
def test_hgt_backward_hidden_sizes(kind, d, heads, use_saved):
    g = graph(kind, T=4, R=7, E=3000)
    t = workloads.tiny_tensors(53, g, d, d, heads=heads)
    t["mu"] = (1.0 + 0.25 * np.arange(7)).astype(np.float32)   # distinct priors
    scale = 1.0 / np.sqrt(d // heads)
    print(f"hgt backward d={d} heads={heads} {kind} saved={use_saved}", flush=True)
    run = Runner(g, t)
    got = run.hgt_backward(heads, scale, use_saved=use_saved)
    run.close()
    ref = oracle.hgt_backward(g, t["h"], t["Wk"], t["Wq"], t["Wv"], t["Wa"], t["Watt"], t["Wmsg"],
                              t["mu"], t["grad_out"], heads=heads, att_scale=scale)
    check_hgt_grads(got, ref, heads, d)


@pytest.mark.parametrize("use_saved", [False, True])
@pytest.mark.parametrize("kind", ["typed", "typedhub"])
@pytest.mark.parametrize("d,heads", [(32, 2), (64, 4), (128, 8)])
def test_hgt_backward_typed_relations(kind, d, heads, use_saved):
    """Typed relations: the backward recomputes the folded segment queries the
    forward used, so the saved statistics match its scores."""
    g = graph(kind, T=4, R=7, E=3000)
    t = workloads.tiny_tensors(57, g, d, d, heads=heads)
    t["mu"] = (1.0 + 0.25 * np.arange(7)).astype(np.float32)
    scale = 1.0 / np.sqrt(d // heads)
    print(f"hgt backward typed d={d} heads={heads} {kind} saved={use_saved}", flush=True)
    run = Runner(g, t)
    got = run.hgt_backward(heads, scale, use_saved=use_saved)
    run.close()
    ref = oracle.hgt_backward(g, t["h"], t["Wk"], t["Wq"], t["Wv"], t["Wa"], t["Watt"], t["Wmsg"],
                              t["mu"], t["grad_out"], heads=heads, att_scale=scale)
    check_hgt_grads(got, ref, heads, d)


@pytest.mark.parametrize("use_saved", [False, True])
@pytest.mark.parametrize("flags", [0, 2, 4])
def test_hgt_backward_flags(flags, use_saved):
    g, t, scale = hgt_case("hub", 4, 34, R=3, T=2)
    print(f"hgt backward flags={flags} saved={use_saved}", flush=True)
    run = Runner(g, t)
    got = run.hgt_backward(4, 0.3, flags=flags, use_saved=use_saved)
    run.close()
    ref = oracle.hgt_backward(g, t["h"], t["Wk"], t["Wq"], t["Wv"], t["Wa"], t["Watt"], t["Wmsg"],
                              t["mu"], t["grad_out"], heads=4, att_scale=0.3,
                              residual=bool(flags & 2), a_linear=bool(flags & 4))
    check_hgt_grads(got, ref, 4)
    if not flags & 4:
        assert got["dWa"] is None


@pytest.mark.parametrize("heads,R", [(2, 12), (4, 24)])
def test_hgt_backward_many_relations(heads, R):
    g, t, scale = hgt_case("random", heads, 35, R=R, T=3, E=5000)
    print(f"hgt backward heads={heads} R={R}", flush=True)
    run = Runner(g, t)
    got = run.hgt_backward(heads, scale)
    run.close()
    ref = oracle.hgt_backward(g, t["h"], t["Wk"], t["Wq"], t["Wv"], t["Wa"], t["Watt"], t["Wmsg"],
                              t["mu"], t["grad_out"], heads=heads, att_scale=scale)
    check_hgt_grads(got, ref, heads)


@pytest.mark.parametrize("kind", ["random", "hub", "isolated", "empty"])
@pytest.mark.parametrize("d,heads", [(64, 4), (128, 8), (32, 2)])
def test_hgt_forward_saved_statistics(kind, d, heads):
    """The forward's optional softmax statistics: the output is the same with
    and without them; per destination and head, the maximum is the largest
    logit (a_e of the layer's definition, formed here in fp64 from the same
    inputs) and the sum is sum_e exp(a_e - max); (0, 0) without in-edges."""
    g = graph(kind, T=4, R=7, E=3000)
    t = workloads.tiny_tensors(54, g, d, d, heads=heads)
    t["mu"] = (1.0 + 0.25 * np.arange(7)).astype(np.float32)
    scale = 1.0 / np.sqrt(d // heads)
    print(f"hgt forward saved d={d} heads={heads} {kind}", flush=True)
    run = Runner(g, t)
    plain = run.hgt(heads, scale)
    out, saved = run.hgt(heads, scale, want_saved=True)
    sv = saved.cpu().numpy()
    run.close()
    np.testing.assert_array_equal(out, plain)
    # logits of the definition: (K_s,i Watt[r,i]) . Q_t,i * mu[r] * scale
    dk = d // heads
    h = t["h"].astype(np.float64)
    nt = g["ntype"]
    K = np.einsum("nd,nde->ne", h, t["Wk"].astype(np.float64)[nt]).reshape(-1, heads, dk)
    Q = np.einsum("nd,nde->ne", h, t["Wq"].astype(np.float64)[nt]).reshape(-1, heads, dk)
    src, dst, rel = g["src"], g["dst"], g["rel"]
    KW = np.einsum("ehk,ehkl->ehl", K[src], t["Watt"].astype(np.float64)[rel])
    a = (KW * Q[dst]).sum(-1) * t["mu"].astype(np.float64)[rel][:, None] * scale   # [E, heads]
    M = np.full((g["N"], heads), -np.inf)
    np.maximum.at(M, dst, a)
    Z = np.zeros((g["N"], heads))
    np.add.at(Z, dst, np.exp(a - M[dst]))
    has = np.bincount(dst, minlength=g["N"]) > 0
    assert np.all(sv[~has] == 0)
    np.testing.assert_allclose(sv[has, :, 0], M[has], rtol=1e-5, atol=1e-5)
    np.testing.assert_allclose(sv[has, :, 1], Z[has], rtol=1e-4)


@pytest.mark.parametrize("kind", ["random", "hub", "dups", "empty"])
@pytest.mark.parametrize("heads", [1, 2])
def test_rgat_ablation_plans(kind, heads):
    """Transform-first with and without compact materialization (graph flag)
    and with and without linear operator reordering of the destination term
    and with the attention term carried in the message rows all give the
    layer's output."""
    g = graph(kind, seed=37)
    t = workloads.tiny_tensors(37, g, 64, 64, heads=heads, att_var=1.0)
    ref = oracle.rgat_forward(g, t["h"], t["W"], t["w_src"], t["w_dst"], heads=heads)
    for compact in (True, False):
        print(f"rgat ablation {kind} heads={heads} compact={compact}", flush=True)
        run = Runner(g, t, compact=compact)
        if not compact:
            assert run.G.info()["num_src_pairs"] == g["E"]
        for plan in (1, 3, 4):
            assert row_err(run.rgat(heads=heads, plan=plan), ref) <= TOL, (compact, plan)
        run.close()


@pytest.mark.parametrize("kind", ["random", "hub"])
def test_rgcn_without_compaction(kind):
    g = graph(kind, seed=38)
    t = workloads.tiny_tensors(38, g, 64, 64)
    print(f"rgcn no compaction {kind}", flush=True)
    run = Runner(g, t, compact=False)
    got = run.rgcn(plan=1)
    run.close()
    assert row_err(got, oracle.rgcn_forward(g, t["h"], t["W"], t["W0"])) <= TOL


def test_forward_bitwise_deterministic():
    g = graph("hub", seed=12)
    t = workloads.tiny_tensors(12, g, 64, 64, heads=4, att_var=1.0)
    print("determinism", flush=True)
    run = Runner(g, t)
    for fn in (lambda: run.rgcn(plan=1), lambda: run.rgcn(plan=2), lambda: run.rgat(plan=1),
               lambda: run.rgat(plan=2), lambda: run.hgt(4, 0.25)):
        a, b = fn(), fn()
        assert np.array_equal(a, b)
    run.close()


def test_plans_agree():
    g = graph("dups", seed=13)
    t = workloads.tiny_tensors(13, g, 64, 64, att_var=1.0)
    print("plans agree", flush=True)
    run = Runner(g, t)
    for fn in (run.rgcn, run.rgat):
        a, b = fn(plan=1), fn(plan=2)
        assert row_err(a, b.astype(np.float64)) <= 1e-5
    run.close()


def degree_graph(seed, degrees, R, T):
    """In-degrees and out-degrees both run through `degrees` (in different
    node orders), repeated over the nodes; relation r has its own edge count."""
    rng = np.random.default_rng(seed)
    deg = np.repeat(np.asarray(degrees), 3)
    N = len(deg)
    dst = np.repeat(rng.permutation(N), deg).astype(np.int32)
    src = np.repeat(rng.permutation(N), deg).astype(np.int32)
    src = src[rng.permutation(len(src))]
    rel = np.minimum(rng.geometric(0.4, len(src)) - 1, R - 1).astype(np.int32)
    return dict(N=N, E=len(src), R=R, T=T, src=src, dst=dst, rel=rel,
                ntype=rng.integers(0, T, N, dtype=np.int32))


@pytest.mark.parametrize("d", [32, 64, 128])
def test_piece_sizes_of_small_graphs(d):
    """Degrees at the edges of the work items of a small graph (bundles of 16
    edges and 8 nodes, whole destinations up to 64 edges, pieces beyond) and
    relations of 1 to several 64-row tiles: forward and backward of every layer."""
    g = degree_graph(61, [0, 1, 7, 8, 9, 15, 16, 17, 31, 33, 63, 64, 65, 128, 129], R=9, T=3)
    heads = d // 16
    t = workloads.tiny_tensors(61, g, d, d, heads=heads)
    print(f"piece sizes d={d}", flush=True)
    run = Runner(g, t)
    assert row_err(run.rgcn(plan=1), oracle.rgcn_forward(g, t["h"], t["W"], t["W0"])) <= TOL
    assert row_err(run.rgcn(plan=2), oracle.rgcn_forward(g, t["h"], t["W"], t["W0"])) <= TOL
    for plan, H in ((1, heads), (2, 1)):
        ref = oracle.rgat_forward(g, t["h"], t["W"], t["w_src"], t["w_dst"], heads=H)
        assert row_err(run.rgat(heads=H, plan=plan), ref) <= TOL
    hgt = [t[k] for k in ("h", "Wk", "Wq", "Wv", "Wa", "Watt", "Wmsg", "mu")]
    assert row_err(run.hgt(heads, 0.25), oracle.hgt_forward(g, *hgt, heads=heads, att_scale=0.25)) <= TOL
    isolated = (np.bincount(g["src"], minlength=g["N"]) + np.bincount(g["dst"], minlength=g["N"])) == 0
    for H in {1, heads}:
        got = run.rgat_backward(heads=H)
        ref = rgat_backward_ref(g, t, heads=H)
        assert row_err(got[0], ref[0], structural_zero=isolated, cancel_floor=1e-6) <= TOL
        for a, b in zip(got[1:], ref[1:]):
            assert row_err(a.reshape(-1, d), b.reshape(-1, d)) <= TOL
    for a, b in zip(run.rgcn_backward(), oracle.rgcn_backward(g, t["h"], t["W"], t["W0"], t["grad_out"])):
        assert row_err(a.reshape(-1, d), b.reshape(-1, d)) <= TOL
    ref = oracle.hgt_backward(g, *hgt, t["grad_out"], heads=heads, att_scale=0.25)
    for use_saved in (False, True):
        check_hgt_grads(run.hgt_backward(heads, 0.25, use_saved=use_saved), ref, heads, d)
    run.close()


@pytest.mark.parametrize("flags", [0, 2, 4, 6])
@pytest.mark.parametrize("d,heads,R,T", [(32, 1, 3, 5), (64, 4, 20, 3), (128, 2, 5, 1), (128, 8, 7, 2)])
def test_hgt_backward_typed_flags(d, heads, R, T, flags):
    """The folded node-type weights with each output option: node types without
    relations (zero dWq and dWa), more relations than the sixteen slices of the
    per-type sums, one node type, d = 128 with and without in-kernel queries."""
    g = graph("typed", seed=71, N=400, E=5000, R=R, T=T)
    t = workloads.tiny_tensors(71, g, d, d, heads=heads)
    t["mu"] = (1.0 + 0.25 * np.arange(R)).astype(np.float32)
    print(f"hgt backward typed d={d} heads={heads} R={R} T={T} flags={flags}", flush=True)
    run = Runner(g, t)
    got = [run.hgt_backward(heads, 0.3, flags=flags, use_saved=s) for s in (False, True)]
    run.close()
    ref = oracle.hgt_backward(g, t["h"], t["Wk"], t["Wq"], t["Wv"], t["Wa"], t["Watt"], t["Wmsg"], t["mu"],
                              t["grad_out"], heads=heads, att_scale=0.3, residual=bool(flags & 2),
                              a_linear=bool(flags & 4))
    for x in got:
        check_hgt_grads(x, ref, heads, d)


@pytest.mark.parametrize("flags", [0, 2, 4, 6])
@pytest.mark.parametrize("kind", ["hub", "typedhub"])
@pytest.mark.parametrize("d,heads,R", [(32, 1, 7), (64, 1, 3), (64, 2, 40), (128, 1, 2), (128, 2, 3), (128, 4, 20)])
def test_hgt_wide_heads(d, heads, R, kind, flags):
    """Heads whose messages come from a GEMM over the segments: hubs of more
    than 32 segments, with and without the output linear (folded into one
    head's weights on typed relations) and the residual, and the statistics."""
    g = graph(kind, seed=77, N=300, E=12000, R=R, T=2)
    t = workloads.tiny_tensors(77, g, d, d, heads=heads)
    print(f"hgt wide heads d={d} heads={heads} R={R} {kind} flags={flags}", flush=True)
    run = Runner(g, t)
    got, saved = run.hgt(heads, 0.2, flags=flags, want_saved=True)
    args = [t[k] for k in ("h", "Wk", "Wq", "Wv", "Wa", "Watt", "Wmsg", "mu")]
    opt = dict(heads=heads, att_scale=0.2, residual=bool(flags & 2), a_linear=bool(flags & 4))
    assert row_err(got, oracle.hgt_forward(g, *args, **opt)) <= TOL
    sv = saved.cpu().numpy()
    deg = np.bincount(g["dst"], minlength=g["N"])
    assert (sv[deg == 0] == 0).all() and (sv[deg > 0][..., 1] >= 1 - 1e-5).all()
    if flags == 6:
        ref = oracle.hgt_backward(g, *args, t["grad_out"], **opt)
        for use_saved in (False, True):
            check_hgt_grads(run.hgt_backward(heads, 0.2, use_saved=use_saved), ref, heads, d)
    run.close()


@pytest.mark.parametrize("R,E,N", [(1, 6000, 40), (2, 2048, 32), (3, 9000, 300)])
@pytest.mark.parametrize("d", [64, 128])
def test_fused_tile_edges(d, R, E, N):
    """Aggregate-first tiles cut by their edges: segments of 64 edges (16-row
    blocks of 1024, 2048 per 128-wide tile) beside short and empty ones."""
    g = workloads.tiny_graph(83, N=N, E=E, R=R, T=1, kind="hub")
    t = workloads.tiny_tensors(83, g, d, d)
    print(f"fused tiles d={d} R={R} E={E}", flush=True)
    run = Runner(g, t)
    assert row_err(run.rgcn(plan=2), oracle.rgcn_forward(g, t["h"], t["W"], t["W0"])) <= TOL
    for scope in (0, 1):
        ref = oracle.rgat_forward(g, t["h"], t["W"], t["w_src"], t["w_dst"], scope=scope)
        assert row_err(run.rgat(plan=2, scope=scope), ref) <= TOL
    run.close()


@pytest.mark.parametrize("K,Nc", [(64, 64), (128, 128)])
@pytest.mark.parametrize("ws_rows", ["more", "least"])
def test_segment_gemm_workspace_of_other_rows(K, Nc, ws_rows):
    """Workspaces made for more rows than the call has, and of the smallest size
    taken (one 16-byte entry per 512 rows and type, a multiple of 256 bytes)."""
    import torch
    from paper_2301_06284_amd import rgnn
    M, T = 49152, 5
    type_ptr = np.array([0, 1, 1, 20000, 49000, M], np.int64)
    least = (((M + 511) // 512 + T) * 16 + 255) // 256 * 256
    n = rgnn.segment_gemm_workspace_size(60000, T) if ws_rows == "more" else least
    print(f"segment_gemm workspace {ws_rows} {n} bytes {K}x{Nc}", flush=True)
    rng = np.random.default_rng(K)
    dev = torch.device("cuda:0")
    X = torch.from_numpy(rng.standard_normal((M, K)).astype(np.float32)).to(dev)
    W = torch.from_numpy(rng.standard_normal((T, K, Nc)).astype(np.float32)).to(dev)
    Y = torch.full((M, Nc), float("nan"), device=dev)
    buf = torch.full((n + 4096,), 7, dtype=torch.uint8, device=dev)
    rgnn.segment_gemm(X, None, type_ptr, W, Y, None, buf[:n], K, Nc)
    torch.cuda.synchronize()
    assert bool((buf[n:] == 7).all())
    Xh, Wh, got = X.cpu().double(), W.cpu().double(), Y.cpu().numpy()
    for t in range(T):
        b, e = type_ptr[t], type_ptr[t + 1]
        if e > b:
            assert row_err(got[b:e], (Xh[b:e] @ Wh[t]).numpy()) <= TOL


@pytest.mark.parametrize("T", [1, 511, 512, 513, 1030])
@pytest.mark.parametrize("K,Nc", [(32, 32), (64, 128), (128, 128)])
def test_segment_gemm_many_types(K, Nc, T):
    """The device-made tile table: type counts around a launch's 512, types of
    0, 1, 63..65 and several hundred rows; eagerly and captured in a graph that is
    replayed with new inputs between eager calls."""
    import torch
    from paper_2301_06284_amd import rgnn
    rng = np.random.default_rng(T + K)
    counts = rng.choice([0, 0, 1, 2, 63, 64, 65, 130, 700], T, p=[.3, .2, .2, .1, .05, .05, .05, .03, .02])
    counts[-1] = 66
    type_ptr = np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)
    M = int(type_ptr[-1])
    print(f"segment_gemm types T={T} M={M} {K}x{Nc}", flush=True)
    dev = torch.device("cuda:0")
    W = torch.from_numpy(rng.standard_normal((T, K, Nc)).astype(np.float32)).to(dev)
    X, Y = torch.empty(M, K, device=dev), torch.empty(M, Nc, device=dev)
    ws = torch.empty(rgnn.segment_gemm_workspace_size(M, T), dtype=torch.uint8, device=dev)
    seg = np.repeat(np.arange(T), counts)

    def check(call):
        x = rng.standard_normal((M, K)).astype(np.float32)
        X.copy_(torch.from_numpy(x))
        Y.fill_(float("nan"))
        call()
        torch.cuda.synchronize()
        got = Y.cpu().numpy()
        for t in rng.permutation(np.flatnonzero(counts))[:40]:
            ref = x[seg == t].astype(np.float64) @ W[t].double().cpu().numpy()
            assert row_err(got[seg == t], ref) <= TOL
        assert np.isfinite(got).all()

    def call():
        rgnn.segment_gemm(X, None, type_ptr, W, Y, None, ws, K, Nc)
    check(call)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        call()
    for _ in range(3):
        check(g.replay)
        check(call)


@pytest.mark.parametrize("flags", [0, 4])
@pytest.mark.parametrize("d", [32, 64, 128])
def test_hgt_wide_heads_nan_row(d, flags):
    """A source row of NaN reaches every destination it has an edge to, also those
    of more than 32 segments whose shares several groups of lanes merge (one item:
    at most 64 in-edges), and no other destination."""
    N, R, bad = 80, 64, 70
    rng = np.random.default_rng(91)
    dst = np.concatenate([np.full(n, v) for v, n in enumerate((33, 40, 64, 48))] + [np.arange(4, 64)])
    rel = np.concatenate([np.arange(n) for n in (33, 40, 64, 48)] + [np.zeros(60, int)])
    src = rng.integers(0, 64, len(dst))
    hit = [0 * 33 + 5, 33 + 39, 33 + 40 + 17, 33 + 40 + 64 + 48 + 3]   # one edge of nodes 0, 1, 2 and 7
    src[hit] = bad
    g = dict(N=N, E=len(src), R=R, T=1, src=src.astype(np.int32), dst=dst.astype(np.int32),
             rel=rel.astype(np.int32), ntype=np.zeros(N, np.int32))
    t = workloads.tiny_tensors(91, g, d, d, heads=1)
    print(f"hgt NaN row d={d} flags={flags}", flush=True)
    run = Runner(g, t)
    clean = run.hgt(1, 0.2, flags=flags)
    run.close()
    t["h"][bad] = np.nan
    run = Runner(g, t)
    got = run.hgt(1, 0.2, flags=flags)
    run.close()
    reached = np.isin(np.arange(N), dst[hit])
    assert np.isnan(got[reached]).all()
    np.testing.assert_array_equal(got[~reached], clean[~reached])


@pytest.mark.parametrize("flags", [2, 6])
@pytest.mark.parametrize("d,heads", [(32, 2), (64, 4), (128, 1)])
def test_hgt_backward_unused_weights(d, heads, flags):
    """The weights of a relation without edges and of a node type without nodes
    have no part in the layer: whatever they hold, the gradients of everything
    else are what they are with ordinary values there."""
    N, R, T = 300, 6, 4
    g = workloads.tiny_graph(93, N=N, E=5000, R=R, T=T, kind="random")
    g["ntype"] = (1 + np.arange(N) % 3).astype(np.int32)                    # none of type 0
    g["rel"] = np.where(g["ntype"][g["dst"]] == 1, g["rel"] % 2, 1 + g["ntype"][g["dst"]]).astype(np.int32)
    assert not (g["rel"] == 5).any() and len(np.unique(g["rel"])) == 4      # 5 (and one type's 4) unused
    unused = np.setdiff1d(np.arange(R), g["rel"])
    t = workloads.tiny_tensors(93, g, d, d, heads=heads)
    print(f"hgt backward unused weights d={d} heads={heads} flags={flags}", flush=True)
    run = Runner(g, t)
    clean = [run.hgt_backward(heads, 0.3, flags=flags, use_saved=s) for s in (False, True)]
    run.close()
    for k in ("Wk", "Wq", "Wv", "Wa"):
        t[k][0] = np.nan
    for k in ("Watt", "Wmsg"):
        t[k][unused] = np.inf
    t["mu"][unused] = np.nan
    run = Runner(g, t)
    got = [run.hgt_backward(heads, 0.3, flags=flags, use_saved=s) for s in (False, True)]
    run.close()
    used = np.setdiff1d(np.arange(R), unused)
    for a, b in zip(got, clean):
        for k in a:
            if a[k] is None:
                continue
            rows = used if k in ("dWatt", "dmu") else slice(None)   # those scale with the weights themselves
            np.testing.assert_array_equal(a[k][rows], b[k][rows], err_msg=k)


@pytest.mark.parametrize("kind", ["hub", "typedhub"])
@pytest.mark.parametrize("R", [12, 13, 25, 26, 32, 33])
def test_hgt_traversal_threads(R, kind):
    """Relation counts at which the d = 64 traversal with heads of 16 changes its
    workgroup (two of 512 threads, one of 1024, one of 512, matrices from L2)."""
    g = graph(kind, seed=95, N=500, E=9000, R=R, T=2)
    t = workloads.tiny_tensors(95, g, 64, 64, heads=4)
    print(f"hgt traversal threads R={R} {kind}", flush=True)
    run = Runner(g, t)
    got, saved = run.hgt(4, 0.25, want_saved=True)
    run.close()
    args = [t[k] for k in ("h", "Wk", "Wq", "Wv", "Wa", "Watt", "Wmsg", "mu")]
    assert row_err(got, oracle.hgt_forward(g, *args, heads=4, att_scale=0.25)) <= TOL
    assert np.isfinite(saved.cpu().numpy()).all()


@pytest.mark.parametrize("flags", [0, 2, 4, 6])
@pytest.mark.parametrize("d,heads,R", [(32, 1, 127), (32, 1, 128), (32, 2, 255), (32, 2, 300), (64, 1, 63), (64, 1, 130),
                                       (64, 4, 254), (64, 4, 260), (128, 1, 27), (128, 1, 31), (128, 1, 40),
                                       (128, 4, 127), (128, 4, 130), (128, 8, 254), (128, 8, 260)])
def test_hgt_folded_weights_rule(d, heads, R, flags):
    """One-type graphs on both sides of the rules that fold the node-type weights
    into the per-relation ones (400 nodes: R dk up to 4075 in the backward, R d^2 up
    to 455 600 for the forward's output linear), many relations without edges."""
    g = workloads.tiny_graph(97, N=400, E=3000, R=R, T=1, kind="hub")
    t = workloads.tiny_tensors(97, g, d, d, heads=heads)
    print(f"hgt folded weights d={d} heads={heads} R={R} flags={flags}", flush=True)
    args = [t[k] for k in ("h", "Wk", "Wq", "Wv", "Wa", "Watt", "Wmsg", "mu")]
    opt = dict(heads=heads, att_scale=0.25, residual=bool(flags & 2), a_linear=bool(flags & 4))
    run = Runner(g, t)
    out = run.hgt(heads, 0.25, flags=flags)
    got = [run.hgt_backward(heads, 0.25, flags=flags, use_saved=s) for s in (False, True)]
    run.close()
    assert row_err(out, oracle.hgt_forward(g, *args, **opt)) <= TOL
    ref = oracle.hgt_backward(g, *args, t["grad_out"], **opt)
    for x in got:
        check_hgt_grads(x, ref, heads, d)


@pytest.mark.parametrize("per_seg", [53, 54, 64, 200])
def test_fused_long_segments(per_seg):
    """Graphs on both sides of the rule for long segments (54 edges on average) at
    128 x 128: RGCN and both softmaxes aggregate-first, RGCN backward (the segment
    means keep the short tiles), with relations of 1 to 40 destinations."""
    rng = np.random.default_rng(per_seg)
    N, R = 200, 5
    pairs = [(v, r) for r, n in enumerate((1, 15, 16, 17, 40)) for v in rng.choice(N, n, replace=False)]
    dst, rel = np.repeat(np.array(pairs), per_seg, axis=0).T
    mix = rng.permutation(len(dst))
    g = dict(N=N, E=len(dst), R=R, T=1, src=rng.integers(0, N, len(dst), dtype=np.int32),
             dst=dst[mix].astype(np.int32), rel=rel[mix].astype(np.int32), ntype=np.zeros(N, np.int32))
    t = workloads.tiny_tensors(per_seg, g, 128, 128)
    print(f"fused long segments {per_seg}", flush=True)
    run = Runner(g, t)
    assert row_err(run.rgcn(plan=2), oracle.rgcn_forward(g, t["h"], t["W"], t["W0"])) <= TOL
    for scope in (0, 1):
        ref = oracle.rgat_forward(g, t["h"], t["W"], t["w_src"], t["w_dst"], scope=scope)
        assert row_err(run.rgat(plan=2, scope=scope), ref) <= TOL
    for a, b in zip(run.rgcn_backward(), oracle.rgcn_backward(g, t["h"], t["W"], t["W0"], t["grad_out"])):
        assert row_err(a.reshape(-1, 128), b.reshape(-1, 128)) <= TOL
    run.close()


@pytest.mark.parametrize("T", [3072, 3073, 9000])
def test_segment_gemm_thousands_of_types(T):
    """Type counts on both sides of the host-made tile table, with empty types and
    some of several tiles: eagerly, and captured (where the table is made on the
    device) and replayed with new inputs between eager calls."""
    import torch
    from paper_2301_06284_amd import rgnn
    rng = np.random.default_rng(T)
    counts = rng.choice([0, 1, 3, 65, 200], T, p=[.5, .3, .15, .04, .01])
    type_ptr = np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)
    M = int(type_ptr[-1])
    print(f"segment_gemm thousands of types T={T} M={M}", flush=True)
    dev = torch.device("cuda:0")
    W = torch.from_numpy(rng.standard_normal((T, 64, 64)).astype(np.float32)).to(dev)
    X, Y = torch.empty(M, 64, device=dev), torch.empty(M, 64, device=dev)
    ws = torch.empty(rgnn.segment_gemm_workspace_size(M, T), dtype=torch.uint8, device=dev)
    seg = torch.from_numpy(np.repeat(np.arange(T), counts)).to(dev)

    def check(call):
        X.copy_(torch.from_numpy(rng.standard_normal((M, 64)).astype(np.float32)))
        Y.fill_(float("nan"))
        call()
        torch.cuda.synchronize()
        for lo in range(0, M, 4096):   # the rows' own weights, in double precision
            x, w = X[lo:lo + 4096].double(), W[seg[lo:lo + 4096]].double()
            ref = (x[:, :, None] * w).sum(1)
            assert row_err(Y[lo:lo + 4096].cpu().numpy(), ref.cpu().numpy()) <= TOL

    def call():
        rgnn.segment_gemm(X, None, type_ptr, W, Y, None, ws, 64, 64)
    check(call)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        call()
    for _ in range(3):
        check(g.replay)
        check(call)


@pytest.mark.parametrize("K,Nc", [(32, 32), (64, 64), (128, 128), (64, 128), (128, 64)])
def test_segment_gemm_full_tiles(K, Nc):
    """Tiles of 512 rows (the smallest workspace the call takes leaves room for no
    others), every wave with several row blocks: gathered and scattered rows, types
    that end inside a block, after one, in the next tile's first; rows over twelve
    decades, each entry within a few fp32 roundoffs of the exact product."""
    import torch
    from paper_2301_06284_amd import rgnn
    rng = np.random.default_rng(7 * K + Nc)
    counts = np.array([511, 0, 512, 513, 1, 1025, 700, 495, 16, 3000])
    type_ptr = np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)
    M, T = int(type_ptr[-1]), len(counts)
    X = (rng.standard_normal((M + 50, K)) * 10.0 ** rng.uniform(-6, 6, (M + 50, 1))).astype(np.float32)
    W = (rng.standard_normal((T, K, Nc)) * 10.0 ** rng.uniform(-3, 3, (T, 1, Nc))).astype(np.float32)
    gather = rng.integers(0, M + 50, M).astype(np.int32)
    scatter = rng.permutation(M + 9)[:M].astype(np.int32)
    least = (((M + 511) // 512 + T) * 16 + 255) // 256 * 256
    print(f"segment_gemm full tiles {K}x{Nc}", flush=True)
    dev = torch.device("cuda:0")
    Y = torch.full((M + 9, Nc), float("nan"), device=dev)
    rgnn.segment_gemm(torch.from_numpy(X).to(dev), torch.from_numpy(gather).to(dev), type_ptr,
                      torch.from_numpy(W).to(dev), Y, torch.from_numpy(scatter).to(dev),
                      torch.empty(least, dtype=torch.uint8, device=dev), K, Nc)
    torch.cuda.synchronize()
    got = Y.cpu().numpy().astype(np.float64)
    assert np.isnan(got[np.setdiff1d(np.arange(M + 9), scatter)]).all()
    for t in range(T):
        rows = np.arange(type_ptr[t], type_ptr[t + 1])
        x, w = X[gather[rows]].astype(np.float64), W[t].astype(np.float64)
        if len(rows):
            err = np.abs(got[scatter[rows]] - x @ w) / (2.0 ** -24 * (np.abs(x) @ np.abs(w)))
            assert err.max() <= 8.0


def check_layers(g, d, heads, hgt_heads, seed):
    """Forward and backward of every layer and plan at width d against the oracle.

    RGAT's dh of a node without out-edges is a sum of softmax Jacobian terms that
    nearly cancel when its relations' vectors point the same way.  The terms are of the
    median row's size, so fp32 leaves about 2^-24 of that (measured: 4e-8): below
    1e-3 of the median that alone can exceed 1e-4 of the row (2^-24 / 1e-4 = 6e-4),
    and such rows are measured against the median row."""
    t = workloads.tiny_tensors(seed, g, d, d, heads=max(hgt_heads))
    isolated = (np.bincount(g["src"], minlength=g["N"]) + np.bincount(g["dst"], minlength=g["N"])) == 0
    run = Runner(g, t)
    ref = oracle.rgcn_forward(g, t["h"], t["W"], t["W0"], relu=True)
    for plan in (1, 2):
        assert row_err(run.rgcn(plan=plan, relu=True), ref) <= TOL
    for a, b in zip(run.rgcn_backward(), oracle.rgcn_backward(g, t["h"], t["W"], t["W0"], t["grad_out"])):
        assert row_err(a.reshape(-1, d), b.reshape(-1, d)) <= TOL
    print("  rgcn", flush=True)
    for plan, H, scope in ((1, heads, 0), (2, 1, 0), (2, 1, 1)):
        ref = oracle.rgat_forward(g, t["h"], t["W"], t["w_src"], t["w_dst"], heads=H, scope=scope)
        assert row_err(run.rgat(heads=H, plan=plan, scope=scope), ref) <= TOL
    for H in {1, heads}:
        got, ref = run.rgat_backward(heads=H), rgat_backward_ref(g, t, heads=H)
        assert row_err(got[0], ref[0], structural_zero=isolated, cancel_floor=1e-3) <= TOL
        for a, b in zip(got[1:], ref[1:]):
            assert row_err(a.reshape(-1, d), b.reshape(-1, d), cancel_floor=1e-6) <= TOL
    run.close()
    print("  rgat", flush=True)
    for H in hgt_heads:
        t = workloads.tiny_tensors(seed, g, d, d, heads=H)
        args = [t[k] for k in ("h", "Wk", "Wq", "Wv", "Wa", "Watt", "Wmsg", "mu")]
        run = Runner(g, t)
        assert row_err(run.hgt(H, 0.25), oracle.hgt_forward(g, *args, heads=H, att_scale=0.25)) <= TOL
        ref = oracle.hgt_backward(g, *args, t["grad_out"], heads=H, att_scale=0.25)
        for use_saved in (False, True):
            check_hgt_grads(run.hgt_backward(H, 0.25, use_saved=use_saved), ref, H, d)
        run.close()
        print(f"  hgt {H}", flush=True)


@pytest.mark.parametrize("kind", ["hub", "srchub", "typedhub"])
@pytest.mark.parametrize("d", [32, 64, 128])
def test_layers_with_several_blocks_per_wave(d, kind):
    """Graphs large enough that a tile gives every wave several 16-row blocks (GEMM
    tiles of 128 to 192 rows and fused ones of 128 to 192 for the narrow shapes, 320
    to 512 and 256 rows at 128 x 128), with ragged ends and hubs: every layer, plan
    and backward, HGT with narrow and wide heads."""
    g = workloads.tiny_graph(101, N=20000, E=200000 if kind != "typedhub" else 400000, R=12, T=3, kind=kind)
    print(f"several blocks per wave d={d} {kind}", flush=True)
    check_layers(g, d, heads=d // 16, hgt_heads=sorted({1, d // 16}), seed=101)


@pytest.mark.parametrize("d_in,d_out", [(64, 128), (128, 64)])
@pytest.mark.parametrize("plan", [1, 2])
def test_rgcn_dims_several_blocks(d_in, d_out, plan):
    g = workloads.tiny_graph(103, N=20000, E=200000, R=12, T=1, kind="hub")
    t = workloads.tiny_tensors(103, g, d_in, d_out)
    print(f"rgcn dims, several blocks {d_in}->{d_out} plan={plan}", flush=True)
    run = Runner(g, t)
    for relu in (False, True):
        ref = oracle.rgcn_forward(g, t["h"], t["W"], t["W0"], relu=relu)
        assert row_err(run.rgcn(plan=plan, relu=relu), ref) <= TOL
    run.close()


def test_layers_of_a_sparse_graph():
    """Far fewer edges than nodes: bundles of many destinations with few edges."""
    g = workloads.tiny_graph(105, N=200000, E=3000, R=5, T=3, kind="random")
    print("sparse graph", flush=True)
    check_layers(g, 32, heads=2, hgt_heads=[1, 2], seed=105)
