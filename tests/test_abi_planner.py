"""CPU-side checks (no GPU): the C-ABI library loads and exports every symbol the header declares,
graph ingest validates and infers shapes, and the optimiser (fusion pre-pass, operator linking,
operator split) produces plans that are structurally sound.  No kernel is launched here."""
import ctypes
import os
import re

import numpy as np
import pytest

from paper_2302_00282_amd import xenos as X
from workloads import cnn_graphs as wg

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def plan_json(g, **kw):
    G = X.graph_from_workload(g)
    try:
        P = X.xenos_plan_link_split(G, **kw)
        try:
            return X.xenos_plan_query(P)
        finally:
            X.xenos_destroy(P)
    finally:
        X.xenos_destroy(G)


def test_library_exports_every_declared_symbol():
    hdr = open(os.path.join(ROOT, "include", "xenos.h")).read()
    names = set(re.findall(r"\b(xenos_[a-z_]+)\s*\(", hdr))
    assert {"xenos_graph_create", "xenos_plan_link_split", "xenos_run", "xenos_destroy"} <= names
    lib = ctypes.CDLL(X.LIB_PATH)
    for n in sorted(names):
        assert hasattr(lib, n), n


def test_missing_library_fails_loudly(monkeypatch):
    monkeypatch.setattr(X, "_lib", None)
    monkeypatch.setattr(X, "LIB_PATH", "/nonexistent/libxenos.so")
    with pytest.raises(ImportError):
        X.lib()


def test_graph_validation_errors():
    g = wg.single_chain(batch=1)
    keep = []
    ops = X.op_descs(g, keep)
    ind = X.TensorDesc(1, 3, 32, 32, X.XENOS_F32, X.XENOS_NCHW)
    with pytest.raises(X.XenosError) as e:
        X.xenos_graph_create(ind, ops, 9)                      # output id out of range
    assert e.value.status == X.XENOS_EINVAL
    bad = X.op_descs(g, keep)
    bad[0].weight = ctypes.cast(None, ctypes.POINTER(ctypes.c_float))
    with pytest.raises(X.XenosError) as e:
        X.xenos_graph_create(ind, bad, 4)
    assert e.value.status == X.XENOS_EINVAL and "weight" in str(e.value)
    bad = X.op_descs(g, keep)
    bad[0].kh = bad[0].kw = 40                                 # kernel larger than the padded map
    with pytest.raises(X.XenosError) as e:
        X.xenos_graph_create(ind, bad, 4)
    assert e.value.status == X.XENOS_ESHAPE
    with pytest.raises(X.XenosError) as e:                     # wrong output descriptor
        X.xenos_graph_create(ind, ops, 4, X.TensorDesc(1, 16, 8, 8, X.XENOS_F32, X.XENOS_NCHW))
    assert e.value.status == X.XENOS_ESHAPE
    b = wg.builder("bad_add", (1, 8, 8, 8), 1)
    t1 = b.conv(0, 8, 3, 1, 1)
    t2 = b.conv(0, 8, 3, 2, 1)
    b.g.ops.append(wg.Op("add", [t1, t2]))
    with pytest.raises(X.XenosError) as e:
        X.xenos_graph_create(X.TensorDesc(1, 8, 8, 8, 0, 0), X.op_descs(b.g, keep), 3)
    assert e.value.status == X.XENOS_ESHAPE
    assert X.xenos_destroy(None) is None


def test_slice_and_shuffle_validation():
    g = wg.single_chain(batch=1)                                   # 16 output channels
    g.ops.append(wg.Op("slice", [len(g.ops)], dict(c_begin=10, out_c=8), {}, "s"))
    g.output = len(g.ops)
    with pytest.raises(X.XenosError) as e:
        X.graph_from_workload(g)
    assert e.value.status == X.XENOS_ESHAPE and "slice" in str(e.value)
    g.ops[-1] = wg.Op("shuffle", [len(g.ops) - 1], dict(groups=3), {}, "s")
    with pytest.raises(X.XenosError) as e:
        X.graph_from_workload(g)
    assert e.value.status == X.XENOS_ESHAPE and "shuffle" in str(e.value)
    g.ops[-1] = wg.Op("shuffle", [len(g.ops) - 1], dict(groups=4), {}, "s")
    j = plan_json(g, link=2)["plan"]
    assert j["linked_shuffles"] == 0 and sum(1 for c in j["chains"] if c["kind"] == "elt") == 4   # one strided copy per group


def test_plan_option_errors():
    G = X.graph_from_workload(wg.single_chain(batch=1))
    try:
        with pytest.raises(X.XenosError):
            X.xenos_plan_link_split(G, link=7)
        with pytest.raises(X.XenosError):
            X.xenos_plan_link_split(G, hw=dict(num_cu=0, lds_bytes_per_cu=0, l2_bytes=0, llc_bytes=0, hbm_bytes=0))
        with pytest.raises(X.XenosError) as e:                 # private memory too small for any parameter split
            X.xenos_plan_link_split(G, hw=dict(num_cu=8, lds_bytes_per_cu=4096, l2_bytes=0, llc_bytes=0, hbm_bytes=0))
        assert e.value.status == X.XENOS_EUNSUPPORTED
    finally:
        X.xenos_destroy(G)


def test_cfg0_links_to_one_chain_and_unlinked_levels():
    g = wg.build(0, 1)
    q2 = plan_json(g, link=2)["plan"]
    q1 = plan_json(g, link=1)["plan"]
    q0 = plan_json(g, link=0)["plan"]
    assert q2["n_chains"] == 1 and q2["chains"][0]["ops"] == [0, 1, 2, 3]       # CBR + MaxPool = one pass (CBRM)
    assert q2["chains"][0]["mode"] == "zigzag"
    assert [c["ops"] for c in q1["chains"] if c["kind"] == "conv"] == [[0, 1, 2]]   # fused CBR, pool separate
    assert sum(1 for c in q0["chains"] if c["ops"]) == 4                            # operator by operator
    assert q0["hbm_bytes"] > q1["hbm_bytes"] > q2["hbm_bytes"]


@pytest.mark.parametrize("cfg,batch", [(1, 1), (2, 1), (2, 32), (4, 1), (4, 32)])
def test_every_operator_runs_exactly_once(cfg, batch):
    g = wg.build(cfg, batch, draw=False)
    for link in (0, 1, 2):
        q = plan_json(g, link=link, compute=X.XENOS_BF16)["plan"]
        # (the summing pass of a reduction split completes the chain of the step before it and names the same operators)
        seen = [o for c in q["chains"] if c["kind"] != "splitk_finish" for o in c["ops"]]
        # a hoisted pooling operator appears once per concat producer; a copied concat once per input
        assert set(seen) == set(range(len(g.ops))) - ({i for i, o in enumerate(g.ops) if o.kind == "concat"} if link >= 2 else set())
        if link < 2:
            non_cat = [o for o in seen if g.ops[o].kind != "concat"]
            assert len(non_cat) == len(set(non_cat))


@pytest.mark.parametrize("compute", [X.XENOS_F32, X.XENOS_BF16])
@pytest.mark.parametrize("hw,rows", [(13, 64), (14, 128), (7, 64), (8, 64), (11, 128), (17, 64)])
def test_global_average_takes_the_tile_that_pads_less(hw, rows, compute):
    b = wg.builder("gap", (32, 64, hw, hw), 3)
    g = b.finish(b.gap(b.cbr(b.cbr(0, 64, 1, name="a"), 1000, 1, name="c")))
    chain = [c for c in plan_json(g, link=2, compute=compute)["plan"]["chains"] if c.get("mode") == "gap"]
    assert len(chain) == 1 and chain[0]["bm"] == rows and chain[0]["bn"] == 64


@pytest.mark.parametrize("hw,ksz,compute,rows", [(20, 1, X.XENOS_F32, 64), (20, 1, X.XENOS_BF16, 128), (17, 3, X.XENOS_F32, 64), (17, 3, X.XENOS_BF16, 128),
                                                  (17, 1, X.XENOS_BF16, 64), (13, 3, X.XENOS_BF16, 64), (20, 3, X.XENOS_F32, 64)])
def test_global_average_near_the_rows_of_the_larger_tile(hw, ksz, compute, rows):
    # 20x20: 448 rows against 512, which pays in fp32 only; 17x17: 320 against 384, which in bf16 pays for 1x1 layers only
    b = undrawn((32, 64, hw, hw))
    g = b.finish(b.gap(b.cbr(b.cbr(0, 64, 1, name="a"), 1000, ksz, 1, ksz // 2, name="c")))
    chain, = [c for c in plan_json(g, link=2, compute=compute)["plan"]["chains"] if c.get("mode") == "gap"]
    assert chain["bm"] == rows and chain["bn"] == 64


def test_linking_patterns_of_the_workloads():
    g2 = wg.build(2, 1, draw=False)
    res = plan_json(g2, link=2, compute=X.XENOS_BF16)["plan"]
    convs = [c for c in res["chains"] if c["kind"] == "conv"]
    # every shortcut add is executed by a conv chain (in its epilogue, or in the summing pass of a reduction split)
    assert sum(any(g2.ops[o].kind == "add" for o in c["ops"]) for c in convs) == 8
    # the 7x7/2 first layer reads the caller's NCHW tensor in place with its 3x3/2 max-pool linked (CBRM): no pass of its own
    assert convs[0]["loader"] == "stem" and any(g2.ops[o].kind == "maxpool" for o in convs[0]["ops"]) and convs[0]["pool"] != 0
    assert all(c["kind"] in ("conv", "splitk_finish") for c in res["chains"])
    # (on the fp32 path the first layer gathers from memory and its pooling is the only stand-alone pass)
    r32 = plan_json(g2, link=2, compute=X.XENOS_F32)["plan"]
    assert r32["chains"][0]["loader"] == "stem" and r32["chains"][1]["kind"] == "pool"
    assert all(c["kind"] in ("conv", "splitk_finish") for c in r32["chains"][2:])
    # last block + global average (CBRA): through the summing pass of a reduction split (batch 1: the gather kernel's
    # split, batch 32: channel chunks shared out inside the halo-staged kernel); without the operator split the average
    # runs in the convolution's own epilogue.  Either way it is an operator of that chain, not a pass of its own
    assert any(g2.ops[o].kind == "gap" for o in convs[-2]["ops"]) and convs[-2]["mode"] == "flat"
    assert res["chains"][convs[-2]["i"] + 1]["kind"] == "splitk_finish"
    res32 = plan_json(wg.build(2, 32, draw=False), link=2, compute=X.XENOS_BF16)["plan"]
    last32 = [c for c in res32["chains"] if c["kind"] == "conv"][-2]
    assert last32["mode"] == "flat" and last32["halo"] == 1 and last32["ksplit"] > 1 and any(g2.ops[o].kind == "gap" for o in last32["ops"])
    assert res32["chains"][last32["i"] + 1]["kind"] == "splitk_finish"
    # the 7x7 x 512 layers at batch 32: 9 pixel tiles x 4 channel tiles would occupy 36 of 256 units; their channel
    # chunks are shared out so that at least half the units work
    shared = [c for c in res32["chains"] if c["kind"] == "conv" and c["halo"] == 1 and c["ksplit"] > 1]
    assert len(shared) == 3 and all(c["H"] == 7 and 2 * c["tiles_m"] * c["tiles_n"] * c["ksplit"] >= 256 for c in shared)
    u32 = plan_json(wg.build(2, 32, draw=False), link=2, split=0, compute=X.XENOS_BF16)["plan"]
    assert [c for c in u32["chains"] if c["kind"] == "conv"][-2]["mode"] == "gap"
    assert not any(c["kind"] == "splitk_finish" for c in u32["chains"])
    sq = plan_json(wg.build(4, 1, draw=False), link=2, compute=X.XENOS_BF16)["plan"]
    # bf16: the 3x3/2 first layer stages its input block in LDS and its 3x3/2 ceil-mode pool is linked into it; fp32: the
    # gather form of the first-layer kernel, then the pool as the only stand-alone pass
    assert sq["chains"][0]["loader"] == "stem" and sq["chains"][0]["pool"] != 0
    assert all(c["kind"] in ("conv", "splitk_finish") for c in sq["chains"])   # concat and the pools cost no pass
    assert sum(c.get("mode") == "patch" for c in sq["chains"][1:]) == 4      # 3x3/2 ceil-mode pools linked into both expand convs, twice
    sq32 = plan_json(wg.build(4, 1, draw=False), link=2, compute=X.XENOS_F32)["plan"]
    assert sq32["chains"][0]["loader"] == "stem" and sq32["chains"][1]["kind"] == "pool"
    assert all(c["kind"] in ("conv", "splitk_finish") for c in sq32["chains"][2:])
    # a first layer of 24 channels (ShuffleNet-style graph) runs on the same kernel, padded to 32
    sh = plan_json(wg.shufflenet_v2(batch=1, draw=False), link=2, compute=X.XENOS_BF16)["plan"]
    assert sh["chains"][0]["loader"] == "stem" and sh["chains"][0]["K"] == 32 and sh["chains"][0]["pool"] != 0
    offs = sorted({(c["out_c_off"], c["out_sP"]) for c in sq["chains"] if c["kind"] == "conv" and c["out_c_off"]})
    assert (64, 128) in offs and (256, 512) in offs            # expand3x3 halves land at their channel offset
    vgg = plan_json(wg.build(3, 2, draw=False), link=2, compute=X.XENOS_BF16)["plan"]
    assert [c["mode"] for c in vgg["chains"] if c["kind"] == "conv"].count("zigzag") == 5
    # the layout transform of the graph input is linked into the first layer: no import pass, the caller's NCHW
    # tensor is read where it lies; un-linked plans convert first
    assert vgg["chains"][0]["kind"] == "conv" and vgg["chains"][0]["loader"] == "stem"
    vgg1 = plan_json(wg.build(3, 2, draw=False), link=1, compute=X.XENOS_BF16)["plan"]
    assert vgg1["chains"][0]["name"] == "import" and vgg1["chains"][1]["loader"] == "vector"


def test_shufflenet_units_link_their_shuffles():
    # ShuffleNet (Section 7.1): every unit ends in concat -> channel shuffle.  Linked, the shuffle is the order in which
    # the concat's parts are stored: no pass of its own.  The last chain of a unit reads the other half (the pass-through
    # half, or the other branch of a down-sampling unit) in its epilogue and stores both, alternating: no copy either.
    g = wg.shufflenet_v2(batch=1, draw=False)
    n_shuffle = sum(1 for op in g.ops if op.kind == "shuffle")
    assert n_shuffle == 16
    plans = {link: plan_json(g, link=link, compute=1)["plan"] for link in (0, 1, 2, 3)}
    for link in (2, 3):
        j = plans[link]
        assert j["linked_shuffles"] == n_shuffle
        assert sum(1 for c in j["chains"] if c["kind"] == "elt") == 0
        assert sum(1 for c in j["chains"] if c.get("shuffle_store")) == n_shuffle
        ran = sorted(o for c in j["chains"] for o in c["ops"])
        gone = {i for i, op in enumerate(g.ops) if op.kind in ("shuffle", "slice")}    # views and store orders: no pass
        cats = {i for i, op in enumerate(g.ops) if op.kind == "concat"}
        assert set(ran) | gone | cats == set(range(len(g.ops))) and not (set(ran) & {i for i in gone if g.ops[i].kind == "shuffle"})
    for link in (0, 1):
        j = plans[link]
        assert j["linked_shuffles"] == 0
        # un-linked: concat copies both parts, the shuffle copies both groups
        assert sum(1 for c in j["chains"] if c["kind"] == "elt" and "group" in c["name"]) == 2 * n_shuffle
    assert plans[2]["hbm_bytes"] < plans[1]["hbm_bytes"] < plans[0]["hbm_bytes"]
    assert plans[2]["n_chains"] < plans[1]["n_chains"] < plans[0]["n_chains"]


@pytest.mark.parametrize("cfg,batch,compute", [(1, 1, 0), (2, 32, 1), (3, 32, 1), (4, 32, 0)])
def test_split_covers_the_output_and_fits_private_memory(cfg, batch, compute):
    g = wg.build(cfg, batch, draw=False)
    q = plan_json(g, link=2, compute=compute)
    for c in q["plan"]["chains"]:
        if c["kind"] != "conv":
            continue
        assert c["lds"] <= X.MI355X["lds_bytes_per_cu"]
        assert c["tiles_n"] * c["bn"] >= c["K"] > (c["tiles_n"] - 1) * c["bn"]      # outC partition, no gap, no overlap
        if c.get("halo"):
            # halo-staged kernel: TH x TW tiles over the images stacked with their two padding rows each
            assert c["th"] * c["tw"] <= c["bm"] == 256
            assert c["tiles_m"] == -(-(c["N"] * (c["H"] + 2)) // c["th"]) * -(-c["W"] // c["tw"])
        elif c["loader"] == "stem" and c["bm"] == 128:
            # first layer with its input block staged on chip: 8 x 16 tiles of output pixels (3 x 8 pooling windows) per image
            if c["pool"]:
                assert c["tiles_m"] == c["N"] * -(-c["PH"] // 3) * -(-c["PW"] // 8)
            else:
                assert c["tiles_m"] == c["N"] * -(-c["OH"] // 8) * -(-c["OW"] // 16)
        elif c["mode"] == "flat":
            m = c["N"] * c["OH"] * c["OW"]
            assert c["tiles_m"] * c["bm"] >= m > (c["tiles_m"] - 1) * c["bm"]
        elif c["mode"] == "zigzag":
            m = c["N"] * c["PH"] * c["PW"] * 4
            assert c["tiles_m"] * c["bm"] >= m > (c["tiles_m"] - 1) * c["bm"]
        elif c["mode"] == "patch":
            assert c["patch_h"] * c["patch_w"] <= c["bm"]
            py, px = -(-c["PH"] // c["pph"]), -(-c["PW"] // c["ppw"])
            assert c["tiles_m"] == c["N"] * py * px
        if c.get("halo"):
            assert 1 <= c["grid"] <= max(8, X.MI355X["num_cu"])      # persistent workgroups walk the tiles
        elif c["loader"] == "stem" and c["bm"] == 128:
            assert c["tiles_n"] == 1 and 1 <= c["grid"] <= c["tiles_m"]                               # persistent workgroups walk the tiles
        elif c["loader"] == "stem":
            assert c["bm"] == 32 and c["tiles_n"] == 1 and 1 <= c["grid"] <= -(-c["tiles_m"] // 4)   # wavefronts stride over 32-pixel blocks
        else:
            assert c["grid"] >= c["tiles_m"] * c["tiles_n"]
    assert q["workspace_bytes"] > 0 and q["weight_bytes"] > 0


def test_unsplit_plan_uses_one_workgroup():
    q = plan_json(wg.build(0, 1), link=2, split=0)["plan"]
    assert all(c["grid"] == 1 for c in q["chains"] if c["kind"] == "conv")


def test_hardware_description_drives_the_split():
    g = wg.build(2, 32, draw=False)
    big = plan_json(g, compute=1)["plan"]
    small = plan_json(g, compute=1, hw=dict(num_cu=8, lds_bytes_per_cu=160 * 1024, l2_bytes=1 << 20, llc_bytes=0, hbm_bytes=1 << 30))["plan"]
    tb = sum(c["tiles_m"] * c["tiles_n"] for c in big["chains"] if c["kind"] == "conv")
    ts = sum(c["tiles_m"] * c["tiles_n"] for c in small["chains"] if c["kind"] == "conv")
    assert ts <= tb            # fewer units -> never a finer split


def test_planning_time_is_reported_scale():
    import time
    g = wg.build(1, 1)
    G = X.graph_from_workload(g)
    t0 = time.perf_counter()
    P = X.xenos_plan_link_split(G, compute=X.XENOS_BF16)
    dt = time.perf_counter() - t0
    X.xenos_destroy(P)
    X.xenos_destroy(G)
    assert dt < 5.0            # the paper reports 0.11 s for MobileNet (Table 2); same order of magnitude


def test_table4_graphs_follow_the_printed_shapes():
    # tests/golden/table4_shapes.txt holds the shapes printed in Table 4 (first row with the stated reading)
    import os
    rows = {}
    for ln in open(os.path.join(os.path.dirname(__file__), "golden", "table4_shapes.txt")):
        if ln.startswith("#") or not ln.strip():
            continue
        f = ln.split()
        rows[f[0]] = [int(x) for x in f[1:8]]
    names = {"cbr_maxpool": "CBR-MaxPooling", "cbr_avgpool": "CBR-AvgPooling", "fully_connected": "FullyConnected", "cbr": "CBR"}
    assert set(names) == set(wg.TABLE4)
    for key, printed in names.items():
        h, w, c, r, s_, c2, k = rows[printed]
        assert wg.TABLE4[key][:6] == (h, w, c, r, s_, k) and c2 == c
        g = wg.table4(key, batch=1, draw=False)
        q = plan_json(g, link=2, compute=X.XENOS_BF16)["plan"]
        assert sum(ch["kind"] == "conv" for ch in q["chains"]) == 1                  # one linked chain each (plus the input conversion)
        assert all(ch["kind"] in ("conv", "cvt", "splitk_finish") for ch in q["chains"])


def test_partition_candidates_and_tune_argument_checks():
    # every convolution chain carries the legal partitions the split planner found (what xenos_plan_tune profiles);
    # chains whose plan structure depends on the choice carry none
    q = plan_json(wg.build(3, 32, draw=False), link=2, compute=X.XENOS_BF16)["plan"]
    convs = [c for c in q["chains"] if c["kind"] == "conv"]
    assert convs[0]["loader"] == "stem" and convs[0]["candidates"] == 0
    assert all(c["candidates"] >= 3 for c in convs[1:13])              # general tiles + halo tiles for the 3x3 layers
    assert all(c["candidates"] == 0 for c in convs if c["ksplit"] > 1)
    assert all(c["tuned"] == 0 for c in convs)
    forced = plan_json(wg.build(0, 1), link=2, tile=3)["plan"]
    assert all(c["candidates"] == 0 for c in forced["chains"] if c["kind"] == "conv")
    G = X.graph_from_workload(wg.build(0, 1))
    P = X.xenos_plan_link_split(G)
    try:
        with pytest.raises(X.XenosError) as e:
            X.xenos_plan_tune(P, 256, 256)                             # not bound: rejected before anything is launched
        assert e.value.status == X.XENOS_EINVAL
        with pytest.raises(X.XenosError):
            X.xenos_plan_tune(P, 0, 256)
    finally:
        X.xenos_destroy(P)
        X.xenos_destroy(G)


def test_kernels_with_a_weight_order_of_their_own_have_candidates_in_it():
    # the variants of the 3x3 kernel whose weights go into registers, and either tile of the fp32 wave kernel
    q = plan_json(wg.build(3, 32, draw=False), link=3, compute=X.XENOS_BF16)["plan"]
    frag = [c for c in q["chains"] if c.get("frag3")]
    assert len(frag) > 6 and all(c["candidates"] == 5 for c in frag)
    wave = [c for c in plan_json(wg.build(4, 32, draw=False), link=3, compute=X.XENOS_F32)["plan"]["chains"] if c.get("wave") and c["loader"] == "vector"]
    assert {c["bm"] for c in wave} == {32, 64}
    for c in wave:                                                     # (raw sums for a summing pass: the plan depends on the tile)
        assert c["candidates"] == (0 if c["out"]["tensor"] < 0 else 2), c


def test_run_entry_points_reject_bad_arguments_before_any_launch():
    # xenos_run / xenos_run_with / xenos_run_static / xenos_run_graph / xenos_run_chain on a plan that is not bound, and
    # null pointers: XENOS_EINVAL with a message, nothing touches the device (there is none here)
    G = X.graph_from_workload(wg.build(0, 1))
    P = X.xenos_plan_link_split(G)
    try:
        for call in (lambda: X.xenos_run(P, 256, 256), lambda: X.xenos_run_with(P, 256, 256, 256), lambda: X.xenos_run_static(P, 256, 256),
                     lambda: X.xenos_run_graph(P, 256, 256), lambda: X.xenos_run_chain(P, 0, 256, 256)):
            with pytest.raises(X.XenosError) as e:
                call()
            assert e.value.status == X.XENOS_EINVAL and "bound" in str(e.value)
        for call in (lambda: X.xenos_run_with(P, 0, 256, 256), lambda: X.xenos_run_with(P, 256, 0, 256), lambda: X.xenos_run_with(P, 256, 256, 0),
                     lambda: X.xenos_run(P, 0, 256)):
            with pytest.raises(X.XenosError) as e:
                call()
            assert e.value.status == X.XENOS_EINVAL
    finally:
        X.xenos_destroy(P)
        X.xenos_destroy(G)


# ------------------------------------------------------------------------------------------ link level 3, one test per pattern
def _kinds(g, c):
    return [g.ops[o].kind for o in c["ops"]]


def test_pattern_pointwise_to_depthwise_on_chip():
    # Section 2.2 / Table 1 (ConvX -> ConvY): a depthwise-separable stack becomes pointwise -> depthwise chains, the
    # tensors that reach memory are the (smaller) depthwise outputs
    g = wg.build(1, 1, draw=False)
    for compute in (X.XENOS_BF16, X.XENOS_F32):
        l2 = plan_json(g, link=2, compute=compute)["plan"]
        l3 = plan_json(g, link=3, compute=compute)["plan"]
        pw = [c for c in l3["chains"] if c.get("loader") == "pwdw"]
        assert len(pw) == 12 and l3["n_chains"] <= l2["n_chains"] - 12
        for c in pw:
            assert _kinds(g, c) == ["conv", "bn", "relu", "conv", "bn", "relu"]
            conv1, conv2 = [o for o in c["ops"] if g.ops[o].kind == "conv"]
            assert g.ops[conv1].attrs["groups"] == 1 and g.ops[conv2].attrs["groups"] == c["K"]
            s = g.ops[conv2].attrs["stride"]
            # tiles of depthwise output pixels cover the output; the staged block of the pointwise output fits the kernel's LDS block
            assert c["tiles_m"] == c["N"] * -(-c["OH"] // c["th"]) * -(-c["OW"] // c["tw"]) and c["tiles_n"] == -(-c["K"] // 64)
            assert ((c["th"] - 1) * s + 3) * ((c["tw"] - 1) * s + 3) <= 400 and c["lds"] <= 160 * 1024
            assert c["out"]["c"] == c["K"] and c["out"]["h"] == c["OH"]
        # only the first depthwise convolution (its producer is the 3x3 first layer) runs as a chain of its own
        assert sum(c["kind"] == "dwconv" for c in l3["chains"]) == 1
        # (the byte counts include the partial sums of the reduction splits of the tail, the same at both levels)
        assert l3["hbm_bytes"] < 0.70 * l2["hbm_bytes"]
    assert all(c.get("loader") != "pwdw" for c in l2["chains"])


@pytest.mark.parametrize("compute,n,hw,c,mid,k,linked", [
    # linked: the widths of the ShuffleNet graph, narrow units at any size, a narrow middle between wide ends
    (1, 32, 28, 88, 88, 88, 1), (1, 32, 14, 176, 176, 176, 1), (1, 32, 7, 352, 352, 352, 1), (0, 32, 14, 88, 88, 88, 1),
    (0, 1, 32, 24, 24, 24, 1), (1, 1, 56, 24, 144, 24, 1), (1, 8, 28, 1024, 128, 1024, 1), (1, 8, 28, 512, 512, 512, 1),
    # apart: wide units, whose tiles of a few pixels read all weights each (measured 1.2 to 5 times the time of the two chains)
    (0, 1, 38, 728, 728, 728, 0), (0, 1, 32, 1024, 1024, 1024, 0), (0, 8, 28, 512, 512, 512, 0), (0, 32, 7, 256, 256, 256, 0),
    (0, 8, 14, 96, 576, 96, 0), (1, 8, 14, 512, 512, 512, 0), (1, 1, 32, 728, 728, 728, 0), (1, 8, 28, 1024, 1024, 1024, 0)])
def test_unit_is_one_chain_only_where_that_is_faster(compute, n, hw, c, mid, k, linked):
    b = wg._Builder("unit", (n, 8, hw, hw), 1, False, False)
    t = b.cbr(0, c, 1, name="pre")
    t = b.cbr(t, mid, 1, name="pw")
    t = b.cbr(t, mid, 3, 1, 1, groups=mid, name="dw", relu=False)
    t = b.cbr(t, k, 1, name="pw2")
    g = b.finish(b.cbr(t, 8, 3, 1, 1, name="post"))
    info = plan_json(g, link=3, compute=compute)["plan"]
    assert sum(ch.get("loader") == "unit" for ch in info["chains"]) == linked, [(ch["kind"], ch.get("loader")) for ch in info["chains"]]
    ran = [o for ch in info["chains"] if ch["kind"] != "splitk_finish" for o in ch["ops"]]
    assert sorted(ran) == list(range(len(g.ops)))


@pytest.mark.parametrize("n,c,hw,mid,k,r1,pool", [(32, 64, 27, 48, 128, 3, 1), (12, 192, 61, 32, 96, 1, 1), (8, 128, 110, 48, 128, 3, 0),
                                                  (4, 128, 150, 32, 40, 3, 1), (32, 256, 55, 48, 192, 3, 0)])
def test_fire_tiles_leave_no_nearly_empty_round(n, c, hw, mid, k, r1, pool):
    # two workgroups to a unit, 512 at a time: a tile size that gives a few more than that costs a round for those few
    b = wg._Builder("pair", (n, 8, hw, hw), 1, False, False)
    t = b.cbr(0, c, 1, name="pre")
    t = b.cbr(t, mid, r1, 1, r1 // 2, name="first")
    t = b.cbr(t, k, 1, name="second")
    t = b.maxpool(t, 3, 2, 0, ceil=1) if pool else t
    g = b.finish(b.cbr(t, 8, 1, name="post"))
    fire, = [ch for ch in plan_json(g, link=3, compute=1)["plan"]["chains"] if ch.get("loader") == "fire"]
    tiles = fire["tiles_m"] * fire["tiles_n"]
    assert tiles <= 512 or tiles >= 0.8 * 256 * -(-tiles // 256), tiles


def test_pattern_depthwise_to_pointwise_on_chip():
    # a depthwise convolution whose pointwise consumer ends the cascade keeps the older link: its result is the
    # operand panel of the pointwise GEMM (ShuffleNet units of the first two stages; the third, 352 channels, is too
    # wide for that kernel and links pointwise -> depthwise instead)
    g = wg.build(5, 1, draw=False)
    l3 = plan_json(g, link=3, compute=X.XENOS_BF16)["plan"]
    dwpw = [c for c in l3["chains"] if c.get("dw_linked") and c.get("loader") == "vector"]
    pwdw = [c for c in l3["chains"] if c.get("loader") == "pwdw"]
    assert len(dwpw) >= 12 and len(pwdw) == 4
    for c in dwpw:
        k = _kinds(g, c)
        assert k[0] == "conv" and g.ops[c["ops"][0]].attrs["groups"] > 1 and k.count("conv") == 2
    for c in pwdw:
        assert c["K"] == 352 and _kinds(g, c).count("conv") == 2


def undrawn(shape):
    """A builder whose tensors are shapes only (the input has no array): for plans of graphs too large to draw."""
    b = wg._Builder("undrawn", (1, 1, 1, 1), 1, False, False)
    b.g.input_shape, b.g.x, b._shapes = tuple(shape), None, [tuple(shape)]
    return b


@pytest.mark.parametrize("compute", [X.XENOS_F32, X.XENOS_BF16])
@pytest.mark.parametrize("ksz,pool", [(3, 1), (7, 0), (7, 1)])
def test_first_layer_of_an_image_beyond_32_bit_offsets_is_gathered(ksz, pool, compute):
    # stem_lds_kernel's offsets inside an image are 32 bits, 4 channels + 64 rows of it: 104 w elements here
    def first(w):
        b = undrawn((1, 3, 8, w))
        t = b.cbr(0, 64, ksz, 2, ksz // 2, name="a")
        t = b.maxpool(t, 3, 2, 1) if pool else t
        return plan_json(b.finish(b.cbr(t, 8, 1, name="b")), link=3, compute=compute)["plan"]["chains"][0]
    fits, beyond = first((1 << 31) // 104 - 2), first((1 << 31) // 104 + 2)
    if compute == X.XENOS_BF16 or (ksz == 3 and pool):
        assert fits["loader"] == "stem" and fits["bm"] == 128
    assert beyond["loader"] == "stem" and beyond["bm"] == 32 and beyond["pool"] == 0


@pytest.mark.parametrize("compute", [X.XENOS_F32, X.XENOS_BF16])
def test_first_layer_whose_windows_pass_32_bits_is_imported(compute):
    # the gather's table holds 32-bit offsets inside a window, here 2 channels + 2 rows + 2: 18 w + 2 elements
    def first(w):
        b = undrawn((1, 3, 8, w))
        return plan_json(b.finish(b.cbr(b.cbr(0, 64, 3, 2, 1, name="a"), 8, 1, name="b")), link=3, compute=compute)["plan"]["chains"][0]
    w = ((1 << 31) - 3) // 18
    assert first(w)["loader"] == "stem" and first(w + 1)["kind"] == "cvt"


def test_large_tensors_keep_the_halo_kernel():
    # the channel-chunk order is conv3x3_kernel's too, which has no 32-bit windows: two fp32 images of 2.2 GB stay on it, a layer that it
    # does not take (stride 2) is planned as before, and so is a forced tile of the general kernel
    def second(stride, **kw):
        b = undrawn((2, 8, 2950, 2950))
        t = b.cbr(b.cbr(0, 64, 1, name="a"), 128, 3, stride, 1, name="b")
        return plan_json(b.finish(b.cbr(t, 8, 1, name="c")), link=2, compute=X.XENOS_F32, **kw)["plan"]["chains"][-2]
    assert second(1)["halo"] and not second(2)["halo"] and not second(1, tile=3)["halo"]


def test_linked_3x3_pair_of_images_just_below_the_limit():
    # two images of 32 KB less than 2 GB: the weights of the first convolution are in channel-chunk order whatever conv_kernel could address
    b = undrawn((2, 8, 257, 65280))
    t = b.cbr(b.cbr(b.cbr(0, 64, 1, name="a"), 32, 3, 1, 1, name="b"), 64, 1, name="c")
    chains = plan_json(b.finish(b.cbr(t, 8, 1, name="d")), link=3, compute=X.XENOS_BF16)["plan"]["chains"]
    assert [c.get("loader") for c in chains].count("fire") == 1


@pytest.mark.parametrize("pattern,compute", [("pwdw", X.XENOS_F32), ("pwdw", X.XENOS_BF16), ("fire", X.XENOS_BF16), ("fire3", X.XENOS_BF16)])
def test_images_beyond_2_gb_stay_linked(pattern, compute):
    # the windows of pw_gemm_phase cover the rows of a block, not an image (2.2 GB here)
    b = undrawn((1, 8, 2950, 2950))
    t = b.cbr(0, 128 if compute else 64, 1, name="a")
    if pattern == "pwdw":
        t = b.cbr(b.cbr(t, 16, 1, name="pw"), 16, 3, 2, 1, groups=16, name="dw")
    else:
        t = b.cbr(t, 32, 3 if pattern == "fire3" else 1, 1, int(pattern == "fire3"), name="sq")
        t = b.concat([b.cbr(t, 16, 1, name="e1"), b.cbr(t, 16, 3, 1, 1, name="e3")]) if pattern == "fire" else b.cbr(t, 16, 1, name="e1")
    chains = plan_json(b.finish(b.cbr(t, 8, 3, 1, 1, name="z")), link=3, compute=compute)["plan"]["chains"]
    assert [c.get("loader") for c in chains].count(pattern[:4]) == 1


@pytest.mark.parametrize("c,k,ksz,pool,n,hw,staged", [(1, 48, 5, 2, 1, 64, 0), (1, 48, 5, 3, 1, 64, 0), (2, 48, 5, 3, 1, 64, 1), (1, 24, 5, 2, 1, 64, 1),
                                                       (3, 48, 3, 2, 1, 64, 0), (3, 48, 3, 3, 1, 64, 1), (3, 32, 3, 2, 1, 64, 1), (1, 64, 5, 2, 1, 64, 1),
                                                       (3, 48, 3, 2, 2, 224, 1), (1, 48, 5, 3, 2, 224, 1)])
def test_small_fp32_first_layers_with_padded_channels(c, k, ksz, pool, n, hw, staged):
    # the general kernel gathers a small input in place: it keeps such a layer of more than 32 channels where that is one reduction step
    # of 16 or more taps, or windows of 2; other layers, and inputs from 100000 pixels on, are staged on chip
    b = undrawn((n, c, hw, hw))
    t = b.maxpool(b.cbr(0, k, ksz, 1, ksz // 2, name="a"), pool, 2, ceil=1)
    chain = plan_json(b.finish(b.cbr(t, 8, 1, name="b")), link=3, compute=X.XENOS_F32)["plan"]["chains"][0]
    assert (chain["loader"] == "stem" and chain["bm"] == 128) if staged else chain["loader"] == "scalar"


def test_pattern_first_layer_pair_on_chip():
    g = wg.build(3, 2, draw=False)
    l3 = plan_json(g, link=3, compute=X.XENOS_BF16)["plan"]
    c0 = l3["chains"][0]
    assert c0["loader"] == "pair" and _kinds(g, c0) == ["conv", "relu", "conv", "relu", "maxpool"] and c0["in"]["mem"] == "input"
    assert plan_json(g, link=3, compute=X.XENOS_F32)["plan"]["chains"][0]["loader"] == "stem"   # the pair kernel is bf16 only


def test_first_layer_pair_of_a_batch_beyond_32_bit_offsets_stays_apart():
    # conv_pair_kernel's offsets in the graph input are 32 bits: n + 4 / 3 images of 3 x 512 x 512
    def first(n):
        b = undrawn((n, 3, 512, 512))
        t = b.cbr(b.cbr(0, 64, 3, 1, 1, name="a"), 64, 3, 1, 1, name="b")
        return plan_json(b.finish(b.cbr(b.maxpool(t, 2, 2), 8, 1, name="c")), link=3, compute=X.XENOS_BF16)["plan"]["chains"][0]["loader"]
    n = ((1 << 31) - 1) // (3 << 18) - 2
    assert first(n) == "pair" and first(n + 2) == "stem"


def test_plan_metadata_names_the_graph_tensor_of_every_view():
    # per-chain checks rely on it: every chain's input / output view says which graph tensor (and channel range) it holds
    for cfg in (1, 2, 4, 5):
        g = wg.build(cfg, 1, draw=False)
        shapes = g.shapes()
        for link in (0, 2, 3):
            q = plan_json(g, link=link, compute=X.XENOS_BF16)["plan"]
            for c in q["chains"]:
                for key in ("in", "in2", "out"):
                    v = c.get(key)
                    if v is None or v["tensor"] < 0:
                        continue
                    n, ch, h, w = shapes[v["tensor"]]
                    assert (v["n"], v["h"], v["w"]) == (n, h, w) and v["c0"] + (v["c"] - 1) * v["cs"] < ch, (cfg, link, c["name"], key, v)
            assert q["chains"][-1]["out"]["tensor"] == g.output and q["chains"][-1]["out"]["mem"] == "output"


@pytest.mark.parametrize("n,hw,c,k,wave", [
    (16, 30, 32, 512, False), (166, 13, 64, 256, False), (4, 56, 64, 192, False),                  # 7200, 7016 and 2352 tiles
    (42, 8, 192, 256, True), (44, 8, 192, 256, False), (44, 8, 256, 256, True),                    # 672 of six steps, 704 of six and of eight
    (87, 8, 64, 256, True), (88, 8, 64, 256, False),                                               # expansions, 1392 and 1408
    (31, 13, 192, 192, False), (16, 16, 192, 288, True),                                           # 984 and 1152 of six steps
    (13, 13, 512, 704, True), (25, 13, 512, 416, False),                                           # 1518 and 1729 of sixteen
    (16, 28, 88, 88, True), (12, 28, 256, 256, True), (12, 28, 192, 256, False),                    # 1176 of 88 channels; 2352 of eight steps and of six
    (102, 14, 256, 256, True), (102, 14, 32, 256, False), (41, 28, 256, 128, False),               # 5000 of eight steps and of one, 4020
    (166, 13, 256, 256, False), (40, 55, 64, 32, True), (58, 35, 96, 96, True)])                   # 7016; half and three quarters of 64 channels
def test_fp32_pointwise_layers_of_many_tiles_keep_the_larger_ones(n, hw, c, k, wave):
    b = undrawn((n, c, hw, hw))
    g = b.finish(b.cbr(b.cbr(b.cbr(0, c, 1, name="pre"), k, 1, name="a"), 8, 1, name="post"))
    chain = [ch for ch in plan_json(g, link=2, compute=X.XENOS_F32)["plan"]["chains"] if ch["kind"] == "conv"][1]
    assert (chain["C"], chain["K"]) == (c, k) and ((chain["bm"], chain["bn"]) == (32, 32)) == wave, chain


@pytest.mark.parametrize("n,hw,c,k,ksz,stride,wave", [
    (75, 14, 128, 256, 3, 1, True), (78, 14, 64, 256, 3, 1, False), (84, 14, 64, 256, 3, 1, True),  # 3680, 3824 and 4120 tiles
    (20, 56, 32, 128, 3, 1, False), (163, 28, 128, 256, 3, 2, False), (75, 56, 32, 32, 3, 1, True), # 7840, 7992; half of 64 channels
    (5, 10, 512, 512, 5, 1, False), (5, 7, 512, 512, 5, 1, False), (3, 14, 512, 512, 5, 1, True),  # 64, 32 and 80 tiles of 64 x 64
    (16, 8, 256, 256, 5, 1, False), (16, 8, 192, 256, 5, 1, True), (20, 14, 1024, 256, 3, 2, False)])   # 200 and 150 steps, 288
def test_fp32_layers_keep_the_larger_tiles_where_those_fill_their_rounds(n, hw, c, k, ksz, stride, wave):
    b = undrawn((n, c, hw, hw))
    g = b.finish(b.cbr(b.cbr(b.cbr(0, c, 1, name="pre"), k, ksz, stride, ksz // 2, name="a"), 8, 1, name="post"))
    chain = [ch for ch in plan_json(g, link=2, compute=X.XENOS_F32)["plan"]["chains"] if ch["kind"] == "conv"][1]
    assert (chain["C"], chain["K"]) == (c, k) and ((chain["bm"], chain["bn"]) == (32, 32)) == wave, chain


@pytest.mark.parametrize("n,hw,c,k,ksz,stride,bm", [
    (16, 10, 192, 384, 1, 1, 32), (16, 10, 256, 416, 1, 1, 0), (16, 10, 192, 416, 1, 1, 32),      # 600 tiles of three steps, 650 of four, an expansion
    (40, 10, 256, 256, 1, 1, 0), (40, 10, 128, 256, 1, 1, 32), (32, 8, 512, 384, 1, 1, 32),       # 1000 of four and, an expansion, of two, 768 of eight
    (17, 15, 512, 512, 1, 1, 0), (12, 14, 640, 448, 1, 1, 64), (27, 7, 576, 1152, 1, 1, 0),       # 1920 of eight, 1036 of ten, 1512 of nine
    (27, 7, 1024, 1152, 1, 1, 64), (128, 8, 4096, 256, 1, 1, 0),                                   # sixteen steps; to a sixteenth of the channels
    (1, 56, 2048, 128, 3, 1, 0), (1, 55, 2048, 384, 3, 1, 0), (1, 56, 1024, 128, 3, 1, 32),       # the halo kernel's shares
    (128, 8, 2048, 256, 3, 2, 0), (128, 10, 2048, 256, 3, 2, 64), (16, 8, 2048, 256, 3, 2, 32)])   # 512, 800 and 64 tiles
def test_bf16_layers_that_other_kernels_run_faster(n, hw, c, k, ksz, stride, bm):
    b = undrawn((n, c, hw, hw))
    g = b.finish(b.cbr(b.cbr(b.cbr(0, c, 1, name="pre"), k, ksz, stride, ksz // 2, name="a"), 8, 1, name="post"))
    chain = [ch for ch in plan_json(g, link=3, compute=X.XENOS_BF16)["plan"]["chains"] if ch["kind"] == "conv"][1]
    wave = chain["halo"] == 0 and chain["bm"] == chain["bn"] and chain["lds"] % (chain["bm"] * 1024) == 0   # (stages of whole tiles, without padding)
    assert (chain["C"], chain["K"]) == (c, k) and chain["bm"] * wave == bm, chain


@pytest.mark.parametrize("compute,rows,hw,c,k,wave", [
    (X.XENOS_F32, 32, 7, 512, 4096, True), (X.XENOS_F32, 40, 7, 512, 4096, False), (X.XENOS_F32, 100, 7, 512, 4096, False), (X.XENOS_F32, 160, 7, 512, 1024, True),
    (X.XENOS_BF16, 160, 7, 512, 1024, True), (X.XENOS_BF16, 256, 7, 512, 1024, True)])
def test_fully_connected_layers_of_many_steps(compute, rows, hw, c, k, wave):
    b = undrawn((rows, c, hw, hw))
    g = b.finish(b.fc(b.fc(b.cbr(0, c, 1, name="pre"), k, "fc"), 8, "post"))
    chain = [ch for ch in plan_json(g, link=3, compute=compute)["plan"]["chains"] if ch["kind"] == "conv"][1]
    assert (chain["C"], chain["K"], bool(chain["wave"])) == (c, k, wave), chain


@pytest.mark.parametrize("rows,c,k,kernel", [
    (8, 1024, 2052, "stream"), (32, 1024, 4100, "stream"), (32, 512, 8196, "tiles"),               # (stores of eight channels: not the wave kernel)
    (1, 2048, 2052, "stream"), (16, 2048, 516, "stream"), (16, 1152, 516, "tiles"), (20, 4096, 4100, "tiles"), (32, 8192, 516, "tiles"),
    (16, 2048, 520, "wave"), (32, 8192, 520, "wave"), (20, 4096, 4104, "wave"),
    (20, 1 << 17, 132, "stream"), (20, 1 << 20, 8, "stream"), (20, (1 << 20) - 128, 8, "wave")])   # (its quotients end at 2^20)
def test_matmul_of_few_rows_streams_its_weights_where_the_wave_kernel_cannot_run(rows, c, k, kernel):
    b = undrawn((rows, c, 1, 1))
    g = b.finish(b.matmul(b.matmul(0, k, "m"), 24, "next"))       # (what the second reads is bf16)
    chain = next(ch for ch in plan_json(g, link=3, compute=X.XENOS_BF16)["plan"]["chains"] if ch.get("K") == k)
    assert (chain["loader"], chain["bm"], chain["bn"]) == dict(stream=("stream", 32, 128), tiles=("vector", 64, 64), wave=("vector", 32, 32))[kernel]


@pytest.mark.parametrize("rows,c,k,stream", [
    (20, 8192, 8192, True), (32, 16384, 4096, True), (32, 16256, 4096, True), (24, 8128, 8192, True), (20, 8192, 4096, True),
    (20, 8192, 4880, False), (32, 8320, 8192, False), (32, 24576, 2048, False), (24, 8192, 2048, False), (32, 4096, 16384, False),
    (4, 1024, 1000, True), (1, 832, 1000, True), (6, 1024, 1000, False), (1, 768, 1000, False), (1, 512, 1000, False)])
def test_matmul_of_few_rows_streams_its_weights_where_the_wave_kernel_is_slower(rows, c, k, stream):
    b = undrawn((rows, c, 1, 1))
    g = b.finish(b.matmul(b.matmul(0, k, "m"), 24, "next"))
    chain = next(ch for ch in plan_json(g, link=3, compute=X.XENOS_BF16)["plan"]["chains"] if ch.get("K") == k)
    assert (chain["loader"], chain["bm"], chain["bn"]) == (("stream", 32, 128) if stream else ("vector", 32, 32))


@pytest.mark.parametrize("k,stream", [(516, True), (520, False)])
def test_matmul_with_a_shortcut_streams_its_weights_where_the_wave_kernel_cannot_run(k, stream):
    b = undrawn((16, 2048, 1, 1))
    side = b.matmul(0, k, "side")
    g = b.finish(b.relu(b.add(b.matmul(0, k, "m"), side)))        # fp32 output: stores of four channels, but the shortcut is read in eights
    chains = [c for c in plan_json(g, link=3, compute=X.XENOS_BF16)["plan"]["chains"] if c["kind"] == "conv"]
    assert len(chains) == 2 and all(c["loader"] == ("stream" if stream else "vector") for c in chains), chains


def test_pattern_matmul_to_matmul_layout_link():
    # Table 1, MatmulX -> MatmulY: the first matmul's chain (+ ReLU) writes the row-major [row][column] tensor the
    # second one reads as its operand, with no pass in between; bias, ReLU and the shortcut add are operators of the
    # matmul chains, not passes of their own
    g = wg.matmul_chain(rows=128, widths=(512, 2048, 512), draw=False)
    for compute in (X.XENOS_BF16, X.XENOS_F32):
        q = plan_json(g, link=2, compute=compute)["plan"]
        mm = [c for c in q["chains"] if c["kind"] == "conv"]
        assert len(mm) == 2 and _kinds(g, mm[0]) == ["matmul", "relu"] and _kinds(g, mm[1]) == ["matmul", "add"]
        assert mm[0]["N"] == 128 and mm[0]["K"] == 2048 and mm[1]["C"] == 2048 and mm[1]["K"] == 512
        # (where the first matmul shares its reduction out over workgroups, its summing pass is the launch that finishes the
        # chain and writes the tensor)
        between = [c for c in q["chains"] if mm[0]["i"] < c["i"] < mm[1]["i"]]
        assert [c["kind"] for c in between] in ([], ["splitk_finish"]) and all(c["ops"] == mm[0]["ops"] for c in between)
        o, i = (between[0] if between else mm[0])["out"], mm[1]["in"]
        assert o["mem"] == i["mem"] == "workspace" and o["byte_off"] == i["byte_off"] and (o["sN"], o["sP"], o["sK"]) == (2048, 2048, 1) == (i["sN"], i["sP"], i["sK"])
        u0 = plan_json(g, link=0, compute=compute)["plan"]
        assert u0["n_chains"] > q["n_chains"] and u0["hbm_bytes"] > q["hbm_bytes"]
    # shape errors of the operator
    keep = []
    bad = wg.matmul_chain(rows=4, widths=(8, 8), residual=False, draw=False)
    ops = X.op_descs(bad, keep)
    with pytest.raises(X.XenosError) as e:
        X.xenos_graph_create(X.TensorDesc(4, 2, 2, 2, X.XENOS_F32, X.XENOS_NCHW), ops, 1)     # not a rows x columns tensor
    assert e.value.status == X.XENOS_ESHAPE


def test_fp32_plans_keep_within_the_static_workspace_where_they_can():
    # the poolings and averages that link level 3 takes apart in fp32 need tensors of their own: not where the linked plan alone fits xenos_run_static
    needs = []
    for batch in (1, 6, 16):
        j = plan_json(wg.vgg16(batch=batch, width=0.25, fc_dim=256, draw=False), link=3, split=1, compute=X.XENOS_F32)
        needs.append((j["workspace_bytes"], sum(c["kind"] == "pool" for c in j["plan"]["chains"])))
    (small, apart), (fits, linked), (large, apart_again) = needs
    assert small <= X.XENOS_STATIC_WORKSPACE_BYTES and apart > 0
    assert fits <= X.XENOS_STATIC_WORKSPACE_BYTES and linked < apart
    assert large > X.XENOS_STATIC_WORKSPACE_BYTES and apart_again > 0


@pytest.mark.parametrize("n,c,hw,k,ksz,pool,apart", [
    (31, 64, 184, 64, 3, 2, 0), (31, 64, 183, 64, 3, 2, 1),                                        # 2^20 pixels and more than the wave kernel's indices hold, and fewer
    (32, 64, 224, 64, 3, 2, 0), (16, 16, 300, 32, 1, 3, 0), (8, 64, 56, 64, 3, 2, 1), (2, 128, 55, 64, 1, 3, 1)])
def test_fp32_window_pooling_stays_linked_where_the_wave_kernel_refuses_the_convolution(n, c, hw, k, ksz, pool, apart):
    b = undrawn((n, 8, hw, hw))
    t = b.cbr(b.cbr(0, c, 1, name="a"), k, ksz, 1, ksz // 2, name="b")
    g = b.finish(b.cbr(b.maxpool(t, pool, 2), 8, 1, name="c"))
    chains = plan_json(g, link=3, compute=X.XENOS_F32)["plan"]["chains"]
    conv, = [ch for ch in chains if ch["kind"] == "conv" and (ch["C"], ch["K"]) == (c, k)]
    assert (conv["pool"] == 0) == bool(apart) and sum(ch["kind"] == "pool" for ch in chains) == apart, chains
    assert conv["wave"] or not apart


@pytest.mark.parametrize("n,hw,c,apart", [
    (32, 200, 256, 0), (31, 184, 256, 0), (31, 100, 256, 0), (20, 100, 256, 1), (32, 13, 256, 1),
    # steps of 32 channels: six on a map of 144 and of 169 pixels, seven; two and three
    (32, 12, 192, 0), (32, 13, 192, 1), (32, 12, 224, 1), (32, 20, 64, 0), (32, 20, 96, 1), (1, 13, 64, 1)])
def test_fp32_global_average_stays_linked_where_that_is_faster(n, hw, c, apart):
    # 2^20 pixels or 2^15 tiles and more, which the wave kernel refuses (31x100x100: 4844 times 8 of 64 x 64): no sums of every pixel for a pass to read.
    # Short reductions of many images neither
    b = undrawn((n, 8, hw, hw))
    t = b.cbr(b.cbr(0, c, 1, name="a"), 512, 1, name="b")
    chains = plan_json(b.finish(b.gap(t)), link=3, compute=X.XENOS_F32)["plan"]["chains"]
    conv, = [ch for ch in chains if ch["kind"] == "conv" and (ch["C"], ch["K"]) == (c, 512)]
    assert (conv["mode"] != "gap") == bool(apart) and bool(conv["wave"]) == bool(apart) and sum(ch["kind"] == "splitk_finish" for ch in chains) == apart


@pytest.mark.parametrize("batch", [5, 6, 8])
def test_fp32_plans_within_the_static_workspace_link_only_the_poolings_of_large_maps(batch):
    # VGG at a quarter of its width: the maps in front of the first two poolings are 16 to 26 MB and half of that; the other three are passes of their own
    # and every layer without one on the wave kernel, as for any other number of images
    j = plan_json(wg.vgg16(batch=batch, width=0.25, fc_dim=256, draw=False), link=3, compute=X.XENOS_F32)
    conv = [c for c in j["plan"]["chains"] if c["kind"] == "conv"]
    linked = [c["OH"] for c in conv if c["pool"]]
    assert j["workspace_bytes"] <= X.XENOS_STATIC_WORKSPACE_BYTES
    assert linked in ([224], [224, 112]) and all(c["wave"] for c in conv if not c["pool"])
    assert sum(c["kind"] == "pool" for c in j["plan"]["chains"]) == 5 - len(linked)


@pytest.mark.parametrize("n,c,hw,k,ksz,pool,last,nhwc,apart", [
    # disjoint windows: four steps of 32 channels and taps, five to nine by the number of 32 x 32 tiles, ten
    (2, 128, 32, 64, 1, 2, 0, 1, 0), (2, 160, 32, 64, 1, 2, 0, 1, 1), (2, 288, 80, 64, 1, 2, 0, 1, 0), (2, 288, 80, 48, 1, 2, 0, 1, 0), (2, 288, 80, 40, 1, 2, 0, 1, 1), (2, 320, 80, 64, 1, 2, 0, 1, 1), (2, 160, 160, 64, 1, 2, 0, 1, 1),
    # overlapping ones
    (2, 64, 33, 64, 1, 3, 0, 1, 0), (2, 96, 33, 64, 1, 3, 0, 1, 1), (8, 64, 80, 64, 1, 3, 0, 1, 1),
    # the graph's output, in the caller's order and in the pooling pass's
    (2, 288, 32, 64, 1, 2, 1, 0, 0), (2, 288, 32, 40, 1, 2, 1, 0, 1), (2, 320, 32, 64, 1, 2, 1, 0, 1), (2, 288, 32, 64, 1, 2, 1, 1, 1),
    (3, 576, 64, 64, 1, 2, 1, 0, 0), (3, 608, 64, 64, 1, 2, 1, 0, 1), (3, 576, 60, 64, 1, 2, 1, 0, 1), (8, 64, 56, 64, 3, 2, 1, 0, 0),
    (2, 192, 33, 64, 1, 3, 1, 0, 0), (2, 224, 33, 64, 1, 3, 1, 0, 1), (4, 288, 64, 64, 1, 3, 1, 0, 0), (4, 320, 64, 64, 1, 3, 1, 0, 1)])
def test_fp32_window_pooling_behind_a_short_reduction_stays_linked(n, c, hw, k, ksz, pool, last, nhwc, apart):
    b = undrawn((n, 8, hw, hw))
    t = b.maxpool(b.cbr(b.cbr(0, c, 1, name="a"), k, ksz, 1, ksz // 2, name="b"), pool, 2)
    G = X.graph_from_workload(b.finish(t if last else b.cbr(t, 8, 1, name="c")), out_layout=X.XENOS_NHWC if nhwc else X.XENOS_NCHW)
    P = X.xenos_plan_link_split(G, link=3, compute=X.XENOS_F32)
    chains = X.xenos_plan_query(P)["plan"]["chains"]
    X.xenos_destroy(P)
    X.xenos_destroy(G)
    assert sum(ch["kind"] == "pool" for ch in chains) == apart, chains
