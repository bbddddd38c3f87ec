"""Resources the compiler gave the kernels of the built library (the metadata of its gfx950 code objects): the kernels named here keep
everything in registers.  A spilled register costs them 10 to 50 % (measured on conv_kernel behind a linked depthwise producer with a
global average, and on fire_kernel), and nothing else shows it: results are the same.  Also what the planner assumes of static LDS."""
import os
import re
import shutil
import struct
import subprocess

import pytest

from paper_2302_00282_amd import xenos as X
from workloads import cnn_graphs as wg

READELF = next((p for p in (shutil.which("llvm-readelf"), "/opt/rocm/llvm/bin/llvm-readelf") if p and os.path.exists(p)), None)
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(data):
    """The gfx950 ELF images of the offload bundles in a shared library."""
    at = data.find(MAGIC)
    while at >= 0:
        n, = struct.unpack_from("<Q", data, at + len(MAGIC))
        pos = at + len(MAGIC) + 8
        for _ in range(n):
            off, size, tlen = struct.unpack_from("<QQQ", data, pos)
            triple = data[pos + 24:pos + 24 + tlen].decode()
            pos += 24 + tlen
            if "gfx950" in triple and size:
                yield data[at + off:at + off + size]
        at = data.find(MAGIC, pos)


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    if READELF is None:
        pytest.skip("no llvm-readelf")
    out = {}
    with open(X.LIB_PATH, "rb") as f:
        images = list(_code_objects(f.read()))
    for i, image in enumerate(images):
        path = tmp_path_factory.mktemp("co") / f"{i}.co"
        path.write_bytes(image)
        notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True, check=True).stdout
        for block in re.split(r"\n\s+- \.agpr_count", notes)[1:]:
            field = lambda k: re.search(r"\." + k + r":\s+(\S+)", block).group(1)
            out[field("name")] = {k: int(field(k)) for k in ("vgpr_spill_count", "private_segment_fixed_size", "group_segment_fixed_size", "vgpr_count")}
    assert out
    return out


@pytest.mark.parametrize("kernel", ["conv_kernel", "fire_kernel", "dwpw_kernel", "pwdw_kernel", "unit_kernel", "dw_kernel", "splitk_finish_kernel", "fc_stream_kernel",
                                    "stem_lds_kernel", "conv3x3_frag_kernel", "conv3x3_first_kernel"])
def test_no_vector_register_is_spilled(kernels, kernel):
    found = {k: v for k, v in kernels.items() if re.search(r"\d" + kernel + r"I|\d" + kernel + r"E", k)}
    assert found, kernel
    assert not {k: v for k, v in found.items() if v["vgpr_spill_count"] or v["private_segment_fixed_size"]}


@pytest.mark.parametrize("kernel,most", [("conv_wave_kernelI\\w+Li1E", 128), ("conv_wave_kernelI\\w+Li2E", 256), ("pwdw_wave_kernelI", 256)])
def test_wave_kernels_keep_everything_in_registers(kernels, kernel, most):
    # (and leave room for four workgroups per unit, or two)
    found = {k: v for k, v in kernels.items() if re.search(r"\d" + kernel, k)}
    assert found and not {k: v for k, v in found.items() if v["vgpr_spill_count"] or v["private_segment_fixed_size"] or v["vgpr_count"] > most}


# first layers that take stem_lds_kernel: (compute type, output channels, kernel size, behind it a pooling)
FIRST_LAYERS = [(1, 32, 3, 1), (1, 64, 3, 1), (1, 24, 3, 0), (1, 32, 3, 0), (1, 48, 3, 0), (1, 64, 3, 0), (1, 24, 5, 1), (1, 32, 5, 0), (1, 64, 4, 0), (1, 64, 5, 1), (1, 32, 7, 1), (1, 32, 7, 0), (1, 48, 7, 1), (1, 64, 7, 0),
                (0, 32, 3, 1), (0, 64, 3, 1), (0, 24, 5, 1), (0, 64, 5, 1)]


def first_layer(kernels, compute, k, ksz, pool, **hw):
    """The first chain of a 32 x 3 x 224 x 224 graph and the metadata of the stem_lds_kernel it would run."""
    b = wg._Builder("first", (1, 1, 1, 1), 1, False, False)
    b.g.input_shape, b.g.x, b._shapes = (32, 3, 224, 224), None, [(32, 3, 224, 224)]
    t = b.cbr(0, k, ksz, 2, ksz // 2, name="a")
    g = b.finish(b.cbr(b.maxpool(t, 3, 2, 1) if pool else t, k, 3, 1, 1, groups=k, name="b"))   # (a depthwise consumer takes no LDS)
    G = X.graph_from_workload(g)
    try:
        P = X.xenos_plan_link_split(G, link=3, compute=compute, hw=dict(X.MI355X, **hw))
    finally:
        X.xenos_destroy(G)
    chain = X.xenos_plan_query(P)["plan"]["chains"][0]
    X.xenos_destroy(P)
    steps = 3 if ksz < 4 else 7 if ksz < 6 else 13
    name = "stem_lds_kernelI%sLi%dELi%dELb%dELi%dE" % ("NS_6bf16_tE" if compute else "f", 1 if k <= 32 else 2, steps, pool, 4 if compute else 3)
    meta, = [v for n, v in kernels.items() if name in n]
    return chain, meta


@pytest.mark.parametrize("compute,k,ksz,pool", FIRST_LAYERS)
def test_first_layer_plans_count_the_lds_they_take(kernels, compute, k, ksz, pool):
    chain, meta = first_layer(kernels, compute, k, ksz, pool)
    lds = meta["group_segment_fixed_size"]
    assert chain["bm"] == 128 and chain["lds"] == lds
    assert first_layer(kernels, compute, k, ksz, pool, lds_bytes_per_cu=lds)[0]["bm"] == 128
    try:
        small = first_layer(kernels, compute, k, ksz, pool, lds_bytes_per_cu=lds - 1)[0]
        assert small.get("lds", 0) < lds and (small.get("loader") != "stem" or small["bm"] != 128)
    except X.XenosError as e:                                      # (nor does any other kernel fit that)
        assert e.status == X.XENOS_EUNSUPPORTED and compute == 1


@pytest.mark.parametrize("compute,k,ksz,pool", FIRST_LAYERS)
def test_first_layer_plans_launch_what_a_unit_holds(kernels, compute, k, ksz, pool):
    # 512 registers per lane and SIMD in granules of 8 (a workgroup has one wavefront on each of the four), 160 KB of LDS in granules of 1280
    chain, meta = first_layer(kernels, compute, k, ksz, pool)
    fit = min(512 // (-(-meta["vgpr_count"] // 8) * 8), 160 * 1024 // (-(-meta["group_segment_fixed_size"] // 1280) * 1280))
    assert chain["grid"] == min(chain["tiles_m"], fit * X.MI355X["num_cu"]) and chain["tiles_m"] > chain["grid"]
