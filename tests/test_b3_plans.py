"""Host checks of the kernels of bf16 part products: their rows of the tile
table against the build, and which shapes the persistent 1x1 kernel takes."""
import json
import os
import random
import re

import pytest

import bench
import workloads
from paper_2307_04941_amd import build, mg3m

RES = "tile=64x64,waves=1x2,kt=32"


def test_b3_table_matches_build():
    """regs and LDS of every tile as compiled, in the form that the table names."""
    with open(os.path.join(build.CSRC, "mg3m_internal.h")) as f:
        body = re.search(r"kTilesB3\[kNumTilesB3\] = \{(.*?)\};", f.read(), re.S).group(1)
    rows = [[int(v) for v in re.findall(r"\d+", r)[:6]] for r in re.findall(r"\{(\d+, \d+, \d+, \d+, \d+, \d+),", body)]
    assert len(rows) == 14
    with open(build.RESOURCES) as f:
        res = json.load(f)
    for i, (mt, nt, kt, wm, wn, regs) in enumerate(rows):
        name = (f"void mg3m::conv_igemm_b3<{2 if i == 8 else 0}, {mt}, {nt}, {kt}, {wn}, {wm}, false>(mg3m::KArgs)"
                if i != 9 else "void mg3m::conv_igemm_b3_res<false>(mg3m::KArgs)")
        got = res[name]
        lds = 12 * kt * mt * wm if i != 9 else 6 * 64 * 384
        assert (got["vgpr_count"], got["lds_bytes"]) == (regs, lds), (i, name, got, regs, lds)
    for name, got in res.items():
        if "conv_igemm_b3" in name:
            assert got["scratch_bytes"] == 0, name


def test_b3_resident_plan():
    """1x1 layers of 64 to 384 channels with work for every CU run on it, and its
    tile, waves and kt read back as an override; the plan needs no workspace."""
    for shape in [(64, 64, 56, 56, 256, 1, 1, 1, 0), (32, 128, 28, 28, 512, 1, 1, 1, 0),
                  (32, 256, 56, 56, 128, 1, 1, 1, 0), (16, 256, 14, 14, 1024, 1, 1, 1, 0)]:
        p = mg3m.conv2d_fwd_f32_plan_info(*shape, "HWCN")
        assert (p["persistent"], p["a_mode"], p["waves_n"], p["grid"], p["workspace_bytes"]) == (1, 3, 2, 256, 0), p
        assert mg3m.conv2d_fwd_f32_plan_info(*shape, "HWCN", RES) == p
        assert mg3m.conv2d_fwd_f32_plan_info(*shape, "HWCN", RES + ",persist=1") == p


@pytest.mark.parametrize("shape", [(4, 32, 65, 65, 64, 1, 1, 1, 0), (4, 448, 65, 65, 64, 1, 1, 1, 0),
                                   (4, 64, 65, 65, 64, 3, 3, 1, 1), (3, 64, 75, 75, 64, 1, 1, 1, 0),
                                   (4, 64, 64, 64, 64, 1, 1, 1, 0)])
def test_b3_resident_refuses(shape):
    """Half a pair of steps, more channels than LDS holds, several taps, an odd
    batch, and 256 tiles (a work-group on every CU is assumed)."""
    with pytest.raises(mg3m.Mg3mError) as e:
        mg3m.conv2d_fwd_f32_plan_info(*shape, "HWCN", RES)
    assert e.value.status == 7


@pytest.mark.parametrize("plan", [RES + ",persist=2", RES + ",split=2", RES + ",sk=300", RES + ",dma=1"])
def test_b3_resident_refuses_other_schedules(plan):
    with pytest.raises(mg3m.Mg3mError) as e:
        mg3m.conv2d_fwd_f32_plan_info(64, 64, 56, 56, 256, 1, 1, 1, 0, "HWCN", plan)
    assert e.value.status == 7


def test_queried_workspace_serves_any_alignment(monkeypatch):
    """A workspace of the queried size (none, where that is 0) is enough whatever
    the alignment of x, w and y.  The calls end at a launch that is made to fail (status 8): status 6 would be
    the refused workspace."""
    monkeypatch.setenv("MG3M_TEST_FAIL_LAUNCH", "1")
    lib = mg3m.load_library()
    x, w, y, ws = 0x7f0000000000, 0x7f2000000000, 0x7f4000000000, 0x7f6000000000
    rng = random.Random(41)
    shapes = [(64, 176, 28, 28, 96, 3, 3, 1, 1), (24, 169, 60, 60, 6, 3, 3, 1, 1), (4, 32, 78, 78, 208, 3, 3, 2, 1),
              (1, 208, 10, 12, 48, 3, 3, 2, 1)]
    while len(shapes) < 250:
        R = rng.choice([1, 1, 3, 3, 5])
        shapes.append((rng.choice([1, 3, 4, 8, 16, 28, 64]), rng.choice([3, 8, 20, 32, 64, 75, 96, 169, 256, 512]),
                       rng.randint(7, 60), rng.randint(7, 60), rng.choice([6, 16, 48, 64, 96, 128, 208, 512]), R, R,
                       rng.choice([1, 1, 2]), R // 2))
    for shape in shapes:
        for layout in (0, 1):
            need = mg3m.conv2d_fwd_f32_workspace_bytes(*shape, layout)
            for off in range(8):
                rc = lib.conv2d_fwd_f32_ex(x + 4 * (off & 1), w + 4 * (off >> 1 & 1), y + 4 * (off >> 2), *shape,
                                           layout, ws if need else None, need, None, None)
                assert rc == 8, (shape, layout, off, need, rc, mg3m.mg3m_last_error())


@pytest.mark.parametrize("shape,layout", [((16, 64, 28, 28, 128, 3, 3, 1, 1), "HWCN"), ((7, 75, 29, 31, 117, 3, 3, 1, 1), "HWCN"),
                                          ((1, 64, 14, 14, 64, 1, 1, 1, 0), "HWCN"), ((8, 64, 28, 28, 96, 3, 3, 1, 1), "NCHW")])
def test_overrides_that_name_fp32_tiles_keep_them(shape, layout):
    """A tile, a depth or dma= without waves means the fp32-MFMA kernel that it meant
    before these kernels came; tile and waves together name one of these."""
    fp32 = ["tile=64x64,kt=32", "tile=64x64,kt=32,split=3", "tile=128x128,kt=32", "tile=128x128,kt=32,tail=2", "kt=32",
            "kt=16", "kt=32,split=2", "waves=2x2", "waves=1x4", "tile=128x128", "tile=64x64,waves=2x2,kt=32"]
    if shape[0] % 4 == 0 and layout == "HWCN":
        fp32 += ["dma=0", "dma=1", "tile=64x64,kt=32,dma=0"]
    for plan in fp32:
        p = mg3m.conv2d_fwd_f32_plan_info(*shape, layout, plan)
        assert p["a_mode"] != 3, (plan, p)
    for plan in ("tile=64x64,waves=1x4,kt=32", "tile=64x64,waves=1x4,kt=32,split=2"):
        assert mg3m.conv2d_fwd_f32_plan_info(*shape, layout, plan)["a_mode"] == 3, plan


@pytest.mark.parametrize("layout", ["HWCN", "NCHW"])
@pytest.mark.parametrize("shape,plan", [((60, 128, 27, 8, 32, 1, 1, 1, 0), "tile=64x64,kt=64"),
                                        ((24, 64, 22, 15, 208, 1, 1, 1, 0), "tile=64x64,kt=64"),
                                        ((60, 64, 25, 30, 64, 1, 1, 1, 0), "tile=64x256,kt=64")])
def test_overrides_that_only_part_products_fit_run_where_they_are_slower(shape, plan, layout):
    """No fp32 tile has this depth: the rules that prefer the fp32-MFMA kernels on
    short reductions choose between kernels and do not refuse a named one."""
    assert mg3m.conv2d_fwd_f32_plan_info(*shape, layout, plan)["a_mode"] == 3


@pytest.mark.parametrize("shape,layout,b3", [
    ((16, 1, 56, 56, 64, 1, 1, 1, 0), "HWCN", 0), ((7, 7, 30, 30, 40, 1, 1, 1, 0), "HWCN", 0),      # under 8 rows
    ((7, 8, 30, 30, 40, 1, 1, 1, 0), "HWCN", 1),
    ((8, 16, 14, 14, 96, 1, 1, 1, 0), "HWCN", 0), ((8, 3, 112, 112, 64, 3, 3, 1, 1), "HWCN", 0),    # a stage, vector loads
    ((8, 24, 14, 14, 96, 1, 1, 1, 0), "HWCN", 1), ((1, 24, 14, 14, 96, 1, 1, 1, 0), "HWCN", 0), ((7, 16, 14, 14, 96, 1, 1, 1, 0), "HWCN", 1),
    ((8, 3, 40, 40, 64, 5, 5, 2, 2), "HWCN", 0),                                                      # rows, under three stages
    ((28, 64, 14, 15, 160, 1, 1, 1, 0), "HWCN", 0), ((64, 64, 56, 56, 256, 1, 1, 1, 0), "HWCN", 1),  # little work, much work
    ((8, 192, 13, 13, 48, 3, 3, 2, 1), "HWCN", 0), ((3, 512, 7, 7, 48, 3, 3, 1, 1), "HWCN", 1),      # many short pieces
    ((16, 128, 64, 64, 16, 3, 3, 1, 1), "HWCN", 0), ((32, 128, 64, 64, 16, 3, 3, 1, 1), "HWCN", 1),   # 16 rows
    ((1, 384, 112, 113, 128, 3, 3, 2, 1), "NCHW", 0), ((32, 128, 57, 57, 128, 3, 3, 2, 1), "NCHW", 1)])   # copies of small batches
def test_selector_keeps_fp32_mfma_where_it_is_faster(shape, layout, b3):
    """Both sides of each line that the selector draws between the two kernel families
    (timed on MI355X), for the caller's call and not for overrides."""
    assert (mg3m.conv2d_fwd_f32_plan_info(*shape, layout)["a_mode"] == 3) == bool(b3)
    assert mg3m.conv2d_fwd_f32_plan_info(*shape, "HWCN", "tile=64x64,waves=1x4,kt=32")["a_mode"] == 3


def test_resident_filter_not_for_an_x_over_the_last_level_cache():
    """It walks x once per filter tile, from memory each time there."""
    big = (120, 384, 82, 82, 176, 1, 1, 1, 0)
    assert mg3m.conv2d_fwd_f32_plan_info(*big, "HWCN")["persistent"] == 0
    assert mg3m.conv2d_fwd_f32_plan_info(24, *big[1:], "HWCN")["persistent"] == 1


def test_benchmark_names_built_kernels():
    """The kernel that the benchmark says a layer runs is one of the build's, by its
    operand form (b= of the plan's string)."""
    with open(build.RESOURCES) as f:
        built = set(json.load(f))
    for name in ("vgg16_n64", "resnet50_n32"):
        for L in workloads.workload(name):
            args = (L.N, L.C, L.H, L.W, L.K, L.R, L.S, L.stride, L.pad, "HWCN")
            kernel = bench.kernel_name(mg3m.conv2d_fwd_f32_plan_info(*args), mg3m.conv2d_fwd_f32_plan_string(*args))
            assert kernel in built, (L.name, kernel)
    for shape, form in [((8, 72, 9, 9, 64, 3, 3, 1, 1), "group"), ((7, 72, 9, 9, 64, 3, 3, 1, 1), "group_n"),
                        ((1, 72, 9, 9, 64, 3, 3, 1, 1), "group_c"), ((8, 75, 9, 9, 64, 3, 3, 1, 1), "row"),
                        ((7, 75, 9, 9, 64, 3, 3, 1, 1), "row_n"), ((8, 64, 9, 9, 64, 3, 3, 1, 1), "slab")]:
        text = mg3m.conv2d_fwd_f32_plan_string(*shape, "HWCN", "tile=64x64,waves=1x4,kt=32")
        assert f",b={form}," in text, (shape, text)
