"""Pieces of the library's code that can run on the host, compiled for the host and run there (no GPU)."""
import json
import os
import re
import subprocess
import sys

import pytest
import test_gpu_parity as gpu

HERE = os.path.join(os.path.dirname(os.path.abspath(__file__)), "host")


@pytest.fixture
def run_host(tmp_path):
    def run(name, language=("-x", "hip", "--offload-host-only")):
        exe = str(tmp_path / name)
        subprocess.run(["hipcc", *language, "-O1", "-std=c++17", os.path.join(HERE, name + ".cpp"), "-o", exe], check=True, timeout=300)
        r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
        return r.returncode, r.stdout.strip()
    return run


def test_raw_weight_loads_stay_inside_the_tensor(run_host):
    """1 to 70 channels against weights that end at a page without access: a load past them ends the program."""
    assert run_host("raw_weights") == (0, "ok")


def test_raw_1x1_weight_loads_stay_inside_the_tensor(run_host):
    """1 to 130 channels, the same way; every 16-byte piece a tile asks for is compared with the bytes, zeros past the row."""
    assert run_host("raw_rows") == (0, "ok")


def test_plan_table_keeps_as_many_problems_as_it_holds(run_host):
    """Plans are made once per problem while no more problems take turns than the table has places."""
    assert run_host("plan_table") == (0, "ok")


def test_window_fills_stay_inside_tensor_and_window(run_host):
    """6000 random layers' input ranges, from NCHW and NHWC tensors that touch a page without access on either side."""
    assert run_host("window_fill", ("-x", "c++", "-D__HIP_PLATFORM_AMD__=1", "-I/opt/rocm/include")) == (0, "ok")


def test_blocked_window_fills_stay_inside_image_and_window(run_host):
    """6000 random layers on blocked images of 16, 32 and 64 channels a block, the same way."""
    assert run_host("block_fill", ("-x", "c++", "-D__HIP_PLATFORM_AMD__=1", "-I/opt/rocm/include")) == (0, "ok")


def test_window_walk_against_its_definition(run_host):
    """The estimates' window sizes: 20000 random problems, up to images of 2^28 pixels, against integer divisions."""
    assert run_host("window_walk", ("-x", "c++")) == (0, "ok")


def test_panel_windows_stay_inside_tensor_and_window(run_host):
    """The panel kernel's windows over random problems: guard pages around the tensor, and every tap's input at its distance."""
    assert run_host("panel_fill", ("-x", "c++", "-D__HIP_PLATFORM_AMD__=1", "-I/opt/rocm/include")) == (0, "ok")


def test_panel_windows_at_the_tensor_s_end(run_host):
    """Small planes without a border, where the last eight slots of a window reach the tensor's last image."""
    assert run_host("panel_fill_end", ("-x", "c++", "-D__HIP_PLATFORM_AMD__=1", "-I/opt/rocm/include")) == (0, "ok")


def test_panel_stage_validation(lib):
    """What the stage refuses, before any device call; no tile asks for more LDS than lets two workgroups share a compute unit."""
    import ctypes
    raw, d, p = lib.load(), lib.ConvDesc(2, 64, 14, 14, 64, 3, 3, 1, 1), 256
    call = lambda x=p, w=p, o=p, cb=64, tile=0, px=64, ws=p, n=1 << 30, dil=1, desc=d: raw.conv2d_int8_panel(ctypes.byref(desc), dil, 0, x, w, cb, o, tile, px, ws, n, None)
    tiles = lib.panel_tiles()
    for bad in (dict(tile=-1), dict(tile=len(tiles)), dict(px=0), dict(px=tiles[0][1] + 1), dict(cb=-1), dict(x=0), dict(w=0), dict(o=0), dict(ws=0), dict(w=264), dict(ws=264), dict(dil=0)):
        assert call(**bad) == lib.ERR_INVALID_ARG, bad
    assert call(n=lib.panel_workspace_bytes((2, 64, 14, 14, 64, 3, 3, 1, 1), 64, 0, 64) - 1) == lib.ERR_WORKSPACE
    assert call(cb=24) == lib.ERR_UNSUPPORTED
    # a border wider than the kernel, rows of fewer than eight slots, a window that fits no compute unit
    for dims in ((2, 64, 14, 14, 64, 3, 3, 1, 3), (2, 64, 14, 5, 64, 3, 3, 1, 1), (1, 64, 700, 700, 64, 3, 3, 1, 1)):
        assert call(desc=lib.ConvDesc(*dims)) == lib.ERR_UNSUPPORTED and lib.panel_workspace_bytes(dims, 64, 0, 64) == 0, dims


# (dims, layout, block): layers whose one-shot and kept-weights calls both take the resident kernel, with different tiles or pixels
SHARED_LAYERS = [((266, 64, 56, 56, 64, 5, 5, 1, 2), 3, 0), ((233, 32, 9, 9, 275, 5, 5, 1, 2), 3, 0), ((161, 64, 32, 32, 59, 5, 5, 1, 2), 3, 0),
                 ((87, 32, 15, 15, 172, 5, 5, 1, 2), 3, 0), ((2, 70, 37, 37, 163, 5, 5, 1, 2), 3, 0), ((215, 64, 7, 7, 432, 5, 5, 1, 2), 3, 0)]


@pytest.fixture
def launches(tmp_path):
    """What calls of conv2d_int8_ex would launch, made one after the other in a process of their own."""
    from paper_2104_04731_amd import build
    recorder = str(tmp_path / "launch_recorder.so")
    subprocess.run(["g++", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__=1", "-I/opt/rocm/include", os.path.join(HERE, "launch_recorder.cpp"), "-o", recorder],
                   check=True, timeout=120)

    def run(calls):
        r = subprocess.run([sys.executable, os.path.join(HERE, "launches.py"), recorder, build.LIB, json.dumps(calls)], capture_output=True, text=True, check=True, timeout=120)
        return json.loads(r.stdout)
    return run


@pytest.mark.parametrize("dims,layout,cb", SHARED_LAYERS)
def test_a_layer_called_both_ways_keeps_a_plan_for_each(lib, launches, dims, layout, cb):
    """Raw and kept weights of one layer, in both orders: each call launches what the query says of it, whichever came first."""
    kept, raw = (dims, layout, cb, 1), (dims, layout, cb, 0)
    first, second = launches([kept, raw]), launches([raw, kept])[::-1]
    assert first == second
    (N, C, H, W, K, R, S, stride, pad), tiles = dims, lib.resident_tiles()
    M = N * ((H + 2 * pad - R) // stride + 1) * ((W + 2 * pad - S) // stride + 1)
    for call in first:
        stage, tile, pixels = call["stage"]
        assert call["rc"] == 0 and stage in (lib.STAGE_RESIDENT, lib.STAGE_RESIDENT_RAW, lib.STAGE_RESIDENT_REWRITE)
        rows, _, threads = tiles[tile]
        assert (call["workgroups"], call["threads"]) == (-(-K // rows) * -(-M // pixels), threads)


@pytest.mark.parametrize("dims", [(144, 128, 28, 28, 128, 3, 3, 2, 1), (451, 450, 7, 8, 64, 3, 3, 1, 1), (100, 300, 14, 14, 20, 5, 5, 1, 2)])
def test_query_names_the_streaming_tile(lib, launches, dims):
    """Kept weights and raw ones: the tile and pixels that the query reports are launched, and the forced call takes them."""
    (N, C, H, W, K, R, S, stride, pad), tiles = dims, lib.stream_tiles()
    M = N * ((H + 2 * pad - R) // stride + 1) * ((W + 2 * pad - S) // stride + 1)
    for call, stage in zip(launches([(dims, 1, 64, 1), (dims, 1, 64, 0)]), (lib.STAGE_STREAM, lib.STAGE_STREAM_REWRITE)):
        got, tile, pixels = call["stage"]
        assert call["rc"] == 0 and got == stage
        rows, most, threads = tiles[tile]
        assert pixels <= most and (call["workgroups"], call["threads"]) == (-(-K // rows) * -(-M // pixels), threads)
        assert lib.resident_applies(dims, 64, tile, pixels)


@pytest.mark.parametrize("dims", [(200, 128, 28, 28, 100, 3, 3, 2, 1), (400, 256, 14, 14, 512, 3, 3, 1, 1), (64, 256, 14, 14, 512, 3, 3, 1, 1)])
def test_query_tells_panels_from_stored_rewrites(lib, launches, dims):
    """Kept weights and raw ones: of the calls that store operands, the tile tells those that read the input as it is from those of the GEMM stage."""
    (N, C, H, W, K, R, S, stride, pad), tiles = dims, lib.panel_tiles()
    M, seen = N * ((H + 2 * pad - R) // stride + 1) * ((W + 2 * pad - S) // stride + 1), set()
    for call in launches([(dims, 1, 64, 1), (dims, 1, 64, 0)]):
        stage, tile, pixels = call["stage"]
        panels = stage == lib.STAGE_STORED and tile >= lib.TILE_PANEL
        assert call["rc"] == 0 and panels == ("conv_panel_kernel" in call["kernel"]) == (lib.stage_name(stage, tile, pixels) == "weights in panels"), call
        if panels:
            rows, most = tiles[tile - lib.TILE_PANEL]
            assert pixels <= most and call["launches"] == 2 and call["workgroups"] == -(-K // rows) * -(-M // pixels)
        elif stage == lib.STAGE_STORED:
            assert (tile, pixels) == (-1, 0) and ("igemm" in call["kernel"] or "conv_band" in call["kernel"])
        seen.add((stage, panels))
    assert (lib.STAGE_STORED, N > 64) in seen


# 1x1 layers that the estimates would send to the resident kernel, but for a stride or for more than 64 output channels.
NOT_BLOCKED_1X1 = [(877, 32, 56, 56, 46, 1, 1, 2, 0), (322, 16, 28, 28, 159, 1, 1, 1, 0)]


def test_fused_activations_that_take_the_resident_kernel(launches):
    """The layers whose results are compared on the GPU do take it, one launch, or two where a border is cleared; deep and small layers, 1x1
    layers with a stride or of many channels, blocks of no power of two and unrolled operands keep the GEMM stages."""
    def kernels(cases):
        got = launches([[dims, layout, cb, "requant", 64 if dims[4] > 32 else 32, pad] for dims, layout, cb in cases for pad in (0, 1)])
        assert [c["rc"] for c in got] == [0] * len(got) and [c["launches"] for c in got] == [1, 2] * len(cases)
        return [c["kernel"] for c in got]

    assert all("conv_resident_kernel" in k and "ResidentBlockedArgs" in k for k in kernels([(dims, 1, 64 if dims[1] > 32 else 32) for dims in gpu.BLOCKED_RESIDENT]))
    first = gpu.BLOCKED_RESIDENT[0]
    others = [(dims, 1, 32) for dims in NOT_BLOCKED_1X1] + [((32, 256, 14, 14, 256, 3, 3, 1, 1), 1, 64), ((1, 64, 14, 14, 64, 3, 3, 1, 1), 1, 64), (first, 1, 48), (first, 2, 0)]
    assert all("igemm" in k or "conv_band" in k for k in kernels(others))


@pytest.mark.parametrize("dims", [(72, 500, 55, 55, 64, 3, 3, 2, 1), (575, 256, 7, 7, 357, 3, 3, 2, 1), (22, 512, 28, 28, 420, 3, 3, 1, 1)])
def test_streaming_tiles_begin_on_whole_sectors(lib, dims):
    """Planes of whole 64-byte sectors: the library's own pixel counts cut none."""
    stage, tile, pixels = lib.query_stage(dims, lib.ENTRY_EX, lib.LAYOUT_PACKED, 64, True)
    assert stage == lib.STAGE_STREAM and pixels % 16 == 0


@pytest.mark.parametrize("dims", [(66, 64, 19, 19, 34, 1, 1, 2, 0), (14, 192, 23, 23, 182, 1, 1, 2, 0), (1, 256, 31, 31, 424, 1, 1, 1, 0), (66, 64, 17, 17, 328, 1, 1, 1, 0),
                                  (197, 384, 9, 9, 56, 1, 1, 1, 0), (109, 448, 17, 17, 47, 1, 1, 1, 0)])
def test_given_and_kept_1x1_weights_take_the_same_launch(lib, dims):
    """A 1x1 layer of whole 64 channels: its raw weights are in depth order as they are, so the two calls read the same bytes."""
    raw = lib.query_stage(dims, lib.ENTRY_ONE_SHOT)
    assert raw[0] == lib.STAGE_RESIDENT and lib.query_stage(dims, lib.ENTRY_EX, lib.LAYOUT_PACKED, 64, True) == raw


@pytest.mark.parametrize("dims,layout,cb", [((8, 256, 14, 14, 512, 3, 3, 1, 1), 1, 64), ((9, 256, 13, 13, 512, 3, 3, 1, 1), 1, 64), ((60, 96, 28, 28, 520, 3, 3, 1, 1), 1, 32),
                                            ((300, 64, 28, 28, 512, 3, 3, 1, 1), 1, 64), ((16, 64, 14, 14, 512, 3, 3, 1, 1), 2, 0)], ids=str)
def test_tile_lds_is_what_the_launch_asks_for(lib, launches, dims, layout, cb):
    """Every tile, the depth whole and split: the ring with its offsets, or the rows of a result that leaves through LDS."""
    pairs = [(t, split) for t in range(lib.num_tiles()) for split in (1, 2, 3) if lib.tile_applies(dims, layout, cb, t, split)]
    calls = launches([(dims, layout, cb, 1, t, split) for t, split in pairs])
    assert pairs and all(c["rc"] == 0 for c in calls)
    assert [c["lds"] for c in calls] == [lib.tile_lds_bytes(dims, layout, cb, t, split) for t, split in pairs]


# (dims, pixels of a tile, three workgroups per compute unit at most), or window: large results of stencil-unrolling layers
STENCIL_RULE = [
    ((15352, 3, 62, 62, 2, 3, 3, 1, 1), 1024, False), ((1198, 1, 89, 109, 6, 3, 3, 1, 0), 1024, False), ((690, 4, 81, 84, 12, 3, 3, 1, 0), 512, False),
    ((678, 1, 76, 79, 32, 3, 3, 1, 1), 512, True), ((92118, 3, 13, 14, 24, 3, 3, 2, 0), 512, False), ((1440, 3, 37, 37, 64, 3, 3, 1, 0), 256, True),
    ((11381, 3, 13, 14, 64, 3, 3, 1, 0), 256, False), ((512, 3, 224, 224, 64, 7, 7, 2, 3), 512, False), ((4340, 3, 48, 48, 8, 3, 3, 1, 1), 1024, False),
    ((495, 2, 40, 41, 64, 3, 3, 1, 1), 256, True), ((73, 3, 86, 87, 96, 3, 3, 1, 1), 256, True), ((60, 4, 95, 115, 128, 3, 3, 1, 1), 0, False),
    # from 190 MB on up to 64 channels whatever the rows, above on rows that leave the window kernel's tiles a fifth empty
    ((185, 1, 151, 268, 64, 5, 5, 2, 0), 256, True), ((67, 1, 161, 328, 64, 5, 5, 2, 1), 256, True), ((69, 3, 69, 117, 94, 3, 3, 1, 1), 0, False),
    # a window of 1024 pixels that is too large (the second one of 512 leaves room for three by itself); deep stems of 36 MB
    ((2087, 8, 91, 260, 6, 3, 3, 2, 1), 512, False), ((772, 12, 322, 109, 10, 3, 3, 2, 0), 512, True), ((9, 1, 161, 504, 64, 20, 5, 2, 1), 0, False),
    ((17, 1, 151, 281, 64, 20, 5, 2, 0), 512, False),
    ((60064, 2, 6, 26, 48, 5, 5, 1, 0), 0, False), ((1302, 3, 32, 32, 64, 3, 3, 1, 1), 0, False), ((557, 4, 240, 384, 24, 3, 3, 2, 1), 0, False),
]


@pytest.mark.parametrize("dims,pixels,few", STENCIL_RULE, ids=str)
def test_large_results_take_the_kernel_that_suits_them(lib, launches, dims, pixels, few):
    """Tiles of consecutive pixels as large as what a workgroup writes allows, three per compute unit only where that is much; rows that fill the
    window kernel's tiles stay there."""
    N, C, H, W, K, R, S, stride, pad = dims
    (call,) = launches([(dims, lib.LAYOUT_IMPLICIT, 0, 0)])
    assert call["rc"] == 0 and call["launches"] == 1
    assert ("conv_stencil_kernel" if pixels else "conv_window_kernel") in call["kernel"]
    if pixels:
        P, Q = lib.out_hw(H, W, R, S, stride, pad)
        assert call["workgroups"] == N * -(-(-(-P * Q // 32)) // (pixels // 32)) * -(-K // 64)
        assert (call["lds"] > 160 * 1024 // 4) == few


def kernel(call):
    """Name and integer template arguments of a recorded launch's kernel."""
    name, args = re.search(r"\d((?:conv|igemm)_\w+?)_kernelI(.*?)EEv", call["kernel"]).groups()
    return name, tuple(int(v) for v in re.findall(r"L(?:[ib]|NS_\d+[A-Za-z]+E)(\d+)E", args))


def test_shapes_of_the_gpu_tests_take_the_kernels_they_are_for(lib, launches):
    """A line of a dispatch that moves does not leave a kernel without its test."""
    def kernels(dims):
        return [kernel(c) for c in launches([(d, lib.LAYOUT_IMPLICIT, 0, packed) for d in dims for packed in (0, 1)])[::2]]

    stencil = dict(zip((c.name for c in gpu.STENCIL), kernels([c.dims() for c in gpu.STENCIL])))
    assert {name for name, k in stencil.items() if k[0] != "conv_stencil"} == set(gpu.STENCIL_NOT)
    past = kernels([(gpu.past_the_cache_batch(d), *d) for d in gpu.PAST_THE_CACHE])
    assert [k[0] for k in past] == ["conv_stencil", "conv_window"] * 2 + ["conv_stencil"] * 5
    # every depth with 32 and with 64 channels to a workgroup
    ran = {k[1] for k in [*stencil.values(), *past] if k[0] == "conv_stencil"}
    assert ran == {(depth, blocks) for depth in (2, 4, 6, 8) for blocks in (1, 2)}
    # the window kernel in several row groups (the fifth argument), through and past the caches (the sixth)
    assert [k[1][1:] for k in kernels([c.dims() for c in gpu.WINDOW_GROUPS])] == [(1, 0, 0, 1, 0)] * 3 + [(2, 0, 0, 1, 0)] + [(1, 0, 0, 1, 2)] * 2
    assert [k[1] for k in kernels([(gpu.window_streamed_batch(K), 3, 32, 32, K, 3, 3, 1, 1) for K in (16, 64)])] == [(2, 1, 0, 0, 1, 1), (2, 2, 0, 0, 0, 1)]
    # the 1x1 kernel past the caches, every depth
    assert set(kernels(gpu.POINTWISE_THROUGH)) == {("conv_pointwise", (n, 0, 1)) for n in range(2, 17, 2)}


def test_raw_1x1_weights_take_the_resident_kernel(lib):
    """... without a launch that rewrites them, in every tile that the library picks; its tile and pixels run on rewritten weights too."""
    tiles = set()
    for N, C, H, W, K, stride, pad in gpu.ROWS_1X1:
        dims = (N, C, H, W, K, 1, 1, stride, pad)
        stage, tile, pixels = lib.query_stage(dims, lib.ENTRY_EX, lib.LAYOUT_PACKED, 64, False)
        assert stage == lib.STAGE_RESIDENT and lib.resident_applies(dims, 16, tile, pixels), dims
        tiles.add(tile)
    assert tiles == {0, 1, 2, 4}


@pytest.fixture(scope="module")
def store_listing(tmp_path_factory):
    """kernel -> its instructions, as lists of words"""
    listing = tmp_path_factory.mktemp("listing") / "store_past.s"
    subprocess.run(["hipcc", "--offload-arch=gfx950", "-O3", "-S", "--cuda-device-only", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                    os.path.join(HERE, "store_past.hip"), "-o", str(listing)], check=True, capture_output=True, timeout=120)

    def code(kernel):
        lines = listing.read_text().split(f"\n{kernel}:")[1].split("\n", 1)[1].split("\n\t.section")[0].splitlines()
        return [s for s in (line.split(";")[0].replace(",", " ").split() for line in lines) if s and not s[0].endswith(":")]
    return code


def wait_states(code):
    return sum(int(s[1]) + 1 if s[0] == "s_nop" else 1 for s in code)


def is_store(s):
    return s[0] in ("global_store_dwordx4", "buffer_store_dwordx4")


def test_stores_past_the_caches_keep_their_wait_states(store_listing):
    """A vector instruction that writes a 16-byte store's registers stands as far behind the store past the caches as behind one of the compiler's."""
    def states(kernel):
        code = store_listing(kernel)
        at = next(i for i, s in enumerate(code) if is_store(s))
        return wait_states(code[at + 1:next(i for i, s in enumerate(code) if i > at and s[0].startswith("v_"))])

    assert states("rewritten_behind_past") >= states("rewritten_behind_compiled") >= 1


def test_stores_past_the_caches_wait_for_their_base(store_listing):
    """A base that a vector instruction writes is five wait states old when the store reads it."""
    code = store_listing("base_written_past")
    at = next(i for i, s in enumerate(code) if is_store(s))
    wrote = [i for i in range(at) if code[i][0] == "v_readfirstlane_b32"]
    assert len(wrote) == 2 and wait_states(code[wrote[-1] + 1:at]) >= 5


def test_stores_past_the_caches_are_not_merged_with_plain_ones(store_listing):
    """One that streams a result past every cache, one that writes it through to the last-level cache, where its reader finds it, a plain one."""
    stores = [s for s in store_listing("three_branches") if is_store(s)]
    assert sorted(("nt" in s, "sc1" in s, "sc0" in s) for s in stores) == [(False, False, False), (False, True, False), (True, False, False)]
