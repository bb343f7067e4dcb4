"""Host-side checks of the C ABI that need no GPU: the library loads, exports every symbol
the header declares, and rejects bad arguments before touching the device."""
import ctypes
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib():
    import paper_2507_07149_amd as daf
    return daf.load_library()


def declared_functions():
    names = set()
    inc = os.path.join(ROOT, "include")
    for header in sorted(os.listdir(inc)):
        if header.endswith(".h"):
            text = re.sub(r"/\*.*?\*/", "", open(os.path.join(inc, header)).read(), flags=re.S)
            names |= set(re.findall(r"\b(daf_[a-z_0-9]+)\s*\(", text))
    return sorted(names)


def test_every_declared_symbol_is_exported(lib):
    names = declared_functions()
    assert {"daf_plan", "daf_quantize_pack", "daf_unpack_dequantize", "daf_plan_destroy", "daf_store_create"} <= set(names)
    for name in names:
        assert hasattr(lib, name), f"{name} is declared in include/*.h but not exported"


def test_python_binding_has_the_same_entry_points():
    import paper_2507_07149_amd as daf
    for name in ("daf_plan", "daf_quantize_pack", "daf_unpack_dequantize"):
        assert callable(getattr(daf, name))


def test_rand_bits_and_status_strings(lib):
    assert lib.daf_rand_bits() == 8
    for code in (0, -1, -2, -3, -4, 77):
        assert lib.daf_status_string(code)


def _plan(lib, shape, gs, bits):
    shp = (ctypes.c_int64 * len(shape))(*shape)
    b = (ctypes.c_uint8 * len(bits))(*bits)
    out = ctypes.c_void_p()
    rc = lib.daf_plan(shp, len(shape), gs, ctypes.cast(b, ctypes.c_void_p), len(bits), None, ctypes.byref(out))
    return rc, out


def test_uniform_plan_needs_no_device(lib):
    rc, p = _plan(lib, (64, 256, 56, 56), 256, [2])
    assert rc == 0
    assert lib.daf_plan_packed_words(p) == 3211264
    assert lib.daf_plan_num_groups(p) == 200704
    assert lib.daf_plan_num_elements(p) == 51380224
    assert lib.daf_plan_group_size(p) == 256 and lib.daf_plan_uniform_bits(p) == 2
    lib.daf_plan_destroy(p)
    rc, p = _plan(lib, (37,), 32, [4])                 # short last group: 4 + 1 words
    assert rc == 0 and lib.daf_plan_packed_words(p) == 5
    off = (ctypes.c_uint32 * 2)()
    assert lib.daf_plan_copy_offsets(p, off) == 0 and list(off) == [0, 4]
    assert lib.daf_plan_set_output_cached(p, 1) == 0 and lib.daf_plan_set_output_cached(p, 0) == 0
    assert lib.daf_plan_set_output_cached(p, 2) == -1 and lib.daf_plan_set_output_cached(p, -1) == -1
    assert lib.daf_plan_set_output_cached(None, 1) == -1
    lib.daf_plan_destroy(p)
    lib.daf_plan_destroy(None)


@pytest.mark.parametrize("shape,gs,bits,want", [
    ((64,), 32, [3], -1), ((64,), 32, [0], -1), ((64,), 32, [16], -1),
    ((64,), 48, [2], -2), ((64,), 0, [2], -2), ((64,), 16, [2], -2),
    ((0,), 32, [2], -1), ((4, -1), 32, [2], -1),
    ((64,), 32, [2, 2, 2], -1),                        # neither 1 nor G widths
    ((1 << 40,), 32, [8], -2),                         # 2^38 words
])
def test_plan_argument_errors(lib, shape, gs, bits, want):
    rc, p = _plan(lib, shape, gs, bits)
    assert rc == want and not p.value


def test_null_arguments(lib):
    out = ctypes.c_void_p()
    assert lib.daf_plan(None, 1, 32, None, 1, None, ctypes.byref(out)) == -1
    shp = (ctypes.c_int64 * 1)(64)
    assert lib.daf_plan(shp, 0, 32, ctypes.cast(shp, ctypes.c_void_p), 1, None, ctypes.byref(out)) == -1
    rc, p = _plan(lib, (64,), 32, [2])
    assert lib.daf_quantize_pack(p, None, 0, 0, None, None, None, None) == -1
    assert lib.daf_unpack_dequantize(p, None, None, None, None, None, 0, None) == -1
    assert lib.daf_quantize_pack(None, 16, 0, 0, 16, 16, 16, None) == -1
    # misaligned x and unknown dtype are rejected before any launch
    assert lib.daf_quantize_pack(p, 20, 0, 0, 16, 16, 16, None) == -1
    assert lib.daf_quantize_pack(p, 16, 7, 0, 16, 16, 16, None) == -2
    assert lib.daf_unpack_dequantize(p, 16, 16, 16, None, 16, 9, None) == -2
    lib.daf_plan_destroy(p)


def test_binding_fails_loudly_without_the_library(monkeypatch, tmp_path):
    from paper_2507_07149_amd import binding
    monkeypatch.setattr(binding, "_lib", None)
    monkeypatch.setattr(binding, "_LIB_PATH", str(tmp_path / "libdaf.so"))
    with pytest.raises(ImportError):
        binding.load_library()


@pytest.mark.parametrize("n,gs,dtype,want", [
    (4096 * 10, 256, 0, 0), (4096 * 10, 4096, 2, 0), (4096 * 10, 32, 1, 0),         # tile
    (768 * 100, 768, 0, 1), (96 * 1000, 96, 1, 1), (4064 * 9, 4064, 2, 1),          # units
    (11008 * 7, 11008, 0, 2), (4128 * 3, 4128, 2, 2), (32736 * 2 + 5, 32736, 1, 2),  # long (not whole tiles)
    (40000 * 3, 40000, 0, 2), (65504 * 2, 65504, 2, 2),                              # long, up to 65536
    (69984 * 3, 69984, 0, 4), (65568 * 2, 65568, 2, 4),                              # group by group
    (100, 256, 0, 4), (700, 768, 1, 4),                                              # no whole group
])
def test_quantize_route_of_uniform_plans(lib, n, gs, dtype, want):
    """The route a plan's quantize call takes, for plans that need no device (one width, no
    statistics pass): tile, units, long, group by group."""
    rc, p = _plan(lib, (n,), gs, [2])
    assert rc == 0
    assert lib.daf_plan_quantize_route(p, dtype) == want
    assert lib.daf_plan_quantize_route(p, 7) == -2 and lib.daf_plan_quantize_route(None, 0) == -1
    lib.daf_plan_destroy(p)


def test_calls_with_another_number_of_looks_check_their_arguments_too(lib):
    classes = (ctypes.c_uint8 * 3)(2, 4, 8)
    wrong = (ctypes.c_uint8 * 3)(2, 3, 8)
    ptr = ctypes.c_void_p

    def select(lo=4096, hi=4096, G=100, cl=classes, n=3, out=4096, ws=4096):
        return lib.daf_internal_select_bits(ptr(lo), ptr(hi), ctypes.c_int64(G), cl, n, ptr(out), ptr(ws), 0, None)
    for bad in (dict(lo=None), dict(hi=None), dict(out=None), dict(ws=None), dict(ws=4104), dict(lo=4098), dict(G=0), dict(n=0),
                dict(n=5), dict(cl=wrong)):
        assert select(**bad) == -1, bad
    assert select(G=1 << 32) == -2
    rc, p = _plan(lib, (64,), 32, [2])
    assert lib.daf_internal_plan_update(None, ptr(16), 0, None) == -1 and lib.daf_internal_plan_update(p, None, 0, None) == -1
    assert lib.daf_internal_plan_update(p, ptr(16), 0, None) == -1                   # one width
    lib.daf_plan_destroy(p)


# m, n, k, element format -> tile of the weight gradient: 512 x 128 only where it is not slower than the general kernel
@pytest.mark.parametrize("m,n,k,dtype,tile", [
    (32768, 4096, 11008, 2, (512, 128)), (32768, 3072, 768, 1, (512, 128)), (128, 4096, 4096, 2, (512, 128)),
    (8192, 832, 4352, 1, (512, 128)), (32768, 320, 768, 2, (512, 128)),
    # the last tile of n mostly outside the output, a last round that is nearly empty
    (32768, 576, 4352, 2, (256, 128)), (32768, 768, 4352, 1, (256, 128)), (8192, 576, 4352, 1, (256, 128)),
    (512, 1088, 11008, 2, (256, 128)),
    # one tile of n: never; enough of them for the wider general tile
    (4096, 256, 4096, 2, (256, 128)), (2048, 256, 65536, 1, (256, 256)), (4096, 128, 65536, 2, (256, 256)),
    (4096, 4096, 4096, 0, (256, 256)), (256, 256, 192, 2, (256, 64)), (512, 1024, 1024, 1, (256, 64)),
    # the narrow tile 8 to 10 % ahead by the model, which is too little in binary32
    (1920, 256, 1152, 0, (256, 128)), (1280, 192, 1920, 0, (256, 128)), (3008, 576, 384, 2, (256, 64))])
def test_weight_gradient_tile(lib, m, n, k, dtype, tile):
    import paper_2507_07149_amd as daf
    import torch
    plan = daf.daf_plan((m, k), 64, 4)
    s = daf.daf_unpack_matmul_schedule(plan, n, k, (torch.float32, torch.float16, torch.bfloat16)[dtype])
    assert (s["tile_n"], s["tile_k"]) == tile
    assert s["tiles"] == -(-n // tile[0]) * (k // tile[1]) and 0 <= s["whole_tiles"] <= s["tiles"]
    assert (s["slices"] > 1) == (s["whole_tiles"] < s["tiles"])
    if s["slices"] > 1:
        need = s["slices"] * (s["tiles"] - s["whole_tiles"]) * tile[0] * tile[1] * 4
        assert need <= daf.daf_unpack_matmul_workspace_bytes(plan, n, k)
    with pytest.raises(daf.DafError):
        daf.daf_unpack_matmul_schedule(plan, n + 1, k, torch.float16)
    plan.destroy()


@pytest.mark.parametrize("m,n,k", [(4096, 4096, 3136), (32768, 4096, 3136), (1024, 2048, 6208)])
def test_weight_gradient_tile_of_an_odd_number_of_64_columns(lib, m, n, k):
    """Outputs of a few 256 x 64 tiles more than whole rounds of 768: the 512 x 128 tile is faster there as well."""
    import paper_2507_07149_amd as daf
    import torch
    assert 0 < (-(-n // 256) * (k // 64)) % 768 <= 24
    plan = daf.daf_plan((m, k), 64, 4)
    for dtype, tile in ((torch.float16, (512, 128)), (torch.bfloat16, (512, 128)), (torch.float32, (256, 64))):
        s = daf.daf_unpack_matmul_schedule(plan, n, k, dtype)
        assert (s["tile_n"], s["tile_k"]) == tile and s["tiles"] == -(-n // tile[0]) * -(-k // tile[1])
    plan.destroy()


@pytest.mark.parametrize("m,n,k,dtype,tile,slices", [
    (1344, 640, 1536, 2, (256, 64), 4), (896, 512, 8064, 1, (256, 64), 1), (672, 320, 5376, 1, (256, 64), 1), (992, 128, 1280, 0, (256, 64), 7),
    # few steps along m
    (512, 640, 1536, 2, (256, 64), 2), (512, 1024, 1024, 1, (256, 64), 4), (64, 512, 256, 2, (256, 64), 1), (32, 256, 1280, 2, (256, 64), 1),
    (96, 192, 8064, 0, (256, 64), 1),
    # below 128 rows, more than a round of such tiles, shapes that have this tile already
    (1344, 64, 1536, 2, (256, 128), None), (4096, 4096, 4352, 0, (256, 256), None),
    (544, 128, 8768, 0, (256, 64), 4), (640, 1344, 960, 2, (256, 64), 3)])
def test_weight_gradient_narrow_tile(lib, m, n, k, dtype, tile, slices):
    """Outputs of few tiles take 256 x 64, in no fewer slices than the wider tile, whose partial sums fit the workspace that callers are told of."""
    import paper_2507_07149_amd as daf
    import torch
    plan = daf.daf_plan((m, k), 64, 4)
    s = daf.daf_unpack_matmul_schedule(plan, n, k, (torch.float32, torch.float16, torch.bfloat16)[dtype])
    assert (s["tile_n"], s["tile_k"]) == tile and s["slices"] == (slices or s["slices"])
    plan.destroy()


def test_weight_gradient_schedules_stay_inside_the_workspace(lib):
    import random
    import paper_2507_07149_amd as daf
    import torch
    rng, narrow = random.Random(3), 0
    for _ in range(600):
        m, n, k = 32 * rng.randint(1, 400), 64 * rng.randint(1, 40), 64 * rng.randint(1, 140)
        plan = daf.daf_plan((m, k), 64, 4)
        room = daf.daf_unpack_matmul_workspace_bytes(plan, n, k)
        for dtype in (torch.float32, torch.float16, torch.bfloat16):
            s = daf.daf_unpack_matmul_schedule(plan, n, k, dtype)
            rest = s["tiles"] - s["whole_tiles"]
            assert s["tiles"] == -(-n // s["tile_n"]) * -(-k // s["tile_k"]) and (s["slices"] > 1) == (rest > 0)
            assert s["slices"] == 1 or (s["slices"] * rest * s["tile_n"] * s["tile_k"] * 4 <= room and m // 32 >= 4 * s["slices"])
            narrow += s["tile_k"] == 64
        plan.destroy()
    assert narrow > 100


# n, group size, width, element format, (relu backward, elements of the list) -> route; plans that need no device
@pytest.mark.parametrize("n,gs,b,dtype,call,want", [
    (1 << 20, 64, 2, 0, (0, 0), 0), (1 << 20, 2048, 8, 0, (0, 0), 0), (1 << 20, 4096, 2, 1, (1, 0), 0),
    # 4096 elements are two tiles in binary32
    (1 << 20, 4096, 2, 0, (0, 0), 1), (1 << 20, 4096, 8, 0, (0, 0), 2), ((1 << 26) + 4096, 4096, 2, 0, (0, 0), 2),
    # groups of 32: 64 to a tile in binary32, half tiles in a 16-bit call on one tensor
    (1 << 20, 32, 2, 0, (0, 0), 0), (1 << 20, 32, 2, 1, (0, 0), 0), (1 << 20, 32, 2, 1, (0, 1 << 20), 2),
    (1 << 20, 32, 2, 2, (1, 0), 2), (1 << 27, 32, 2, 2, (1, 0), 0),
    # not a power of two
    (768 * 4000, 768, 4, 1, (0, 0), 1), (768 * 4000, 768, 8, 0, (0, 0), 2), (96 * 40000, 96, 1, 0, (1, 0), 1),
    (768 * 4000, 768, 1, 0, (0, 5 << 23), 1), (768 * 4000, 768, 1, 0, (0, (5 << 23) + 1), 2), (768 * 70000, 768, 1, 0, (0, 0), 1),
    # longer than a tile
    (40000 * 1677, 40000, 2, 1, (0, 0), 1), (40000 * 1677, 40000, 1, 1, (0, 0), 2), (40000 * 1678, 40000, 1, 1, (0, 0), 1),
    (40000 * 1677, 40000, 4, 2, (0, 0), 1), (40000 * 1678, 40000, 4, 2, (0, 0), 2), (40000 * 1678, 40000, 8, 2, (0, 0), 1),
    (40000 * 1677, 40000, 2, 0, (0, 0), 1), (40000 * 1678, 40000, 2, 0, (0, 0), 2),
    (40000 * 419, 40000, 2, 1, (1, 0), 1), (40000 * 420, 40000, 2, 1, (1, 0), 2), (40000 * 209, 40000, 2, 0, (1, 0), 1),
    (40000 * 210, 40000, 2, 0, (1, 0), 2), (40000 * 1048, 40000, 1, 0, (0, 0), 1), (40000 * 1049, 40000, 1, 0, (0, 0), 2),
    (100, 64, 2, 1, (0, 0), 2)])
def test_dequantize_route_of_uniform_plans(lib, n, gs, b, dtype, call, want):
    rc, p = _plan(lib, (n,), gs, [b])
    assert rc == 0
    assert lib.daf_plan_dequantize_route(p, dtype, *call) == want
    assert lib.daf_plan_dequantize_route(p, 7, 0, 0) == -2 and lib.daf_plan_dequantize_route(None, 0, 0, 0) == -1
    assert lib.daf_plan_dequantize_route(p, dtype, 1, 5) == -1 and lib.daf_plan_dequantize_route(p, dtype, 0, -1) == -1
    lib.daf_plan_destroy(p)
