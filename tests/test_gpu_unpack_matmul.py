"""GPU parity of the fused weight gradient: daf_unpack_matmul_grad_weight (unpack + dequantize
inside the matrix product) against the oracle's dequantized activation multiplied out in double
precision.  The additions happen in binary32 in an unspecified order, so the bar is the
accumulation bound M * 2^-24 * sum_m |grad_y| |xhat| (with a factor 2 of slack)."""
import numpy as np
import pytest
import torch

from daf_inputs import BF16, F16, F32, to_numpy_bits, torch_dtype

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import paper_2507_07149_amd as daf
    from oracle import daf_oracle as orc
    assert torch.cuda.is_available()
    return daf, orc


def _case(daf, orc, M, N, K, gs, bits, dtype, seed):
    g = torch.Generator().manual_seed(seed)
    x = (torch.randn(M, K, generator=g) * (1 + torch.rand(M, 1, generator=g))).to(torch_dtype(dtype))
    gy = (torch.randn(M, N, generator=g) * 0.5).to(torch_dtype(dtype))
    G = M * K // gs
    b = (np.random.default_rng(seed).choice([1, 2, 4, 8], G).astype(np.uint8) if bits == "mixed"
         else np.array([bits], np.uint8))
    ow, omn, osc, _ = orc.quantize_pack(to_numpy_bits(x), dtype, gs, b, seed)
    oxh, _ = orc.unpack_dequantize(ow, omn, osc, b, M * K, gs, dtype)
    want = orc.grad_weight(oxh, to_numpy_bits(gy), M, K, N, dtype)
    mag = orc.grad_weight(np.abs(orc.widen(oxh, dtype)), np.abs(orc.widen(to_numpy_bits(gy), dtype)), M, K, N, F32)

    dbits = torch.from_numpy(b).cuda() if b.size > 1 else None
    plan = daf.daf_plan((M, K), gs, dbits if dbits is not None else int(b[0]))
    ws_bytes = daf.daf_unpack_matmul_workspace_bytes(plan, N, K)
    assert ws_bytes >= 0
    ws = torch.empty(max(ws_bytes, 16), dtype=torch.uint8, device="cuda:0")
    out = torch.full((N, K), float("nan"), device="cuda:0")
    daf.daf_unpack_matmul_grad_weight(plan, torch.from_numpy(ow.view(np.int32)).cuda(), torch.from_numpy(omn).cuda(),
                                      torch.from_numpy(osc).cuda(), gy.cuda(), out, ws)
    torch.cuda.synchronize()
    got = out.cpu().numpy().astype(np.float64)
    bound = 2.0 * M * 2.0 ** -24 * mag + 1e-30
    err = np.abs(got - want)
    assert np.all(err <= bound), (f"worst {err.max():.3e} at {np.unravel_index(err.argmax(), err.shape)}, "
                                  f"bound there {bound.flat[err.argmax()]:.3e}, share outside {np.mean(err > bound):.4f}")
    plan.destroy()
    return ws_bytes


@pytest.mark.parametrize("dtype", [BF16, F16, F32])
@pytest.mark.parametrize("bits", [1, 2, 4, 8, "mixed"])
@pytest.mark.parametrize("gs", [32, 128])
def test_grad_weight_small(env, dtype, bits, gs):
    daf, orc = env
    print("case small", dtype, bits, gs, flush=True)
    _case(daf, orc, 128, 256, 256, gs, bits, dtype, 7)                 # two k-tiles, m in several slices


# K a multiple of 128 runs the 128-column tile, any other multiple of 64 the 64-column one.
@pytest.mark.parametrize("shape", [(32, 256, 128), (64, 256, 128), (96, 256, 256), (192, 512, 384), (1024, 256, 128),
                                   (2048, 512, 1024), (32, 256, 64), (96, 256, 192), (160, 512, 320),
                                   (1024, 256, 448), (1088, 256, 128)])         # the last: 34 steps in 7 slices
@pytest.mark.parametrize("bits", [2, "mixed"])
def test_grad_weight_shapes(env, shape, bits):
    daf, orc = env
    M, N, K = shape
    print("case shape", shape, bits, flush=True)
    _case(daf, orc, M, N, K, 64, bits, BF16, 11)


# N a multiple of 64 but not of 256: the last tile of n has waves outside the output
@pytest.mark.parametrize("case", [(64, 256, 768, 768, "mixed", BF16), (96, 256, 768, 384, 4, F16), (64, 64, 704, 704, "mixed", F32),
                                  (128, 512, 3072, 3072, "mixed", BF16), (64, 256, 1536, 96, "mixed", F16),
                                  (32, 256, 2816, 1408, 2, BF16)])
def test_grad_weight_groups_that_are_rows_or_not_a_power_of_two(env, case):
    """One group per row of the activation (768, 3072), half rows, and small odd multiples of 32."""
    daf, orc = env
    M, N, K, gs, bits, dtype = case
    print("case", case, flush=True)
    _case(daf, orc, M, N, K, gs, bits, dtype, 19)


@pytest.mark.parametrize("case", [(256, 64, 256, 64, "mixed", BF16), (128, 320, 384, 32, 2, F16), (512, 192, 128, 128, "mixed", F32),
                                  (8192, 64, 256, 64, 4, F32), (2048, 448, 192, 64, "mixed", BF16),
                                  (32, 4160, 4096, 64, "mixed", BF16)])       # the last: 512 x 128 tile, 9 tiles of n
def test_grad_weight_n_not_a_multiple_of_256(env, case):
    daf, orc = env
    M, N, K, gs, bits, dtype = case
    print("case n % 256 != 0", case, flush=True)
    _case(daf, orc, M, N, K, gs, bits, dtype, 29)


def test_grad_weight_tall_and_skinny(env):
    """A long reduction into one or two tiles: m is cut into far more than 16 slices."""
    daf, orc = env
    print("case tall and skinny", flush=True)
    ws = _case(daf, orc, 16384, 256, 256, 128, "mixed", BF16, 19)
    assert ws > 16 * 2 * 256 * 128 * 4                                        # more than 16 slices of the 2 tiles
    _case(daf, orc, 8192, 256, 128, 64, 2, F32, 23)


# The sum over the slices starts the loads of up to eight slices at a time: every remainder, once and twice eight, and two
# levels (more than 16 slices) whose last group is short or whole.  One tile that N ends inside of; bound as in _case.
@pytest.mark.parametrize("slices", [*range(2, 18), 25, 33, 40])
def test_grad_weight_every_number_of_slices(env, slices):
    daf, orc = env
    print("case slices", slices, flush=True)
    M, N, K = 128 * slices, 192, 64
    plan = daf.daf_plan((M, K), 32, 4)
    assert daf.daf_unpack_matmul_schedule(plan, N, K, torch.float32)["slices"] == slices
    plan.destroy()
    _case(daf, orc, M, N, K, 32, 4, F32, slices)


def test_grad_weight_without_split_needs_no_workspace(env):
    daf, orc = env
    print("case no split", flush=True)
    ws = _case(daf, orc, 64, 4096, 4096, 256, 4, BF16, 3)              # 256 tiles of 512 x 128: one slice of m
    assert ws == 0


# 256 or more 256 x 256 tiles: 8 waves per work-group, the 256-column tile in binary32, 512 x 128 in the 16-bit formats
@pytest.mark.parametrize("case", [(32, 4096, 4096, 64, "mixed", BF16), (96, 4096, 4096, 128, "mixed", F16),
                                  (64, 8192, 2048, 32, "mixed", BF16), (64, 2048, 8192, 256, 8, F16),
                                  (32, 4096, 4096, 64, 1, BF16), (64, 4096, 4096, 64, "mixed", F32),
                                  (32, 2048, 8192, 128, 2, F32)])
def test_grad_weight_wide_tile(env, case):
    daf, orc = env
    M, N, K, gs, bits, dtype = case
    print("case wide tile", case, flush=True)
    ws = _case(daf, orc, M, N, K, gs, bits, dtype, 13)
    assert ws == 0


# 16-bit formats, 256 or more tiles of 512 x 128, or enough steps: the pipeline of 32 values of m per step is four deep and
# unrolled by four, so every remainder; N with a last tile of n that is mostly outside the output, groups that do not
# coincide with the 128 columns of a tile.
@pytest.mark.parametrize("steps,N,K,gs,bits,dtype", [(4, 2368, 6912, 96, "mixed", BF16), (5, 3648, 4096, 4096, 2, F16),
                                                     (6, 2560, 6912, 384, "mixed", F16), (7, 3648, 4096, 32, 8, BF16),
                                                     (8, 3648, 4096, 64, "mixed", BF16), (9, 3648, 4096, 2048, 1, F16),
                                                     (2561, 320, 128, 32, "mixed", BF16), (1283, 576, 128, 128, 4, F16)])
def test_grad_weight_512_by_128_tile(env, steps, N, K, gs, bits, dtype):
    _steps_case(env, steps, N, K, gs, bits, dtype, 512, 128)


# The general kernel in the 16-bit formats: a few tiles of 512 x 128 more than a round of work-groups holds (the general
# kernel's tiles are one round), one tile of n with 128 columns of k, the last of them in slices of m, and with 256.
@pytest.mark.parametrize("steps,N,K,gs,bits,dtype,bk", [(4, 2112, 6912, 96, "mixed", BF16, 128), (5, 2112, 6656, 6656, 2, F16, 128),
                                                        (7, 2112, 6912, 32, 8, BF16, 128), (9, 4160, 3840, 1920, 1, F16, 128),
                                                        (16, 256, 128 * 513, 64, "mixed", BF16, 128), (16, 192, 128 * 513, 384, 2, F16, 128),
                                                        (3, 256, 65536, 128, "mixed", F16, 256), (2, 128, 65536, 32, 4, BF16, 256)])
def test_grad_weight_general_kernel(env, steps, N, K, gs, bits, dtype, bk):
    _steps_case(env, steps, N, K, gs, bits, dtype, 256, bk)


# K an odd multiple of 64: the last tile of k reaches 64 columns past the output, in both kernels, over all of m (the second
# and third) and in slices; groups that end with the row inside that tile, one group per row among them.
@pytest.mark.parametrize("steps,N,K,gs,bits,dtype,bn,bk", [(1280, 320, 192, 192, "mixed", BF16, 512, 128), (33, 4096, 2112, 32, "mixed", F16, 512, 128),
                                                           (34, 2048, 4160, 64, 8, BF16, 512, 128), (512, 1024, 448, 64, 1, F16, 512, 128),
                                                           (169, 64, 10176, 32, "mixed", BF16, 256, 128), (270, 64, 5824, 5824, 4, F16, 256, 128)])
def test_grad_weight_odd_multiple_of_64_columns(env, steps, N, K, gs, bits, dtype, bn, bk):
    _steps_case(env, steps, N, K, gs, bits, dtype, bn, bk)


# Outputs of few tiles: 256 x 64, over all of m and in slices, from one step along m; ends of n inside the tile.
@pytest.mark.parametrize("steps,N,K,gs,bits,dtype", [(20, 1344, 960, 32, "mixed", BF16), (17, 128, 640, 64, 2, F16), (42, 640, 768, 768, "mixed", F16),
                                                     (21, 320, 5376, 64, "mixed", BF16), (31, 128, 640, 128, 8, F32),
                                                     (1, 256, 1280, 64, "mixed", BF16), (2, 192, 1280, 32, 4, F16), (3, 192, 8064, 32, "mixed", F32),
                                                     (15, 320, 768, 768, "mixed", BF16), (16, 1024, 1024, 128, 1, F16)])
def test_grad_weight_few_tiles(env, steps, N, K, gs, bits, dtype):
    _steps_case(env, steps, N, K, gs, bits, dtype, 256, 64)


def _steps_case(env, steps, N, K, gs, bits, dtype, bn, bk):
    daf, orc = env
    print("case", bn, bk, steps, N, K, gs, bits, dtype, flush=True)
    M = 32 * steps
    g = torch.Generator().manual_seed(steps)
    x = (torch.randn(M, K, generator=g) * (1 + torch.rand(M, 1, generator=g))).to(torch_dtype(dtype))
    gy = (torch.randn(M, N, generator=g) * 0.5).to(torch_dtype(dtype))
    b = _widths(M * K // gs, bits, steps)
    ow, omn, osc, _ = orc.quantize_pack(to_numpy_bits(x), dtype, gs, b, steps)
    xh = orc.widen(orc.unpack_dequantize(ow, omn, osc, b, M * K, gs, dtype)[0], dtype).reshape(M, K).astype(np.float64)
    gd = gy.double().numpy()
    plan = daf.daf_plan((M, K), gs, torch.from_numpy(b).cuda() if b.size > 1 else int(b[0]))
    how = daf.daf_unpack_matmul_schedule(plan, N, K, torch_dtype(dtype))
    assert (how["tile_n"], how["tile_k"]) == (bn, bk)
    assert (K != 128 * 513) or (how["slices"] > 1 and how["whole_tiles"] == 512)
    ws = torch.empty(max(daf.daf_unpack_matmul_workspace_bytes(plan, N, K), 16), dtype=torch.uint8, device="cuda:0")
    out = torch.full((N, K), float("nan"), device="cuda:0")
    daf.daf_unpack_matmul_grad_weight(plan, torch.from_numpy(ow.view(np.int32)).cuda(), torch.from_numpy(omn).cuda(),
                                      torch.from_numpy(osc).cuda(), gy.cuda(), out, ws)
    torch.cuda.synchronize()
    bound = 2.0 * M * 2.0 ** -24 * (np.abs(gd).T @ np.abs(xh)) + 1e-30
    assert np.all(np.abs(out.cpu().numpy() - gd.T @ xh) <= bound)
    plan.destroy()


# The same kernel where a wave's loads are furthest from its neighbours': many work-groups, grad_y from memory, and a number
# of steps that leaves three after the last whole four (32768 x 3072 x 768: slices of 146 and 147 steps; 352 x 4096 x 4096:
# 256 tiles, not sliced, 11 steps), with one width, whose steps have the fewest waits of their own, and with several.
@pytest.mark.timeout(300)
@pytest.mark.parametrize("M,N,K,gs,bits,dtype", [(32768, 3072, 768, 128, 2, F16), (32768, 3072, 768, 128, "mixed", F16),
                                                 (32768, 3072, 768, 64, 4, BF16), (352, 4096, 4096, 64, 8, F16),
                                                 (352, 4096, 4096, 128, 1, BF16)])
def test_grad_weight_512_by_128_tile_three_steps_left(env, M, N, K, gs, bits, dtype):
    daf, orc = env
    print("case three steps left", M, N, K, gs, bits, dtype, flush=True)
    g = torch.Generator().manual_seed(M + K)
    x = torch.randn(M, K, generator=g).to(torch_dtype(dtype))
    gy = (torch.randn(M, N, generator=g) * 0.5).to(torch_dtype(dtype))
    b = _widths(M * K // gs, bits, M)
    ow, omn, osc, _ = orc.quantize_pack(to_numpy_bits(x), dtype, gs, b, M)
    xh = orc.widen(orc.unpack_dequantize(ow, omn, osc, b, M * K, gs, dtype)[0], dtype).reshape(M, K).astype(np.float64)
    plan = daf.daf_plan((M, K), gs, torch.from_numpy(b).cuda() if b.size > 1 else int(b[0]))
    ws = torch.empty(max(daf.daf_unpack_matmul_workspace_bytes(plan, N, K), 16), dtype=torch.uint8, device="cuda:0")
    words, mn, sc, gyd = torch.from_numpy(ow.view(np.int32)).cuda(), torch.from_numpy(omn).cuda(), torch.from_numpy(osc).cuda(), gy.cuda()
    outs = [torch.full((N, K), float("nan"), device="cuda:0") for _ in range(3)]
    for out in outs:
        daf.daf_unpack_matmul_grad_weight(plan, words, mn, sc, gyd, out, ws)
    torch.cuda.synchronize()
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
    gd = gy.double().numpy()
    want, mag = gd.T @ xh, np.abs(gd).T @ np.abs(xh)
    assert np.all(np.abs(outs[0].cpu().numpy() - want) <= 2.0 * M * 2.0 ** -24 * mag + 1e-30)
    plan.destroy()


@pytest.mark.parametrize("start", [1, 2, 3])
def test_grad_weight_512_by_128_tile_widths_at_any_address(env, start):
    """The widths may be handed in at any byte address: the same result as with the plan's own copy."""
    daf, orc = env
    M, N, K, gs = 160, 4096, 4096, 96 if start == 2 else 32
    K = 3840 if gs == 96 else K                                               # (groups end with the rows)
    N = 4608 if gs == 96 else N
    print("case widths at", start, flush=True)
    g = torch.Generator().manual_seed(start)
    x = torch.randn(M * K, generator=g).to(torch.bfloat16).cuda()
    gy = torch.randn(M, N, generator=g).to(torch.bfloat16).cuda()
    G = M * K // gs
    store = torch.zeros(G + start + 4, dtype=torch.uint8, device="cuda:0")
    bits = store[start: start + G]
    bits.copy_(torch.from_numpy(_widths(G, "mixed", start)))
    plan = daf.daf_plan((M, K), gs, bits.clone())
    words = torch.zeros(plan.packed_words, dtype=torch.int32, device="cuda:0")
    mn, sc = torch.empty(G, device="cuda:0"), torch.empty(G, device="cuda:0")
    daf.daf_quantize_pack(plan, x, 5, words, mn, sc)
    ws = torch.empty(max(daf.daf_unpack_matmul_workspace_bytes(plan, N, K), 16), dtype=torch.uint8, device="cuda:0")
    own, given = torch.empty(N, K, device="cuda:0"), torch.empty(N, K, device="cuda:0")
    daf.daf_unpack_matmul_grad_weight(plan, words, mn, sc, gy, own, ws)
    daf.daf_unpack_matmul_grad_weight(plan, words, mn, sc, gy, given, ws, bits=bits)
    torch.cuda.synchronize()
    assert torch.equal(own, given) and bool(own.abs().sum() > 0)
    plan.destroy()


def _widths(G, bits, seed):
    return (np.random.default_rng(seed).choice([1, 2, 4, 8], G).astype(np.uint8) if bits == "mixed"
            else np.array([bits], np.uint8))


# A few tiles more than whole rounds of work-groups (256 per round for the 512 x 128 and the 256 x 256 tile, 512 for 256 x 128,
# 768 for 256 x 64): the tiles of the last round are cut into slices of m, the others are not.  The 16-bit cases take the
# 512 x 128 tile (K = 4160: the last one of a row half outside the output), the binary32 ones the tile of 256 x bk (which
# the workspace is sized by).
@pytest.mark.timeout(300)
@pytest.mark.parametrize("K,bk,bits,dtype", [(4352, 256, "mixed", BF16), (4224, 128, "mixed", F16), (4160, 64, 4, BF16),
                                             (4352, 256, "mixed", F32), (4224, 128, 2, F32), (3136, 64, "mixed", F32)])
def test_grad_weight_sliced_last_round(env, K, bk, bits, dtype):
    daf, orc = env
    M, N = 4096, 4096
    print("case sliced last round", K, bk, bits, dtype, flush=True)
    plan = daf.daf_plan((M, K), 64, 4)
    how = daf.daf_unpack_matmul_schedule(plan, N, K, torch_dtype(dtype))
    plan.destroy()
    assert (how["tile_n"], how["tile_k"]) == ((512, 128) if dtype != F32 else (256, bk))
    assert how["slices"] > 1 and 0 < how["whole_tiles"] < how["tiles"]
    ws = _case(daf, orc, M, N, K, 64, bits, dtype, 17)
    tile_bytes = 256 * bk * 4
    # 16 tiles, each in a few slices (K = 4160: 272 binary32 tiles in 5)
    assert ws > 0 and ws % (16 * tile_bytes) == 0 and ws <= (64 if K != 4160 else 85) * 16 * tile_bytes


def test_grad_weight_argument_errors(env):
    daf, _ = env
    plan = daf.daf_plan((512, 256), 64, 2)
    words = torch.zeros(plan.packed_words, dtype=torch.int32, device="cuda:0")
    mn = torch.zeros(plan.num_groups, device="cuda:0")
    gy = torch.zeros(512, 256, dtype=torch.bfloat16, device="cuda:0")
    out = torch.zeros(256, 256, device="cuda:0")
    assert daf.daf_unpack_matmul_workspace_bytes(plan, 256, 256) > 0
    assert daf.daf_unpack_matmul_workspace_bytes(plan, 100, 256) == -1       # N not a multiple of 64
    assert daf.daf_unpack_matmul_workspace_bytes(plan, 256, 96) == -1        # K does not divide the tensor
    with pytest.raises(daf.DafError) as e:                                    # split, but no workspace
        daf.daf_unpack_matmul_grad_weight(plan, words, mn, mn, gy, out, None)
    assert e.value.status == -1
    plan2 = daf.daf_plan((80, 256), 64, 2)                                    # M not a multiple of 32
    with pytest.raises(daf.DafError) as e:
        daf.daf_unpack_matmul_grad_weight(plan2, words, mn, mn, gy[:80], out, torch.empty(1 << 22, dtype=torch.uint8, device="cuda:0"))
    assert e.value.status == -2


@pytest.mark.parametrize("dtype", [BF16, F16, F32])
@pytest.mark.parametrize("bits", [1, 2, 4, 8, "mixed"])
@pytest.mark.parametrize("K", [384, 192])                                      # 128- and 64-column tiles
def test_identity_gradient_returns_xhat_bit_for_bit(env, dtype, bits, K):
    _identity_case(env, dtype, bits, 256, K)


@pytest.mark.parametrize("dtype,bits", [(BF16, "mixed"), (F16, "mixed"), (BF16, 8), (F16, 2), (F32, "mixed"), (F32, 4)])
def test_identity_gradient_wide_tile(env, dtype, bits):
    _identity_case(env, dtype, bits, 4096, 4096)                               # 256 tiles of 512 x 128 (binary32: 256 x 256)


def _identity_case(env, dtype, bits, M, K):
    """With grad_y = identity every output is a sum with exactly one non-zero term, so
    out[n, k] must equal xhat[n, k] exactly: the dequantization inside the product produces the
    same 16-bit patterns as the oracle's unpack_dequantize (tiny and huge scales included)."""
    daf, orc = env
    N = M
    gs = 32
    print("case identity", dtype, bits, M, K, flush=True)
    g = torch.Generator().manual_seed(5)
    mag = torch.exp(torch.randn(M, K // gs, 1, generator=g) * 6.0)              # group scales over many octaves
    x = (torch.randn(M, K // gs, gs, generator=g) * mag).reshape(M, K).to(torch_dtype(dtype))
    x[torch.isinf(x.float())] = 0
    G = M * K // gs
    b = (np.random.default_rng(1).choice([1, 2, 4, 8], G).astype(np.uint8) if bits == "mixed"
         else np.array([bits], np.uint8))
    ow, omn, osc, _ = orc.quantize_pack(to_numpy_bits(x), dtype, gs, b, 2)
    oxh, _ = orc.unpack_dequantize(ow, omn, osc, b, M * K, gs, dtype)
    finite = np.isfinite(orc.widen(oxh, dtype))
    dbits = torch.from_numpy(b).cuda() if b.size > 1 else None
    plan = daf.daf_plan((M, K), gs, dbits if dbits is not None else int(b[0]))
    ws = torch.empty(max(daf.daf_unpack_matmul_workspace_bytes(plan, N, K), 16), dtype=torch.uint8, device="cuda:0")
    out = torch.empty(N, K, device="cuda:0")
    gy = torch.eye(M, dtype=torch_dtype(dtype), device="cuda:0")
    daf.daf_unpack_matmul_grad_weight(plan, torch.from_numpy(ow.view(np.int32)).cuda(), torch.from_numpy(omn).cuda(),
                                      torch.from_numpy(osc).cuda(), gy, out, ws)
    torch.cuda.synchronize()
    got = out.cpu().numpy().reshape(-1)
    want = orc.widen(oxh, dtype)
    assert finite.all()
    assert np.array_equal((got + np.float32(0)).view(np.uint32), (want + np.float32(0)).view(np.uint32))
    plan.destroy()


@pytest.mark.timeout(600)
@pytest.mark.parametrize("cfg,N", [(5, 4096), (3, 3072)])
def test_grad_weight_at_benchmark_size_sampled(env, cfg, N):
    """The shapes bench.py --fused-matmul times (the LLM MLP activation with per-group widths
    {2,4,8}; the ViT activation with {1,2,4,8}, m in slices): sampled
    outputs against the oracle, which quantizes and dequantizes only the groups those outputs
    read, one group at a time; and every output against the plain dequantize kernel's xhat
    multiplied by the library in binary32 (a property that holds at any size)."""
    from daf_inputs import make_config
    daf, orc = env
    (w,) = make_config(cfg)
    K = w.x.shape[-1]
    M = w.numel // K
    gs, dtype = w.group_size, w.dtype
    gpr = K // gs
    print("case benchmark size", w.name, M, N, K, flush=True)
    g = torch.Generator().manual_seed(100 + cfg)
    gy = (torch.randn(M, N, generator=g) * 0.5).to(torch_dtype(dtype))

    dev = "cuda:0"
    x = w.x.reshape(-1).to(dev)
    dbits = torch.from_numpy(w.bits).to(dev)
    plan = daf.daf_plan((M, K), gs, dbits)
    words = torch.empty(plan.packed_words, dtype=torch.int32, device=dev)
    mn = torch.empty(plan.num_groups, device=dev)
    sc = torch.empty(plan.num_groups, device=dev)
    daf.daf_quantize_pack(plan, x, w.seed, words, mn, sc)
    ws = torch.empty(max(daf.daf_unpack_matmul_workspace_bytes(plan, N, K), 16), dtype=torch.uint8, device=dev)
    out = torch.full((N, K), float("nan"), device=dev)
    gyd = gy.to(dev)
    daf.daf_unpack_matmul_grad_weight(plan, words, mn, sc, gyd, out, ws)
    torch.cuda.synchronize()
    print("ran; oracle on sampled columns", flush=True)

    # ---- sampled outputs: 6 group columns (first, last, 4 random), all their k, 8 values of n ----
    rng = np.random.default_rng(cfg)
    gcols = np.unique(np.concatenate([[0, gpr - 1], rng.integers(0, gpr, 4)]))
    ns = np.unique(np.concatenate([[0, N - 1], rng.integers(0, N, 6)]))
    xb = to_numpy_bits(w.x).reshape(-1)
    off, total = orc.plan(w.numel, gs, w.bits)
    ow = np.zeros(total, dtype=np.uint32)
    omn = np.zeros(plan.num_groups, dtype=np.float32)
    osc = np.zeros(plan.num_groups, dtype=np.float32)
    oxh = np.zeros(w.numel, dtype=xb.dtype)
    for gc in gcols:
        for m in range(M):
            gi = m * gpr + int(gc)
            orc.quantize_pack_range(xb, dtype, gs, w.bits, off, w.seed, gi, gi + 1, ow, omn, osc)
            orc.unpack_dequantize_range(ow, omn, osc, w.bits, off, w.numel, gs, gi, gi + 1, oxh, dtype)
    gy64 = orc.widen(to_numpy_bits(gy), dtype).reshape(M, N)[:, ns].astype(np.float64)         # [M, ns]
    got = out.cpu().numpy()
    for gc in gcols:
        ks = np.arange(int(gc) * gs, (int(gc) + 1) * gs)
        xh64 = orc.widen(oxh, dtype).reshape(M, K)[:, ks].astype(np.float64)                     # [M, gs]
        want = gy64.T @ xh64                                                                      # [ns, gs]
        mag = np.abs(gy64).T @ np.abs(xh64)
        err = np.abs(got[np.ix_(ns, ks)].astype(np.float64) - want)
        bound = 2.0 * M * 2.0 ** -24 * mag + 1e-30
        assert np.all(err <= bound), f"group column {gc}: worst {err.max():.3e}, bound there {bound.flat[err.argmax()]:.3e}"
    print("sampled outputs agree; every output against dequantize + binary32 product", flush=True)

    # ---- every output: the fused kernel against xhat from the plain kernel times grad_y ----
    xh = torch.empty_like(x)
    daf.daf_unpack_dequantize(plan, words, mn, sc, xh)
    ref = torch.zeros(N, K, device=dev)
    mag = torch.zeros(N, K, device=dev)
    step = 4096
    for m0 in range(0, M, step):                       # slabs of m keep the binary32 copies small
        a = gyd[m0:m0 + step].float()
        b = xh.view(M, K)[m0:m0 + step].float()
        ref += a.t() @ b
        mag += a.abs().t() @ b.abs()
    torch.cuda.synchronize()
    # both sides add M products in binary32 in their own order
    assert bool(((out - ref).abs() <= 4.0 * M * 2.0 ** -24 * mag + 1e-30).all())
    plan.destroy()
