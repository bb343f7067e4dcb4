"""GPU parity of the several-tensors-per-call entry points: every tensor of a list must come
out exactly as the oracle (and therefore the single-tensor calls) produce it, whatever mix of
plans the list holds (shared launches, separate launches, remainders after the last tile)."""
import numpy as np
import pytest
import torch

from daf_inputs import BF16, F16, F32, make_config, to_numpy_bits, torch_dtype

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import paper_2507_07149_amd as daf
    from oracle import daf_oracle as orc
    assert torch.cuda.is_available()
    return daf, orc


def _roundtrip(daf, orc, dtype, specs):
    """specs: list of (n, gs, bits) with bits an int or 'mixed'."""
    g = torch.Generator().manual_seed(123 + dtype)
    tensors, q_items, d_items, keep = [], [], [], []
    for i, (n, gs, bits) in enumerate(specs):
        x = (torch.randn(n, generator=g) * (1 + i)).to(torch_dtype(dtype))
        G = (n + gs - 1) // gs
        b = (np.random.default_rng(i).choice([1, 2, 4, 8], G).astype(np.uint8) if bits == "mixed"
             else np.array([bits], np.uint8))
        dbits = torch.from_numpy(b).cuda() if b.size > 1 else None
        plan = daf.daf_plan((n,), gs, dbits if dbits is not None else int(b[0]))
        xd = x.cuda()
        words = torch.full((max(plan.packed_words, 1),), -1, dtype=torch.int32, device="cuda:0")[: plan.packed_words]
        mn = torch.full((G,), float("nan"), device="cuda:0")
        sc = torch.full((G,), float("nan"), device="cuda:0")
        xh = torch.zeros_like(xd)
        tensors.append((x, gs, b, 40 + i, words, mn, sc, xh))
        q_items.append((plan, xd, 40 + i, words, mn, sc))
        d_items.append((plan, words, mn, sc, xh, None))
        keep.append((plan, xd, dbits))
    print("case", dtype, specs, flush=True)
    daf.daf_quantize_pack_batch(q_items)
    daf.daf_unpack_dequantize_batch(d_items)
    torch.cuda.synchronize()
    for i, (x, gs, b, seed, words, mn, sc, xh) in enumerate(tensors):
        ow, omn, osc, _ = orc.quantize_pack(to_numpy_bits(x), dtype, gs, b, seed)
        oxh, _ = orc.unpack_dequantize(ow, omn, osc, b, x.numel(), gs, dtype)
        assert np.array_equal(words.cpu().numpy().view(np.uint32), ow), f"tensor {i}: words differ"
        assert np.array_equal(mn.cpu().numpy().view(np.uint32), omn.view(np.uint32)), f"tensor {i}: min differs"
        assert np.array_equal(sc.cpu().numpy().view(np.uint32), osc.view(np.uint32)), f"tensor {i}: scale differs"
        assert np.array_equal(to_numpy_bits(xh.cpu()).view(oxh.dtype), oxh), f"tensor {i}: xhat differs"
    for plan, _, _ in keep:
        plan.destroy()


@pytest.mark.parametrize("dtype", [F32, F16, BF16])
def test_batch_of_like_tensors_shares_launches(env, dtype):
    daf, orc = env
    _roundtrip(daf, orc, dtype, [(4096 * 3, 256, 2), (4096 * 7, 256, 2), (4096, 256, 2), (4096 * 2 + 256 * 3 + 40, 256, 2)])


@pytest.mark.parametrize("dtype", [F32, F16, BF16])
def test_batch_of_unlike_tensors(env, dtype):
    daf, orc = env
    _roundtrip(daf, orc, dtype, [(4096 * 2, 128, 4), (4096 * 2, 128, 8), (4096 * 3, 64, "mixed"), (4096 * 5 + 64, 64, "mixed"),
                                 (1000, 96, 2), (20000, 8192, 1), (4096 * 2, 128, 4), (33, 32, "mixed")])


@pytest.mark.parametrize("dtype", [F32, F16, BF16])
def test_batch_of_tensors_with_row_sized_groups(env, dtype):
    """Group sizes that are not a power of two share one launch whatever their size, as long as
    the width kind is the same; power-of-two items in between keep their own batches."""
    daf, orc = env
    _roundtrip(daf, orc, dtype, [(768 * 40, 768, 2), (3072 * 9 + 5, 3072, 2), (96 * 100 + 96 * 3, 96, 2), (4096 * 3, 256, 2),
                                 (160 * 77 + 33, 160, 2), (768 * 11, 768, "mixed"), (4064 * 3 + 1500, 4064, "mixed"),
                                 (4096 * 2, 64, "mixed"), (2080 * 7, 2080, 8), (11008 * 3 + 100, 11008, 8)])


@pytest.mark.parametrize("dtype", [F32, BF16])
def test_batch_of_tensors_with_long_groups(env, dtype):
    """Groups of 4128 ... 65536 elements: items with the same number of waves per group and the same
    width kind share a launch; others, and the short last groups, get their own."""
    daf, orc = env
    _roundtrip(daf, orc, dtype, [(11008 * 5, 11008, 2), (11008 * 3 + 700, 11008, 2), (12288 * 2 + 5, 12288, 2), (4128 * 7, 4128, 2),
                                 (8192 * 300, 8192, 2), (4096 * 3, 256, 2), (11008 * 4, 11008, "mixed"), (9600 * 6 + 9000, 9600, "mixed"),
                                 (32736 * 2 + 1, 32736, 8), (768 * 9, 768, 8), (32768 * 3, 32768, 8), (65504 * 2 + 9, 65504, 8),
                                 (40000 * 3, 40000, 2)])


def test_batch_of_many_row_sized_tensors(env):
    daf, orc = env
    _roundtrip(daf, orc, BF16, [(768 * (5 + i % 4), 768 if i % 3 else 3072, 4) for i in range(40)])


def test_batch_longer_than_one_launch(env):
    daf, orc = env
    _roundtrip(daf, orc, F32, [(4096 * (1 + i % 3), 256, 2) for i in range(70)])


@pytest.mark.timeout(400)
def test_batch_resnet18_step_at_full_size(env):
    """The 17 tensors of the ResNet-18 configuration at full size, one call per direction;
    compared with the single-tensor calls (which the full-size parity tests tie to the oracle)."""
    daf, _ = env
    ws = make_config(4, 1.0)
    q_items, d_items, ref = [], [], []
    for w in ws:
        x = w.x.reshape(-1).cuda()
        plan = daf.daf_plan(tuple(w.x.shape), w.group_size, int(w.bits[0]))
        bufs = [torch.empty(plan.packed_words, dtype=torch.int32, device="cuda:0"),
                torch.empty(plan.num_groups, device="cuda:0"), torch.empty(plan.num_groups, device="cuda:0")]
        xh = torch.empty_like(x)
        q_items.append((plan, x, w.seed, *bufs))
        d_items.append((plan, *bufs, xh, None))
        ref.append((plan, x, w.seed, bufs, xh))
    print("case resnet18 step, 17 tensors", flush=True)
    daf.daf_quantize_pack_batch(q_items)
    daf.daf_unpack_dequantize_batch(d_items)
    torch.cuda.synchronize()
    for plan, x, seed, bufs, xh in ref:
        w2, m2, s2 = torch.empty_like(bufs[0]), torch.empty_like(bufs[1]), torch.empty_like(bufs[2])
        daf.daf_quantize_pack(plan, x, seed, w2, m2, s2)
        xh2 = torch.empty_like(xh)
        daf.daf_unpack_dequantize(plan, w2, m2, s2, xh2)
        torch.cuda.synchronize()
        assert torch.equal(w2, bufs[0]) and torch.equal(m2.view(torch.int32), bufs[1].view(torch.int32))
        assert torch.equal(s2.view(torch.int32), bufs[2].view(torch.int32))
        assert torch.equal(xh2.view(torch.int32), xh.view(torch.int32))
        plan.destroy()


def test_batch_argument_errors(env):
    daf, _ = env
    plan = daf.daf_plan((4096,), 256, 2)
    x = torch.zeros(4096 + 1, device="cuda:0")
    words = torch.zeros(plan.packed_words, dtype=torch.int32, device="cuda:0")
    mn = torch.zeros(plan.num_groups, device="cuda:0")
    with pytest.raises(daf.DafError) as e:                       # second item misaligned: nothing is launched
        daf.daf_quantize_pack_batch([(plan, x[:4096], 0, words, mn, mn), (plan, x[1:], 0, words, mn, mn)])
    assert e.value.status == -1
    lib = daf.load_library()
    assert lib.daf_quantize_pack_batch(None, 1, 0, None) == -1
    assert lib.daf_unpack_dequantize_batch(None, 0, 0, None) == -1


@pytest.mark.parametrize("dtype", [F32, F16, BF16])
@pytest.mark.parametrize("bits", [1, 2, 4, 8, "mixed"])
def test_long_groups_and_groups_of_32_dequantize_through_tiles(env, dtype, bits):
    """Groups longer than a tile: a tile inside one group, a group boundary in a tile's first, middle or last chunk,
    a last group of one element, one group for the tensor; groups of 32 elements; tensors that end inside a
    tile.  Each as a call of its own and all in one list call.  By rule the chunk kernel still takes: binary32 with 8
    bits; 1 bit in a 16-bit format up to 2^26 elements (the tile route has a test of its own below); 16-bit groups of 32
    with several widths or in a list."""
    daf, orc = env
    cases = [(8192 * 3, 8192), (8192 * 2 + 4096 + 1, 8192), (40000 * 3 + 8, 40000), (36896 * 4 + 1000, 36896),
             (65536 + 96 + 4096, 65536 + 96), (4096 * 9 + 77, 4096 * 10), (131072 + 1, 131072), (2048 * 5, 32), (2048 * 4 + 40, 32)]
    _roundtrip(daf, orc, dtype, [(n, gs, bits) for n, gs in cases])
    for n, gs in cases:
        print("case", dtype, bits, n, gs, flush=True)
        _roundtrip(daf, orc, dtype, [(n, gs, bits)])
        g = torch.Generator().manual_seed(n)
        x = torch.randn(n, generator=g).to(torch_dtype(dtype))
        G = -(-n // gs)
        b = (np.random.default_rng(n).choice([1, 2, 4, 8], G).astype(np.uint8) if bits == "mixed" else np.array([bits], np.uint8))
        ow, omn, osc, _ = orc.quantize_pack(to_numpy_bits(x), dtype, gs, b, 3)
        plan = daf.daf_plan((n,), gs, torch.from_numpy(b).cuda() if b.size > 1 else int(b[0]))
        if gs == 32:
            route = "chunk" if dtype != F32 and b.size > 1 else "tile"
        else:                                                    # (every other group size here is longer than a tile)
            route = "chunk" if b.size == 1 and b[0] == (8 if dtype == F32 else 1) else "tile_any"
        assert plan.dequantize_route(torch_dtype(dtype)) == route
        out = torch.full_like(x, 7.0, device="cuda:0")
        daf.daf_unpack_dequantize(plan, torch.from_numpy(ow.view(np.int32)).cuda(), torch.from_numpy(omn).cuda(),
                                  torch.from_numpy(osc).cuda(), out)
        want, _ = orc.unpack_dequantize(ow, omn, osc, b, n, gs, dtype)
        assert np.array_equal(to_numpy_bits(out.cpu()), want)
        plan.destroy()


def _xhat_one_bit(words, mn, scale, n, gs, dtype):
    """xhat of a tensor of 1-bit codes: the first code of a word in its most significant bit.  With codes 0 and 1
    fma(code, scale, min) is min + scale rounded once."""
    shift = torch.arange(31, -1, -1, device="cuda:0", dtype=torch.int32)
    lo, hi = mn.to(torch_dtype(dtype)), (mn.double() + scale.double()).float().to(torch_dtype(dtype))
    code = ((words[:, None] >> shift) & 1).bool().view(-1)[:n]
    g = torch.arange(n, device="cuda:0") // gs if mn.numel() > 1 else None
    return torch.where(code, hi if g is None else hi[g], lo if g is None else lo[g])


@pytest.mark.parametrize("dtype,n,gs", [(F16, (1 << 26) + 4096 + 77, 0), (BF16, (1 << 26) + 9, 40000), (F16, (1 << 26), 8192),
                                        (F32, 5 << 23, 40000), (F32, (5 << 23) + 2048 + 5, 0)])
def test_one_bit_long_groups_either_side_of_the_limit(env, dtype, n, gs):
    """1 bit: a 16-bit format takes tiles beyond 2^26 elements only, binary32 up to 5 * 2^23 only."""
    daf, _ = env
    print("case one bit", dtype, n, gs, flush=True)
    gs = gs or -(-n // 32) * 32
    x = torch.randn(n, device="cuda:0").to(torch_dtype(dtype))
    plan = daf.daf_plan((n,), gs, 1)
    words = torch.empty(plan.packed_words, dtype=torch.int32, device="cuda:0")
    mn, sc = torch.empty(plan.num_groups, device="cuda:0"), torch.empty(plan.num_groups, device="cuda:0")
    out = torch.full_like(x, 9.0)
    daf.daf_quantize_pack(plan, x, 3, words, mn, sc)
    daf.daf_unpack_dequantize(plan, words, mn, sc, out)
    assert torch.equal(out, _xhat_one_bit(words, mn, sc, n, gs, dtype))
    plan.destroy()


@pytest.mark.parametrize("sizes", [(9 << 20, 5 << 22, 11 << 20), ((9 << 20) + 7, 5 << 22, (11 << 20) + 12000)])
def test_one_bit_lists_either_side_of_the_limit(env, sizes):
    """binary32 with 1 bit: a list takes tiles up to 5 * 2^23 elements in all."""
    daf, _ = env
    print("case one bit list", sizes, sum(sizes) - (5 << 23), flush=True)
    items, outs = [], []
    for i, n in enumerate(sizes):
        x = torch.randn(n, device="cuda:0")
        plan = daf.daf_plan((n,), 768, 1)
        words = torch.empty(plan.packed_words, dtype=torch.int32, device="cuda:0")
        mn, sc = torch.empty(plan.num_groups, device="cuda:0"), torch.empty(plan.num_groups, device="cuda:0")
        daf.daf_quantize_pack(plan, x, i, words, mn, sc)
        outs.append(torch.full_like(x, 9.0))
        items.append((plan, words, mn, sc, outs[-1], None))
    daf.daf_unpack_dequantize_batch(items)
    for (plan, words, mn, sc, out, _), n in zip(items, sizes):
        assert torch.equal(out, _xhat_one_bit(words, mn, sc, n, 768, F32))
        plan.destroy()


@pytest.mark.parametrize("dtype", [F32, F16])
@pytest.mark.parametrize("bits", [2, 8, "mixed"])
@pytest.mark.parametrize("gs", [128, 96])
def test_list_left_over_chunks(env, dtype, bits, gs):
    """A tensor's chunks after its last whole tile of 512 go to waves of 128: none, one, and the edges of a wave and of a tile
    in one list, with and without elements after the last chunk; then a list without any left over."""
    daf, orc = env
    epl = 4 if dtype == F32 else 8
    print("case left over", dtype, bits, gs, flush=True)
    left = [0, 1, 63, 127, 128, 129, 255, 256, 257, 384, 385, 511]
    _roundtrip(daf, orc, dtype, [((512 * (1 + i % 3) + c) * epl + (i % 2) * 3, gs, bits) for i, c in enumerate(left)])
    _roundtrip(daf, orc, dtype, [(512 * k * epl, gs, bits) for k in (1, 2, 7)])


@pytest.mark.timeout(400)
@pytest.mark.parametrize("gs,bits", [(64, "mixed"), (256, 2)])
def test_binary16_list_above_the_limit_for_four_waves(env, gs, bits):
    """Two tensors of 6 << 11 tiles, one of them with a short one behind, and a third."""
    daf, orc = env
    _roundtrip(daf, orc, F16, [(4096 * (6 << 11), gs, bits), (4096 * (6 << 11) + 2 * gs + 9, gs, bits), (4096 * 3, gs, bits)])


def test_list_of_more_tensors_than_a_launch_takes(env):
    """Forty ragged tensors: two launches per kind, every tensor's short last tile in one of them."""
    daf, orc = env
    _roundtrip(daf, orc, F16, [(4096 * (i % 3) + 8 * i + 8, 64, "mixed") for i in range(40)])
    _roundtrip(daf, orc, F32, [(2048 * (i % 3) + 4 * i + 5, 96, 2) for i in range(40)])


def _per_tensor(daf, orc, dtype, bits, n):
    g = torch.Generator().manual_seed(n)
    x = (torch.randn(n, generator=g) * 3).to(torch_dtype(dtype))
    x[n // 2] = -41.0
    x[-1] = 57.0                                           # the last element holds the maximum: the tail counts
    gs = -(-n // 32) * 32
    b = np.array([bits], np.uint8)
    plan = daf.daf_plan((n,), gs, bits)
    words = torch.full((plan.packed_words,), -1, dtype=torch.int32, device="cuda:0")
    mn, sc = torch.full((1,), float("nan"), device="cuda:0"), torch.full((1,), float("nan"), device="cuda:0")
    xd = x.cuda()
    ow, omn, osc, _ = orc.quantize_pack(to_numpy_bits(x), dtype, gs, b, 77)
    for call in (daf.daf_quantize_pack, daf.daf_quantize_pack_static):
        words.fill_(-1)
        call(plan, xd, 77, words, mn, sc)
        torch.cuda.synchronize()
        assert np.array_equal(words.cpu().numpy().view(np.uint32), ow), n
        assert np.array_equal(mn.cpu().numpy().view(np.uint32), omn.view(np.uint32))
        assert np.array_equal(sc.cpu().numpy().view(np.uint32), osc.view(np.uint32))
    plan.destroy()


@pytest.mark.parametrize("dtype", [F32, F16, BF16])
@pytest.mark.parametrize("bits", [1, 2, 4, 8])
def test_one_group_per_tensor_at_tile_and_workgroup_edges(env, dtype, bits):
    """Around one tile, four tiles (a workgroup of the quantize pass) and eight (one of the statistics pass)."""
    daf, orc = env
    print("case per tensor", dtype, bits, flush=True)
    for n in (31, 4095, 4096, 4097, 4096 * 3 + 4095, 4096 * 4, 4096 * 5 + 33, 4096 * 8 - 1, 4096 * 8, 4096 * 9 + 2, 4096 * 33 + 4000):
        _per_tensor(daf, orc, dtype, bits, n)


@pytest.mark.parametrize("n", [2048 * 8 * 4096, 2048 * 8 * 4096 + 1])
def test_one_group_per_tensor_at_the_limit_of_the_folded_reduction(env, n):
    daf, orc = env
    print("case per tensor limit", n, flush=True)
    _per_tensor(daf, orc, BF16, 2, n)
