"""The tile in which a tensor ends: every length around its edges, through every call that has such a tile (quantize, the
same with metrics, with relu in and out of place, in a list; group statistics), against the oracle bit for bit, and
nothing written behind the outputs."""
import numpy as np
import pytest
import torch

from daf_inputs import BF16, F16, F32, to_numpy_bits, torch_dtype

pytestmark = pytest.mark.gpu
GUARD = 64


def _guarded(n, dtype, fill):
    whole = torch.full((n + GUARD,), fill, dtype=dtype, device="cuda:0")
    return whole, whole[:n]


def _packed(plan):
    return [_guarded(plan.packed_words, torch.int32, -1), _guarded(plan.num_groups, torch.float32, 7.0),
            _guarded(plan.num_groups, torch.float32, 7.0)]


def _check_packed(bufs, want, what):
    for (whole, part), ref, fill, name in zip(bufs, want, (-1, 7.0, 7.0), ("words", "min", "scale")):
        got = part.cpu().numpy().view(np.uint32)
        assert np.array_equal(got, ref.view(np.uint32)), (what, name, np.nonzero(got != ref.view(np.uint32))[0][:4])
        assert bool((whole[part.numel():] == fill).all()), (what, name, "written behind its end")


@pytest.mark.parametrize("dtype", [F32, F16, BF16])
@pytest.mark.parametrize("gs", [32, 64, 256, 1024, 2048, 4096, 96, 768, 3072])
@pytest.mark.parametrize("bits", [1, 2, 4, 8, "mixed"])
def test_every_end(dtype, gs, bits):
    import paper_2507_07149_amd as daf
    from oracle import daf_oracle as orc
    tile = 4096 if gs & (gs - 1) == 0 else 4096 // gs * gs
    if dtype == F32 and gs <= 1024:
        tile = 1024
    per_load = 4 if dtype == F32 else 8
    ends = {1, per_load - 1, per_load, per_load + 1, 31, 33, gs - 1, gs, gs + 1, 2 * gs + 17, tile - gs - 1, tile - 1, tile - gs}
    lengths = sorted({base + e for e in ends if 0 < e < tile for base in (0, tile, 5 * tile) if base + e >= gs})
    rng = np.random.default_rng(gs + 11 * dtype)
    items, checks, plans = [], [], []
    for n in lengths:
        print("case", dtype, gs, bits, n, flush=True)
        x = (torch.randn(n, generator=torch.Generator().manual_seed(n)) * 2).to(torch_dtype(dtype))
        x[-1] = (9.0, -9.0, 0.0)[n % 3]                     # the last element decides the short group's range, or not
        G = -(-n // gs)
        b = rng.choice([1, 2, 4, 8], G).astype(np.uint8) if bits == "mixed" else np.array([bits], np.uint8)
        xd = x.cuda()
        plan = daf.daf_plan((n,), gs, torch.from_numpy(b).cuda() if bits == "mixed" else int(bits))
        xb = to_numpy_bits(x)
        ow, omn, osc, codes = orc.quantize_pack(xb, dtype, gs, b, 77, want_codes=True)

        bufs = _packed(plan)
        daf.daf_quantize_pack(plan, xd, 77, *(p for _, p in bufs))
        _check_packed(bufs, (ow, omn, osc), "quantize")

        bufs = _packed(plan)
        met_all, met = _guarded(3 * G, torch.float32, 5.0)
        daf.daf_quantize_pack_metrics(plan, xd, 77, *(p for _, p in bufs), met)
        _check_packed(bufs, (ow, omn, osc), "metrics")
        got = met.cpu().numpy().reshape(G, 3)
        want = np.concatenate([orc.group_metrics(xb, dtype, gs, codes, omn, osc).reshape(G, 2),
                               orc.group_variance(xb, dtype, gs, b).reshape(G, 1)], axis=1)
        # the variance: an exact integer times scale^2; the sums: binary32 over at most 4096 terms, in any order
        assert np.allclose(got, want, rtol=4096 * 2.0 ** -24, atol=1e-30), (n, np.abs(got - want).max())
        assert bool((met_all[3 * G:] == 5.0).all()), "metrics written behind their end"

        oy = orc.relu(xb, dtype)
        want_relu = orc.quantize_pack(oy, dtype, gs, b, 78)[:3]
        for in_place in (False, True):
            z_all, z = _guarded(n, xd.dtype, -3.0)
            z.copy_(xd)
            y_all, y = (z_all, z) if in_place else _guarded(n, xd.dtype, -3.0)
            bufs = _packed(plan)
            daf.daf_relu_quantize_pack(plan, z, 78, y, *(p for _, p in bufs))
            _check_packed(bufs, want_relu, "relu")
            assert np.array_equal(to_numpy_bits(y.cpu()).view(oy.dtype), oy), (n, "y")
            assert bool((y_all[n:] == -3.0).all()), "y written behind its end"

        (lo_all, lo), (hi_all, hi) = _guarded(G, torch.float32, 7.0), _guarded(G, torch.float32, 7.0)
        daf.daf_group_minmax(plan, xd, lo, hi)
        olo, ohi = orc.group_minmax(xb, dtype, gs)
        assert np.array_equal(lo.cpu().numpy().view(np.uint32), olo.view(np.uint32))
        assert np.array_equal(hi.cpu().numpy().view(np.uint32), ohi.view(np.uint32))
        assert bool((lo_all[G:] == 7.0).all() and (hi_all[G:] == 7.0).all())

        bufs = _packed(plan)
        items.append((plan, xd, 77, *(p for _, p in bufs)))
        checks.append((bufs, (ow, omn, osc)))
        plans.append(plan)
    daf.daf_quantize_pack_batch(items)
    for bufs, want in checks:
        _check_packed(bufs, want, "list")
    for plan in plans:
        plan.destroy()


@pytest.mark.parametrize("dtype", [F32, F16, BF16])
@pytest.mark.parametrize("gs", [32, 64, 256, 2048, 4096])
def test_statistics_of_ends_around_the_parts_that_waves_take(dtype, gs):
    """The statistics of such a tile are taken by up to four waves, 1024 elements each."""
    import paper_2507_07149_amd as daf
    from oracle import daf_oracle as orc
    for n in sorted({base + 1024 * part + d for base in (4096, 8192) for part in range(4) for d in (-1, 0, 1, 7, 9)}):
        print("case", dtype, gs, n, flush=True)
        x = (torch.randn(n, generator=torch.Generator().manual_seed(n)) * 2).to(torch_dtype(dtype))
        x[-1] = (9.0, -9.0, 0.0)[n % 3]
        G = -(-n // gs)
        plan = daf.daf_plan((n,), gs, 2)
        (lo_all, lo), (hi_all, hi) = _guarded(G, torch.float32, 7.0), _guarded(G, torch.float32, 7.0)
        daf.daf_group_minmax(plan, x.cuda(), lo, hi)
        olo, ohi = orc.group_minmax(to_numpy_bits(x), dtype, gs)
        assert np.array_equal(lo.cpu().numpy().view(np.uint32), olo.view(np.uint32))
        assert np.array_equal(hi.cpu().numpy().view(np.uint32), ohi.view(np.uint32))
        assert bool((lo_all[G:] == 7.0).all() and (hi_all[G:] == 7.0).all())
        plan.destroy()
