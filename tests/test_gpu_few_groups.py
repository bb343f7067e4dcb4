"""Width selection and plan scan in their one-launch forms, around the sizes where their workgroups, loads and forms change,
against the oracle: ties, equal ranges, widths replaced in place, widths outside the classes, unaligned widths."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import paper_2507_07149_amd as daf
    from oracle import daf_oracle as orc
    assert torch.cuda.is_available()
    return daf, orc


@pytest.mark.parametrize("G", [1, 31, 32, 33, 63, 64, 65, 1023, 1024, 1025, 8191, 8192, 8193, 15359, 15360, 15361, 16351, 16383, 16384, 16385])
@pytest.mark.parametrize("kind", ["random", "ties", "equal", "sorted"])
@pytest.mark.parametrize("classes", [(1, 2, 4, 8), (2, 4, 8), (4, 8), (2,)])
def test_select_bits(env, G, kind, classes):
    daf, orc = env
    rng = np.random.default_rng(G)
    lo = rng.standard_normal(G).astype(np.float32)
    span = {"random": rng.random(G, dtype=np.float32), "ties": rng.choice(np.array([0.0, 0.5, 0.5, 2.0], np.float32), G),
            "equal": np.ones(G, np.float32), "sorted": np.linspace(3, 0, G, dtype=np.float32)}[kind]
    lo = lo if kind == "random" else np.zeros(G, np.float32)
    hi = lo + span
    ws = daf.daf_select_bits_workspace(G)
    whole = torch.full((G + 64,), 77, dtype=torch.uint8, device="cuda:0")
    print("case", G, kind, classes, flush=True)
    daf.daf_select_bits(torch.from_numpy(lo).cuda(), torch.from_numpy(hi).cuda(), classes, whole[:G], ws)
    want = orc.select_bits(lo, hi, classes)
    assert np.array_equal(whole[:G].cpu().numpy(), want)
    assert bool((whole[G:] == 77).all())
    prev = rng.choice([1, 2, 4, 8], G).astype(np.uint8)
    scale = span / ((1 << prev.astype(np.int64)) - 1).astype(np.float32)
    want = orc.select_bits(np.zeros(G, np.float32), scale * ((1 << prev.astype(np.int64)) - 1).astype(np.float32), classes)
    bits = torch.from_numpy(prev).cuda()
    daf.daf_select_bits_from_scale(torch.from_numpy(scale).cuda(), bits, classes, whole[:G], ws)
    assert np.array_equal(whole[:G].cpu().numpy(), want)
    daf.daf_select_bits_from_scale(torch.from_numpy(scale).cuda(), bits, classes, bits, ws)           # in place
    assert np.array_equal(bits.cpu().numpy(), want)


@pytest.mark.parametrize("G", [33, 8192, 8193, 16384])
@pytest.mark.parametrize("over", ["min", "max", "scale", "scale, one width"])
def test_select_bits_over_an_input(env, G, over):
    """The widths may be written over the statistics that they come from."""
    daf, orc = env
    rng = np.random.default_rng(G)
    lo, span = rng.standard_normal(G).astype(np.float32), rng.random(G, dtype=np.float32)
    prev = rng.choice([1, 2, 4, 8], G).astype(np.uint8) if over == "scale" else np.full(G, 2, np.uint8)
    ws = daf.daf_select_bits_workspace(G)
    print("case", G, over, flush=True)
    if over in ("min", "max"):
        hi = lo + span
        a, b = torch.from_numpy(lo).cuda(), torch.from_numpy(hi).cuda()
        out = (a if over == "min" else b).view(torch.uint8)[:G]
        daf.daf_select_bits(a, b, (2, 4, 8), out, ws)
        want = orc.select_bits(lo, hi, (2, 4, 8))
    else:
        a = torch.from_numpy(span).cuda()
        out = a.view(torch.uint8)[3 * G:]
        daf.daf_select_bits_from_scale(a, torch.from_numpy(prev).cuda() if over == "scale" else 2, (2, 4, 8), out, ws)
        want = orc.select_bits(np.zeros(G, np.float32), span * ((1 << prev.astype(np.int64)) - 1).astype(np.float32), (2, 4, 8))
    assert np.array_equal(out.cpu().numpy(), want)


@pytest.mark.parametrize("G", [2, 8, 8191, 8192, 8193, 16384, 16391, 65533, 65536, 65537, 200003])
@pytest.mark.parametrize("skew", [0, 4, 1])
@pytest.mark.parametrize("bad", [None, "first", "last"])
def test_plan_scan(env, G, skew, bad):
    """`skew`: the widths start so many bytes past a 16-byte boundary; `bad`: one width that is none."""
    daf, orc = env
    gs, n = 96, G * 96 - 37
    rng = np.random.default_rng(G + skew)
    b = rng.choice([1, 2, 4, 8], G).astype(np.uint8)
    whole = torch.zeros(G + 32, dtype=torch.uint8, device="cuda:0")
    start = (-whole.data_ptr()) % 16 + skew
    print("case", G, skew, bad, flush=True)
    plan = daf.daf_plan((n,), gs, torch.from_numpy(np.ones(G, np.uint8)).cuda())
    if bad:
        b[0 if bad == "first" else G - 1] = (0, 3, 16, 255)[G % 4]
    whole[start: start + G] = torch.from_numpy(b).cuda()
    plan.update(whole[start: start + G])
    if bad:
        with pytest.raises(daf.DafError):
            plan.finish()
    else:
        plan.finish()
        off, total = orc.plan(n, gs, b)
        assert plan.packed_words == total
        assert np.array_equal(plan.offsets().numpy().view(np.uint32), off)
    plan.destroy()
