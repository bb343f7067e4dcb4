"""Width updates and width selection whose workgroups tell each other their sums inside one launch, around the numbers of groups
where a workgroup ends and the forms change, against the oracle: called again and again on one plan and one workspace, with every
workgroup left to work the others' sums out for itself (no look at the posts), and replayed from a graph."""
import ctypes

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
# one round of 4096 groups to a workgroup, two (from 5 << 18), four (from 13 << 18)
GROUPS = [14337, 4096 * 4, 32769, 65536, 65537, 4096 * 17 - 1, 4096 * 17, 4096 * 17 + 1, (1 << 20) - 7, (1 << 20) + 1, 8192 * 200 + 5, (13 << 18) + 4096 + 3]


@pytest.fixture(scope="module")
def env():
    import paper_2507_07149_amd as daf
    from oracle import daf_oracle as orc
    assert torch.cuda.is_available()
    return daf, orc, daf.load_library()


def _stream():
    return ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)


def _update(lib, plan, bits, polls):
    return lib.daf_internal_plan_update(ctypes.c_void_p(plan.handle),
                                        ctypes.c_void_p(bits.data_ptr()), polls, _stream())


@pytest.mark.parametrize("G", GROUPS)
@pytest.mark.parametrize("skew", [0, 3])
def test_update(env, G, skew):
    daf, orc, lib = env
    gs, n = 64, G * 64 - 37
    rng = np.random.default_rng(G)
    plan = daf.daf_plan((n,), gs, torch.ones(G, dtype=torch.uint8, device="cuda:0"))
    # a wrong width (reported, and counted as 8): in the first workgroup with no look at its post, and in the middle
    for polls, wrong in [(256, None), (0, 5), (0, None), (256, G // 2), (1, None), (0, G - 1), (256, None)]:
        b = rng.choice([1, 2, 4, 8], G).astype(np.uint8)
        if wrong is not None:
            b[wrong] = 3
        whole = torch.zeros(G + 32, dtype=torch.uint8, device="cuda:0")
        whole[skew: skew + G] = torch.from_numpy(b).cuda()
        print("case", G, skew, polls, wrong, flush=True)
        assert _update(lib, plan, whole[skew: skew + G], polls) == 0
        assert lib.daf_plan_finish(ctypes.c_void_p(plan.handle), _stream()) == (0 if wrong is None else -1)
        b[b == 3] = 8
        off, total = orc.plan(n, gs, b)
        assert lib.daf_plan_packed_words(ctypes.c_void_p(plan.handle)) == total
        assert np.array_equal(plan.offsets().numpy().view(np.uint32), off)
    plan.destroy()


@pytest.mark.parametrize("G", [4096 * 21 + 9, (5 << 18) + 9, (13 << 18) + 9])
def test_update_replayed(env, G):
    daf, orc, _ = env
    gs = 32
    rng = np.random.default_rng(5)
    bits = torch.from_numpy(rng.choice([1, 2, 4, 8], G).astype(np.uint8)).cuda()
    plan = daf.daf_plan((G * gs,), gs, bits)
    plan.update(bits)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        plan.update(bits)
    for i in range(6):
        b = rng.choice([1, 2, 4, 8], G).astype(np.uint8)
        bits.copy_(torch.from_numpy(b))
        graph.replay()
        if i % 2:
            torch.cuda.synchronize()
            plan.update(bits)
        torch.cuda.synchronize()
        assert np.array_equal(plan.offsets().numpy().view(np.uint32), orc.plan(G * gs, gs, b)[0])
    plan.destroy()


@pytest.mark.parametrize("G", [14337, 65537, 4096 * 40 + 3, (13 << 18) + 77])
def test_update_after_overlapping_updates(env, G):
    """Updates of one plan that overlap give no defined offsets (equal widths: the right ones), but leave nothing behind: the next
    update alone is right."""
    daf, orc, _ = env
    gs = 32
    rng = np.random.default_rng(G)
    host = [rng.choice([1, 2, 4, 8], G).astype(np.uint8) for _ in range(3)]
    bits = [torch.from_numpy(b).cuda() for b in host]
    want = [orc.plan(G * gs, gs, b)[0] for b in host]
    plan = daf.daf_plan((G * gs,), gs, bits[0])
    streams = [torch.cuda.Stream() for _ in range(3)]
    torch.cuda.synchronize()
    for same in (False, True):
        print("case", G, same, flush=True)
        for i in range(60):
            for k, s in enumerate(streams):
                plan.update(bits[1 if same else (i + k) % 3], stream=s)
            if i % 10 == 9:
                torch.cuda.synchronize()
                if same:
                    assert np.array_equal(plan.offsets().numpy().view(np.uint32), want[1])
                for k in (0, 2):
                    plan.update(bits[k])
                    torch.cuda.synchronize()
                    assert np.array_equal(plan.offsets().numpy().view(np.uint32), want[k]), (same, i, k)
    plan.destroy()


@pytest.mark.parametrize("G", [16385, 4096 * 5 - 1, 4096 * 5 + 1, 197000, 1500001, (7 << 18) + 8192 + 3])
@pytest.mark.parametrize("kind", ["random", "ties", "equal", "half zero"])
@pytest.mark.parametrize("polls", [256, 0])
def test_select(env, G, kind, polls):
    daf, orc, lib = env
    rng = np.random.default_rng(G)
    hi = {"random": rng.random(G, dtype=np.float32), "ties": rng.choice(np.array([0.0, 0.5, 0.5, 2.0], np.float32), G),
          "equal": np.ones(G, np.float32), "half zero": np.maximum(rng.standard_normal(G), 0).astype(np.float32)}[kind]
    lo = np.zeros(G, np.float32)
    ws = daf.daf_select_bits_workspace(G)
    out = torch.full((G + 64,), 77, dtype=torch.uint8, device="cuda:0")
    a, b = torch.from_numpy(lo).cuda(), torch.from_numpy(hi).cuda()
    for classes in ((1, 2, 4, 8), (2, 8)):
        print("case", G, kind, polls, classes, flush=True)
        assert lib.daf_internal_select_bits(ctypes.c_void_p(a.data_ptr()), ctypes.c_void_p(b.data_ptr()), ctypes.c_int64(G),
                                            (ctypes.c_uint8 * len(classes))(*classes), len(classes), ctypes.c_void_p(out.data_ptr()),
                                            ctypes.c_void_p(ws.data_ptr()), polls, _stream()) == 0
        assert np.array_equal(out[:G].cpu().numpy(), orc.select_bits(lo, hi, classes))
        assert bool((out[G:] == 77).all())
