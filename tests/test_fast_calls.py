"""The native step of the inner loop's calls (csrc/fast_calls.cpp): it takes the usual arguments, and leaves everything else to the
general checks without having done anything."""
import os
import subprocess
import types

import pytest
import torch

import paper_2507_07149_amd as daf
from paper_2507_07149_amd import binding, build


needs_the_module = pytest.mark.skipif(binding._fast_calls is None, reason="the module does not compile here (test_the_module_is_built)")


class Tagged(torch.Tensor):
    pass


def _case(device):
    n, gs = 8192, 128
    G = n // gs
    t = {"x": torch.randn(n, device=device), "y": torch.empty(n, device=device), "bits": torch.full((G,), 4, dtype=torch.uint8, device=device),
         "next": torch.empty(G, dtype=torch.uint8, device=device), "words": torch.zeros(n // 4, dtype=torch.int32, device=device),
         "min": torch.empty(G, device=device), "scale": torch.empty(G, device=device), "metrics": torch.empty(3 * G, device=device),
         "lo": torch.empty(G, device=device), "hi": torch.empty(G, device=device), "ws": daf.daf_select_bits_workspace(G, device)}
    plan = daf.daf_plan((n,), gs, t["bits"] if device != "cpu" else 4)
    calls = {
        "quantize_pack": [plan, "x", 3, "words", "min", "scale", None],
        "quantize_pack_static": [plan, "x", 3, "words", "min", "scale", None],
        "unpack_dequantize": [plan, "words", "min", "scale", "y", None, None],
        "quantize_pack_metrics": [plan, "x", 3, "words", "min", "scale", "metrics", None],
        "relu_quantize_pack": [plan, "x", 3, "y", "words", "min", "scale", None],
        "unpack_relu_backward": [plan, "words", "min", "scale", "x", "y", "bits", None],
        "group_minmax": [plan, "x", "lo", "hi", None],
        "select_bits": ["lo", "hi", (2, 4, 8), "next", "ws", None],
        "select_bits_from_scale": ["scale", "bits", [2, 4, 8], "next", "ws", None],
        "plan_update": [plan, "bits", None],
    }
    return plan, t, calls


def _call(name, args, t, **other):
    return getattr(binding._fast_calls, name)(*[other.get(a, t.get(a)) if isinstance(a, str) else a for a in args])


def test_the_module_is_built():
    if not os.path.exists(build.FAST_CALLS):
        try:
            build._compile_fast_calls()
        except (ImportError, OSError, subprocess.CalledProcessError) as e:
            pytest.skip(f"does not compile here: {e}")
    assert binding._fast_calls is not None and binding._fast is binding._fast_calls


def test_the_library_is_linked_where_the_module_does_not_compile(monkeypatch, tmp_path, capsys):
    steps = []
    stale = tmp_path / "_fast_calls.so"
    stale.write_bytes(b"")
    monkeypatch.setattr(build, "HERE", str(tmp_path))
    monkeypatch.setattr(build, "OBJ", str(tmp_path / "obj"))
    monkeypatch.setattr(build, "_compile", lambda item: item[1])

    def run(command, **other):
        steps.append(command[0])
        if command[0] == "g++":
            raise subprocess.CalledProcessError(1, command)
    monkeypatch.setattr(build.subprocess, "run", run)
    assert build.build() == build.LIB
    assert sorted(steps) == sorted(["g++", build.HIPCC]) and not stale.exists()
    assert "was not built" in capsys.readouterr().err


def test_a_module_of_another_torch_is_not_used():
    assert binding._of_this_torch(types.SimpleNamespace(torch_version=torch.__version__)) is not None
    for other in (types.SimpleNamespace(torch_version="1.0"), types.SimpleNamespace(), None):
        assert binding._of_this_torch(other) is None
    assert binding._fast_calls is None or binding._fast_calls.torch_version == torch.__version__


PUBLIC = {"group_minmax": "daf_group_minmax", "quantize_pack": "daf_quantize_pack", "quantize_pack_static": "daf_quantize_pack_static",
          "quantize_pack_metrics": "daf_quantize_pack_metrics", "relu_quantize_pack": "daf_relu_quantize_pack",
          "unpack_dequantize": "daf_unpack_dequantize", "unpack_relu_backward": "daf_unpack_relu_backward",
          "select_bits": "daf_select_bits", "select_bits_from_scale": "daf_select_bits_from_scale"}


def _public_call(name, args, t):
    plan, args = args[0], [t.get(a) if isinstance(a, str) else a for a in args]
    (plan.update if name == "plan_update" else getattr(daf, PUBLIC[name]))(*(args[1:] if name == "plan_update" else args))


def test_without_the_module_the_general_checks_refuse(monkeypatch):
    monkeypatch.setattr(binding, "_fast", binding._NoFastCalls())
    plan, t, calls = _case("cpu")
    for name, args in calls.items():
        with pytest.raises(ValueError):
            _public_call(name, args, t)
    plan.destroy()


@pytest.mark.gpu
def test_without_the_module_every_call_does_the_same(monkeypatch):
    plan, t, calls = _case("cuda:0")
    torch.manual_seed(0)
    t["x"].copy_(torch.randn(t["x"].numel()))
    order = ("group_minmax", "select_bits", "quantize_pack", "quantize_pack_static", "quantize_pack_metrics", "unpack_dequantize",
             "unpack_relu_backward", "relu_quantize_pack", "select_bits_from_scale", "plan_update")
    assert set(order) == set(calls)
    seen = []
    for fast in (binding._fast, binding._NoFastCalls()):
        monkeypatch.setattr(binding, "_fast", fast)
        for key in set(t) - {"x", "bits", "ws"}:
            t[key].zero_()
        for name in order:
            _public_call(name, calls[name], t)
            torch.cuda.synchronize()
            seen.append({k: v.clone() for k, v in t.items() if k != "ws"})
    n = len(order)
    for name, a, b in zip(order, seen[:n], seen[n:]):
        assert all(torch.equal(a[k], b[k]) for k in a), name
    plan.destroy()


@needs_the_module
def test_host_tensors_are_left_to_the_general_checks():
    plan, t, calls = _case("cpu")
    for name, args in calls.items():
        assert _call(name, args, t) is None, name
    plan.destroy()
    assert _call("quantize_pack", calls["quantize_pack"], t) is None


@needs_the_module
@pytest.mark.gpu
def test_usual_arguments_are_taken_and_others_left():
    plan, t, calls = _case("cuda:0")
    for name, args in calls.items():
        assert _call(name, args, t) == 0, name
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    assert _call("quantize_pack", calls["quantize_pack"][:-1] + [side], t) == 0
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    want = [t[k].clone() for k in ("words", "min", "scale")]
    binding._general_quantize_pack(plan, t["x"], 3, t["words"].zero_(), t["min"], t["scale"], None)
    assert all(torch.equal(a, t[k]) for a, k in zip(want, ("words", "min", "scale")))
    for name, args in calls.items():
        for i, a in enumerate(args):
            if not isinstance(a, str):
                continue
            good = t[a]
            for bad in (good.cpu(), good[:-1], torch.stack([good, good], 1)[:, 0], good.view(torch.int16), good.as_subclass(Tagged), [0], None):
                if (bad is None and a == "bits") or (a == "words" and bad is not None and getattr(bad, "is_cuda", False)
                                                     and type(bad) is torch.Tensor and bad.dtype == torch.int32 and bad.is_contiguous()):
                    continue                                         # (the words' buffer is larger than it has to be)
                if a == "lo" and name == "select_bits" and bad is not None and getattr(bad, "is_cuda", False) and len(bad) == len(good) - 1:
                    continue                                         # (there the first argument says how many groups; the second differs then)
                assert getattr(binding._fast_calls, name)(*[bad if j == i else t.get(b) if isinstance(b, str) else b
                                                            for j, b in enumerate(args)]) is None, (name, a, type(bad))
    assert binding._fast_calls.quantize_pack(plan, t["x"], 3.0, t["words"], t["min"], t["scale"], None) is None
    assert binding._fast_calls.quantize_pack(object(), t["x"], 3, t["words"], t["min"], t["scale"], None) is None
    assert binding._fast_calls.quantize_pack(plan, t["x"], 3) is None

    seen = []

    def traced(x):
        seen.append(binding._fast_calls.quantize_pack(plan, x, 3, t["words"], t["min"], t["scale"], None))
        return x
    torch.vmap(traced)(t["x"].unsqueeze(0))
    assert seen == [None]
    torch.cuda.synchronize()
    plan.destroy()


@needs_the_module
@pytest.mark.gpu
def test_operands_of_products_that_are_taken_and_left():
    """The linear layer and the weight gradient: shapes, sizes taken from the operands and the workspace's bytes."""
    m, k, n, gs = 4096, 128, 256, 64
    fast, dev = binding._fast_calls, "cuda:0"
    full = lambda *shape, dtype=torch.bfloat16: torch.zeros(shape, dtype=dtype, device=dev)
    y_plan, x_plan = daf.daf_plan((m, n), gs, 4), daf.daf_plan((m, k), gs, 4)

    def packed(plan):
        return [full(plan.packed_words, dtype=torch.int32), full(plan.num_groups, dtype=torch.float32), full(plan.num_groups, dtype=torch.float32)]
    linear = [y_plan, full(m, k), full(n, k), 3, full(m, n), *packed(y_plan), None]
    need = daf.daf_unpack_matmul_workspace_bytes(x_plan, n, k)
    assert need >= 16
    grad = [x_plan, *packed(x_plan), full(m, n), full(n, k, dtype=torch.float32), full(need, dtype=torch.uint8), None, None]

    def left(call, args, i, *bad):
        for b in bad:
            assert call(*args[:i], b, *args[i + 1:]) is None, (call.__name__, i, getattr(b, "shape", b))
    assert fast.linear_quantize_pack(*linear) == 0 and fast.unpack_matmul_grad_weight(*grad) == 0
    assert fast.unpack_matmul_grad_weight(*grad[:6], full(need // 4, dtype=torch.float32), None, None) == 0
    for i in (1, 2, 4, 5, 6, 7):
        left(fast.linear_quantize_pack, linear, i, None, [0], linear[i].cpu(), linear[i][:-1], linear[i].double(), linear[i].as_subclass(Tagged))
    left(fast.linear_quantize_pack, linear, 1, full(m, 2 * k), full(m * k), full(1, m, k), full(k, m).t(), full(m, 2 * k)[:, :k],
         full(m, k, dtype=torch.float16), full(m, k, dtype=torch.int16))
    left(fast.linear_quantize_pack, linear, 2, full(n, 2 * k), full(n * k), full(k, n).t(), full(2 * n, k), full(n, k, dtype=torch.float16))
    left(fast.linear_quantize_pack, linear, 4, full(m, n, dtype=torch.float16), full(n, m).t())
    left(fast.linear_quantize_pack, linear, 0, x_plan, None)
    for i in (1, 2, 3, 4, 5, 6):
        left(fast.unpack_matmul_grad_weight, grad, i, [0], grad[i].cpu(), grad[i][:-1], grad[i].as_subclass(Tagged))
    for i in (1, 2, 3, 4, 5):
        left(fast.unpack_matmul_grad_weight, grad, i, None)
    left(fast.unpack_matmul_grad_weight, grad, 4, full(m, n // 2), full(m // 2, n), full(m * n), full(n, m).t(), full(m, n, dtype=torch.float64))
    left(fast.unpack_matmul_grad_weight, grad, 5, full(n, k), full(n * k, dtype=torch.float32), full(2 * n, k, dtype=torch.float32),
         full(n, k // 2, dtype=torch.float32), full(n, 2 * k, dtype=torch.float32), full(k, n, dtype=torch.float32).t())
    left(fast.unpack_matmul_grad_weight, grad, 6, full(need // 4 - 1, dtype=torch.float32), full(2 * need, dtype=torch.uint8)[::2])
    left(fast.unpack_matmul_grad_weight, grad, 7, full(x_plan.num_groups - 1, dtype=torch.uint8), full(x_plan.num_groups, dtype=torch.int32))
    left(fast.unpack_matmul_grad_weight, grad, 0, y_plan, None)
    torch.cuda.synchronize()
    for plan in (x_plan, y_plan):
        plan.destroy()
        assert fast.linear_quantize_pack(plan, *linear[1:]) is None and fast.unpack_matmul_grad_weight(plan, *grad[1:]) is None
