"""What a training program has this library do, as cases that can be timed and compared.

Every case goes through the public entry points of `paper_2507_07149_amd`, with buffers and plans
that a training loop allocates once and keeps.  Shapes and value distributions are those of the
repository's five benchmark configurations (a small convolution activation, a ResNet-50 convolution, a
ViT/BERT activation, the 17 activations of a ResNet-18 step, an LLM MLP activation) and of its tests;
`draw` gives further sizes, group sizes, widths and element formats of the same ranges.

Kinds of case
  tensor      save one activation and restore it: quantize+pack, then unpack+dequantize
  resnet      the same for the activations of a ResNet-18 step, one list call per direction
  vit         the same for the activations of some transformer layers, rows as groups
  relu        a layer whose activation function is fused: relu+quantize+pack in the forward pass,
              relu's backward from the packed words
  controller  one iteration with widths chosen on the device: statistics, widths, plan, quantize+pack
  metrics     the same with the importance metrics and the widths for the next iteration
              taken from the scales of this one
  linear      forward pass of a linear layer with the output saved in its epilogue
  wgrad       weight gradient of a linear layer from its packed input
"""
import math

import torch

import paper_2507_07149_amd as daf

DTYPES = {"float32": torch.float32, "float16": torch.float16, "bfloat16": torch.bfloat16}
BYTES = {"float32": 4, "float16": 2, "bfloat16": 2}


def _case(kind, dtype, values, group, widths, **sizes):
    return {"kind": kind, "dtype": dtype, "values": values, "group": group, "widths": widths, **sizes}


def listed():
    """`group` 0: one group for the whole tensor.  `widths`: one number = all groups, several = per-group widths by
    rank of the group's range."""
    named = {
        # the smallest call of a step (a CIFAR-size convolution activation): launches and host work count
        "tiny_f32": _case("tensor", "float32", "relu", 128, "2", rows=4 * 64 * 32, cols=32),
        # a ResNet-50 activation at batch 64 whose relu is fused, forward and backward
        "conv_relu_f32": _case("relu", "float32", "signed", 256, "2", rows=64 * 256, cols=56 * 56),
        # the paper's own granularity, one minimum and maximum per tensor, on the same activation
        "per_tensor_f32": _case("tensor", "float32", "relu", 0, "2", rows=64 * 256, cols=56 * 56),
        # a ViT/BERT activation in half precision with all four widths
        "vit_f16": _case("tensor", "float16", "gelu", 128, "1248", rows=32 * 1024, cols=768),
        # the activations of a whole ResNet-18 training step at batch 256
        "resnet18_step_f32": _case("resnet", "float32", "relu", 256, "2", batch=256),
        # the MLP activation of an LLM at 16 sequences of 2048 tokens, with outlier channels
        "llm_bf16": _case("tensor", "bfloat16", "heavy", 64, "248", rows=16 * 2048, cols=11008),
        # two activations of each of 12 layers of a ViT at 8 images of 197 tokens, one group per row: ragged sizes, a list
        "vit_rows_f16": _case("vit", "float16", "gelu", 768, "1248", images=8, tokens=197, layers=12),
        # one iteration of a width controller on the ViT activation: many short launches
        "controller_f16": _case("controller", "float16", "gelu", 128, "1248", rows=32 * 1024, cols=768),
        # one iteration on the LLM activation, with importance metrics and the next widths from the scales
        "metrics_bf16": _case("metrics", "bfloat16", "heavy", 64, "248", rows=16 * 2048, cols=11008),
        # the LLM MLP's up-projection with its output saved in the epilogue
        "linear_bf16": _case("linear", "bfloat16", "heavy", 64, "248", rows=16 * 2048, cols=11008, inner=4096),
        # the weight gradient of the LLM MLP's down-projection, and of a ViT/BERT layer
        "wgrad_bf16": _case("wgrad", "bfloat16", "heavy", 64, "248", rows=16 * 2048, cols=11008, inner=4096),
        "wgrad_f16": _case("wgrad", "float16", "gelu", 128, "1248", rows=32 * 1024, cols=768, inner=3072),
    }
    return [dict(c, name=n) for n, c in named.items()]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["tensor", "tensor", "tensor", "resnet", "vit", "relu", "controller", "metrics", "linear", "wgrad"])
    dtype = rng.choice(list(DTYPES))
    values = {"float32": "relu", "float16": "gelu", "bfloat16": "heavy"}[dtype]
    widths = rng.choice(["1", "2", "4", "8", "1248", "248", "28", "124"])
    if kind == "resnet":
        return _case(kind, dtype, values, rng.choice([64, 128, 256, 768]), widths, batch=_log_uniform(rng, 1, 256))
    if kind == "vit":
        group = rng.choice([768, 256, 128, 64])
        return _case(kind, dtype, values, group, widths, images=_log_uniform(rng, 1, 32), tokens=rng.choice([128, 197, 577]), layers=rng.randint(1, 12))
    if kind == "linear":
        # whole tiles of 256 x 256 outputs and 64 inner values are what the entry point takes
        rows, cols, inner = 256 * _log_uniform(rng, 1, 128), 256 * _log_uniform(rng, 1, 43), 64 * _log_uniform(rng, 4, 64)
        return _case(kind, rng.choice(["float16", "bfloat16"]), "heavy", rng.choice([32, 64, 128]), widths, rows=rows, cols=cols, inner=inner)
    if kind == "wgrad":
        rows, cols, inner = 32 * _log_uniform(rng, 16, 1024), 64 * _log_uniform(rng, 4, 172), 64 * _log_uniform(rng, 1, 64)
        if dtype == "float32":                       # the binary32 matrix cores are a sixteenth as fast
            rows, inner = 32 * _log_uniform(rng, 16, 256), 64 * _log_uniform(rng, 1, 16)
        group = rng.choice([g for g in (32, 64, 128, 256) if cols % g == 0])
        return _case(kind, dtype, values, group, widths, rows=rows, cols=cols, inner=inner)
    cols = rng.choice([49, 196, 784, 3136, 768, 3072, 4096, 11008])      # a channel's pixels, or a token's features
    most = 300_000_000 if dtype != "float32" else 200_000_000
    rows = max(1, _log_uniform(rng, 1 << 15, most) // cols)
    if kind in ("controller", "metrics"):
        if len(widths) == 1:
            widths = "248"
        return _case(kind, dtype, values, rng.choice([32, 64, 128, 256, 768]), widths, rows=rows, cols=cols)
    if kind == "relu":
        return _case(kind, dtype, "signed", rng.choice([64, 128, 256, 768]), widths, rows=rows, cols=cols)
    group = rng.choice([32, 64, 96, 128, 256, 256, 768, 3072, 11008, 0])
    if group == 0 and len(widths) > 1:
        widths = "8"
    return _case(kind, dtype, values, group, widths, rows=rows, cols=cols)


# ---- shapes of a case -------------------------------------------------------------------------------------------------

# (count, channels, pixels) of the activations that a ResNet-18 step saves, forward order
_RESNET18 = [(1, 64, 112 * 112), (4, 64, 56 * 56), (4, 128, 28 * 28), (4, 256, 14 * 14), (4, 512, 7 * 7)]


def _tensors(case):
    """(elements, group size) of every activation that the case saves."""
    group = case["group"]
    if case["kind"] == "resnet":
        return [(case["batch"] * c * p, group) for n, c, p in _RESNET18 for _ in range(n)]
    if case["kind"] == "vit":
        rows = case["images"] * case["tokens"]
        wide = 3072 if group == 768 else group       # a group per row, or the same groups for both
        return [(rows * cols, g) for _ in range(case["layers"]) for cols, g in ((768, group), (3072, wide))]
    n = case["rows"] * case["cols"]
    return [(n, group if group else -(-n // 32) * 32)]


def _classes(case):
    return [int(c) for c in case["widths"]]


# ---- inputs -----------------------------------------------------------------------------------------------------------

def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _values(case, n, g, cols=None):
    """Activations as they come out of a relu, a gelu, or an LLM's gated MLP (heavy tails, one channel in a hundred 20 times
    as large); "signed": before a relu."""
    kind = case["values"]
    x = torch.randn(n, generator=g, device="cuda")
    if kind == "relu":
        x = torch.relu_(x)
    elif kind == "gelu":
        x = torch.nn.functional.gelu(x)
    elif kind == "heavy":
        chi2 = torch.randn(n, generator=g, device="cuda").square_()
        for _ in range(2):
            chi2 += torch.randn(n, generator=g, device="cuda").square_()
        x /= chi2.div_(3).sqrt_()
        del chi2
        if cols:
            channel = torch.ones(cols, device="cuda")
            channel[torch.randperm(cols, generator=g, device="cuda")[: cols // 100]] = 20.0
            x = (x.view(-1, cols) * channel).view(-1)
    return x.to(DTYPES[case["dtype"]])


def _padded(x, group):
    """[groups, group] with the last value repeated to fill a short last group."""
    pad = -x.numel() % group
    if pad:
        x = torch.cat([x, x[-1:].expand(pad)])
    return x.view(-1, group)


def _by_rank(ranges, classes):
    """Equal shares of the groups by (range, index), smallest ranges first."""
    G = ranges.numel()
    order = torch.sort(ranges, stable=True).indices
    table = torch.tensor(classes, dtype=torch.uint8, device="cuda")
    bits = torch.empty(G, dtype=torch.uint8, device="cuda")
    bits[order] = table[torch.arange(G, device="cuda") * len(classes) // G]
    return bits


def _ranges(x, group):
    rows = _padded(x, group)
    return rows.amax(1).float() - rows.amin(1).float()


def _widths(case, x, group):
    classes = _classes(case)
    if len(classes) == 1:
        return classes[0]
    return _by_rank(_ranges(x, group), classes)


def _arena(parts, filled=False):
    """One buffer with a place for every part, each on a boundary of 64 elements, and the places; `filled`: the buffer with
    the parts in it."""
    starts, at = [], 0
    for p in parts:
        starts.append(at)
        at += -(-p.numel() // 64) * 64
    whole = torch.zeros(at, dtype=parts[0].dtype, device="cuda")
    places = [whole[i: i + p.numel()] for i, p in zip(starts, parts)]
    if not filled:
        return whole, places
    for place, p in zip(places, parts):
        place.copy_(p.view(-1))
    return whole


class _Saved:
    """One activation, its plan and the buffers that hold its packed form."""

    def __init__(self, case, x, group, words=None):
        self.x, self.group = x, group
        self.bits = _widths(case, x, group)
        self.plan = daf.daf_plan((x.numel(),), group, self.bits)
        size = self.plan.packed_words if words is None else words(self.plan)
        self.words = torch.zeros(size, dtype=torch.int32, device="cuda")
        self.min = torch.empty(self.plan.num_groups, dtype=torch.float32, device="cuda")
        self.scale = torch.empty_like(self.min)

    def packed(self):
        return self.words, self.min, self.scale


def prepare(case, seed):
    g = _gen(seed)
    kind = case["kind"]
    state = {"case": case, "seed": seed}
    dtype = DTYPES[case["dtype"]]
    if kind == "tensor":
        (n, group), = _tensors(case)
        state["saved"] = s = _Saved(case, _values(case, n, g, case["cols"]), group)
        state["restored"] = torch.empty_like(s.x)
        return state
    if kind in ("resnet", "vit"):
        # what the step saves lives in one arena of each kind: words, minima, scales, restored values
        saved = [_Saved(case, _values(case, n, g), group) for n, group in _tensors(case)]
        words, mins, scales = (_arena([getattr(s, name) for s in saved]) for name in ("words", "min", "scale"))
        restored = _arena([s.x for s in saved])
        for s, w, lo, sc in zip(saved, words[1], mins[1], scales[1]):
            s.words, s.min, s.scale = w, lo, sc
        state["out"] = {"words": words[0], "min": mins[0], "scale": scales[0], "restored": restored[0]}
        state["saved"] = saved
        state["save"] = daf.quantize_items([(s.plan, s.x, seed + i, *s.packed()) for i, s in enumerate(saved)])
        backward = list(zip(saved, restored[1]))[::-1]
        state["restore"] = daf.dequantize_items([(s.plan, *s.packed(), out, None) for s, out in backward])
        return state
    (n, group), = _tensors(case)
    if kind == "relu":
        z = _values(case, n, g, case["cols"])
        state["saved"] = _Saved(case, torch.relu(z), group)
        state["saved"].x = None
        state["z"], state["y"] = z, torch.empty_like(z)
        state["grad_y"] = torch.randn(n, generator=g, device="cuda").mul_(1e-2).to(dtype)
        state["grad_z"] = torch.empty_like(z)
    elif kind in ("controller", "metrics"):
        state["saved"] = s = _Saved(case, _values(case, n, g, case["cols"]), group, words=lambda p: p.packed_words_bound)
        state["next_bits"] = torch.empty_like(s.bits)
        state["workspace"] = daf.daf_select_bits_workspace(s.plan.num_groups)
        if kind == "controller":
            state["lo"], state["hi"] = torch.empty_like(s.min), torch.empty_like(s.min)
        else:
            state["metrics"] = torch.empty(3 * s.plan.num_groups, dtype=torch.float32, device="cuda")
    elif kind == "linear":
        x, w = _linear_inputs(case, g)
        state["x"], state["w"] = x, w
        # the widths were chosen from an earlier batch: any fixed choice with equal shares
        classes = _classes(case)
        G = n // group
        bits = classes[0] if len(classes) == 1 else _by_rank(torch.rand(G, generator=g, device="cuda"), classes)
        plan = daf.daf_plan((n,), group, bits)
        state["plan"], state["bits"] = plan, bits
        state["y"] = torch.empty(case["rows"], case["cols"], dtype=dtype, device="cuda")
        state["words"] = torch.zeros(plan.packed_words, dtype=torch.int32, device="cuda")
        state["min"] = torch.empty(plan.num_groups, dtype=torch.float32, device="cuda")
        state["scale"] = torch.empty_like(state["min"])
    else:
        codes, lo, scale, bits, grad_y = _wgrad_inputs(case, g)
        state["plan"] = plan = daf.daf_plan((n,), group, bits)
        state["words"], state["min"], state["scale"] = _pack(codes, bits), lo, scale
        state["bits"], state["grad_y"] = bits, grad_y
        del codes
        state["grad_w"] = torch.empty(case["inner"], case["cols"], dtype=torch.float32, device="cuda")
        need = daf.daf_unpack_matmul_workspace_bytes(plan, case["inner"], case["cols"])
        state["workspace"] = torch.empty(max(need, 16), dtype=torch.uint8, device="cuda")
    return state


def _linear_inputs(case, g):
    rows, cols, inner, dtype = case["rows"], case["cols"], case["inner"], DTYPES[case["dtype"]]
    x = torch.randn(rows, inner, generator=g, device="cuda").to(dtype)               # a normalised input
    w = torch.randn(cols, inner, generator=g, device="cuda").div_(math.sqrt(inner)).to(dtype)
    return x, w


def _wgrad_inputs(case, g):
    """Codes of an activation that the forward pass saved (stochastic rounding), group minima and scales, and the gradient."""
    (n, group), = _tensors(case)
    x = _values(case, n, g, case["cols"])
    bits = _widths(case, x, group)
    rows = x.view(-1, group).float()
    lo, hi = rows.amin(1), rows.amax(1)
    top = (2.0 ** bits.float() - 1) if isinstance(bits, torch.Tensor) else torch.full_like(lo, 2.0 ** bits - 1)
    scale = (hi - lo) / top
    v = (rows - lo[:, None]) / torch.where(scale > 0, scale, 1.0)[:, None]
    codes = torch.floor(v + torch.rand(v.shape, generator=g, device="cuda"))
    codes = torch.minimum(codes, top[:, None]).to(torch.uint8)
    grad_y = torch.randn(case["rows"], case["inner"], generator=g, device="cuda").mul_(1e-2).to(DTYPES[case["dtype"]])
    return codes, lo, scale, bits, grad_y


def _pack(codes, bits):
    """The packed words of [groups, group] codes: first code in the most significant bits, groups one after the other."""
    G, group = codes.shape
    per_group = bits.long() if isinstance(bits, torch.Tensor) else torch.full((G,), bits, device="cuda")
    sizes = per_group * (group // 32)
    ends = torch.cumsum(sizes, 0)
    words = torch.empty(int(ends[-1]), dtype=torch.int32, device="cuda")
    for b in (1, 2, 4, 8):
        which = torch.nonzero(per_group == b).view(-1)
        if which.numel() == 0:
            continue
        c = codes[which].view(-1, group * b // 32, 32 // b)
        acc = torch.zeros(c.shape[:2], dtype=torch.int32, device="cuda")
        for j in range(32 // b):
            acc |= c[:, :, j].int() << (32 - b * (j + 1))
        place = (ends - sizes)[which][:, None] + torch.arange(group * b // 32, device="cuda")
        words[place.view(-1)] = acc.view(-1)
    return words


# ---- one pass ---------------------------------------------------------------------------------------------------------

def run(state):
    case = state["case"]
    kind, seed = case["kind"], state["seed"]
    if kind == "tensor":
        s = state["saved"]
        daf.daf_quantize_pack(s.plan, s.x, seed, *s.packed())
        daf.daf_unpack_dequantize(s.plan, *s.packed(), state["restored"])
        return {"words": s.words, "min": s.min, "scale": s.scale, "restored": state["restored"]}
    if kind in ("resnet", "vit"):
        daf.daf_quantize_pack_batch(state["save"])
        daf.daf_unpack_dequantize_batch(state["restore"])
        return state["out"]
    if kind == "relu":
        s = state["saved"]
        daf.daf_relu_quantize_pack(s.plan, state["z"], seed, state["y"], *s.packed())
        daf.daf_unpack_relu_backward(s.plan, *s.packed(), state["grad_y"], state["grad_z"])
        return {"y": state["y"], "words": s.words, "min": s.min, "scale": s.scale, "grad_z": state["grad_z"]}
    if kind == "controller":
        s = state["saved"]
        daf.daf_group_minmax(s.plan, s.x, state["lo"], state["hi"])
        daf.daf_select_bits(state["lo"], state["hi"], _classes(case), state["next_bits"], state["workspace"])
        s.plan.update(state["next_bits"])
        daf.daf_quantize_pack(s.plan, s.x, seed, *s.packed())
        return {"bits": state["next_bits"], "words": s.words, "min": s.min, "scale": s.scale}
    if kind == "metrics":
        s = state["saved"]
        s.plan.update(s.bits)                        # the widths that the last iteration chose
        daf.daf_quantize_pack_metrics(s.plan, s.x, seed, *s.packed(), state["metrics"])
        daf.daf_select_bits_from_scale(s.scale, s.bits, _classes(case), state["next_bits"], state["workspace"])
        return {"bits": state["next_bits"], "words": s.words, "min": s.min, "scale": s.scale, "metrics": state["metrics"]}
    if kind == "linear":
        daf.daf_linear_quantize_pack(state["plan"], state["x"], state["w"], seed, state["y"], state["words"], state["min"], state["scale"])
        return {"y": state["y"], "words": state["words"], "min": state["min"], "scale": state["scale"]}
    daf.daf_unpack_matmul_grad_weight(state["plan"], state["words"], state["min"], state["scale"], state["grad_y"], state["grad_w"], state["workspace"])
    return state["grad_w"]


# ---- what a pass cannot do without ------------------------------------------------------------------------------------

def work(case):
    size, classes = BYTES[case["dtype"]], _classes(case)
    mean = sum(classes) / len(classes) / 8           # packed bytes per element
    per_group = 8 if len(classes) == 1 else 13       # minimum and scale; with per-group widths a width and an offset
    kind = case["kind"]
    total, flops = 0.0, 0.0
    for n, group in _tensors(case):
        groups = -(-n // group)
        packed = n * mean + groups * per_group
        if kind == "wgrad":
            total += packed + case["rows"] * case["inner"] * size + case["inner"] * case["cols"] * 4
            flops += 2.0 * case["rows"] * case["inner"] * case["cols"]
        elif kind == "linear":
            total += packed + (n + (case["rows"] + case["cols"]) * case["inner"]) * size
            flops += 2.0 * n * case["inner"]
        elif kind == "relu":
            total += 2 * packed + 4 * n * size
        elif kind == "controller":                   # widths come out of the statistics, so the activation is read twice
            total += 2 * n * size + packed + groups * 12
        elif kind == "metrics":
            total += n * size + packed + groups * (12 + 6)
        elif group >= n:
            total += 2 * packed + 3 * n * size       # one group: nothing can be quantized before all has been read
        else:
            total += 2 * packed + 2 * n * size
    return {"bytes": total, "flops": flops}


def tolerance(case):
    """Everything but the two contractions and the metrics is defined to the bit.  The others: about four times what the
    path differs by from the same sums in 64 bits.

    metrics: sums of one group in binary32 (2e-7 on the sum of squares).
    wgrad: sums over `rows` products in binary32, in any order (1.0e-6, largest 4.7e-5, at 32768 rows).
    linear: the same sums rounded to 16 bits (4.1e-5, largest one unit in the last place of bfloat16, 7.8e-3); where the
    rounding falls the other way the codes can follow (8.4e-5 of the packed words with bfloat16; binary16's finer grid
    has eight times as many such places)."""
    if case["kind"] == "metrics":
        return {"rel": 1e-6, "differ": 0.0}
    if case["kind"] == "wgrad":
        return {"rel": 4e-6, "max": 2e-4}
    if case["kind"] == "linear":
        return {"rel": 2e-4, "max": 0.04, "differ": 3e-3}
    return "exact"


# ---- 64-bit results ---------------------------------------------------------------------------------------------------

def _philox_part(first, n, seed):
    """Bytes of elements first .. first + n - 1; `first` is a multiple of 16."""
    m32 = 0xFFFFFFFF
    blocks = torch.arange(first // 16, -(-(first + n) // 16), device="cuda", dtype=torch.int64)
    c = [blocks & m32, blocks >> 32, torch.zeros_like(blocks), torch.zeros_like(blocks)]
    k0, k1 = seed & m32, (seed >> 32) & m32

    def product(a, const):                           # high and low half of a 32 x 32 bit product, within 63 bits
        q, r = (a >> 16) * const, (a & 0xFFFF) * const
        low = ((q & 0xFFFF) << 16) + (r & m32)
        return ((q >> 16) + (r >> 32) + (low >> 32)) & m32, low & m32

    for _ in range(10):
        h0, l0 = product(c[0], 0xD2511F53)
        h1, l1 = product(c[2], 0xCD9E8D57)
        c = [h1 ^ c[1] ^ k0, l1, h0 ^ c[3] ^ k1, l0]
        k0, k1 = (k0 + 0x9E3779B9) & m32, (k1 + 0xBB67AE85) & m32
    return torch.stack([((w >> (8 * j)) & 0xFF).to(torch.uint8) for w in c for j in range(4)], 1).view(-1)[:n]


def _quantized(x, group, bits, seed):
    """(min, scale, codes [groups, group], fractional parts before rounding) in 64 bits."""
    n = x.numel()
    rows = _padded(x.double(), group)
    lo, hi = rows.amin(1), rows.amax(1)
    top = (2.0 ** bits.double() - 1) if isinstance(bits, torch.Tensor) else torch.full_like(lo, 2.0 ** bits - 1)
    scale = (hi - lo) / top
    v = (rows - lo[:, None]) / torch.where(scale > 0, scale, 1.0)[:, None]
    del rows
    byte = torch.zeros(v.numel(), dtype=torch.uint8, device="cuda")
    step = 1 << 26
    for i in range(0, n, step):                      # a block of bytes at a time
        byte[i: min(i + step, n)] = _philox_part(i, min(step, n - i), seed)
    up = v - torch.floor(v)
    codes = torch.floor(v) + ((byte.view(v.shape).double() + 0.5) < up * 256)
    codes = torch.minimum(codes, top[:, None])
    return lo, scale, codes, up


def _exact_saved(x, group, bits, seed):
    lo, scale, codes, _ = _quantized(x, group, bits, seed)
    codes.mul_(scale[:, None]).add_(lo[:, None])
    return lo, scale, codes.view(-1)[: x.numel()]


def exact(case, seed):
    g = _gen(seed)
    kind = case["kind"]
    if kind in ("tensor", "resnet", "vit"):
        parts = []
        for i, (n, group) in enumerate(_tensors(case)):
            x = _values(case, n, g, case.get("cols"))
            parts.append(_exact_saved(x, group, _widths(case, x, group), seed + i))
        lo, scale, back = zip(*parts)
        if kind == "tensor":
            return {"words": None, "min": lo[0], "scale": scale[0], "restored": back[0]}
        return {"words": None, "min": _arena(lo, True), "scale": _arena(scale, True), "restored": _arena(back, True)}
    (n, group), = _tensors(case)
    if kind == "relu":
        z = _values(case, n, g, case["cols"])
        y = torch.relu(z)
        grad = torch.randn(n, generator=g, device="cuda").mul_(1e-2).to(DTYPES[case["dtype"]])
        lo, scale, back = _exact_saved(y, group, _widths(case, y, group), seed)
        return {"y": y.double(), "words": None, "min": lo, "scale": scale, "grad_z": torch.where(back > 0, grad.double(), 0.0)}
    if kind in ("controller", "metrics"):
        x = _values(case, n, g, case["cols"])
        bits = _widths(case, x, group)
        lo, scale, codes, up = _quantized(x, group, bits, seed)
        out = {"bits": None, "words": None, "min": lo, "scale": scale}
        if kind == "metrics":
            rows = _padded(x.double(), group)
            inside = (torch.arange(rows.numel(), device="cuda") < n).view(rows.shape)
            err = ((rows - codes.mul_(scale[:, None]).add_(lo[:, None])).square() * inside).sum(1)
            p = torch.ceil(up * 256 - 0.5).clamp_(0, 256) / 256
            var = (p * (1 - p) * inside).sum(1) * scale.square()
            out["metrics"] = torch.stack([err, (rows.square() * inside).sum(1), var], 1).view(-1)
        return out
    if kind == "linear":
        x, w = _linear_inputs(case, g)
        y = x.double() @ w.double().t().contiguous()
        classes = _classes(case)
        bits = classes[0] if len(classes) == 1 else _by_rank(torch.rand(n // group, generator=g, device="cuda"), classes)
        rows = y.view(-1, group)
        lo, hi = rows.amin(1), rows.amax(1)
        top = (2.0 ** bits.double() - 1) if isinstance(bits, torch.Tensor) else 2.0 ** bits - 1
        return {"y": y, "words": None, "min": lo, "scale": (hi - lo) / top}
    codes, lo, scale, bits, grad_y = _wgrad_inputs(case, g)
    x = torch.addcmul(lo.double()[:, None], codes.double(), scale.double()[:, None]).float()     # one rounding to binary32,
    x = x.to(DTYPES[case["dtype"]]).double().view(case["rows"], case["cols"])                   # one to the element format
    return grad_y.double().t().contiguous() @ x
