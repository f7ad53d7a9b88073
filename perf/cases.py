"""What the speed of this library is measured on: passes through its public
entry points (``PackedWeight.run``, ``quantize_act``), as a serving program
makes them.

A case is a dict of plain values. ``op`` says what one pass is:

    linear    one sparse linear on int8 activations
    quantize  one quantisation of fp32 activations
    ffn       quantise the input, FFN1 (GELU, int8), FFN2 (fp32)
    layer     the four linears of an encoder layer (QKV, attention output,
              FFN1, FFN2); the attention core between them is not this
              library's, so QKV and the attention output each read an int8
              tensor of their own
    stack     the linears of several such layers, FFN2 of one feeding the QKV
              of the next

``m`` tokens, ``n`` output and ``k`` input features (of a linear), ``hidden``
and ``inter`` (of the others), ``sparsity`` of the 4x1 blocks, ``epi`` the
epilogue, ``layout`` of the int8 activations (``rows``: the entry points'
default; ``blocks``: the 16-token x 32-feature layout, in which activations
stay from one linear to the next), ``graph``: the pass is captured in a HIP
graph once and replayed, as a program that serves one fixed shape does.

Weights are block-sparse with masks of the given density; values are normal,
as trained weights and activations nearly are, on the int8 range that
quantising by the largest magnitude leaves them. Output scales are calibrated
on a sample of the tokens, by largest magnitude.
"""
import math

import torch

import paper_2211_07715_amd as sl

F32, F32_GELU, I8, I8_GELU, ACC = sl.EPI_F32, sl.EPI_F32_GELU, sl.EPI_I8, sl.EPI_I8_GELU, sl.EPI_ACC_I32
INT8_KINDS = (I8, I8_GELU)
SX = 0.02            # scale of the int8 activations that a pass starts from
SAMPLE = 256         # tokens that output scales are calibrated on


def listed():
    return [
        # the smallest call: one projection of one short sequence, defaults throughout
        dict(name="linear_b1_s128", op="linear", m=128, n=768, k=768, sparsity=0.8, epi="f32", layout="rows",
             graph=False),
        # batch-1 latency of a whole encoder's linears, replayed from a graph
        dict(name="stack_b1_s128_graph", op="stack", m=128, hidden=768, inter=3072, layers=6, sparsity=0.8,
             layout="blocks", graph=True),
        # the same encoder on a long sequence, called eagerly with the default layout
        dict(name="stack_b1_s384", op="stack", m=384, hidden=768, inter=3072, layers=6, sparsity=0.9, layout="rows",
             graph=False),
        # odd sizes: a batch of unpadded sequences through a layer whose widths are no multiple of 16
        dict(name="linear_ragged", op="linear", m=1531, n=1000, k=1001, sparsity=0.8, epi="i8", layout="rows",
             graph=False),
        # raw accumulators, for a program with an epilogue of its own
        dict(name="qkv_acc_b16_s128", op="linear", m=2048, n=2304, k=768, sparsity=0.7, epi="acc_i32", layout="rows",
             graph=False),
        # FFN1 whose activations leave the int8 chain (a layer kept in fp32)
        dict(name="ffn1_f32gelu_b8_s384", op="linear", m=3072, n=3072, k=768, sparsity=0.8, epi="f32_gelu",
             layout="rows", graph=False),
        # the headline workload: quantisation and FFN pair of a DistilBERT layer at batch 32
        dict(name="ffn_b32_s128", op="ffn", m=4096, hidden=768, inter=3072, sparsity=0.9, layout="blocks",
             graph=False),
        # the same sizes in the default layout, at a lower sparsity
        dict(name="ffn_rows_b32_s128", op="ffn", m=4096, hidden=768, inter=3072, sparsity=0.7, layout="rows",
             graph=False),
        # all linears of one layer at batch 32
        dict(name="layer_b32_s128", op="layer", m=4096, hidden=768, inter=3072, sparsity=0.8, layout="blocks",
             graph=False),
        # throughput serving of long sequences: one layer at batch 128
        dict(name="layer_b128_s384", op="layer", m=49152, hidden=768, inter=3072, sparsity=0.9, layout="blocks",
             graph=False),
        # the largest: a BERT-large FFN pair at batch 128, default layout
        dict(name="bertl_ffn_b128_s384", op="ffn", m=49152, hidden=1024, inter=4096, sparsity=0.8, layout="rows",
             graph=False),
        # the first step of every chain, at the size of a large batch
        dict(name="quantize_b128_s384", op="quantize", m=49152, k=768, layout="rows"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the same ranges: 1 to 49152 tokens, up to 4096 features, 70 to
    90 % sparsity, every epilogue and both layouts."""
    op = rng.choice(["linear"] * 5 + ["ffn"] * 2 + ["layer"] * 2 + ["quantize"])
    m = _log_int(rng, 1, 49152)
    layout = rng.choice(["rows", "blocks"])
    sparsity = round(rng.uniform(0.7, 0.9), 2)
    if op == "quantize":
        return dict(op=op, m=m, k=rng.choice([768, 1024, 3072, 4096, rng.randrange(1, 4097)]), layout=layout)
    if op in ("ffn", "layer"):
        hidden, inter = rng.choice([(768, 3072), (1024, 4096)])
        if op == "layer" and hidden == 1024:
            m = min(m, 24576)
        if op == "layer" and layout == "blocks":
            m = (m + 15) // 16 * 16  # its int8 QKV output is returned whole, so it has no padding tokens
        return dict(op=op, m=m, hidden=hidden, inter=inter, sparsity=sparsity, layout=layout, graph=rng.random() < 0.2)
    epi = rng.choice(["f32", "f32", "i8", "i8", "i8_gelu", "i8_gelu", "f32_gelu", "acc_i32"])
    if rng.random() < 0.6:
        n, k = rng.choice([(2304, 768), (768, 768), (3072, 768), (768, 3072), (1024, 1024), (4096, 1024), (1024, 4096)])
    else:
        n, k = 4 * _log_int(rng, 4, 1024), _log_int(rng, 32, 4096)
    return dict(op=op, m=m, n=n, k=k, sparsity=sparsity, epi=epi, layout=layout, graph=rng.random() < 0.2)


# --- inputs -----------------------------------------------------------------

def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed) * 7919 + 17)


def _codes(shape, g):
    """int8 codes of a normal tensor quantised by its largest magnitude (about 4 standard deviations)."""
    return torch.randn(shape, generator=g, device="cuda").mul_(127 / 4).round_().clamp_(-127, 127).to(torch.int8)


def _weight(n, k, sparsity, g):
    keep = torch.rand((n // 4, k), generator=g, device="cuda") >= sparsity
    w = _codes((n, k), g) * keep.repeat_interleave(4, dim=0).to(torch.int8)
    sw = torch.empty(n, device="cuda").uniform_(0.001, 0.01, generator=g)
    b = torch.randn(n, generator=g, device="cuda").mul_(0.02)
    return {"w": w, "sw": sw, "b": b}


def _f32(v):
    return float(torch.tensor(v, dtype=torch.float32))


def _ops(case):
    """(name, n, k, epilogue, source) of the pass's linears; a source is an
    input of the pass ("in.<name>") or the name of an earlier linear."""
    if case["op"] == "linear":
        return [("y", case["n"], case["k"], sl.EPI_BY_NAME[case["epi"]], "in.x")]
    h, i = case["hidden"], case["inter"]
    if case["op"] == "ffn":
        return [("ffn1", i, h, I8_GELU, "in.x"), ("ffn2", h, i, F32, "ffn1")]
    layers, ops = case.get("layers", 1), []
    for l in range(layers):
        last = l == layers - 1
        ops += [("qkv%d" % l, 3 * h, h, I8, "in.x" if l == 0 else "ffn2%d" % (l - 1)),
                ("attn%d" % l, h, h, I8, "in.a%d" % l),
                ("ffn1%d" % l, i, h, I8_GELU, "attn%d" % l),
                ("ffn2%d" % l, h, i, F32 if last else I8, "ffn1%d" % l)]
    return ops


def _returned(name):
    """What a pass hands on: a linear's or pair's output, a layer's QKV and final output."""
    return not name.startswith(("attn", "ffn1"))


def _inputs(case, seed):
    """Weights and activations of a pass, and the scale of every linear's input and output, as plain tensors."""
    g = _gen(seed)
    m = case["m"]
    if case["op"] == "quantize":
        return {"f": torch.randn((m, case["k"]), generator=g, device="cuda").mul_(0.6)}
    ops = _ops(case)
    d = {"ops": ops, "w": {}, "x": {}, "sx": {}, "so": {}}
    if case["op"] == "ffn":  # the pass quantises its fp32 input
        d["f"] = torch.randn((m, case["hidden"]), generator=g, device="cuda").mul_(0.6)
    sample = {}
    for name, n, k, kind, src in ops:
        d["w"][name] = _weight(n, k, case["sparsity"], g)
        if src.startswith("in."):
            if "f" in d:
                sample[src] = torch.round(d["f"][:SAMPLE].double() / _f32(SX)).clamp(-127, 127)
            else:
                d["x"][src] = _codes((m, k), g)
                sample[src] = d["x"][src][:SAMPLE].double()
            d["sx"][name] = _f32(SX)
        else:
            d["sx"][name] = d["so"][src]
        d["so"][name] = 1.0
        y = _reference(sample[src], d["w"][name], d["sx"][name], kind, None)
        if kind in INT8_KINDS:
            d["so"][name] = _f32(max(float(y.abs().max()), 1e-3) / 127)
            sample[name] = torch.round(y / d["so"][name]).clamp(-127, 127)
    return d


def _blocks(x):
    """An int8 [m, k] tensor in the block layout, zeros for padding."""
    m, k = x.shape
    rb, cb, _, _ = sl.t16x32_shape(m, k)
    p = torch.zeros((rb * 16, cb * 32), dtype=torch.int8, device=x.device)
    p[:m, :k] = x
    return p.reshape(rb, 16, cb, 32).permute(0, 2, 1, 3).contiguous()


def prepare(case, seed):
    d = _inputs(case, seed)
    layout = sl.LAYOUT_T16X32 if case["layout"] == "blocks" else sl.LAYOUT_ROWS
    s = {"op": case["op"], "m": case["m"], "layout": layout, "f": d.get("f"), "graph": None}
    if case["op"] != "quantize":
        s["x"] = {n: _blocks(x) if layout else x for n, x in d["x"].items()}
        s["steps"] = []
        for name, n, k, kind, src in d["ops"]:
            w = d["w"][name]
            pw = sl.PackedWeight.pack(w["w"].cpu().numpy(), w["sw"].cpu().numpy(), w["b"].cpu().numpy())
            # int8 outputs stay in the chain's layout; a lone linear's only where it leaves no padding
            whole = case["m"] % 16 == 0 and n % 32 == 0
            yl = layout if kind in INT8_KINDS and (whole or not _returned(name)) else sl.LAYOUT_ROWS
            s["steps"].append((name, src, pw, d["sx"][name], kind, d["so"][name], yl))
    if case.get("graph"):
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            _pass(s)
        torch.cuda.current_stream().wait_stream(side)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            s["out"] = _pass(s)
        s["graph"] = graph
    return s


# --- one pass ---------------------------------------------------------------

def _pass(s):
    m, layout = s["m"], s["layout"]
    if s["op"] == "quantize":
        return sl.quantize_act(s["f"], SX, layout=layout)
    have = dict(s["x"])
    if s["f"] is not None:
        have["in.x"] = sl.quantize_act(s["f"], SX, layout=layout)
    out = {}
    for name, src, pw, sx, kind, so, yl in s["steps"]:
        have[name] = pw.run(have[src], sx, kind, out_scale=so, x_layout=layout, y_layout=yl, m_tokens=m)
        if _returned(name):
            out[name] = have[name]
    return out


def run(state):
    if state["graph"] is not None:
        state["graph"].replay()
        return state["out"]
    return _pass(state)


# --- what a pass cannot do without, and what it has to give -----------------

def _linear_work(m, n, k, sparsity, kind):
    blocks = (1 - sparsity) * (n // 4) * k
    out = 1 if kind in INT8_KINDS else 4
    # X, Y, the canonical block-sparse weight (4 values and a 16-bit column a block, row pointers), scales and biases
    return m * k + m * n * out + 6 * blocks + n + 8 * n, 2.0 * m * 4 * blocks


def work(case):
    if case["op"] == "quantize":
        return {"bytes": 5.0 * case["m"] * case["k"], "flops": 0.0}
    nbytes, flops = 0.0, 0.0
    if case["op"] == "ffn":
        nbytes += 5.0 * case["m"] * case["hidden"]
    for _, n, k, kind, _ in _ops(case):
        b, f = _linear_work(case["m"], n, k, case["sparsity"], kind)
        nbytes, flops = nbytes + b, flops + f
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    if case["op"] == "quantize" or case.get("epi") == "acc_i32":
        return "exact"
    # about four times what the path differs by from the same arithmetic in 64 bits, measured over listed and drawn cases
    if case["op"] == "linear":
        # int8 (1.1e-6 of the codes): a code rounds the other way where fp32 falls on a tie;
        # fp32 (6.5e-8, largest 2.8e-7): three roundings, and erf's
        return {"differ": 1e-5} if case["epi"] in ("i8", "i8_gelu") else {"rel": 4e-7, "max": 2e-6}
    # (2.1e-4, largest 4.9e-2, 6e-4 of the codes) a code that rounds the other way travels into the next linears' sums
    return {"rel": 8e-4, "max": 2e-1, "differ": 2.4e-3}


def _reference(x, w, sx, kind, so):
    """One linear in 64 bits on int8 codes held as float64."""
    acc = x @ w["w"].double().t()
    if kind == ACC:
        return acc.to(torch.int32)
    y = acc.mul_(w["sw"].double() * sx).add_(w["b"].double())
    if kind in (F32_GELU, I8_GELU):
        y = 0.5 * y * (1 + torch.erf(y / math.sqrt(2.0)))
    return torch.round(y / so).clamp_(-127, 127) if kind in INT8_KINDS and so is not None else y


def exact(case, seed):
    d = _inputs(case, seed)
    blocks = case["layout"] == "blocks"

    def laid(q):
        return _blocks(q.to(torch.int8)) if blocks else q.to(torch.int8)

    if case["op"] == "quantize":
        return laid(torch.round(d["f"].double() / _f32(SX)).clamp(-127, 127))
    have = {n: x.double() for n, x in d["x"].items()}
    if "f" in d:
        have["in.x"] = torch.round(d["f"].double() / _f32(SX)).clamp(-127, 127)
    out = {}
    for name, n, k, kind, src in d["ops"]:
        y = _reference(have[src], d["w"][name], d["sx"][name], kind, d["so"][name])
        if kind in INT8_KINDS:
            have[name] = y
        if _returned(name):
            whole = case["m"] % 16 == 0 and n % 32 == 0
            out[name] = y if kind not in INT8_KINDS else laid(y) if whole else y.to(torch.int8)
    return out
