"""The calls whose speed matters to a program that keeps its weights compressed, as cases to be timed.

A program encodes its weights once (on the device, at load time), keeps the blobs resident, and then, layer by layer,
either decodes them into a buffer or multiplies by them directly.  The cases are those calls, through the Python binding:

  decode   one tensor, ``ecf8_decode`` / ``ecfw_decode``
  batch    the tensors of a layer or of a whole stack in one launch, ``ecf8_decode_batched`` / ``ecfw_decode_batched``
  gemm     decode fused into the product with a few rows of activations (a decode step of serving)
  grouped  the same for the routed experts of a mixture-of-experts layer, one launch
  encode   a matrix that is on the device, ``ecf8_encode_gpu`` / ``ecfw_encode_gpu`` (a checkpoint being loaded)

Weights are seeded draws from the symmetric alpha-stable family (what trained weights look like to an exponent coder),
made on the device.  Shapes are those of the 8B-class LLM layer, the 14B-class diffusion-transformer block and the
671B-class mixture-of-experts layer that the package's own benchmark uses.
"""
import math

import torch

from paper_2510_02676_amd import ecf8, ecfw, synth

DEV = "cuda:0"
MOE_SHAPES = [("gate", 2048, 7168), ("up", 2048, 7168), ("down", 7168, 2048)]
# size of the blob over the size of the raw tensor, as the encoders give it on these weights (it moves by a percent or
# two with the draw): what a decode has to read and an encode has to write
RATIO = {"e4m3": 0.893, "dit": 0.851, "plain": 0.906, "tiled": 0.915, "bf16": 0.684, "e5m2": 0.726}


def listed():
    return [
        # one small matrix by itself: router, norm-sized projection, adapter.  Launch and start-up are all of it.
        {"name": "decode_1024x1024", "op": "decode", "fmt": "e4m3", "rows": 1024, "cols": 1024, "cap": 0, "tiled": False},
        # a matrix whose size is no multiple of anything: padded vocabularies, pruned or odd heads, biases joined on
        {"name": "decode_ragged_4099x5127", "op": "decode", "fmt": "e4m3", "rows": 4099, "cols": 5127, "cap": 0, "tiled": False},
        # just-in-time decode of one LLM layer (7 matrices) into a shared buffer: the use the method is meant for
        {"name": "layer_llm8b", "op": "batch", "fmt": "e4m3", "set": "llm8b", "copies": 1, "cap": 0, "tiled": False},
        # a stack of diffusion-transformer blocks in one launch: the headline, and the largest
        {"name": "stack_dit_8_blocks", "op": "batch", "fmt": "e4m3", "set": "dit", "copies": 8, "cap": 0, "tiled": False},
        # the LLM layer with the plain Huffman code (no cap on codewords): blobs made for the smallest size
        {"name": "layer_llm8b_plain_huffman", "op": "batch", "fmt": "e4m3", "set": "llm8b", "copies": 1, "cap": 15, "tiled": False},
        # the LLM layer in the layout the fused product reads, decoded into a buffer: prefill of a program whose
        # decode steps use the fused product, so that it keeps one compressed copy
        {"name": "layer_llm8b_row_tiled", "op": "batch", "fmt": "e4m3", "set": "llm8b", "copies": 1, "cap": 0, "tiled": True},
        # the LLM layer held in BF16
        {"name": "layer_llm8b_bf16", "op": "batch", "fmt": "bf16", "set": "llm8b", "copies": 1, "cap": 0, "tiled": False},
        # the LLM layer held in E5M2
        {"name": "layer_llm8b_e5m2", "op": "batch", "fmt": "e5m2", "set": "llm8b", "copies": 1, "cap": 0, "tiled": False},
        # one projection of a decode step with 16 sequences, weights never written out
        {"name": "gemm_14336x4096_m16", "op": "gemm", "rows": 14336, "cols": 4096, "m": 16, "way": "fp8"},
        # eight routed experts, four tokens each, block scales of W and row scales of X
        {"name": "experts_8_m4_scaled", "op": "grouped", "experts": 8, "m": 4, "scaled": True},
        # a matrix of a checkpoint encoded on the device, FP8 and BF16
        {"name": "encode_14336x4096", "op": "encode", "fmt": "e4m3", "rows": 14336, "cols": 4096, "cap": 0, "tiled": False},
        {"name": "encode_14336x4096_bf16", "op": "encode", "fmt": "bf16", "rows": 14336, "cols": 4096, "cap": 0, "tiled": False},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _shape(rng, tiled):
    """From a bias-sized matrix up to the largest projection of the configurations; row-tiled blobs want whole blocks."""
    if tiled:
        return 16 * _log(rng, 2, 1024), 256 * _log(rng, 1, 96)
    return _log(rng, 8, 16384), _log(rng, 256, 16384)


def draw(rng):
    op = rng.choice(["decode", "decode", "batch", "batch", "gemm", "gemm", "grouped", "encode", "encode"])
    if op == "gemm":
        return {"op": op, "rows": 16 * _log(rng, 4, 1024), "cols": rng.choice([4096, 256 * _log(rng, 1, 64)]), "m": _log(rng, 1, 64),
                "way": rng.choice(["fp8", "exact", "scaled", "scaled_groups", "splitk"])}
    if op == "grouped":
        return {"op": op, "experts": _log(rng, 2, 20), "m": _log(rng, 1, 64), "scaled": rng.random() < 0.5}
    fmt = rng.choice(["e4m3", "e4m3", "e4m3", "bf16", "e5m2"])
    tiled = fmt == "e4m3" and rng.random() < 0.25
    # caps: the encoders' own default, the plain code, and one between
    cap = 0 if tiled or fmt != "e4m3" else rng.choice([0, 0, 15, 10])
    if op == "batch" and rng.random() < 0.5:
        return {"op": op, "fmt": fmt, "set": rng.choice(["llm8b", "moe"] if tiled else ["llm8b", "dit", "moe"]), "copies": 1,
                "take": _log(rng, 2, 32), "cap": cap, "tiled": tiled}
    rows, cols = _shape(rng, tiled)
    case = {"op": op, "fmt": fmt, "rows": rows, "cols": cols, "cap": cap, "tiled": tiled}
    if op == "batch":
        case["copies"] = _log(rng, 2, 24) if rows * cols < 1 << 24 else rng.randint(2, 4)
    return case


def _shapes(case):
    if case["op"] == "grouped":
        return [(r, c) for _, r, c in MOE_SHAPES] * case["experts"]
    if case["op"] != "batch":
        return [(case["rows"], case["cols"])]
    one = {"llm8b": synth.LLM8B_SHAPES, "dit": synth.DIT_SHAPES, "moe": MOE_SHAPES}.get(case.get("set"), [("w", case.get("rows"), case.get("cols"))])
    shapes = [(r, c) for _, r, c in one] * case["copies"]
    return [shapes[i % len(shapes)] for i in range(case.get("take", len(shapes)))]      # take: so many tensors, over and over


def _weights(case, seed):
    """The raw tensors, one at a time."""
    fmt = case.get("fmt", "e4m3")
    dit = case.get("set") == "dit"
    for i, (r, c) in enumerate(_shapes(case)):
        # tail index and scale differ from matrix to matrix as in the configurations (1.6 .. 2.0; 0.01 .. 0.03)
        alpha = 1.9 if dit else 1.6 + 0.1 * ((i + seed) % 5)
        scale = 0.015 if dit else 0.01 + 0.005 * ((i + seed) % 4)
        if fmt == "bf16":
            yield synth.make_bf16(r, c, alpha, scale, seed, i, DEV).view(torch.bfloat16)
        elif fmt == "e5m2":
            yield synth.make_e5m2(r, c, alpha, scale, seed, i, DEV)
        else:
            yield synth.make_weight(r, c, alpha, scale, seed, i, "tensor" if dit else "block128", DEV)


def _encode(case, w):
    fmt = case.get("fmt", "e4m3")
    if fmt == "e4m3":
        tiled = case["op"] in ("gemm", "grouped") or case["tiled"]
        hdr, blob = ecf8.ecf8_encode_gpu(w, max_code_len=case.get("cap", 0), lane_syms=64 if tiled else 0, tile_rows=16 if tiled else 0)
    else:
        hdr, blob = ecfw.ecfw_encode_gpu(ecfw.FMT_BF16 if fmt == "bf16" else ecfw.FMT_E5M2, w, max_code_len=case.get("cap", 0))
    return hdr, blob.clone()                     # keep the blob's bytes, not the worst-case buffer they were written to


def _scales(rows, cols, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return torch.rand((rows, cols) if cols else (rows,), generator=g, device=DEV) * 0.01 + 0.001


def _operands(case, seed):
    """Per product: X and the scales (or None)."""
    out = []
    for i, (rows, cols) in enumerate(_shapes(case)):
        x = synth.activations(case["m"], cols, seed * 1000 + i, DEV)
        ws = xs = None
        way = case.get("way", "scaled" if case.get("scaled") else "fp8")
        if way.startswith("scaled"):
            ws = _scales((rows + 127) // 128, cols // 128, seed + i)
            xs = _scales(case["m"], cols // 128 if way == "scaled_groups" else 0, seed + i + 500)
        out.append((x, ws, xs))
    return out


def _nbytes(t):
    return t.numel() * t.element_size()


def prepare(case, seed):
    op, fmt = case["op"], case.get("fmt", "e4m3")
    if op == "encode":
        # the blob goes to a buffer of the program's own, with room for the worst of these weights; what it does not fill stays zero
        w = next(_weights(case, seed))
        room = (_nbytes(w) + _nbytes(w) // 4 + (1 << 17)) // 256 * 256
        return {"op": op, "fmt": fmt, "w": w, "cap": case["cap"], "tiled": case["tiled"], "out": torch.zeros(room, dtype=torch.uint8, device=DEV)}
    hdrs, blobs, sizes = [], [], []
    for w in _weights(case, seed):
        h, b = _encode(case, w)
        hdrs.append(h)
        blobs.append(b)
        sizes.append(_nbytes(w))
        del w
    if op == "gemm":
        (x, ws, xs), = _operands(case, seed)
        state = {"op": op, "way": case["way"], "hdr": hdrs[0], "blob": blobs[0], "x": x, "ws": ws, "xs": xs}
        state["y"] = torch.empty((case["m"], case["rows"]), dtype=torch.float32, device=DEV)
        if case["way"] == "splitk":
            state["work"] = ecf8.gemm_splitk_workspace(case["rows"], case["cols"], case["m"], DEV)
        return state
    if op == "grouped":
        members = []
        for h, b, (x, ws, xs) in zip(hdrs, blobs, _operands(case, seed)):
            m = {"hdr": h, "blob": b, "x": x}
            if ws is not None:
                m.update(w_scale=ws, x_scale=xs)
            members.append(m)
        return {"op": op, "group": ecf8.GemmGroup(members)}
    # the layer buffer: tensors one behind the other at multiples of 256 bytes, as the just-in-time manager lays them out
    at = [0]
    for n in sizes:
        at.append((at[-1] + n + 255) // 256 * 256)
    out = torch.zeros(at[-1], dtype=torch.uint8, device=DEV)
    outs = [out[a:a + n] for a, n in zip(at, sizes)]
    if op == "decode":
        return {"op": op, "fmt": fmt, "hdr": hdrs[0], "blob": blobs[0], "out": out, "view": outs[0]}
    batch = ecf8.Batch(hdrs, blobs, outs) if fmt == "e4m3" else ecfw.WBatch(hdrs, blobs, outs)
    return {"op": op, "fmt": fmt, "batch": batch, "out": out}


def run(state):
    op = state["op"]
    if op == "decode":
        if state["fmt"] == "e4m3":
            ecf8.ecf8_decode(state["hdr"], state["blob"], state["view"])
        else:
            ecfw.ecfw_decode(state["blob"], state["hdr"], state["view"])
        return state["out"]
    if op == "batch":
        if state["fmt"] == "e4m3":
            ecf8.ecf8_decode_batched(state["batch"])
        else:
            ecfw.ecfw_decode_batched(state["batch"])
        return state["out"]
    if op == "encode":
        if state["fmt"] == "e4m3":
            ecf8.ecf8_encode_gpu(state["w"], max_code_len=state["cap"], lane_syms=64 if state["tiled"] else 0,
                                 tile_rows=16 if state["tiled"] else 0, d_blob=state["out"])
        else:
            ecfw.ecfw_encode_gpu(ecfw.FMT_BF16 if state["fmt"] == "bf16" else ecfw.FMT_E5M2, state["w"], max_code_len=state["cap"],
                                 d_blob=state["out"])
        return state["out"]
    if op == "grouped":
        return ecf8.ecf8_gemm_fp8_grouped(state["group"])
    way, hdr, blob, x, y = state["way"], state["hdr"], state["blob"], state["x"], state["y"]
    if way == "fp8":
        return ecf8.ecf8_gemm_fp8(hdr, blob, x, y)
    if way == "exact":
        return ecf8.ecf8_gemm_fp8_exact(hdr, blob, x, d_y=y)
    if way == "splitk":
        return ecf8.ecf8_gemm_fp8_splitk(hdr, blob, x, state["work"], d_y=y)
    return ecf8.ecf8_gemm_fp8_scaled(hdr, blob, x, state["ws"], state["xs"], y)


def work(case):
    """Decode reads the blob and writes the tensor, encode the other way round; a product reads W's blob, X and its scales
    once and writes Y.  The codec has no floating-point work."""
    fmt = case.get("fmt", "e4m3")
    elems = sum(r * c for r, c in _shapes(case))
    if case["op"] in ("gemm", "grouped"):
        m = case["m"]
        scaled = 4 * elems // 16384 if case.get("scaled") or case.get("way", "").startswith("scaled") else 0
        io = sum(m * c + 4 * m * r for r, c in _shapes(case))
        return {"bytes": RATIO["tiled"] * elems + io + scaled, "flops": 2.0 * m * elems}
    raw = elems * (2 if fmt == "bf16" else 1)
    key = fmt
    if fmt == "e4m3":
        key = "tiled" if case["tiled"] else "plain" if case["cap"] > 7 else "dit" if case.get("set") == "dit" else "e4m3"
    return {"bytes": raw * (1 + RATIO[key]), "flops": 0}


def tolerance(case):
    """Bytes are exact: the codec is lossless, and a container is one sequence of bytes.  The products' sums are fp32; the
    FP8 matrix core drops bits that lie 13 places below the largest product of a group of eight, the F16 one does not.
    Measured against 64 bits over the sizes that draw() gives: 5e-5 and 1e-7; allowed: four times that."""
    if case["op"] not in ("gemm", "grouped"):
        return "exact"
    return {"rel": 5e-7} if case.get("way") == "exact" else {"rel": 2e-4}


def exact(case, seed):
    """The tensors themselves where the call decodes; the product of the dequantised operands in 64 bits where it multiplies."""
    if case["op"] == "encode":
        return None
    if case["op"] in ("decode", "batch"):
        out = []
        for w in _weights(case, seed):
            b = w.contiguous().reshape(-1).view(torch.uint8)
            out.append(torch.nn.functional.pad(b, (0, -b.numel() % 256)))
        return torch.cat(out)
    ys = []
    for w, (x, ws, xs) in zip(_weights(case, seed), _operands(case, seed)):
        wf = w.view(torch.float8_e4m3fn).double()
        xf = x.view(torch.float8_e4m3fn).double()
        if ws is not None:
            wf *= ws.double().repeat_interleave(128, 0)[:wf.shape[0]].repeat_interleave(128, 1)
            xf *= xs.double()[:, None] if xs.dim() == 1 else xs.double().repeat_interleave(128, 1)
        ys.append(xf @ wf.T)
    return ys if case["op"] == "grouped" else ys[0]
