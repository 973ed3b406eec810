"""The work a user of this package has it do, as cases that can be timed.

Three kinds:
  layer     the four quantised linears of a decoder layer (fused QKV, O, fused gate/up, down) times `layers`:
            token generation at small M, prompt processing at large M.  `graph` = the launch sequence is
            captured once into a HIP graph and replayed, as a serving loop does; otherwise the plain calls.
  linear    one linear called the plain way, output and scratch allocated by the call.
  quantize  a weight matrix turned into what the GEMM reads: learn the tables, pack, re-lay-out.

Fields of a GEMM case: M rows of activations; bits 4 / 3 / 2; weights "table" (a table per row), "one_table"
(one for the matrix) or "int4" (no table); dtype "bf16" / "f16"; group (weights per scale along K); layout
"plain" / "repacked".  A layer is given by hidden (K of QKV, O, gate/up), qkv (rows of QKV) and ffn.
"""
import torch

import paper_2507_04610_amd as any4
from paper_2507_04610_amd import inputs


def _layer(name, M, layers, hidden=4096, qkv=6144, ffn=14336, bits=4, weights="table", dtype="bf16", group=128,
           layout="plain", graph=True):
    c = {"kind": "layer", "M": M, "layers": layers, "hidden": hidden, "qkv": qkv, "ffn": ffn, "bits": bits,
         "weights": weights, "dtype": dtype, "group": group, "layout": layout, "graph": graph}
    return dict(c, name=name) if name else c


def _linear(name, M, N, K, bits=4, weights="table", dtype="bf16", group=128, layout="plain"):
    c = {"kind": "linear", "M": M, "N": N, "K": K, "bits": bits, "weights": weights, "dtype": dtype, "group": group,
         "layout": layout, "graph": False}
    return dict(c, name=name) if name else c


def _quantize(name, N, K, bits=4, symmetric=False):
    c = {"kind": "quantize", "N": N, "K": K, "bits": bits, "symmetric": symmetric, "iters": 20}
    return dict(c, name=name) if name else c


def listed():
    return [
        # one small linear, one token: what a single call costs
        _linear("linear_1k_m1", 1, 1024, 1024),
        # a ragged shard of a linear with 3-bit weights and a handful of tokens in flight
        _linear("linear_ragged_any3_m5", 5, 5003, 2944, bits=3),
        # token generation, one sequence: four Llama-3-8B layers, so that the weights come from HBM as in a whole model
        _layer("8b_m1", 1, 4),
        # token generation, eight sequences, fp16 models
        _layer("8b_m8_f16", 8, 4, dtype="f16"),
        # token generation, sixteen sequences
        _layer("8b_m16", 16, 4),
        # token generation with many sequences in flight: between the memory-bound and the compute-bound end
        _layer("8b_m64", 64, 4),
        # token generation, one sequence, one Llama-3-70B layer, weights in the offline re-layout
        _layer("70b_m1_repacked", 1, 1, hidden=8192, qkv=10240, ffn=28672, layout="repacked"),
        # a prompt (or a chunk of one) of 512 tokens through one Llama-3-8B layer
        _layer("8b_m512", 512, 1, graph=False),
        # a prompt of 2048 tokens through one Llama-3-8B layer: the largest call
        _layer("8b_m2048", 2048, 1, graph=False),
        # a prompt of odd length through a smaller layer of ragged sizes, groups of 64
        _layer("ragged_m777_g64", 777, 1, hidden=2944, qkv=4421, ffn=7808, group=64, graph=False),
        # converting a checkpoint: the fused QKV matrix of Llama-3-8B ...
        _quantize("quantize_qkv", 6144, 4096),
        # ... and its down projection (long rows)
        _quantize("quantize_down", 4096, 14336),
    ]


def _log(rng, lo, hi):
    """an integer of [lo, hi], its logarithm spread evenly"""
    return min(hi, max(lo, int(round(lo * (hi / lo) ** rng.random()))))


def _option(rng):
    """4 bits, bf16, groups of 128 and a table per row are the common choice; each of the others is in use"""
    r = rng.random()
    if r < 0.40:
        return {}
    if r < 0.52:
        return {"bits": rng.choice((3, 2))}
    if r < 0.64:
        return {"dtype": "f16", "bits": rng.choice((4, 4, 3))}
    if r < 0.74:
        return {"group": rng.choice((64, 64, 256, 512)), "bits": rng.choice((4, 4, 3))}
    if r < 0.82:
        return {"weights": "int4"}
    if r < 0.88:
        return {"weights": "one_table"}
    return {"layout": "repacked", "bits": rng.choice((4, 4, 3, 2))}


def draw(rng):
    kind = rng.choice(("linear", "decode", "decode", "batched", "prefill", "prefill", "quantize"))
    if kind == "quantize":
        K = 128 * _log(rng, 8, 120)
        return _quantize(None, _log(rng, 512, min(28672, 58720256 // K)), K, bits=rng.choice((4, 4, 4, 3, 2)),
                         symmetric=rng.random() < 0.25)
    opt = _option(rng)
    unit = max(128, opt.get("group", 128))
    if kind == "linear":
        M, K = _log(rng, 1, 64), unit * _log(rng, 1024 // unit, 8192 // unit)
        return _linear(None, M, _log(rng, 512, 16384), K, **opt)
    hidden = unit * _log(rng, 2048 // unit, 8192 // unit)
    ffn = unit * max(1, int(hidden * rng.uniform(2.5, 3.6)) // unit)
    qkv = int(hidden * rng.uniform(1.1, 2.0))
    per_layer = hidden * (qkv + hidden + 3 * ffn)
    if kind == "prefill":
        most = 2 * 2048 * 218103808 // (2 * per_layer)   # the work of the largest listed one
        return _layer(None, _log(rng, 129, max(129, min(4096, most))), 1, hidden, qkv, ffn, graph=False, **opt)
    layers = max(1, 872415232 // per_layer)              # the weights of four Llama-3-8B layers
    M = _log(rng, 1, 16) if kind == "decode" else _log(rng, 17, 128)
    return _layer(None, M, layers, hidden, qkv, ffn, **opt)


def _linears(case):
    """(N, K) of every GEMM of one pass"""
    if case["kind"] == "linear":
        return [(case["N"], case["K"])]
    h, f = case["hidden"], case["ffn"]
    return [(case["qkv"], h), (h, h), (2 * f, h), (h, f)] * case["layers"]


def _problem(case, N, K, seed):
    """one linear as a program holds it: packed (and re-laid-out) codes, table, scales, offsets, activations"""
    bits, group = case["bits"], case["group"]
    f16 = case["dtype"] == "f16"
    t = inputs.make_case_device(case["M"], N, K, bits, seed=seed, f16=f16)
    codes = any4.any4_pack(t["codes_u8"], bits)
    scale, offset = t["scale"], t["offset"]
    if group < 128:
        more = inputs.make_case_device(1, N, K, 2, seed=seed + 500000, f16=f16)
        scale = torch.stack((scale, more["scale"]), dim=2).reshape(N, K // group).contiguous()
        offset = torch.stack((offset, more["offset"]), dim=2).reshape(N, K // group).contiguous()
    elif group > 128:
        scale, offset = scale[:, :: group // 128].contiguous(), offset[:, :: group // 128].contiguous()
    lut = None if case["weights"] == "int4" else t["lut"][:1].contiguous() if case["weights"] == "one_table" else t["lut"]
    p = {"x": t["x"], "codes": codes, "lut": lut, "scale": scale, "offset": offset, "out": None, "ws": None}
    if case["layout"] == "repacked":
        p["codes"] = any4.any4_repack(codes, bits)
    if case["graph"]:
        ws = any4.any4_gemm_workspace_bytes(case["M"], N, K, bits)
        p["out"] = torch.empty((case["M"], N), dtype=t["x"].dtype, device=codes.device)
        p["ws"] = torch.empty(max(ws, 16), dtype=torch.uint8, device=codes.device)
    return p


def _gemm(case, p):
    if case["layout"] == "repacked":
        return any4.any4_gemm_repacked(p["x"], p["codes"], p["lut"], p["scale"], p["offset"], case["bits"],
                                       out=p["out"], workspace=p["ws"])
    return any4.any4_gemm(p["x"], p["codes"], p["lut"], p["scale"], p["offset"], case["bits"], out=p["out"],
                          workspace=p["ws"], group=case["group"])


def prepare(case, seed):
    if case["kind"] == "quantize":
        return dict(inputs.make_quant_case_device(case["N"], case["K"], case["bits"], seed=seed), case=case)
    problems = [_problem(case, N, K, seed * 1000 + i) for i, (N, K) in enumerate(_linears(case))]
    state = {"case": case, "problems": problems}
    if case["graph"]:
        for p in problems:
            _gemm(case, p)
        torch.cuda.synchronize()
        state["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(state["graph"]):
            for p in problems:
                _gemm(case, p)
    return state


def run(state):
    case = state["case"]
    if case["kind"] == "quantize":
        q = any4.any4_quantize(state["w"], state["act"], state["u"], case["bits"], case["symmetric"], case["iters"])
        codes = any4.any4_pack(q["codes_u8"], case["bits"])
        return {"codes": codes, "rcodes": any4.any4_repack(codes, case["bits"]), **q}
    if case["graph"]:
        state["graph"].replay()
        return [p["out"] for p in state["problems"]]
    return [_gemm(case, p) for p in state["problems"]]


def work(case):
    if case["kind"] == "quantize":
        N, K, bits = case["N"], case["K"], case["bits"]
        L = 1 << bits
        # in: weights, activations, draws; out: codes as bytes, packed and re-laid-out, tables, scales, offsets, counts
        by = 4 * N * K + 4 * K + 4 * N * L + N * K + N * K * bits // 8 + (N + 15) // 16 * 16 * K * bits // 8 \
            + 2 * N * L + 4 * N * (K // 128) + 4 * N
        # per weight: the scaling, and for every centre of the start its distance and sampling mass
        return {"bytes": by, "flops": N * K * (4 + 4 * L)}
    M, bits = case["M"], case["bits"]
    by = fl = 0
    for N, K in _linears(case):
        table = 0 if case["weights"] == "int4" else (1 if case["weights"] == "one_table" else N) * (1 << bits) * 2
        by += N * K * bits // 8 + table + 2 * N * (K // case["group"]) * 2 + M * K * 2 + M * N * 2
        fl += 2 * M * N * K
    return {"bytes": by, "flops": fl}


def tolerance(case):
    if case["kind"] == "quantize":
        # codes, counts, tables and scales are decided in fp64; only the association of its sums is free, and a
        # value within its rounding of a decision boundary may then fall to the other side (a row in ten thousand)
        return {"rel": 1e-4, "max": 2e-2, "differ": 1e-4}
    # fp32 accumulation, then one rounding to 16 bits: another order of the sums moves an output by at most one
    # unit in the last place (2^-7 of the value in bf16, 2^-10 in fp16)
    return {"rel": 5e-4, "max": 2e-3} if case["dtype"] == "f16" else {"rel": 4e-3, "max": 1e-2}
