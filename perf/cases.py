"""Timed cases: the calls an actor update makes through the binding, over the sizes it meets.

Per microbatch a trainer forms the GRPO coefficients, encodes its L units, scores
their exposure and risk, allocates H/L/R, and in backward reconstructs L units or
consumes them directly (weight gradient, adapter gradient, gated-MLP backward).
Each listed case is one of these calls at a size of that work; the first is the
whole chain on a small batch.  Widths are those of the package's workloads (896,
3584, 4096, 14336, 18944 and the 512-wide key/value projection that goes with
3584); token counts run from a thousand to a complete 16384-token microbatch, and
drawn cases take odd ones.

prepare() keeps what a trainer keeps between steps (output buffers, the workspaces
that a call requires); calls whose workspace the binding takes by itself are made
without one.
"""
import math

import numpy as np
import torch

from paper_2609_33570_amd import hilore as hl
from paper_2609_33570_amd import workloads as wl

DEV = "cuda"
CLIP, ADV_EPS = 0.2, 1e-6
EPS_ALPHA, EPS_REL = 1e-8, 1e-8
N_GRID = 1024
QMAX = {"int8": 127.0, "e4m3fn": 448.0}
LARGEST_FLOPS = 2.0 * 16384 * 3584 * 18944  # of a drawn contraction
LARGEST_ELEMS = 16384 * (3584 + 18944)      # of a drawn streaming call


# ------------------------------------------------------------------- cases --
def listed():
    return [
        # a small batch through every step: launches and host work count
        {"name": "microbatch_small", "kind": "chain", "P": 4, "G": 8, "T": 32, "cols": 896,
         "n": 256, "code": "int8", "block": 128},
        # coefficients of a complete rollout batch (padded, K3 term, N counted in the call)
        {"name": "coeffs_rollout", "kind": "coeffs", "P": 64, "G": 16, "T": 4096, "pad": 0.3,
         "beta": 1e-3, "given_n": False},
        # post-forward encode of one layer's hidden state and MLP intermediate, with row sums
        {"name": "encode_layer", "kind": "encode", "rows": 16384, "cols": 3584, "units": 1,
         "cols2": 18944, "units2": 1, "code": "e4m3fn", "block": 128},
        # batched reconstruction of a plan's L units (a third of a 28-layer plan's 78)
        {"name": "decode_plan", "kind": "decode", "rows": 16384, "cols": 3584, "units": 26,
         "cols2": 0, "units2": 0, "code": "int8", "block": 64},
        # exposure and risk of all L units of a 28-layer plan
        {"name": "risk_plan", "kind": "risk", "rows": 16384, "units": 78, "pad": 0.3},
        # weight gradient of a square projection
        {"name": "wgrad_4096", "kind": "wgrad", "K": 16384, "M": 4096, "N": 4096,
         "code": "e4m3fn", "block": 128, "accumulate": False},
        # weight gradient of the gate/up projection, accumulated over microbatches
        {"name": "wgrad_gate", "kind": "wgrad", "K": 16384, "M": 3584, "N": 18944,
         "code": "int8", "block": 64, "accumulate": True},
        # weight gradient of a key/value projection over a ragged microbatch, literal cast codes
        {"name": "wgrad_kv", "kind": "wgrad", "K": 11987, "M": 3584, "N": 512,
         "code": "e4m3fn_cast", "block": 0, "accumulate": True},
        # rank-16 adapter of the down projection (its input is the MLP intermediate)
        {"name": "lora_down", "kind": "lora", "K": 16384, "M": 18944, "r": 16,
         "code": "e4m3fn", "block": 128, "accumulate": True},
        # three rank-16 adapters that share the hidden state (q, k, v), ragged tokens
        {"name": "lora_qkv", "kind": "lora", "K": 13001, "M": 3584, "r": 48,
         "code": "int8", "block": 64, "accumulate": True},
        # gated-MLP backward with the gate activation in L
        {"name": "swiglu_gate", "kind": "swiglu", "rows": 16384, "cols": 18944,
         "code": "e4m3fn", "block": 128, "gate_l": True, "up_l": False},
        # joint H/L/R allocation of a 28-layer model's 196 units on the paper's grid
        {"name": "allocate_model", "kind": "allocate", "layers": 28, "tokens": 16384},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _code(rng):
    code = rng.choice(["int8", "e4m3fn", "e4m3fn", "e4m3fn_cast"])
    return code, 0 if code == "e4m3fn_cast" else rng.choice([32, 64, 128, 128, 256])


def _width(rng, block, lo=256, hi=18944, step=16):
    """A feature width: one of the models' or any multiple of the block (of `step` with cast codes)."""
    b = max(block, step)
    if rng.random() < 0.5:
        w = rng.choice([w for w in (896, 3584, 4096, 14336, 18944) if lo <= w <= hi])
    else:
        w = _log(rng, lo, hi)
    return max(b, (w + b // 2) // b * b)


def draw(rng):
    kind = rng.choice(["chain", "coeffs", "encode", "decode", "risk", "wgrad", "wgrad", "wgrad",
                       "lora", "lora", "swiglu", "allocate"])
    if kind == "chain":
        code, block = rng.choice([("int8", 128), ("int8", 64), ("e4m3fn", 128), ("e4m3fn", 32)])
        return {"kind": kind, "P": rng.randint(1, 6), "G": rng.choice([4, 5, 8, 16]),
                "T": rng.randint(17, 96), "cols": _width(rng, block, 256, 4096),
                "n": 8 * rng.randint(4, 128), "code": code, "block": block}
    if kind == "coeffs":
        G = rng.choice([4, 7, 8, 16, 32])
        T = _log(rng, 32, 4100)
        slots = _log(rng, 1 << 10, 1 << 22)
        return {"kind": kind, "P": max(1, slots // (G * T)), "G": G, "T": T,
                "pad": rng.choice([0.0, 0.1, 0.3]), "beta": rng.choice([0.0, 1e-3]),
                "given_n": rng.random() < 0.4}
    code, block = _code(rng)
    if kind in ("encode", "decode"):
        step = 1 if code == "e4m3fn_cast" else 16
        cols = _width(rng, block, step=step)
        rows = _log(rng, 256, 16384)
        units = rng.randint(1, 12)
        while rows * cols * units > LARGEST_ELEMS:
            rows, units = max(1, rows // 2), max(1, units - 1)
        return {"kind": kind, "rows": rows, "cols": cols, "units": units, "cols2": 0, "units2": 0,
                "code": code, "block": block}
    if kind == "risk":
        return {"kind": kind, "rows": _log(rng, 256, 32768), "units": rng.randint(1, 130),
                "pad": rng.choice([0.0, 0.3])}
    if kind == "wgrad":
        M, K = _width(rng, block), _log(rng, 512, 16384)
        N = (rng.choice([512, 896, 1024, 3584, 4096, 14336, 18944]) if rng.random() < 0.6
             else 8 * _log(rng, 32, 2368))
        while 2.0 * K * M * N > LARGEST_FLOPS:
            K //= 2
        return {"kind": kind, "K": K, "M": M, "N": N, "code": code, "block": block,
                "accumulate": rng.random() < 0.5}
    if kind == "lora":
        return {"kind": kind, "K": _log(rng, 512, 16384), "M": _width(rng, block),
                "r": rng.choice([8, 16, 16, 32, 32, 48, 64, 80]), "code": code, "block": block,
                "accumulate": rng.random() < 0.5}
    if kind == "swiglu":
        cols = _width(rng, block, 896, 18944)
        rows = _log(rng, 256, 16384)
        gate = rng.random() < 0.6
        return {"kind": kind, "rows": rows, "cols": cols, "code": code, "block": block,
                "gate_l": gate, "up_l": not gate or rng.random() < 0.5}
    return {"kind": "allocate", "layers": rng.randint(2, 28), "tokens": _log(rng, 512, 16384)}


# ------------------------------------------------------------------ inputs --
def _empty(shape, dtype):
    return torch.empty(shape, dtype=dtype, device=DEV)


def _f32(*shape):
    return _empty(shape, torch.float32)


def _u8(*shape):
    return _empty(shape, torch.uint8)


def _bf16(*shape):
    return _empty(shape, torch.bfloat16)


def _gen(seed, stream):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 1000003 + stream)
    return g


def _activation(rows, cols, seed, stream):
    """A decoder activation: N(0, 1) with 0.5% of the channels x30, bf16; rows padded to 16 bytes."""
    ld = (cols + 7) // 8 * 8
    x = wl.activation_device(rows, ld, int(seed) * 1009 + stream, outliers=("channels", 0.005, 30.0))
    return x[:, :cols]


def _dense(rows, cols, sigma, seed, stream):
    z = torch.randn((rows, cols), generator=_gen(seed, stream), device=DEV)
    return z.mul_(sigma).to(torch.bfloat16)


def _scales(rows, cols, block):
    return _f32(rows, cols // block) if block else None


def _stored(rows, cols, code, block, seed, stream, x=None):
    """Codes and scales of an activation, as the forward pass left them."""
    x = _activation(rows, cols, seed, stream) if x is None else x
    codes, scales = _u8(rows, cols), _scales(rows, cols, block)
    hl.hilore_compress([hl.unit_desc(x=x, codes=codes, scales=scales)], code, block)
    return codes, scales


def _tokens(c, seed):
    R, T = c["P"] * c["G"], c["T"]
    rew, new, old, mask = wl.grpo_batch_device(c["P"], c["G"], T, int(seed), pad_frac=c.get("pad") or None)
    ref = None
    if c.get("beta"):
        ref = old + 0.05 * torch.randn(R * T, generator=_gen(seed, 7), device=DEV)
    return rew, new, old, ref, mask


def _shapes(c):
    return [(c["rows"], c["cols"])] * c["units"] + [(c["rows"], c["cols2"])] * c["units2"]


def prepare(case, seed):
    c = dict(case)
    s = {"c": c, "kind": c["kind"]}
    kind = c["kind"]
    if kind in ("coeffs", "chain"):
        s["tok"] = _tokens(c, seed)
        R, n = c["P"] * c["G"], c["P"] * c["G"] * c["T"]
        s["out"] = {"adv": _f32(R), "ratio": _f32(n), "flags": _u8(n), "coeff": _f32(n)}
        s["n_norm"] = 0.0
        if c.get("given_n"):
            mask = s["tok"][4]
            s["n_norm"] = float(n if mask is None else int(mask.sum()))
    if kind == "chain":
        rows, cols, block = n, c["cols"], c["block"]
        s["x"] = _activation(rows, cols, seed, 1)
        s["dy"] = _dense(rows, c["n"], 0.02, seed, 2)
        s["out"].update(codes=_u8(rows, cols), scales=_scales(rows, cols, block),
                        ss_x=_f32(rows), ss_err=_f32(rows), score=_f32(3),
                        xhat=_bf16(rows, cols), dw=_f32(cols, c["n"]))
    elif kind in ("encode", "decode"):
        block, s["units"], s["out"] = c["block"], [], []
        for i, (rows, cols) in enumerate(_shapes(c)):
            x = _activation(rows, cols, seed, i)
            if kind == "encode":
                o = {"codes": _u8(rows, cols), "scales": _scales(rows, cols, block),
                     "ss_x": _f32(rows), "ss_err": _f32(rows)}
                u = hl.unit_desc(x=x, codes=o["codes"], scales=o["scales"], row_ss_x=o["ss_x"],
                                 row_ss_err=o["ss_err"])
                s.setdefault("keep", []).append(x)
            else:
                codes, scales = _stored(rows, cols, c["code"], block, seed, i, x)
                o = {"xhat": _bf16(rows, cols)}
                u = hl.unit_desc(codes=codes, scales=scales, xhat=o["xhat"])
                s.setdefault("keep", []).append((codes, scales))
            s["units"].append(u)
            s["out"].append(o)
        s["out"] = [o[k] for o in s["out"] for k in o if o[k] is not None]
    elif kind == "risk":
        n, U = c["rows"], c["units"]
        g = _gen(seed, 3)
        width = [wl.UnitShape(str(u), n, 18944 if u % 7 > 3 else 3584) for u in range(U)]
        # row sums as the encoder leaves them: chi-square like sums of squares, a 2% row error
        ss_x = torch.stack([w.cols * (1.0 + 0.1 * torch.randn(n, generator=g, device=DEV)).abs_()
                            for w in width])
        ss_err = ss_x * 4e-4 * (0.5 + torch.rand((U, n), generator=g, device=DEV))
        s["coeff"] = torch.randn(n, generator=g, device=DEV).mul_(1e-4)
        s["mask"] = None
        if c["pad"]:
            s["mask"] = (torch.rand(n, generator=g, device=DEV) >= c["pad"]).to(torch.uint8)
            s["coeff"] *= s["mask"]
        pad = (n + 3) // 4 * 4  # 16-byte rows
        s["ss_x"], s["ss_err"] = (torch.nn.functional.pad(t, (0, pad - n)).contiguous()
                                  for t in (ss_x, ss_err))
        s["units"] = [hl.unit_desc(row_ss_x=s["ss_x"][u][:n], row_ss_err=s["ss_err"][u][:n], rows=n,
                                   cols=w.cols, ld=w.cols) for u, w in enumerate(width)]
        s["width"] = [w.cols for w in width]
        s["out"] = {"exposure": _f32(U), "risk": _f32(U), "rel_err": _f32(U)}
    elif kind == "wgrad":
        s["codes"], s["scales"] = _stored(c["K"], c["M"], c["code"], c["block"], seed, 1)
        s["dy"] = _dense(c["K"], c["N"], 0.02, seed, 2)
        s["dw0"] = torch.randn((c["M"], c["N"]), generator=_gen(seed, 3), device=DEV)
        s["dw"] = s["dw0"] if c["accumulate"] else _f32(c["M"], c["N"])
    elif kind == "lora":
        s["codes"], s["scales"] = _stored(c["K"], c["M"], c["code"], c["block"], seed, 1)
        s["dh"] = _dense(c["K"], c["r"], 0.02, seed, 2)
        s["da"] = torch.randn((c["r"], c["M"]), generator=_gen(seed, 3), device=DEV)
        s["ws"] = _u8(hl.hilore_lora_grad_workspace_bytes(c["K"], c["M"], c["r"]))
    elif kind == "swiglu":
        rows, cols, block = c["rows"], c["cols"], c["block"]
        g, u = (_activation(rows, cols, seed, i) for i in (1, 2))
        s["dh"] = _dense(rows, cols, 0.02, seed, 3)
        s["ops"] = []
        for x, low in ((g, c["gate_l"]), (u, c["up_l"])):
            if low:
                codes, scales = _stored(rows, cols, c["code"], block, seed, 0, x)
                s["ops"].append((None, codes, scales))
            else:
                s["ops"].append((x, None, None))
        s["gate"], s["up"] = (hl.unit_desc(x=x, codes=k, scales=t) for x, k, t in s["ops"])
        s["out"] = {"dgate": _bf16(rows, cols), "dup": _bf16(rows, cols)}
    elif kind == "allocate":
        inst = _instance(c, seed)
        s["inst"] = inst
        s["dev"] = [torch.from_numpy(np.ascontiguousarray(a)).to(DEV) for a in inst.arrays()]
        s["out"] = {"action": _u8(inst.U), "totals": _empty(3, torch.float64),
                    "jk": _empty(2, torch.int64)}
        s["ws"] = _u8(hl.hilore_allocate_workspace_bytes(inst.U, N_GRID, N_GRID))
    return s


def _instance(c, seed):
    return wl.alloc_instance(wl.qwen2_7b_unit_mix(c["layers"], c["tokens"]), int(seed))


# --------------------------------------------------------------------- run --
def _coeffs(s):
    c, o = s["c"], s["out"]
    rew, new, old, ref, mask = s["tok"]
    hl.hilore_grpo_coeffs(rew, new, old, ref, mask, c["P"], c["G"], c["T"], CLIP, ADV_EPS,
                          c.get("beta", 0.0), s["n_norm"], o["adv"], o["ratio"], o["flags"],
                          o["coeff"])


def run(state):
    s = state
    c, kind = s["c"], s["kind"]
    if kind == "coeffs":
        _coeffs(s)
        return s["out"]
    if kind == "chain":
        o, block, code = s["out"], c["block"], c["code"]
        rows, cols = o["codes"].shape
        unit = hl.unit_desc(x=s["x"], codes=o["codes"], scales=o["scales"], xhat=o["xhat"],
                            row_ss_x=o["ss_x"], row_ss_err=o["ss_err"])
        hl.hilore_compress([unit], code, block)
        _coeffs(s)
        sc = o["score"]
        hl.hilore_unit_exposure_risk(o["coeff"], s["tok"][4], rows, [unit], EPS_ALPHA, EPS_REL,
                                     sc[0:1], sc[1:2], sc[2:3])
        hl.hilore_decompress([unit], code, block)
        hl.hilore_dequant_wgrad(o["codes"], o["scales"], code, block, s["dy"], o["dw"], rows, cols,
                                c["n"], False)
        return o
    if kind == "encode":
        hl.hilore_compress(s["units"], c["code"], c["block"])
        return s["out"]
    if kind == "decode":
        hl.hilore_decompress(s["units"], c["code"], c["block"])
        return s["out"]
    if kind == "risk":
        o = s["out"]
        hl.hilore_unit_exposure_risk(s["coeff"], s["mask"], c["rows"], s["units"], EPS_ALPHA,
                                     EPS_REL, o["exposure"], o["risk"], o["rel_err"])
        return o
    if kind == "wgrad":
        hl.hilore_dequant_wgrad(s["codes"], s["scales"], c["code"], c["block"], s["dy"], s["dw"],
                                c["K"], c["M"], c["N"], c["accumulate"])
        return s["dw"]
    if kind == "lora":
        hl.hilore_dequant_lora_grad(s["codes"], s["scales"], c["code"], c["block"], s["dh"], s["da"],
                                    c["K"], c["M"], c["r"], _lora_scale(c), c["accumulate"], s["ws"])
        return s["da"]
    if kind == "swiglu":
        o = s["out"]
        hl.hilore_dequant_swiglu_bwd(s["gate"], s["up"], c["code"], c["block"], s["dh"], o["dgate"],
                                     o["dup"])
        return o
    o, inst = s["out"], s["inst"]
    hl.hilore_allocate(*s["dev"], inst.m_res, inst.delta_b, N_GRID, N_GRID, o["action"],
                       o["totals"], o["jk"], s["ws"])
    return o


def _lora_scale(c):
    return 32.0 / 16.0  # alpha / rank of each adapter


# ---------------------------------------------------------- work, tolerance --
def _code_bytes(rows, cols, block):
    return rows * cols * (1.0 + (4.0 / block if block else 0.0))


def work(case):
    c = case
    kind, block = c["kind"], c.get("block", 0)
    if kind in ("coeffs", "chain"):
        R = c["P"] * c["G"]
        n = R * c["T"]
        b = 8.0 * R + n * (8 + 9 + (1 if c.get("pad") else 0) + (4 if c.get("beta") else 0))
        if kind == "coeffs":
            return {"bytes": b, "flops": 0.0}
        w = _code_bytes(n, c["cols"], block)
        b += 2.0 * n * c["cols"] + w + 8.0 * n                    # encode with row sums
        b += w + 2.0 * n * c["cols"]                              # decode
        b += 12.0 * n + 12                                        # exposure and risk
        b += w + 2.0 * n * c["n"] + 4.0 * c["cols"] * c["n"]      # weight gradient
        return {"bytes": b, "flops": 2.0 * n * c["cols"] * c["n"]}
    if kind in ("encode", "decode"):
        b = 0.0
        for rows, cols in _shapes(c):
            b += 2.0 * rows * cols + _code_bytes(rows, cols, block)
            b += 8.0 * rows if kind == "encode" else 0.0
        return {"bytes": b, "flops": 0.0}
    if kind == "risk":
        return {"bytes": c["rows"] * (8.0 * c["units"] + 4 + (1 if c["pad"] else 0)) + 12.0 * c["units"],
                "flops": 0.0}
    if kind == "wgrad":
        K, M, N = c["K"], c["M"], c["N"]
        return {"bytes": _code_bytes(K, M, block) + 2.0 * K * N + (8.0 if c["accumulate"] else 4.0) * M * N,
                "flops": 2.0 * K * M * N}
    if kind == "lora":
        K, M, r = c["K"], c["M"], c["r"]
        return {"bytes": _code_bytes(K, M, block) + 2.0 * K * r + (8.0 if c["accumulate"] else 4.0) * M * r,
                "flops": 2.0 * K * M * r}
    if kind == "swiglu":
        rows, cols = c["rows"], c["cols"]
        b = 6.0 * rows * cols
        for low in (c["gate_l"], c["up_l"]):
            b += _code_bytes(rows, cols, block) if low else 2.0 * rows * cols
        return {"bytes": b, "flops": 0.0}
    U = 7 * c["layers"]
    # the table of one unit after the other: one candidate per action and state
    return {"bytes": 43.0 * U + 40, "flops": 4.0 * U * (N_GRID + 1) ** 2}


def tolerance(case):
    kind = case["kind"]
    if kind in ("decode", "allocate"):
        return "exact"
    if kind == "swiglu":
        return {"rel": 4e-3}   # one bf16 rounding of each output
    if kind in ("wgrad", "chain"):
        return {"rel": 4e-6}   # fp32 accumulation over the tokens (8e-7 from fp64 at 16384)
    if kind == "lora":
        return {"rel": 1e-6}   # the same in parts (2e-7 from fp64)
    return {"rel": 5e-7, "max": 1e-5}  # fp32 sums and exponentials; codes and flags are exact


# ------------------------------------------------------------------- exact --
def _value(codes, code):
    """Code values in fp64."""
    if code == "int8":
        return codes.view(torch.int8).double()
    return codes.view(torch.float8_e4m3fn).float().double()


def _xhat(codes, scales, code, block):
    """The bf16 reconstruction (one fp32 product, rounded once), as fp64."""
    v = _value(codes, code)
    if block:
        v = (v.float() * scales.repeat_interleave(block, 1)).to(torch.bfloat16).double()
    return v


def _encode(x, code, block):
    """(codes, scale in fp64) of a bf16 block: the codes are defined by fp32 steps."""
    if not block:
        return x.contiguous().to(torch.float8_e4m3fn).view(torch.uint8), None
    xf = x.float().reshape(x.shape[0], -1, block)
    amax = xf.abs().amax(2, keepdim=True)
    live = amax >= 2.0 ** -64
    q = torch.where(live, torch.full_like(amax, QMAX[code]) / amax, torch.zeros_like(amax))
    v = xf * q
    if code == "int8":
        codes = v.round().clamp_(-127, 127).to(torch.int8).view(torch.uint8)
    else:
        codes = v.clamp_(-448, 448).to(torch.float8_e4m3fn).view(torch.uint8)
    scale = torch.where(live, amax.double() / QMAX[code], torch.zeros_like(amax, dtype=torch.float64))
    return codes.reshape(x.shape), scale[..., 0]


def _exact_encode(x, code, block):
    scales, ss_x, ss_err = [], [], []
    for part in x.split(2048):
        codes, sc = _encode(part, code, block)
        xd = part.double()
        e = _xhat(codes, None if sc is None else sc.float(), code, block) - xd
        ss_x.append(xd.square().sum(1))
        ss_err.append(e.square().sum(1))
        scales.append(sc)
    return (torch.cat(scales) if block else None), torch.cat(ss_x), torch.cat(ss_err)


def _exact_coeffs(c, tok, n_norm):
    rew, new, old, ref, mask = tok
    R, T = c["P"] * c["G"], c["T"]
    r = rew.double().reshape(c["P"], c["G"])
    adv = (r - r.mean(1, keepdim=True)) / (r.std(1, unbiased=False, keepdim=True) + ADV_EPS)
    adv = adv.reshape(R, 1)
    m = torch.ones(R, T, device=DEV, dtype=torch.float64) if mask is None else (mask != 0).double().reshape(R, T)
    n = n_norm if n_norm > 0 else float(m.sum())
    delta = (new - old).reshape(R, T)  # the clip decision is made on this fp32 difference
    hi, lo = np.float32(math.log1p(np.float32(CLIP))), np.float32(math.log1p(-float(np.float32(CLIP))))
    chi = torch.where(adv >= 0, delta <= float(hi), delta >= float(lo))
    ratio = torch.exp(new.double() - old.double()).reshape(R, T)
    w = -torch.where(chi, ratio * adv, torch.zeros_like(ratio))
    if ref is not None:
        w = w - c["beta"] * torch.expm1(ref.double() - new.double()).reshape(R, T)
    coeff = w * m / max(n, 1.0)
    return {"adv": adv.reshape(-1), "ratio": ratio.reshape(-1), "flags": None, "coeff": coeff.reshape(-1)}


def _exact_risk(coeff, mask, ss_x, ss_err, cols):
    w = coeff.double().abs()
    t = torch.ones_like(w) if mask is None else (mask != 0).double()
    a = (ss_x.double() / cols).sqrt()
    n = t.sum()
    mean = (a * t).sum() / n if float(n) else torch.zeros((), device=DEV, dtype=torch.float64)
    return (float((w * t * (a + EPS_ALPHA)).sum() / (mean + EPS_ALPHA)),
            float((w * t * ss_err.double().sqrt()).sum()),
            float(ss_err.double().sum().sqrt() / (ss_x.double().sum().sqrt() + EPS_REL)))


def _mm_t(a, b):
    """a^T b in fp64, over row chunks."""
    out = torch.zeros((a.shape[1], b.shape[1]), dtype=torch.float64, device=DEV)
    for i in range(0, a.shape[0], 4096):
        out += a[i:i + 4096].t().contiguous() @ b[i:i + 4096].double()
    return out


def _exact_allocate(inst):
    """The dynamic programme over the (memory, risk) grid, one unit after the other."""
    inf = float("inf")
    S = N_GRID + 1
    f = torch.full((S, S), -inf, dtype=torch.float64, device=DEV)  # [risk, memory]
    f[0, 0] = 0.0
    back = []

    def grid(cost, budget):
        c = math.ceil(cost / (budget / N_GRID))
        return int(c) if c <= N_GRID else None

    for u in range(inst.U):
        best, act = f.clone(), torch.zeros((S, S), dtype=torch.uint8, device=DEV)
        bh = bl = rl = 0
        if inst.q[u] == 1 and inst.verified[u] & 2 and inst.tau_h[u] > 0:
            bh = grid(inst.dm_h[u], inst.m_res)
            if bh is not None:
                v = f[:, :S - bh] + inst.tau_h[u]
                up = v > best[:, bh:]
                best[:, bh:][up] = v[up]
                act[:, bh:][up] = 1
        if inst.q[u] in (1, 2) and inst.verified[u] & 4 and inst.tau_l[u] > 0:
            bl, rl = grid(inst.dm_l[u], inst.m_res), grid(inst.psi[u], inst.delta_b)
            if bl is not None and rl is not None:
                v = f[:S - rl, :S - bl] + inst.tau_l[u]
                up = v > best[rl:, bl:]
                best[rl:, bl:][up] = v[up]
                act[rl:, bl:][up] = 2
        back.append((act, bh, bl, rl))
        f = best
    top = f.max()
    k, j = (int(i) for i in (f == top).nonzero()[0])
    jk = [j, k]
    action = np.zeros(inst.U, dtype=np.uint8)
    for u in range(inst.U - 1, -1, -1):
        act, bh, bl, rl = back[u]
        a = int(act[k, j])
        action[u] = a
        if a == 1:
            j -= bh
        elif a == 2:
            j, k = j - bl, k - rl
    mem = risk = 0.0
    for u in range(inst.U):
        mem += inst.dm_h[u] if action[u] == 1 else inst.dm_l[u] if action[u] == 2 else 0.0
        risk += inst.psi[u] if action[u] == 2 else 0.0
    return {"action": action, "totals": np.array([float(top), mem, risk]), "jk": np.array(jk)}


def exact(case, seed):
    c = dict(case)
    s = prepare(c, seed)
    kind = c["kind"]
    if kind == "coeffs":
        return _exact_coeffs(c, s["tok"], s["n_norm"])
    if kind == "chain":
        o = _exact_coeffs(c, s["tok"], 0.0)
        codes, sc = _encode(s["x"], c["code"], c["block"])
        _, ss_x, ss_err = _exact_encode(s["x"], c["code"], c["block"])
        xh = _xhat(codes, sc.float(), c["code"], c["block"])
        o.update(codes=None, scales=sc, ss_x=ss_x, ss_err=ss_err,
                 score=np.array(_exact_risk(o["coeff"], s["tok"][4], ss_x, ss_err, c["cols"])),
                 xhat=_value(codes, c["code"]) * sc.repeat_interleave(c["block"], 1),
                 dw=_mm_t(xh, s["dy"]))
        return o
    if kind == "encode":
        out = []
        for x in s["keep"]:
            sc, ss_x, ss_err = _exact_encode(x, c["code"], c["block"])
            out += [None] + ([sc] if c["block"] else []) + [ss_x, ss_err]
        return out
    if kind == "decode":
        out = []
        for codes, scales in s["keep"]:
            v = _value(codes, c["code"])
            out.append(v * scales.double().repeat_interleave(c["block"], 1) if c["block"] else v)
        return out
    if kind == "risk":
        n = c["rows"]
        rows = [_exact_risk(s["coeff"], s["mask"], s["ss_x"][u][:n], s["ss_err"][u][:n], w)
                for u, w in enumerate(s["width"])]
        e, k, r = (np.array(v) for v in zip(*rows))
        return {"exposure": e, "risk": k, "rel_err": r}
    if kind == "wgrad":
        out = torch.zeros((c["M"], c["N"]), dtype=torch.float64, device=DEV)
        for i in range(0, c["K"], 4096):
            sc = s["scales"][i:i + 4096] if c["block"] else None
            out += _mm_t(_xhat(s["codes"][i:i + 4096], sc, c["code"], c["block"]), s["dy"][i:i + 4096])
        return out + s["dw0"].double() if c["accumulate"] else out
    if kind == "lora":
        out = torch.zeros((c["r"], c["M"]), dtype=torch.float64, device=DEV)
        for i in range(0, c["K"], 4096):
            sc = s["scales"][i:i + 4096] if c["block"] else None
            out += s["dh"][i:i + 4096].double().t().contiguous() @ _xhat(
                s["codes"][i:i + 4096], sc, c["code"], c["block"])
        out *= _lora_scale(c)
        return out + s["da"].double() if c["accumulate"] else out
    if kind == "swiglu":
        dg, du = [], []
        for i in range(0, c["rows"], 2048):
            at = slice(i, i + 2048)
            g, u = (x[at].double() if x is not None else
                    _xhat(k[at], t[at] if t is not None else None, c["code"], c["block"])
                    for x, k, t in s["ops"])
            h = s["dh"][at].double()
            sig = torch.sigmoid(g)
            du.append((h * g * sig).float())
            dg.append((h * u * sig * (1.0 + g * (1.0 - sig))).float())
        return {"dgate": torch.cat(dg), "dup": torch.cat(du)}
    return _exact_allocate(s["inst"])
