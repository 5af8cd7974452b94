"""The work that this framework's users have it do, as cases that can be timed.

Kinds of case (``kind``):
  call    one online call of the masked product for M tokens against one
          prepared weight (protocol.run_call: Init X, mask, server, unmask),
          into call buffers that the program keeps, as a decode or prefill
          loop does;
  linear  one floating-point linear layer through Pi_Sec-Linear
          (SecureLinear.__call__), which allocates its own buffers;
  weight  Init W of one weight (MaskedWeight), once per layer when a model is
          loaded, with the check vectors of the integrity check;
  verify  the integrity check of one server output (protocol.verify), some
          entries of which were changed;
  rotate  the random Hadamard rotation of activations, forward, and the
          inverse rotation of as many others;
  input   the separate client passes of an input that the fused pass does not
          take: quantisation of every row, then the mask pass into digits.

Parameters of the mask (``params``): the sets of synthetic_inputs by name.
Sizes are those of the decode, prefill and decoder-stack workloads, of the
client-overhead sweep, and ragged ones. Every input is made from the seed on
the GPU.
"""
from __future__ import annotations

import math

import torch

import synthetic_inputs as si
from paper_2607_29221_amd import mosaic as m
from paper_2607_29221_amd import protocol as gp
from paper_2607_29221_amd.secure_linear import SecureLinear, rotation_block

PARAMS = {
    "d1": si.PARAMS_PAPER_D1,            # deployed: LWE rank 1536, sigma = 0.5
    "d2": si.PARAMS_PAPER_D2_SPARSE,     # decode workload: one LPN level, no E
    "d2_t80": si.PARAMS_PAPER_D2_T80,
    "d3_t80": si.PARAMS_PAPER_D3_T80,    # Example 4.1 in full
}


def listed():
    return [
        # token-by-token generation, one sequence: an attention projection
        {"name": "call_1tok", "kind": "call", "M": 1, "K": 4096, "N": 4096, "params": "d2"},
        # a few sequences, the MLP's up projection under the deepest mask
        {"name": "call_8tok", "kind": "call", "M": 8, "K": 4096, "N": 14336, "params": "d3_t80"},
        # a full decode batch, the MLP's down projection
        {"name": "call_64tok", "kind": "call", "M": 64, "K": 14336, "N": 4096, "params": "d2"},
        # a short prompt (ragged token count), attention output projection
        {"name": "call_200tok", "kind": "call", "M": 200, "K": 4096, "N": 4608, "params": "d1"},
        # prefill at a 70B layer's up projection: the largest call
        {"name": "call_2048tok", "kind": "call", "M": 2048, "K": 8192, "N": 28672, "params": "d1"},
        # a small model's up projection for four sequences
        {"name": "linear_4tok", "kind": "linear", "M": 4, "K": 2048, "N": 8192, "params": "d1", "bias": True},
        # ragged in every size: a short prompt, a width with 512-long rotation
        # blocks, an odd number of outputs
        {"name": "linear_333tok", "kind": "linear", "M": 333, "K": 4608, "N": 5003, "params": "d1", "bias": False},
        # the decoder stack's fused q|k|v projection, 4 x 1024 tokens
        {"name": "linear_4096tok", "kind": "linear", "M": 4096, "K": 8192, "N": 10240, "params": "d1", "bias": False},
        # loading one weight of a model that decodes under the deepest mask
        {"name": "weight_4096", "kind": "weight", "K": 4096, "N": 4096, "params": "d3_t80", "t": 32},
        # checking a prefill output
        {"name": "verify_2048tok", "kind": "verify", "M": 2048, "K": 8192, "N": 8192, "params": "d1", "t": 32},
        # the rotation workload
        {"name": "rotate_8192", "kind": "rotate", "rows": 4096, "n": 8192, "block": 8192, "kron28": False},
        # rows of an odd length through the separate passes
        {"name": "input_odd", "kind": "input", "rows": 1000, "n": 5003, "qmax": 1997, "noise": True},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _width(rng, lo, hi):
    """A matrix dimension: a multiple of 64 mostly, any number at times."""
    v = _log(rng, lo, hi)
    return v if rng.random() < 0.35 else max(64, 64 * round(v / 64))


def draw(rng):
    kind = rng.choice(("call", "call", "call", "linear", "linear", "weight", "verify", "rotate", "input"))
    if kind == "call":
        M = _log(rng, 1, 2048)
        top = 14336 if M > 512 else 16384
        c = {"M": M, "K": _width(rng, 1024, top), "N": _width(rng, 1024, top),
             "params": rng.choice(("d1", "d2", "d2_t80", "d3_t80"))}
    elif kind == "linear":
        b = 2 ** rng.randint(8, 13)
        c = {"M": _log(rng, 1, 2048), "K": b * rng.choice([q for q in (1, 3, 5, 7, 9, 11) if 1024 <= b * q <= 14336] or [5]),
             "N": _width(rng, 1024, 14336), "params": "d1", "bias": rng.random() < 0.5}
    elif kind == "weight":
        c = {"K": _width(rng, 1024, 6144), "N": _width(rng, 1024, 6144),
             "params": rng.choice(("d1", "d2", "d3_t80")), "t": rng.choice((0, 32))}
    elif kind == "verify":
        c = {"M": _log(rng, 8, 2048), "K": _width(rng, 1024, 8192), "N": 64 * _log(rng, 16, 128),
             "params": "d1", "t": rng.choice((16, 32, 64))}
    elif kind == "rotate":
        if rng.random() < 0.25:
            b = 2 ** rng.randint(8, 10)
            c = {"rows": _log(rng, 64, 4096), "n": 28 * b, "block": b, "kron28": True}
        else:
            b = 2 ** rng.randint(4, 15)
            c = {"rows": _log(rng, 64, 4096), "n": b * max(1, _log(rng, 1024, 28672) // b), "block": b, "kron28": False}
    else:
        c = {"rows": _log(rng, 16, 4096), "n": _width(rng, 512, 16384), "qmax": rng.choice((127, 567, 1997)),
             "noise": rng.random() < 0.7}
    return dict(c, kind=kind)


# ---------------------------------------------------------------------------
# inputs

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) & 0x7FFFFFFFFFFFFFFF)
    return g


def _int8(rows, cols, g):
    return torch.randint(-127, 128, (rows, cols), generator=g, device="cuda", dtype=torch.int8)


def _activations(rows, n, g):
    """N(0, 1) entries, one in a thousand times 50."""
    x = torch.randn((rows, n), generator=g, device="cuda")
    return torch.where(torch.rand((rows, n), generator=g, device="cuda") < 1e-3, 50.0 * x, x)


def _linear_inputs(c, seed):
    g = _gen(seed)
    x = _activations(c["M"], c["K"], g)
    W = torch.randn((c["N"], c["K"]), generator=g, device="cuda").mul_(0.02)
    bias = torch.randn(c["N"], generator=g, device="cuda").mul_(0.1) if c["bias"] else None
    return x, W, bias


def _rotate_inputs(c, seed):
    g = _gen(seed)
    x, y = _activations(c["rows"], c["n"], g), _activations(c["rows"], c["n"], g)
    signs = (2 * torch.randint(0, 2, (c["n"],), generator=g, device="cuda") - 1).to(torch.int8)
    return x, y, signs


def prepare(case, seed):
    c, p = case, PARAMS.get(case.get("params"))
    s = {"case": dict(c)}
    if c["kind"] in ("call", "verify"):
        g = _gen(seed)
        s["A"], W = _int8(c["M"], c["K"], g), _int8(c["N"], c["K"], g)
        s["w"] = gp.MaskedWeight(W, p, seed=seed + 77, weight_id=1, check_vectors=c.get("t", 0))
        s["buf"] = gp.alloc_call(s["w"], c["M"])
        if c["kind"] == "verify":
            gp.run_call(s["w"], s["A"], 5, s["buf"])
            yq = s["buf"].YQ                      # the server's output, changed in a few places
            part = c["M"] * c["N"] // 16
            at = part * torch.arange(16, device="cuda") + torch.randint(0, part, (16,), generator=g, device="cuda")
            yq[at // c["N"], at % c["N"]] += 1 + 2 * torch.randint(0, 2 ** 20, (16,), generator=g, device="cuda",
                                                                   dtype=torch.int32)
    elif c["kind"] == "linear":
        s["x"], W, bias = _linear_inputs(c, seed)
        s["layer"] = SecureLinear(W, p, seed=seed + 77, weight_id=1, bias=bias)
    elif c["kind"] == "weight":
        s["W"], s["seed"] = _int8(c["N"], c["K"], _gen(seed)), seed + 77
    elif c["kind"] == "rotate":
        s["x"], s["y"], s["signs"] = _rotate_inputs(c, seed)
        s["fwd"], s["inv"] = torch.empty_like(s["x"]), torch.empty_like(s["y"])
    else:
        g = _gen(seed)
        s["x"] = _activations(c["rows"], c["n"], g)
        s["u"] = torch.randint(-2 ** 31, 2 ** 31, (c["rows"], c["n"]), generator=g, device="cuda", dtype=torch.int32)
        s["codes"] = torch.empty((c["rows"], c["n"]), dtype=torch.int32, device="cuda")
        s["scale"] = torch.empty(c["rows"], dtype=torch.float32, device="cuda")
        s["dig"] = m.Digits.empty(c["rows"], c["n"])
        s["noise"] = m.rng(seed + 77, 0x50, 5, m.DIST_DGAUSS, sigma=0.5, bound=4) if c["noise"] else None
    return s


def run(s):
    c = s["case"]
    if c["kind"] == "call":
        buf = gp.run_call(s["w"], s["A"], 5, s["buf"])
        return {"Y": buf.Y, "YQ": buf.YQ}
    if c["kind"] == "linear":
        return {"y": s["layer"](s["x"], 5)}
    if c["kind"] == "weight":
        w = gp.MaskedWeight(s["W"], PARAMS[c["params"]], s["seed"], weight_id=1, check_vectors=c["t"])
        out = {"Bext": w.Bext.buf, "Lcat": w.Lcat[0].buf, "Bx": w.Bx.buf}
        for lv, S in w.S.items():
            out["S%d" % lv] = [S.row_ptr, S.col_idx, S.values]
            out["D%d" % lv] = w.D[lv]
        if w.t:
            out["key"] = w.cT.buf
        return out
    if c["kind"] == "verify":
        count = gp.verify(s["w"], c["M"], s["buf"])
        return {"count": count, "diff": s["buf"].check_diff}
    if c["kind"] == "rotate":
        if c["kron28"]:
            m.mosaic_hadamard28_rotate(s["x"], s["fwd"], signs=s["signs"])
            m.mosaic_hadamard28_rotate(s["y"], s["inv"], signs=s["signs"], inverse=True)
        else:
            m.mosaic_hadamard_rotate(s["x"], s["fwd"], block=c["block"], signs=s["signs"])
            m.mosaic_hadamard_rotate(s["y"], s["inv"], block=c["block"], signs=s["signs"], inverse=True)
        return {"fwd": s["fwd"], "inv": s["inv"]}
    m.mosaic_quantize_rows(s["x"], c["qmax"], q=s["codes"], scale=s["scale"])
    m.mosaic_mask(s["codes"], s["u"], s["noise"], c["rows"], c["n"], out_dig=s["dig"])
    return {"codes": s["codes"], "scale": s["scale"], "digits": s["dig"].buf}


# ---------------------------------------------------------------------------
# what a pass cannot do without

def work(case):
    """Bytes: each operand read once (4 bytes of digits or ring word per
    element), each result written once. Operations: 20 int8 ones per ring
    multiply-accumulate (the ten limb products that survive mod 2^32). Of the
    sparse LPN levels of a call with few tokens only the nonzeros count."""
    c = case
    if c["kind"] in ("call", "linear", "weight", "verify"):
        K, N, M, p = c["K"], c["N"], c.get("M", 0), PARAMS[c["params"]]
        r = list(p.ranks)
        R, rd = sum(r), r[-1]
        nnz = [p.lpn_weights[i] if p.lpn_weights else ri / 2.0 ** p.sparse_log2_inv_density
               for i, ri in enumerate(r[:-1])]            # nonzeros per row of each LPN level
    if c["kind"] in ("call", "linear"):
        server = {"bytes": 4.0 * (N + R) * K, "macs": 1.0 * M * (N + R) * K}
        dense = {"bytes": 4.0 * (K + N) * R + 4.0 * N * R, "macs": 1.0 * M * (K + 2 * N) * R}
        sparse = {"bytes": 4.0 * (K + 2 * N) * rd + sum(4.0 * M * t * (K + N) + 8.0 * N * t for t in nnz),
                  "macs": 1.0 * M * (K + 2 * N) * rd + sum(1.0 * M * t * (K + 2 * N) for t in nnz)}
        client = min((dense, sparse), key=lambda w: w["bytes"] / 6e12 + 20 * w["macs"] / 2.8e15)
        io = M * K * (4.0 if c["kind"] == "linear" else 1.0) + 4.0 * M * N
        return {"bytes": server["bytes"] + client["bytes"] + io, "flops": 20.0 * (server["macs"] + client["macs"])}
    if c["kind"] == "weight":
        # U_w and the J_i, one product each per level, and each chain once
        chains = sum(2.0 * K * r[i] * r[i - 1] for i in range(1, len(r)))
        lpn = sum(1.0 * N * K * t for t in nnz)
        macs = N * K * rd + lpn + N * K * R + chains + c["t"] * K * (N + R)
        out = 4.0 * (N + R) * K + 4.0 * N * R + 4.0 * (K + N) * R + sum(4.0 * ri * (K + N) for ri in r[:-1])
        return {"bytes": N * K + out, "flops": 20.0 * macs}
    if c["kind"] == "verify":
        return {"bytes": 4.0 * (M + c["t"]) * (K + N + R) + 4.0 * M * c["t"],
                "flops": 20.0 * c["t"] * M * (K + N + R)}
    e = 1.0 * c["rows"] * c["n"]
    if c["kind"] == "rotate":
        return {"bytes": 16 * e + c["n"], "flops": 2 * e * (math.log2(c["block"]) + (15 if c["kron28"] else 0))}
    return {"bytes": 4 * e + 4 * e + 4 * e + 4 * e, "flops": 4 * e}


def tolerance(case):
    if case["kind"] in ("call", "weight", "verify"):
        return "exact"                     # residues mod 2^32: every order of the sums gives the same words
    if case["kind"] == "linear":
        # codes within fp32 rounding of a tie may differ by one between
        # correct rotations; measured with the codes of a float64 rotation
        return {"rel": 5e-5, "max": 8e-4}
    if case["kind"] == "rotate":
        return {"rel": 5e-7, "max": 4e-6}  # fp32 butterflies in another order
    return {"rel": 1e-6, "max": 1e-6, "differ": 0.0}   # codes: correctly rounded fp32 division


# ---------------------------------------------------------------------------
# the same values in 64 bits

def _hadamard64(x, b):
    rows, n = x.shape
    v = x.double().reshape(rows * (n // b), b)
    h = 1
    while h < b:
        v = v.reshape(-1, b // (2 * h), 2, h)
        v = torch.stack((v[:, :, 0] + v[:, :, 1], v[:, :, 0] - v[:, :, 1]), dim=2)
        h *= 2
    return v.reshape(rows, n)


def _paley28():
    """I + S over GF(27) = GF(3)[t] / (t^3 + 2 t + 1), S = [[0, 1], [-1, Q]]."""
    coef = lambda a: (a % 3, (a // 3) % 3, a // 9)  # noqa: E731

    def mul(a, b):
        p = [0] * 5
        for i, u in enumerate(coef(a)):
            for j, v in enumerate(coef(b)):
                p[i + j] += u * v
        for k in (4, 3):
            p[k - 2] += p[k]
            p[k - 3] += 2 * p[k]
        return p[0] % 3 + 3 * (p[1] % 3) + 9 * (p[2] % 3)

    squares = {mul(a, a) for a in range(1, 27)}
    H = torch.eye(28, dtype=torch.float64)
    H[0, 1:] += 1
    H[1:, 0] -= 1
    for i in range(27):
        for k in range(27):
            d = sum(((u - v) % 3) * 3 ** e for e, (u, v) in enumerate(zip(coef(i), coef(k))))
            if d:
                H[1 + i, 1 + k] += 1 if d in squares else -1
    return H


def exact(case, seed):
    c = case
    if c["kind"] == "call" and PARAMS[c["params"]].noise.kind == "zero":
        g = _gen(seed)                     # without E the protocol returns the plain product
        A, W = _int8(c["M"], c["K"], g), _int8(c["N"], c["K"], g)
        Y = (A.double() @ W.double().t().contiguous()).to(torch.int64)
        return {"Y": ((Y + 2 ** 31) % 2 ** 32 - 2 ** 31).to(torch.int32), "YQ": None}
    if c["kind"] == "linear":
        x, W, bias = _linear_inputs(c, seed)
        y = x.double() @ W.double().t().contiguous()
        return {"y": y if bias is None else y + bias.double()}
    if c["kind"] == "rotate":
        x, y, signs = _rotate_inputs(c, seed)
        d, b, rows, n = signs.double(), c["block"], c["rows"], c["n"]
        fwd, inv, norm = _hadamard64(x.double() * d, b), _hadamard64(y, b), math.sqrt(n if c["kron28"] else b)
        if c["kron28"]:
            H = _paley28().to(fwd.device)
            mix = lambda h, v: (v.reshape(rows, 28, b).transpose(1, 2).reshape(-1, 28)  # noqa: E731
                                @ h.t().contiguous()).reshape(rows, b, 28).transpose(1, 2).reshape(rows, n)
            fwd, inv = mix(H, fwd), mix(H.t().contiguous(), inv)
        return {"fwd": fwd / norm, "inv": d * inv / norm}
    if c["kind"] == "input":
        x = _activations(c["rows"], c["n"], _gen(seed))
        return {"codes": None, "scale": x.double().abs().amax(dim=1) / c["qmax"], "digits": None}
    return None
