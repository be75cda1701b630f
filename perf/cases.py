"""The work a user of this library has it do, as cases that can be timed and compared.

Two kinds.  "layer" and "linear": forward calls (y = x.What^T + (x.A^T).B^T, arXiv 2410.21271, Sec. 3) of the
linears of decoder layers, or of one linear (or one group of linears that share x), from one token to a long
prompt, over every stored format of the backbone (w4, w3, w2, 2:4 fp16, 2:4 with 4-bit kept values) and of the
factors (fp16, 4-bit, 3-bit).  "factors": Algorithm 1 steps 1-6, the calibration that produces the factors.

Token-by-token generation runs from a captured HIP graph, as a serving loop does ("graph": True): prepare() holds
the stored weights, the workspace, the buffers and the graph of the entry points' launches, run() replays it.
Prompts, the smallest single call and the calibration are called directly.

Inputs are synthetic: LLaMA-3-shaped linears, Gaussian weights quantised by round-to-nearest (or pruned 2:4 by
magnitude), Gaussian factors, activations with 1 % outlier channels.
"""
import math

import numpy as np
import torch

import paper_2410_21271_amd as eora

LLAMA3_8B = {"d": 4096, "kv": 1024, "ff": 14336}
LLAMA3_70B = {"d": 8192, "kv": 1024, "ff": 28672}


def listed():
    return [
        # the smallest call a program makes: one small linear, one token, called directly; launch and host time count
        dict(name="one small linear, 1 token", kind="linear", fmt="w4", ab=4, r=64, M=1, d_in=1024, d_outs="1024", graph=False),
        # generation for one request: the decoder layers' linears with a 3-bit backbone (two layers, four launches each)
        dict(name="8B layers w3, 1 token", kind="layer", fmt="w3", ab=16, r=128, M=1, layers=2, graph=True, **LLAMA3_8B),
        # generation for a handful of requests, everything in 4 bits
        dict(name="8B layers w4 q4, 8 tokens", kind="layer", fmt="w4", ab=4, r=128, M=8, layers=2, graph=True, **LLAMA3_8B),
        # a serving batch
        dict(name="8B layers w4, 64 tokens", kind="layer", fmt="w4", ab=16, r=128, M=64, layers=2, graph=True, **LLAMA3_8B),
        # a serving batch whose requests choose among four adapters: one call per linear
        dict(name="8B layer w4 multi, 24 tokens", kind="layer", fmt="w4", ab=16, r=64, multi=4, M=24, layers=1, graph=True, **LLAMA3_8B),
        # sizes that are no powers of two, an odd number of requests and a rank that is no multiple of 128
        dict(name="ragged layers w3, 37 tokens", kind="layer", fmt="w3", ab=16, r=96, M=37, layers=3, graph=True, d=2688, kv=896, ff=7296),
        # generation for one request with the 2:4 backbone of a 70B model
        dict(name="70B layer 2:4, 1 token", kind="layer", fmt="sp24", ab=16, r=128, M=1, layers=1, graph=True, **LLAMA3_70B),
        # a serving batch on the 2:4 backbone with 4-bit kept values
        dict(name="70B layer 2:4 q4, 64 tokens", kind="layer", fmt="sp24q4", ab=16, r=128, M=64, layers=1, graph=True, **LLAMA3_70B),
        # a short prompt of odd length, 3-bit backbone and 4-bit factors
        dict(name="8B layer w3 q4, 333 tokens", kind="layer", fmt="w3", ab=4, r=128, M=333, layers=1, graph=False, **LLAMA3_8B),
        # a prompt, rank 256
        dict(name="8B layer w4, 2048 tokens", kind="layer", fmt="w4", ab=16, r=256, M=2048, layers=1, graph=False, **LLAMA3_8B),
        # a long prompt through the MLP's first two linears, backbone alone (adapter switched off)
        dict(name="8B gate+up w4 bare, 8192 tok", kind="linear", fmt="w4", ab=16, r=0, M=8192, d_in=4096, d_outs="14336,14336", graph=False),
        # calibration of one attention projection
        dict(name="factors 4096x4096", kind="factors", d_in=4096, d_out=4096, r=128, n_tokens=8192),
    ]


def _log(rng, lo, hi):
    """A whole number, uniform over its logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.49)))))))


def draw(rng):
    """One more case of the same ranges: any shape the entry points take, odd ones among them."""
    what = rng.choice(("decode", "decode", "batch", "batch", "batch", "sparse", "prompt", "prompt", "factors"))
    if what == "factors":
        # multiples of 128 as in every model here, now and then other even sizes
        if rng.random() < 0.7:
            d_in, d_out = 128 * _log(rng, 4, 24), 128 * _log(rng, 4, 24)
        else:
            d_in, d_out = 2 * _log(rng, 150, 450), 2 * _log(rng, 150, 450)
        return dict(kind="factors", d_in=d_in, d_out=d_out, r=min(32 * _log(rng, 1, 8), d_in, d_out), n_tokens=_log(rng, d_in, 8192))
    d_in = 128 * _log(rng, 8, 112)
    if rng.random() < 0.4:
        d_in = max(1024, d_in // 1024 * 1024)
    n = rng.choice((1, 1, 2, 3))
    d_outs = [16 * _log(rng, 32, 896) for _ in range(n)]
    fmt = rng.choice(("w4", "w4", "w3", "w3", "w2")) if what != "sparse" else rng.choice(("sp24", "sp24q4"))
    ab = rng.choice((16, 16, 4, 3)) if what != "sparse" else 16
    r = 32 * rng.randint(0, 8) if ab == 16 else (rng.choice((64, 128, 256)) if ab == 4 else 128)
    M = {"decode": rng.randint(1, 4), "batch": _log(rng, 5, 127), "sparse": _log(rng, 1, 127), "prompt": _log(rng, 128, 2048)}[what]
    if r == 0:
        ab = 16
    case = dict(kind="linear", fmt=fmt, ab=ab, r=r, M=M, d_in=d_in, d_outs=",".join(str(v) for v in d_outs),
                graph=what != "prompt" and rng.random() < 0.9)
    if fmt in ("w4", "w3", "w2") and rng.random() < 0.15:
        case["group"] = d_in                                 # channel-wise quantisation
    if what == "batch" and n == 1 and ab == 16 and 0 < r <= 128 and rng.random() < 0.5:
        case["multi"] = rng.choice((2, 3, 4))
    return case


# ---------------------------------------------------------------------------------------------- logical operands
def _calls(case):
    """(d_in, d_outs) of the case's forward calls, in order."""
    if case["kind"] == "linear":
        return [(case["d_in"], [int(v) for v in case["d_outs"].split(",")])]
    d, kv, ff = case["d"], case["kv"], case["ff"]
    one = [(d, [d, kv, kv]), (d, [d]), (d, [ff, ff]), (ff, [d])]
    if case.get("multi"):                                    # linear_q_multi serves one linear per call
        one = [(d_in, [d_out]) for d_in, d_outs in one for d_out in d_outs]
    return one * case["layers"]


def _generator(seed, *index):
    g = torch.Generator(device="cuda")
    s = seed
    for i in index:
        s = (s * 1000003 + i + 1) % (1 << 62)
    g.manual_seed(s)
    return g


def _randn(g, *shape):
    return torch.randn(*shape, generator=g, device="cuda", dtype=torch.float32)


def _rtn(W, bits, per):
    """Asymmetric round-to-nearest over `per` consecutive columns: codes u8, zeros u8, scales fp16."""
    rows, K = W.shape
    qmax = (1 << bits) - 1
    Wg = W.view(rows, K // per, per)
    lo, hi = Wg.amin(2).clamp(max=0.0), Wg.amax(2).clamp(min=0.0)
    sc = ((hi - lo) / qmax).to(torch.float16)
    sc = torch.where(sc == 0, torch.ones_like(sc), sc)
    s = sc.float()
    z = torch.round(-lo / s).clamp(0, qmax)
    q = (torch.round(Wg / s[:, :, None]) + z[:, :, None]).clamp(0, qmax)
    return q.view(rows, K).to(torch.uint8), z.to(torch.uint8), sc


def _symmetric(Mat, bits):
    """Symmetric round-to-nearest per row and min(128, K) columns: codes u8 (zero-point 2^(bits-1)), scales fp16."""
    rows, K = Mat.shape
    kt, zp = min(128, K), 1 << (bits - 1)
    Mg = Mat.view(rows, K // kt, kt)
    sc = (Mg.abs().amax(2) / (zp - 1)).to(torch.float16)
    sc = torch.where(sc == 0, torch.ones_like(sc), sc)
    q = (torch.round(Mg / sc.float()[:, :, None]) + zp).clamp(1, 2 * zp - 1)
    return q.view(rows, K).to(torch.uint8), sc


def _prune(W):
    """2:4 by magnitude (ties keep the lower column): kept values fp16 and positions, both rows x K/2."""
    rows, K = W.shape
    w = W.to(torch.float16).view(rows, K // 4, 4)
    g = w.abs()
    first = g.argmax(2, keepdim=True)
    second = g.masked_fill(torch.zeros_like(g, dtype=torch.bool).scatter_(2, first, True), -1.0).argmax(2, keepdim=True)
    pos = torch.cat((torch.minimum(first, second), torch.maximum(first, second)), 2)
    return w.gather(2, pos).view(rows, K // 2), pos.to(torch.uint8).view(rows, K // 2)


def _member(case, g, d_in, d_out):
    """One linear's operands before packing, and nothing that depends on the library."""
    fmt, r = case["fmt"], case["r"] * case.get("multi", 1)
    W = _randn(g, d_out, d_in) * 0.02
    m = {}
    if fmt in ("w4", "w3", "w2"):
        m["codes"], m["zeros"], m["scales"] = _rtn(W, int(fmt[1]), case.get("group", 128))
    else:
        vals, m["pos"] = _prune(W)
        if fmt == "sp24":
            m["vals"] = vals
        else:                                                # 64 kept values per 128 dense columns
            m["codes"], m["zeros"], m["scales"] = _rtn(vals.float(), 4, 64)
    del W
    if r:
        A, B = _randn(g, r, d_in) * 0.01, _randn(g, d_out, r) * 0.01
        if case["ab"] == 16:
            m["A"], m["B"] = A.to(torch.float16), B.to(torch.float16)
        else:
            m["A"], m["B"] = _symmetric(A, case["ab"]), _symmetric(B, case["ab"])
    return m


def _inputs(case, seed):
    """Per forward call: x, the adapter of each token (or None), and a function that makes its members one by one."""
    for c, (d_in, d_outs) in enumerate(_calls(case)):
        g = _generator(seed, c)
        x = _randn(g, case["M"], d_in)
        hot = torch.randperm(d_in, generator=g, device="cuda")[: max(1, d_in // 100)]
        x[:, hot] *= 20.0
        sel = None
        if case.get("multi"):
            sel = torch.randint(-1, case["multi"], (case["M"],), generator=g, device="cuda", dtype=torch.int32)
        members = ((_member(case, _generator(seed, c, 1 + i), d_in, d_out), d_out) for i, d_out in enumerate(d_outs))
        yield d_in, x.to(torch.float16), sel, members


# ---------------------------------------------------------------------------------------------- stored formats
def _words(parts, shifts):
    """Small integers (last dimension) at the given bit positions of one 32-bit word each."""
    sh = torch.tensor(shifts, dtype=torch.int32, device=parts.device)
    return (parts.to(torch.int32) << sh).sum(-1, dtype=torch.int32)


def _lanes(a, kt):
    """rows x K -> (row block, tile, quarter j, row n, kt/4 columns): the order of the lanes in the stored tiles."""
    rows, K = a.shape
    return a.view(rows // 16, 16, K // kt, 4, kt // 4).permute(0, 2, 3, 1, 4)


def _pack_codes(codes, bits):
    kt = min(128, codes.shape[1])
    L = _lanes(codes, kt)
    if bits == 4:
        w = _words(L.reshape(*L.shape[:4], kt // 32, 8), [4 * (4 * (k % 2) + k // 2) for k in range(8)])
    elif bits == 2:
        w = _words(L.reshape(*L.shape[:4], 2, 16), [16 * (c % 2) + 2 * (c // 2) for c in range(16)])
    else:
        body = L[..., :30].reshape(*L.shape[:4], 3, 10)
        w = _words(body, [16 * (c % 2) + 3 * (c // 2) for c in range(10)])
        last = L[..., 30:]
        bit = torch.stack([_words((last >> b) & 1, [15, 31]) for b in range(3)], -1)
        w = w | bit
    return w.reshape(-1).contiguous()


def _pack_zeros(zeros):
    rows, ng = zeros.shape
    pad = torch.zeros(rows, (ng + 7) // 8 * 8, dtype=torch.uint8, device=zeros.device)
    pad[:, :ng] = zeros
    return _words(pad.view(rows, -1, 8), [4 * e for e in range(8)]).reshape(-1).contiguous()


def _pack_f16(a):
    return _lanes(a, 32).reshape(-1).contiguous()


def _kept(a):
    """rows x K/2 kept entries -> (row block, tile, half s, quarter j, row n, 8)."""
    rows, half = a.shape
    return a.view(rows // 16, 16, half // 64, 2, 4, 8).permute(0, 2, 3, 4, 1, 5)


def _pack_positions(pos):
    p = _kept(pos).permute(0, 1, 3, 4, 2, 5).reshape(-1, 16)
    return _words(p, [2 * e for e in range(16)])


def _pack_member(case, m):
    """(backbone operands..., A, B, A_scales, B_scales) as the entry points read them."""
    fmt = case["fmt"]
    if fmt in ("w4", "w3", "w2"):
        bb = (_pack_codes(m["codes"], int(fmt[1])), m["scales"].contiguous(), _pack_zeros(m["zeros"]))
    elif fmt == "sp24":
        bb = (_kept(m["vals"]).reshape(-1).contiguous(), _pack_positions(m["pos"]))
    else:
        codes = _words(_kept(m["codes"]).permute(0, 1, 3, 4, 2, 5), [4 * (4 * (e % 2) + e // 2) for e in range(8)])   # (.., n, s)
        tiles = torch.cat((codes.reshape(-1, 2), _pack_positions(m["pos"])[:, None]), 1).reshape(-1).contiguous()
        meta = m["scales"].view(torch.int16).to(torch.int32).bitwise_and(0xFFFF) | (m["zeros"].to(torch.int32) << 16)
        rows, G = meta.shape
        bb = (tiles, meta.view(rows // 16, 16, G).permute(0, 2, 1).reshape(-1).contiguous())
    if "A" not in m:
        return bb + (None,) * 4
    if case["ab"] == 16:
        return bb + (_pack_f16(m["A"]), _pack_f16(m["B"]), None, None)
    (ca, sa), (cb, sb) = m["A"], m["B"]
    return bb + (_pack_codes(ca, case["ab"]), _pack_codes(cb, case["ab"]), sa.contiguous(), sb.contiguous())


# ---------------------------------------------------------------------------------------------- the cases
def prepare(case, seed):
    if case["kind"] == "factors":
        d_in, d_out, n = case["d_in"], case["d_out"], case["n_tokens"]
        W, W_hat, Xt = _calibration(case, seed)
        f64 = dict(dtype=torch.float64, device="cuda")
        ws = torch.empty(eora.factors_workspace_bytes(d_in, d_out, case["r"]), dtype=torch.uint8, device="cuda")
        return dict(case=case, W=W, W_hat=W_hat, Xt=Xt, n=n, B=torch.empty(d_out, case["r"], **f64),
                    A=torch.empty(case["r"], d_in, **f64), sigma=torch.empty(case["r"], **f64), ws=ws)
    M, r_all = case["M"], case["r"] * case.get("multi", 1)
    calls, need = [], 0
    for d_in, x, sel, members in _inputs(case, seed):
        packed = []
        for m, d_out in members:
            packed.append(_pack_member(case, m) + (torch.zeros(M, d_out, dtype=torch.float16, device="cuda"), d_out))
            need = max(need, eora.workspace_bytes(M, d_in, d_out, r_all))
        need = max(need, eora.workspace_bytes_group(M, d_in, r_all, len(packed)))
        calls.append((d_in, x, sel, packed))
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    eora.workspace_init(ws)
    state = dict(case=case, calls=calls, ws=ws, graph=None)
    if case["graph"]:
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            _forward(state)
        torch.cuda.current_stream().wait_stream(side)
        torch.cuda.synchronize()
        state["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(state["graph"]):
            _forward(state)
    return state


def _forward(state):
    case, ws = state["case"], state["ws"]
    M, r, ab = case["M"], case["r"], case["ab"]
    for d_in, x, sel, members in state["calls"]:
        if case["fmt"] in ("w4", "w3", "w2"):
            bits, group = int(case["fmt"][1]), case.get("group", 128)
            if sel is not None:
                qw, sc, qz, A, B, As, Bs, y, d_out = members[0]
                eora.linear_q_multi(x, qw, sc, qz, A, B, As, Bs, sel, y, M, d_in, d_out, r, case["multi"], bits, group, ab, ws)
            elif len(members) == 1:
                qw, sc, qz, A, B, As, Bs, y, d_out = members[0]
                eora.linear_q(x, qw, sc, qz, A, B, As, Bs, y, M, d_in, d_out, r, bits, group, ab, ws)
            else:
                eora.linear_q_group(x, members, M, d_in, r, bits, group, ab, ws)
        elif len(members) == 1:
            w0, w1, A, B, _, _, y, d_out = members[0]
            (eora.linear_sp24 if case["fmt"] == "sp24" else eora.linear_sp24q4)(x, w0, w1, A, B, y, M, d_in, d_out, r, ws)
        else:
            none = (None, None)
            eora.linear_sp24_group(x, [(m[:2] + none if case["fmt"] == "sp24" else none + m[:2]) + (m[2], m[3], m[6], m[7]) for m in members],
                                   M, d_in, r, ws)


def run(state):
    case = state["case"]
    if case["kind"] == "factors":
        s = state
        eora.factors(s["W"], s["W_hat"], s["Xt"], s["B"], s["A"], s["sigma"], s["n"], case["d_in"], case["d_out"], case["r"], 1e-12, s["ws"])
        # the sign of a component is arbitrary, so the pair is handed on as the correction it stands for
        return {"sigma": s["sigma"], "correction": s["B"] @ s["A"]}
    if state["graph"] is not None:
        state["graph"].replay()
    else:
        _forward(state)
    return [m[-2] for _, _, _, members in state["calls"] for m in members]


def _calibration(case, seed):
    g = _generator(seed, 0)
    d_in, d_out = case["d_in"], case["d_out"]
    W = _randn(g, d_out, d_in) * 0.02
    per = 128 if d_in % 128 == 0 else d_in
    codes, zeros, scales = _rtn(W, 4, per)
    W_hat = (codes.view(d_out, -1, per).float() - zeros[:, :, None].float()) * scales[:, :, None].float()
    spread = torch.exp(torch.rand(d_in, generator=g, device="cuda") * 2.0 - 1.0)
    spread[torch.randperm(d_in, generator=g, device="cuda")[: max(1, d_in // 100)]] *= 20.0
    return W, W_hat.view(d_out, d_in), _randn(g, d_in, case["n_tokens"]) * spread[:, None]


def work(case):
    if case["kind"] == "factors":
        k, d, n, r = case["d_in"], case["d_out"], case["n_tokens"], case["r"]
        s = min(k, d)
        # Gram matrix (one triangle), its square root, dW times it, the r leading components, A
        return {"bytes": 4.0 * (2 * k * d + k * n) + 8.0 * r * (k + d + 1),
                "flops": 1.0 * k * k * n + k ** 3 / 3.0 + 1.0 * d * k * k + 4.0 * s * max(k, d) * r + 2.0 * r * k * d}
    M, total, flops = case["M"], 0.0, 0.0
    r = case["r"] * case.get("multi", 1)
    for d_in, d_outs in _calls(case):
        total += 2.0 * M * d_in + (4.0 * M if case.get("multi") else 0.0)
        for d_out in d_outs:
            if case["fmt"] == "sp24":
                total += 1.125 * d_in * d_out
            elif case["fmt"] == "sp24q4":
                total += 0.375 * d_in * d_out + d_out * (d_in // 128) * 4.0
            else:
                total += d_in * d_out * int(case["fmt"][1]) / 8.0 + d_out * (d_in // case.get("group", 128)) * 2.5
            total += r * (d_in + d_out) * case["ab"] / 8.0 + 2.0 * M * d_out
            if r and case["ab"] != 16:
                total += 2.0 * r * (d_in // 128) + 2.0 * d_out * (r // min(128, r))
            flops += 2.0 * M * d_in * d_out * (0.5 if case["fmt"] in ("sp24", "sp24q4") else 1.0) + 2.0 * M * r * (d_in + d_out)
    return {"bytes": total, "flops": flops}


def tolerance(case):
    if case["kind"] == "factors":
        # 64-bit sums of some thousand terms, and a division by the gap between the r-th and the next singular value
        return {"rel": 1e-8, "max": 1e-6}
    # y is rounded to fp16 once (2.1e-4 against 64 bits); where a dequantised weight or t is rounded to fp16 too it is
    # 2.8e-4.  Four times the larger; the largest single difference is four times two roundings and their tails.
    return {"rel": 1.2e-3, "max": 8e-3}


# ---------------------------------------------------------------------------------------------- 64 bits
def _dense(case, m, d_in):
    """The stored backbone as the numbers it stands for, float64."""
    fmt = case["fmt"]
    if fmt in ("w4", "w3", "w2"):
        rows, per = m["codes"].shape[0], case.get("group", 128)
        q = m["codes"].view(rows, -1, per).double() - m["zeros"][:, :, None].double()
        return (q * m["scales"][:, :, None].double()).view(rows, d_in)
    if fmt == "sp24":
        vals = m["vals"].double()
    else:
        rows = m["codes"].shape[0]
        vals = ((m["codes"].view(rows, -1, 64).double() - m["zeros"][:, :, None].double()) * m["scales"][:, :, None].double()).view(rows, -1)
    rows = vals.shape[0]
    dense = torch.zeros(rows, d_in // 4, 4, dtype=torch.float64, device=vals.device)
    dense.scatter_(2, m["pos"].view(rows, -1, 2).long(), vals.view(rows, -1, 2))
    return dense.view(rows, d_in)


def _factor64(f, bits):
    if bits == 16:
        return f.double()
    codes, scales = f
    rows, K = codes.shape
    kt = min(128, K)
    return ((codes.view(rows, -1, kt).double() - (1 << (bits - 1))) * scales[:, :, None].double()).view(rows, K)


def exact(case, seed):
    if case["kind"] == "factors":
        if max(case["d_in"], case["d_out"]) > 2048:
            return None                                      # LAPACK takes longer than 20 seconds
        W, W_hat, Xt = (t.double().cpu().numpy() for t in _calibration(case, seed))
        dW = W - W_hat
        lam, Q = np.linalg.eigh(Xt @ Xt.T)
        root = np.sqrt(np.maximum(lam, 1e-12 * lam.max()))
        U, sig, Vt = np.linalg.svd((dW @ Q) * root[None, :], full_matrices=False)
        r = case["r"]
        A = (Vt[:r] / root[None, :]) @ Q.T
        return {"sigma": sig[:r], "correction": (U[:, :r] * sig[None, :r]) @ A}
    out = []
    for d_in, x, sel, members in _inputs(case, seed):
        x = x.double()
        for m, _ in members:
            y = x @ _dense(case, m, d_in).T
            if "A" in m:
                t = x @ _factor64(m["A"], case["ab"]).T
                if sel is not None:
                    own = torch.arange(t.shape[1], device=t.device)[None, :] // case["r"] == sel[:, None]
                    t = t * own
                y = y + t @ _factor64(m["B"], case["ab"]).T
            out.append(y)
    return out
