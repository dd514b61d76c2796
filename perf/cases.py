"""Timed cases of the library's public calls: training steps of single layers and deployment steps.

A case is one call, or one forward with its backward, as a training or
serving program makes it through the Python binding.  Inputs follow the
seeded workloads of this repository (unit-norm or 1/sqrt(d) inputs, small
proposed costates, gate-family retentions and step sizes, packed documents),
drawn on the GPU.  The reference values are the sequential definition in
float64, token by token.

Kinds:
  scan     forward + backward of the unit-retention scan, plain calls or the
           save-for-backward pair; scalar or per-token eta; either read
           convention; fp32 or bf16 inputs; 64/128-wide maps
  reset    the unit-retention pair with document resets (64 x 64 maps)
  gated    forward + backward with retention, per-token eta and resets,
           plain calls or the save-for-backward pair, every gradient
  mlp      the two-map online MLP, forward + reverse targets + the MLP's own
           gradients, at 64/128 widths or at LM widths (wide maps)
  decode   one deployment step over resident states, plain or gated
"""

import math

import torch

import paper_2609_34174_amd as gl


# ---------------------------------------------------------------------------
# Cases
# ---------------------------------------------------------------------------

def _scan(name, B, H, T, d, m, dtype, pair, eta, prefix="exclusive"):
    return {"name": name, "kind": "scan", "B": B, "H": H, "T": T, "d": d, "m": m, "dtype": dtype, "pair": pair,
            "eta": eta, "prefix": prefix}


def _reset(name, B, H, T, dtype, doc):
    return {"name": name, "kind": "reset", "B": B, "H": H, "T": T, "d": 64, "m": 64, "dtype": dtype, "doc": doc}


def _gated(name, B, H, T, d, m, dtype, pair, doc):
    return {"name": name, "kind": "gated", "B": B, "H": H, "T": T, "d": d, "m": m, "dtype": dtype, "pair": pair,
            "doc": doc}


def _mlp(name, B, H, T, d, hidden, o, dtype, act, retention, doc):
    return {"name": name, "kind": "mlp", "B": B, "H": H, "T": T, "d": d, "hidden": hidden, "o": o, "dtype": dtype,
            "act": act, "retention": retention, "doc": doc}


def _decode(name, S, H, d, m, gated):
    return {"name": name, "kind": "decode", "S": S, "H": H, "d": d, "m": m, "gated": gated}


def listed():
    return [
        # The smallest layer of the workloads (small-f32): one short sequence, launches and latency.
        _scan("small-f32", 1, 1, 256, 64, 64, "f32", "plain", "scalar"),
        # The LM layer of the workloads (lm-bf16) as a training step runs it.
        _scan("lm-bf16-saved", 8, 16, 2048, 64, 64, "bf16", "saved", "scalar"),
        # An LM layer whose step sizes come from the write gate, an odd length, plain calls.
        _scan("lm-bf16-eta-odd", 3, 12, 1999, 64, 64, "bf16", "plain", "token"),
        # One layer of the headline 24-layer stack.
        _scan("stack-bf16-layer", 4, 32, 4096, 64, 64, "bf16", "saved", "scalar"),
        # Long context, 128-wide heads (long-bf16).
        _scan("long-bf16", 2, 16, 16384, 128, 128, "bf16", "saved", "scalar"),
        # fp32 activations, unequal widths, ragged length, the inclusive read.
        _scan("rect-f32-incl", 2, 8, 1000, 64, 128, "f32", "plain", "token", "inclusive"),
        # Packed documents at unit retention (the paper's LM regime), documents of mean length 512.
        _reset("lm-bf16-docs", 8, 16, 2048, "bf16", 512),
        # Retention, per-token gates and packed documents, every gradient.
        _gated("lm-bf16-gated", 8, 16, 2048, 64, 64, "bf16", "saved", 512),
        # The same with 128-wide heads, few sequences and an odd length, plain calls.
        _gated("gated-128-odd", 2, 8, 1500, 128, 128, "bf16", "plain", 300),
        # The online MLP inside a head: 64 -> 128 -> 64.
        _mlp("mlp-head", 2, 16, 1024, 64, 128, 64, "bf16", "tanh", "token", 300),
        # The paper's adapted final MLP, 1024 -> 4096 -> 1024, context 1024, unit retention, documents.
        _mlp("mlp-lm", 2, 1, 1024, 1024, 4096, 1024, "bf16", "gelu_tanh", "one", 512),
        # Deployment: one token for 256 sequences x 16 heads (decode-f32).
        _decode("decode-f32", 256, 16, 64, 64, False),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _heads(rng, T, wmax, limit):
    """B and H with B * H * T * wmax at most `limit`."""
    most = max(1, min(256, limit // (T * wmax)))
    BH = _log_int(rng, 1, most)
    H = min(BH, rng.choice([1, 2, 4, 6, 8, 12, 16, 32]))
    return max(1, BH // H), H


# Elements B * H * T * width of the largest drawn scan (the largest listed one has 67 M at 128-wide maps in bf16).
_LIMIT = 16 << 20


def draw(rng):
    kind = rng.choice(["scan", "scan", "scan", "reset", "gated", "gated", "mlp", "decode"])
    if kind == "decode":
        if rng.random() < 0.3:  # LM-width maps, a few sequences
            d, m = rng.choice([(1024, 4096), (4096, 1024), (512, 2048), (2048, 512)])
            return {"kind": "decode", "S": rng.randint(1, 24), "H": 1, "d": d, "m": m, "gated": rng.random() < 0.5}
        d, m = rng.choice([(64, 64), (128, 128), (64, 128), (128, 64)])
        return {"kind": "decode", "S": _log_int(rng, 1, 1024), "H": rng.choice([1, 4, 8, 16]), "d": d, "m": m,
                "gated": rng.random() < 0.5}
    if kind == "mlp" and rng.random() < 0.5:  # LM widths
        d, hidden = rng.choice([(256, 1024), (512, 2048), (768, 3072), (1024, 4096)])
        return {"kind": "mlp", "B": rng.randint(1, 2), "H": 1, "T": _log_int(rng, 100, 1024), "d": d,
                "hidden": hidden, "o": d, "dtype": "bf16", "act": "gelu_tanh",
                "retention": rng.choice(["one", "one", "token"]), "doc": rng.choice([0, 128, 512])}
    T = _log_int(rng, 64, 8192)
    dtype = rng.choice(["bf16", "bf16", "bf16", "f32"])
    limit = _LIMIT if dtype == "bf16" else _LIMIT // 4
    if kind == "mlp":
        T = _log_int(rng, 64, 2048)
        B, H = _heads(rng, T, 128, limit // 4)
        d, hidden, o = rng.choice([(64, 128, 64), (64, 64, 64), (128, 128, 128)])
        return {"kind": "mlp", "B": B, "H": H, "T": T, "d": d, "hidden": hidden, "o": o, "dtype": dtype,
                "act": rng.choice(["tanh", "gelu", "gelu_tanh"]), "retention": "token",
                "doc": rng.choice([0, 128, 512])}
    if kind == "reset":
        B, H = _heads(rng, T, 64, limit)
        return {"kind": "reset", "B": B, "H": H, "T": T, "d": 64, "m": 64, "dtype": dtype,
                "doc": rng.choice([128, 512, 2048])}
    d, m = rng.choice([(64, 64), (64, 64), (128, 128), (128, 128), (64, 128), (128, 64)])
    pair = rng.choice(["plain", "saved", "saved"])
    if kind == "gated":
        T = _log_int(rng, 64, 4096)
        B, H = _heads(rng, T, max(d, m), limit // 2)
        return {"kind": "gated", "B": B, "H": H, "T": T, "d": d, "m": m, "dtype": dtype, "pair": pair,
                "doc": rng.choice([0, 128, 512])}
    B, H = _heads(rng, T, max(d, m), limit)
    return {"kind": "scan", "B": B, "H": H, "T": T, "d": d, "m": m, "dtype": dtype, "pair": pair,
            "eta": rng.choice(["scalar", "token"]),
            "prefix": rng.choice(["exclusive", "exclusive", "inclusive"])}


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------

_DT = {"bf16": torch.bfloat16, "f32": torch.float32}


class _Gen:
    def __init__(self, seed):
        self.dev = torch.device("cuda")
        self.g = torch.Generator(device=self.dev)
        self.g.manual_seed(seed)

    def normal(self, *shape, std=1.0, mean=0.0):
        return torch.randn(*shape, device=self.dev, generator=self.g) * std + mean

    def documents(self, B, T, mean_len):
        """Packed rows: a document starts with probability 1 / mean_len per token, and at token 0."""
        if not mean_len:
            return None
        r = (torch.rand(B, T, device=self.dev, generator=self.g) < 1.0 / mean_len).to(torch.uint8)
        r[:, 0] = 1
        return r

    def inputs(self, B, H, T, d, dt):
        """Layer inputs: unit-norm rows at 64 wide, N(0, 1/d) at other widths."""
        x = self.normal(B, H, T, d)
        x = x / x.norm(dim=-1, keepdim=True) if d == 64 else x * d ** -0.5
        return x.to(dt)

    def retention(self, B, H, T):
        return torch.sigmoid(self.normal(B, H, T, std=0.5, mean=1.5))

    def write_strength(self, B, H, T):
        """mu = 4 sigmoid(b), starting at 0.9."""
        return 4.0 * torch.sigmoid(self.normal(B, H, T, std=0.5, mean=math.log(0.9 / 3.1)))


def prepare(case, seed):
    r = _Gen(seed)
    k = case["kind"]
    s = {"case": case}
    if k == "decode":
        S, H, d, m = case["S"], case["H"], case["d"], case["m"]
        s["W"] = r.normal(S, H, m, d, std=d ** -0.5)
        s["x"] = r.normal(S, H, d, std=d ** -0.5)
        s["g"] = r.normal(S, H, m, std=0.1)
        if case["gated"]:
            s["W0"] = r.normal(H, m, d, std=d ** -0.5)
            s["eta"] = (r.write_strength(S, H, 1) / d)[:, :, 0].contiguous()
            s["alpha"] = r.retention(S, H, 1)[:, :, 0].contiguous()
            s["reset"] = (torch.rand(S, device=r.dev, generator=r.g) < 1.0 / 64).to(torch.uint8)
        return s
    B, H, T, d, dt = case["B"], case["H"], case["T"], case["d"], _DT[case["dtype"]]
    if k == "mlp":
        hid, o = case["hidden"], case["o"]
        s["W1"] = r.normal(H, hid, d, std=d ** -0.5)
        s["W2"] = r.normal(H, o, hid, std=hid ** -0.5)
        s["X"] = r.normal(B, H, T, d).to(dt)
        s["Gz"] = r.normal(B, H, T, hid, std=0.3).to(dt)
        s["Gy"] = r.normal(B, H, T, o, std=0.3).to(dt)
        s["gY"] = r.normal(B, H, T, o).to(dt)
        s["mu"] = r.write_strength(B, H, T)
        s["alpha"] = 1.0 if case["retention"] == "one" else r.retention(B, H, T)
        s["reset"] = r.documents(B, T, case["doc"])
        s["grads"] = ("dmu", "dw10", "dw20") if case["retention"] == "one" else gl.MLP_GRADS
        return s
    m = case["m"]
    s["W0"] = r.normal(H, m, d, std=d ** -0.5)
    s["X"] = r.inputs(B, H, T, d, dt)
    s["G"] = r.normal(B, H, T, m, std=0.1 if d == 64 else 0.05).to(dt)
    s["dY"] = r.normal(B, H, T, m).to(dt)
    if k == "gated":
        s["eta"] = r.write_strength(B, H, T) / d
        s["alpha"] = r.retention(B, H, T)
        s["reset"] = r.documents(B, T, case["doc"])
    elif k == "reset":
        s["eta"] = 0.1
        s["reset"] = r.documents(B, T, case["doc"])
    else:
        s["eta"] = (0.1 if d == 64 else 0.05) if case["eta"] == "scalar" else r.write_strength(B, H, T) / d
    return s


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------

def run(s):
    c = s["case"]
    k = c["kind"]
    if k == "decode":
        if c["gated"]:
            y = gl.decode_step_gated(s["W"], s["W0"], s["x"], s["g"], s["eta"], s["alpha"], s["reset"])
        else:
            y = gl.decode_step(s["W"], s["x"], s["g"], 0.1)
        return {"y": y, "W": s["W"]}
    if k == "mlp":
        a = (s["mu"], s["alpha"], s["reset"])
        Z, Hid, Y = gl.mlp_fwd(s["W1"], s["W2"], s["X"], s["Gz"], s["Gy"], *a, act=c["act"])
        gZ, gX, g = gl.mlp_reverse(s["W1"], s["W2"], s["X"], s["Gz"], s["Gy"], Z, Hid, s["gY"], *a, act=c["act"],
                                   grads=s["grads"])
        return {"Z": Z, "Hid": Hid, "Y": Y, "gZ": gZ, "gX": gX, **g}
    W0, X, G, dY, eta = s["W0"], s["X"], s["G"], s["dY"], s["eta"]
    if k == "reset":
        Y, saved = gl.scan_fwd_reset_save(W0, X, G, eta, s["reset"])
        return {"Y": Y, **gl.scan_bwd_reset_saved(W0, X, G, dY, saved, eta, s["reset"])}
    if k == "gated":
        a = (eta, s["alpha"], s["reset"])
        if c["pair"] == "saved":
            Y, saved = gl.scan_fwd_gated_save(W0, X, G, *a)
            return {"Y": Y, **gl.scan_bwd_gated_saved(W0, X, G, dY, saved, *a)}
        Y = gl.scan_fwd_gated(W0, X, G, *a)
        return {"Y": Y, **gl.scan_bwd_gated(W0, X, G, dY, *a)}
    if c["pair"] == "saved":
        Y, saved = gl.scan_fwd_save(W0, X, G, eta, prefix=c["prefix"])
        return {"Y": Y, **gl.scan_bwd_saved(W0, X, G, dY, saved, eta, prefix=c["prefix"])}
    Y = gl.scan_fwd(W0, X, G, eta, prefix=c["prefix"])
    return {"Y": Y, **gl.scan_bwd(W0, X, G, dY, eta, prefix=c["prefix"])}


# ---------------------------------------------------------------------------
# What a pass cannot do without
# ---------------------------------------------------------------------------

def _pass_flops(T, d, m, gated):
    """Per token, forward + backward of one scan with every output: the lesser
    of the recurrent form (read, write, transpose read, dG, dX and dW0: 2 m d
    each) and the parallel form (W_0 reads, dW0 and causal pair sums)."""
    rec = (12 + (2 if gated else 0)) * m * d
    par = 6 * m * d + (T - 1) * 3 * (d + m)
    return min(rec, par)


def work(case):
    k = case["kind"]
    if k == "decode":
        S, H, d, m = case["S"], case["H"], case["d"], case["m"]
        b = S * H * (2 * m * d + d + 2 * m) * 4 + ((H * m * d + 2 * S * H) * 4 + S if case["gated"] else 0)
        return {"bytes": b, "flops": S * H * m * d * (6 if case["gated"] else 4)}
    B, H, T, d = case["B"], case["H"], case["T"], case["d"]
    n, e = B * H * T, 2 if case["dtype"] == "bf16" else 4
    if k == "mlp":
        hid, o = case["hidden"], case["o"]
        token = case["retention"] == "token"
        # in: X, Gz, Gy, gY, mu, alpha; out: Z, Hid, Y, gZ, gX, dmu, dalpha
        per = (d + hid + 2 * o) * e + 4 * (2 if token else 1) + 4 * hid + e * hid + 4 * o + 4 * hid + 4 * d + \
            4 * (2 if token else 1)
        fl = 0
        for a, b in ((d, hid), (hid, o)):  # forward read/write, transpose read, dW0, dmu (and dalpha)
            fl += min((10 + (2 if token else 0)) * a * b, 6 * a * b + (T - 1) * 2 * (a + b))
        return {"bytes": n * per + 4 * H * 2 * (hid * d + o * hid) + (B * T if case["doc"] else 0), "flops": n * fl}
    m = case["m"]
    per = (d + 2 * m) * e + 4 * m + 4 * (2 * d + m) + 4  # X, G, dY; Y; gtilde, dX, dG, deta
    rows = 0
    if k == "gated":
        per += 4 * 3  # eta, alpha, dalpha
        rows = B * T if case["doc"] else 0
    elif k == "reset":
        rows = B * T
    elif case["eta"] == "token":
        per += 4
    return {"bytes": n * per + 2 * 4 * H * m * d + rows, "flops": n * _pass_flops(T, d, m, k == "gated")}


def tolerance(case):
    """About four times the error that the path shows against exact().

    Measured: 3e-8 to 1e-7 for decode; up to 5e-7 for fp32 scans; 2e-6 to
    1.2e-4 for bf16 ones, whose operands are exact and whose states are split
    into two bf16 terms, but whose intra-chunk score tiles may be rounded to
    bf16; 6e-4 for the MLP, whose hidden activations and hidden targets are
    stored in bf16 between the maps."""
    if case["kind"] == "decode":
        return {"rel": 5e-7}
    if case["dtype"] == "f32":
        return {"rel": 2e-6}
    return {"rel": 2.5e-3 if case["kind"] == "mlp" else 5e-4}


# ---------------------------------------------------------------------------
# Reference: the sequential definition in float64, token by token
# ---------------------------------------------------------------------------

_BLOCK = 64  # tokens between kept states of the reference's sweeps


def _gates64(eta, alpha, reset, B, H, T, dev):
    """eta, alpha and the mask of kept gate gradients as [BH, T]: a document
    start at t drops the write of t - 1 and the state it would carry."""
    def full(v):
        v = v.double() if torch.is_tensor(v) else torch.full((B, H, T), float(torch.tensor(v, dtype=torch.float32)),
                                                             dtype=torch.float64, device=dev)
        return v.reshape(B * H, T).clone()

    e, a = full(eta), full(alpha)
    keep = torch.ones_like(e)
    if reset is not None:
        cut = torch.zeros(B, T, dtype=torch.bool, device=dev)
        cut[:, :-1] = reset[:, 1:] != 0
        cut = cut[:, None, :].expand(B, H, T).reshape(B * H, T)
        e[cut] = 0.0
        a[cut] = 0.0
        keep[cut] = 0.0
    return e, a, keep


def _step(D, g, x, e, a):
    """Delta after one write, in place: a Delta - e g x^T."""
    D.mul_(a[:, None, None])
    return D.baddbmm_((g * -e[:, None])[:, :, None], x[:, None, :])


def _scan64(W0, X, G, eta, alpha, reset, dY=None, inclusive=False, want=()):
    """Y and, with dY, the wanted gradients (unit retention: alpha 1.0)."""
    B, H, T, d = X.shape
    m, dev = G.shape[3], X.device
    BH = B * H
    x, g = X.double().reshape(BH, T, d), G.double().reshape(BH, T, m)
    w0 = W0.double()[None].expand(B, H, m, d).reshape(BH, m, d)
    e, a, keep = _gates64(eta, alpha, reset, B, H, T, dev)
    dy = None if dY is None else dY.double().reshape(BH, T, m)
    Y = x @ w0.transpose(1, 2).contiguous()
    gt = None if dy is None else dy @ w0
    D = torch.zeros(BH, m, d, dtype=torch.float64, device=dev)
    kept = []
    for t in range(T):
        if "dalpha" in want and t % _BLOCK == 0:
            kept.append(D.clone())
        if inclusive:
            _step(D, g[:, t], x[:, t], e[:, t], a[:, t])
        Y[:, t] += (D @ x[:, t, :, None])[:, :, 0]
        if gt is not None:
            gt[:, t] += (dy[:, t, None, :] @ D)[:, 0]
        if not inclusive:
            _step(D, g[:, t], x[:, t], e[:, t], a[:, t])
    out = {"Y": Y.reshape(B, H, T, m)}
    if dy is None:
        return out
    out["gtilde"] = gt.reshape(B, H, T, d)
    if "dw0" in want:
        out["dw0"] = (dy.transpose(1, 2).contiguous() @ x).reshape(B, H, m, d).sum(0)
    if not any(k in want for k in ("dg", "dx", "deta", "dalpha")):
        return out
    U = torch.empty_like(g)
    V = torch.empty_like(x)
    da = torch.zeros_like(e)
    L = torch.zeros(BH, m, d, dtype=torch.float64, device=dev)  # dL/dDelta after token t
    states = []
    for t in range(T - 1, -1, -1):
        if "dalpha" in want:
            if not states:  # the states before each token of this block, recomputed from the kept one
                s0 = t // _BLOCK * _BLOCK
                D = kept[s0 // _BLOCK].clone()
                for u in range(s0, t + 1):
                    states.append(D.clone())
                    _step(D, g[:, u], x[:, u], e[:, u], a[:, u])
            da[:, t] = (L * states.pop()).sum((1, 2))
        if inclusive:
            L.baddbmm_(dy[:, t, :, None], x[:, t, None, :])
        U[:, t] = -(L @ x[:, t, :, None])[:, :, 0]
        V[:, t] = (g[:, t, None, :] @ L)[:, 0]
        if not inclusive:
            L.mul_(a[:, t, None, None]).baddbmm_(dy[:, t, :, None], x[:, t, None, :])
    out["dg"] = (U * e[:, :, None]).reshape(B, H, T, m)
    out["dx"] = out["gtilde"] - (V * e[:, :, None]).reshape(B, H, T, d)
    out["deta"] = ((g * U).sum(-1) * keep).reshape(B, H, T)
    out["dalpha"] = (da * keep).reshape(B, H, T)
    return out


def _act64(z, act):
    """sigma(z) and sigma'(z)."""
    if act == "tanh":
        h = torch.tanh(z)
        return h, 1 - h * h
    if act == "gelu":
        cdf = 0.5 * (1 + torch.erf(z / math.sqrt(2)))
        return z * cdf, cdf + z * torch.exp(-0.5 * z * z) / math.sqrt(2 * math.pi)
    k = math.sqrt(2 / math.pi)
    th = torch.tanh(k * (z + 0.044715 * z ** 3))
    return 0.5 * z * (1 + th), 0.5 * (1 + th) + 0.5 * z * (1 - th * th) * k * (1 + 3 * 0.044715 * z * z)


def exact(case, seed):
    k = case["kind"]
    s = prepare(case, seed)
    if k == "decode":
        W, x, g = s["W"].double(), s["x"].double(), s["g"].double()
        if case["gated"]:
            w0 = s["W0"].double()[None]
            W = torch.where(s["reset"][:, None, None, None] != 0, w0, W)
            y = (W @ x[..., None])[..., 0]
            W = w0 + s["alpha"].double()[..., None, None] * (W - w0)
            e = s["eta"].double()
        else:
            y = (W @ x[..., None])[..., 0]
            e = torch.full(x.shape[:2], float(torch.tensor(0.1, dtype=torch.float32)), dtype=torch.float64,
                           device=x.device)
        return {"y": y, "W": W - e[..., None, None] * g[..., :, None] * x[..., None, :]}
    if k == "mlp":
        d, hid, dt = case["d"], case["hidden"], _DT[case["dtype"]]
        want = ("deta", "dw0", "dalpha") if "dalpha" in s["grads"] else ("deta", "dw0")
        al, rs = s["alpha"], s["reset"]
        e1, e2 = s["mu"].double() / d, s["mu"].double() / hid
        Z = _scan64(s["W1"], s["X"], s["Gz"], e1, al, rs)["Y"]
        h, dh = _act64(Z, case["act"])
        Hid = h.to(dt)  # stored in the input type between the two maps
        second = _scan64(s["W2"], Hid, s["Gy"], e2, al, rs, s["gY"], want=want)
        gZ = dh * second["gtilde"]
        first = _scan64(s["W1"], s["X"], s["Gz"], e1, al, rs, gZ.to(dt), want=want)
        out = {"Z": Z, "Hid": Hid, "Y": second["Y"], "gZ": gZ, "gX": first["gtilde"],
               "dmu": first["deta"] / d + second["deta"] / hid}
        if "dalpha" in want:
            out["dalpha"] = first["dalpha"] + second["dalpha"]
        out["dw10"], out["dw20"] = first["dw0"], second["dw0"]
        return out
    names = gl.GATED_OUTPUTS if k == "gated" else gl.BWD_OUTPUTS
    o = _scan64(s["W0"], s["X"], s["G"], s["eta"], s.get("alpha", 1.0), s.get("reset"), s["dY"],
                case.get("prefix") == "inclusive", want=names)
    return {"Y": o["Y"], **{n: o[n] for n in names}}
