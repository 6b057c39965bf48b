"""The framework's work as its users call it: the cases that its speed is judged on.

Every case goes through the public entry points of ``paper_2608_29539_amd``
with device tensors, as a program that holds its inputs, workspaces and
(where the entry point takes them) output buffers calls them:

  layer   one LoGo attention layer's forward (``logo_attn_fwd``): serving
          prefill, ratio mode, a host threshold or a device threshold
  prefill the layer with its inputs' side: gate projection, branch transforms
          of K and V, the layer with the query transform on load
  train   training step of the layer (``logo_attn_fwd_train`` +
          ``logo_attn_bwd``)
  sparse  training step of the query-sparse global operator alone (the object
          of the paper's speed measurement, Sec. 4.3)
  dense   training step of the dense causal baseline
  decode  one autoregressive decoding step (``logo_decode``)

All tensors are bf16 with fp32 gates (the only types the entry points take).
"""
import math

import numpy as np
import torch

import paper_2608_29539_amd as pk

EPS = 1e-6


# --- the cases ---------------------------------------------------------------
def _case(name, op, lens, hq, hkv, d, window, ratio, **kw):
    c = dict(op=op, lens=lens, hq=hq, hkv=hkv, d=d, window=window, ratio=ratio,
             gate="uniform", mode="ratio", distinct=False, gains=False, d_model=0)
    if name:
        c["name"] = name
    c.update(kw)
    return c


def listed():
    return [
        # the smallest call: a short prompt, few heads; launches and latency
        _case("layer-1k-mha-d64", "layer", "1024", 4, 4, 64, 128, 0.25),
        # two medium sequences, one query head per KV head (the paper's models)
        _case("layer-2x8k-mha", "layer", "8192,8192", 16, 16, 128, 512, 0.125,
              gate="logit_normal"),
        # long-context prefill with grouped heads: the headline shape
        _case("layer-32k-gqa", "layer", "32768", 32, 8, 128, 1024, 0.125, gate="burst"),
        # a ragged serving batch routed by the threshold kept on the device,
        # with the global branch's own tensors and learned gains
        _case("layer-varlen-gqa", "layer", "3971,12288,16381,32768", 16, 4, 128, 512, 0.125,
              mode="device", distinct=True, gains=True),
        # the longest context
        _case("layer-128k-gqa", "layer", "131072", 32, 8, 128, 4096, 0.0625),
        # the layer with the steps that feed it: gate projection, LP transforms
        _case("prefill-8k-gqa", "prefill", "8192", 32, 8, 128, 1024, 0.125, d_model=4096,
              gains=True),
        # training step at the headline shape
        _case("train-32k-gqa", "train", "32768", 32, 8, 128, 1024, 0.125, gate="burst"),
        # a small packed training batch of odd lengths, d = 64, everything learned
        _case("train-varlen-mha-d64", "train", "1501,777,2048,63", 8, 8, 64, 256, 0.25,
              distinct=True, gains=True),
        # the paper's operator benchmark: 8 heads, half of the rows selected
        _case("sparse-train-16k-mha", "sparse", "16384", 8, 8, 128, 16384, 0.5),
        # the dense baseline's training step (warm-up phases, comparisons)
        _case("dense-train-8k-gqa", "dense", "8192", 32, 8, 128, 8192, 1.0),
        # serving: 16 long caches, an eighth of the new tokens selected
        _case("decode-16x32k-gqa", "decode", ",".join(["32768"] * 16), 32, 8, 128, 1024, 0.125),
        # serving: few short caches of odd lengths, latency
        _case("decode-4x2k-mha", "decode", "2047,513,1200,31", 16, 16, 128, 256, 0.5,
              gains=True),
    ]


_HEADS = ((4, 4), (8, 8), (16, 16), (8, 4), (16, 8), (8, 2), (16, 4), (32, 8), (16, 2))


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _lens(rng, total, n):
    """n lengths (at least 1) of about `total` tokens together, uneven."""
    w = [rng.uniform(0.2, 1.0) for _ in range(n)]
    return ",".join(str(max(1, int(total * x / sum(w)) - rng.randint(0, 3))) for x in w)


def draw(rng):
    while True:
        op = rng.choice(["layer"] * 5 + ["prefill", "train", "train", "sparse", "dense",
                                         "decode", "decode"])
        hq, hkv = rng.choice(_HEADS)
        d = rng.choice([64, 128, 128])
        if op == "decode":
            n = rng.randint(1, 24)
            lens = ",".join(str(_log_int(rng, 16, 32768)) for _ in range(n))
        else:
            top = {"layer": 65536, "prefill": 16384, "train": 32768, "sparse": 32768,
                   "dense": 16384}[op]
            lens = _lens(rng, _log_int(rng, 512, top), rng.randint(1, 6))
        c = _case(None, op, lens, hq, hkv, d, _log_int(rng, 32, 4096),
                  round(math.exp(rng.uniform(math.log(1 / 32), math.log(0.75))), 4),
                  gate=rng.choice(["uniform", "logit_normal", "burst"]),
                  mode=rng.choice(["ratio", "threshold", "device"]),
                  distinct=rng.random() < 0.4, gains=rng.random() < 0.4)
        if op == "prefill":
            c.update(d_model=rng.choice([512, 1000, 2048, 4096]), mode="ratio", distinct=False)
        if op in ("train", "sparse"):
            c["mode"] = "ratio"          # (every saved row is then defined)
        if op == "dense":
            c.update(window=max(_ints(lens)), ratio=1.0)
        if op == "decode":
            c["mode"] = rng.choice(["threshold", "device"])
        if work(c)["flops"] <= 4e12:
            return c


# --- inputs ------------------------------------------------------------------
def _ints(lens):
    return [int(x) for x in lens.split(",")]


def _burst(rng, T):
    """A two-state chain: on-runs of mean 8 (p in [0.5, 1)), off-runs of mean
    56 (p in [0, 0.5))."""
    runs, n, on = [], 0, rng.random() < 0.125
    while n < T:
        r = rng.geometric(1 / 8 if on else 1 / 56)
        runs.append((r, on))
        n += r
        on = not on
    s = np.concatenate([np.full(r, o) for r, o in runs])[:T]
    u = rng.random(T, dtype=np.float32)
    half = np.float32(0.5)
    return np.where(s, half + half * u, half * u).astype(np.float32)


def _gate(rng, lens, kind):
    parts = []
    for T in lens:
        if kind == "burst":
            parts.append(_burst(rng, T))
        elif kind == "logit_normal":
            parts.append((1.0 / (1.0 + np.exp(-rng.standard_normal(T)))).astype(np.float32))
        else:
            parts.append(rng.random(T, dtype=np.float32))
    return np.concatenate(parts)


def _threshold(gate, ratio):
    """The threshold that about `ratio` of these gates pass."""
    s = np.sort(gate)[::-1]
    return float(s[min(int(ratio * gate.size), gate.size - 1)])


def prepare(case, seed):
    dev = "cuda"
    g = torch.Generator(device=dev)
    g.manual_seed(seed)
    rng = np.random.default_rng(seed)
    lens, op = _ints(case["lens"]), case["op"]
    N, B, Hq, Hkv, d = sum(lens), len(lens), case["hq"], case["hkv"], case["d"]
    rows = B if op == "decode" else N

    def normal(*shape):
        return torch.randn(shape, generator=g, device=dev, dtype=torch.float32).to(torch.bfloat16)

    def uniform(lo, hi, *shape):
        return lo + (hi - lo) * torch.rand(shape, generator=g, device=dev, dtype=torch.float32)

    s = dict(case=case)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    s["prob"] = pk.Problem(torch.from_numpy(cu).to(dev), Hq, Hkv, d, case["window"],
                           cu_seqlens_host=cu)
    prob = s["prob"]
    s["q"], s["k"], s["v"] = normal(rows, Hq, d), normal(N, Hkv, d), normal(N, Hkv, d)
    gate = _gate(rng, [rows] if op == "decode" else lens, case["gate"])
    thr = _threshold(gate, case["ratio"]) if op != "decode" else 1.0 - case["ratio"]
    s["gate"] = torch.from_numpy(gate).to(dev)
    s["sel"] = {"ratio": dict(ratio=case["ratio"]), "threshold": dict(threshold=thr)}.get(
        case["mode"])
    if case["mode"] == "device":
        s["sel"] = dict(threshold_device=torch.full((B,), thr, device=dev))
    if op == "decode" and case["mode"] == "ratio":
        s["sel"] = dict(threshold=thr)
    s["kw"] = {}
    if case["distinct"]:
        s["kw"].update(q_g=normal(rows, Hq, d), k_g=normal(N, Hkv, d), v_g=normal(N, Hkv, d))
    if case["gains"]:
        s["kw"].update(gain_local=uniform(0.5, 1.5, Hq, d), gain_global=uniform(0.5, 1.5, Hq, d))

    def ws(entry, cap=0):
        return torch.empty(max(pk.logo_workspace_bytes(prob, entry, cap), 256),
                           dtype=torch.uint8, device=dev)

    def ints(n):
        return torch.full((n,), -1, dtype=torch.int32, device=dev)

    if op in ("layer", "prefill", "train", "sparse"):
        cap = pk.logo_ratio_capacity(prob, case["ratio"]) if case["mode"] == "ratio" else N
        s["cap"] = cap = max(cap, 1)
    if op in ("layer", "prefill"):
        s["bufs"] = dict(out=torch.empty((N, Hq, d), dtype=torch.bfloat16, device=dev),
                         sel_idx=ints(cap), cu_sel=ints(B + 1), tok2sel=ints(N))
        if case["mode"] != "device":
            s["bufs"]["thr_out"] = torch.empty(B, dtype=torch.float32, device=dev)
        s["ws"] = ws(pk.LOGO_ENTRY_FWD if op == "layer" else pk.LOGO_ENTRY_FWD_QPHI, cap)
    if op == "prefill":
        dm = case["d_model"]
        s["x"], s["w_g"] = normal(N, dm), (normal(dm).float() / math.sqrt(dm)).to(torch.bfloat16)
        eye = torch.eye(d, device=dev)

        def near_identity(H):
            return (eye + 0.5 / math.sqrt(d) * torch.randn(
                (H, d, d), generator=g, device=dev, dtype=torch.float32)).to(torch.bfloat16)
        s["A_q"], s["A_k"] = near_identity(Hq), near_identity(Hkv)
        s["s_v"], s["b_v"] = uniform(0.5, 1.5, Hkv, d), uniform(-0.2, 0.2, Hkv, d)
        s["p"] = torch.empty(N, dtype=torch.float32, device=dev)
        s["k_g"], s["v_g"] = torch.empty_like(s["k"]), torch.empty_like(s["v"])
    if op == "train":
        s["dout"] = normal(N, Hq, d)
        s["ws_f"], s["ws_b"] = ws(pk.LOGO_ENTRY_FWD_TRAIN, cap), ws(pk.LOGO_ENTRY_BWD, cap)
    if op == "sparse":
        s["dout"] = normal(cap, Hq, d)
        s["ws_s"] = ws(pk.LOGO_ENTRY_SELECT)
        s["ws_f"], s["ws_b"] = ws(pk.LOGO_ENTRY_GLOBAL, cap), ws(pk.LOGO_ENTRY_GLOBAL_BWD, cap)
    if op == "dense":
        s["dout"], s["ws_b"] = normal(N, Hq, d), ws(pk.LOGO_ENTRY_DENSE_BWD)
    if op == "decode":
        s["bufs"] = dict(out=torch.empty((B, Hq, d), dtype=torch.bfloat16, device=dev),
                         active=ints(B), n_active=ints(1))
        s["ws"] = ws(pk.LOGO_ENTRY_DECODE)
    return s


# --- one pass ----------------------------------------------------------------
def run(s):
    op, prob = s["case"]["op"], s["prob"]
    q, k, v, gate = s["q"], s["k"], s["v"], s["gate"]
    if op == "layer":
        r = pk.logo_attn_fwd(prob, q, k, v, gate, **s["sel"], **s["kw"], sel_capacity=s["cap"],
                             ws=s["ws"], **s["bufs"])
        return dict(zip(("out", "sel_idx", "cu_sel", "tok2sel", "thr"), r))
    if op == "prefill":
        p = pk.logo_gate_proj(s["x"], s["w_g"], out=s["p"])
        k_g = pk.logo_branch_transform(k, pk.LOGO_PHI_LP, A=s["A_k"], out=s["k_g"])
        v_g = pk.logo_branch_transform(v, pk.LOGO_PHI_SO, s=s["s_v"], b=s["b_v"], out=s["v_g"])
        r = pk.logo_attn_fwd_qphi(prob, q, k, v, p, pk.LOGO_PHI_LP, A=s["A_q"], k_g=k_g, v_g=v_g,
                                  **s["sel"], **s["kw"], sel_capacity=s["cap"], ws=s["ws"],
                                  **s["bufs"])
        return dict(p=p, k_g=k_g, v_g=v_g, out=r[0], cu_sel=r[2])
    if op == "train":
        st = pk.logo_attn_fwd_train(prob, q, k, v, gate, **s["sel"], **s["kw"],
                                    sel_capacity=s["cap"], ws=s["ws_f"])
        grads = pk.logo_attn_bwd(prob, q, k, v, gate, st, s["dout"], **s["kw"], ws=s["ws_b"])
        return dict(out=st["out"], tok2sel=st["tok2sel"], **grads)
    if op == "sparse":
        sel_idx, cu_sel, tok2sel, _ = pk.logo_select(prob, gate, **s["sel"],
                                                     sel_capacity=s["cap"], ws=s["ws_s"])
        o, lse = pk.logo_global_attn_sparse_q_fwd_train(prob, q, k, v, sel_idx, cu_sel, s["cap"],
                                                        ws=s["ws_f"])
        grads = pk.logo_global_attn_sparse_q_bwd(prob, q, k, v, sel_idx, cu_sel, s["cap"], o, lse,
                                                 s["dout"], ws=s["ws_b"])
        return dict(o=o, lse=lse, tok2sel=tok2sel, **grads)
    if op == "dense":
        out, lse = pk.logo_dense_causal_attn_fwd_train(prob, q, k, v)
        grads = pk.logo_dense_causal_attn_bwd(prob, q, k, v, out, lse, s["dout"], ws=s["ws_b"])
        return dict(out=out, lse=lse, **grads)
    out, _, n_active = pk.logo_decode(prob, q, k, v, gate, **s["sel"], **s["kw"], ws=s["ws"],
                                      **s["bufs"])
    return dict(out=out, n_active=n_active)


# --- the least work of one pass ------------------------------------------------
def _pairs(T, w):
    """Visible (query, key) pairs of T causal rows with a window of w keys."""
    w = min(w, T)
    return w * (w + 1) // 2 + (T - w) * w


def work(case):
    lens, op = _ints(case["lens"]), case["op"]
    N, B, Hq, Hkv, d = sum(lens), len(lens), case["hq"], case["hkv"], case["d"]
    w, rho = case["window"], case["ratio"]
    local = Hq * sum(_pairs(T, w) for T in lens)
    glob = Hq * rho * sum(_pairs(T, T) for T in lens)
    q_b, kv_b = 2 * N * Hq * d, 2 * 2 * N * Hkv * d
    nsel = rho * N
    dist = 1 if case["distinct"] else 0
    if op == "layer":
        return dict(flops=4 * d * (local + glob),
                    bytes=2 * q_b + kv_b * (1 + dist) + dist * rho * q_b + 8 * N + 4 * nsel)
    if op == "prefill":
        lp = 2 * d * d * (N * Hkv + nsel * Hq)
        return dict(flops=4 * d * (local + glob) + lp + 2 * N * case["d_model"],
                    bytes=2 * N * case["d_model"] + 2 * q_b + 2 * kv_b + 8 * N +
                    2 * d * d * (Hq + Hkv))
    if op == "train":
        # forward 2 products, backward 5, per visible pair; out and fp32 gradients
        return dict(flops=14 * d * (local + glob),
                    bytes=(1 + dist) * (q_b + kv_b) + 2 * q_b + 2 * (1 + dist) * (q_b + kv_b) +
                    12 * N)
    if op == "sparse":
        return dict(flops=14 * d * glob,
                    bytes=rho * q_b + kv_b + 3 * rho * q_b + 2 * (q_b + kv_b) + 8 * N)
    if op == "dense":
        pairs = Hq * sum(_pairs(T, T) for T in lens)
        return dict(flops=14 * d * pairs, bytes=5 * q_b + 3 * kv_b + 4 * N * Hq)
    rows_l, rows_g = sum(min(T, w) for T in lens), rho * sum(lens)
    if not dist:                       # a selected token's window is part of its cache
        rows_g -= rho * rows_l
    return dict(flops=4 * d * Hq * (rows_l + rows_g),
                bytes=4 * Hkv * d * (rows_l + rows_g) + 4 * B * Hq * d)


# Relative errors: bf16 outputs carry 2^-9 each, P and dS are rounded to bf16
# for the matrix products.  Measured against `exact`: layer and dense outputs
# 2.0e-3 to 2.3e-3, decoding and transforms 1.7e-3, gradients 1.5e-3 to 2.6e-3,
# fp32 LSEs 1e-5; four times the largest is stated.
def tolerance(case):
    return {"rel": 0.01}


# --- the same in 64 bits -------------------------------------------------------
def _select64(case, s, gate, lens, z_known=None):
    """z [N] bool, thr [B] as the selection defines them."""
    z, thr, off = torch.zeros_like(gate, dtype=torch.bool), [], 0
    for T in lens:
        gs = gate[off:off + T]
        if "ratio" in s["sel"]:
            kk = int(math.floor(case["ratio"] * T))
            t = torch.sort(gs, descending=True)[0][kk] if kk < T else torch.tensor(
                -math.inf, device=gate.device, dtype=gate.dtype)
        elif "threshold" in s["sel"]:
            t = torch.tensor(s["sel"]["threshold"], device=gate.device, dtype=torch.float32).to(
                gate.dtype)
        else:
            t = s["sel"]["threshold_device"][0].to(gate.dtype)
        z[off:off + T] = gs > t
        thr.append(t)
        off += T
    return z, torch.stack(thr)


def _attn64(q, k, v, pos, window, scale, dout=None, out=None, lse=None):
    """Softmax attention of query rows q [R, Hq, d] at positions pos [R]
    (ascending) over one sequence's k, v [T, Hkv, d]; keys pos-window < j <= pos.
    Without dout: (o, base-2 lse [Hq, R]).  With dout: (dq, dk, dv)."""
    R, Hq, d = q.shape
    T, Hkv, _ = k.shape
    G = Hq // Hkv
    o = torch.zeros_like(q)
    ls = torch.zeros((Hq, R), dtype=q.dtype, device=q.device)
    dk, dv = torch.zeros_like(k), torch.zeros_like(v)
    step = 1024
    for r0 in range(0, R, step):
        r1 = min(R, r0 + step)
        p = pos[r0:r1]
        lo, hi = max(0, int(p[0]) - window + 1), int(p[-1]) + 1
        j = torch.arange(lo, hi, device=q.device)
        hide = (j[None, :] > p[:, None]) | (j[None, :] <= p[:, None] - window)
        for h in range(Hkv):
            kk, vv = k[lo:hi, h].contiguous(), v[lo:hi, h].contiguous()
            kt = kk.t().contiguous()
            for hq in range(h * G, (h + 1) * G):
                qq = q[r0:r1, hq].contiguous()
                sc = (qq @ kt) * scale
                sc.masked_fill_(hide, -math.inf)
                if dout is None:
                    m = torch.logsumexp(sc, dim=1)
                    o[r0:r1, hq] = (sc - m[:, None]).exp_() @ vv
                    ls[hq, r0:r1] = m / math.log(2.0)
                    continue
                pr = (sc - lse[hq, r0:r1, None] * math.log(2.0)).exp_()
                do = dout[r0:r1, hq].contiguous()
                dv[lo:hi, h] += pr.t().contiguous() @ do
                ds = do @ vv.t().contiguous()
                ds -= (do * out[r0:r1, hq]).sum(1)[:, None]
                ds *= pr
                o[r0:r1, hq] = (ds @ kk) * scale
                dk[lo:hi, h] += (ds.t().contiguous() @ qq) * scale
    return (o, ls) if dout is None else (o, dk, dv)


def _norm64(o, gain):
    r = torch.sqrt((o * o).mean(-1, keepdim=True) + EPS)
    return o / r * (1.0 if gain is None else gain)


def _norm_bwd64(o, gain, dy):
    """(do, dgain) of _norm64."""
    g = 1.0 if gain is None else gain
    r = torch.sqrt((o * o).mean(-1, keepdim=True) + EPS)
    gd = dy * g
    do = gd / r - o * (gd * o).mean(-1, keepdim=True) / r ** 3
    return do, (dy * o / r).sum(0)


def exact(case, seed):
    s = prepare(case, seed)
    lens, op = _ints(case["lens"]), case["op"]
    N, B, Hq, Hkv, d = sum(lens), len(lens), case["hq"], case["hkv"], case["d"]
    w, scale, dev = case["window"], 1.0 / math.sqrt(d), s["q"].device
    q, k, v = s["q"].double(), s["k"].double(), s["v"].double()
    gate = s["gate"]
    kw = {n: t.double() for n, t in s["kw"].items()}
    gl, gg = kw.get("gain_local"), kw.get("gain_global")
    qg, kg, vg = kw.get("q_g", q), kw.get("k_g", k), kw.get("v_g", v)
    offs = [sum(lens[:b]) for b in range(B)]
    res = {}
    if op == "decode":
        out = torch.zeros_like(q)
        thr = s["sel"].get("threshold")
        thr = s["sel"]["threshold_device"][0] if thr is None else torch.tensor(
            thr, dtype=torch.float32, device=dev)
        z = gate > thr
        for b in range(B):
            a0, a1 = offs[b], offs[b] + lens[b]
            pos = torch.tensor([lens[b] - 1], device=dev)
            y = _norm64(_attn64(q[b:b + 1], k[a0:a1], v[a0:a1], pos, w, scale)[0], gl)
            if z[b]:
                o = _attn64(qg[b:b + 1], kg[a0:a1], vg[a0:a1], pos, lens[b], scale)[0]
                p = gate[b].double()
                y = (1 - p) * y + p * _norm64(o, gg)
            out[b:b + 1] = y
        return dict(out=out, n_active=z.sum().reshape(1).to(torch.int32))
    if op == "dense":
        out, lse = torch.zeros_like(q), torch.zeros((Hq, N), dtype=q.dtype, device=dev)
        dq, dk, dv = torch.zeros_like(q), torch.zeros_like(k), torch.zeros_like(v)
        dout = s["dout"].double()
        for b in range(B):
            a0, a1 = offs[b], offs[b] + lens[b]
            pos = torch.arange(lens[b], device=dev)
            o, l = _attn64(q[a0:a1], k[a0:a1], v[a0:a1], pos, lens[b], scale)
            out[a0:a1], lse[:, a0:a1] = o, l
            dq[a0:a1], dk[a0:a1], dv[a0:a1] = _attn64(q[a0:a1], k[a0:a1], v[a0:a1], pos, lens[b],
                                                     scale, dout[a0:a1], o, l)
        return dict(out=out, lse=lse, dq=dq, dk=dk, dv=dv)
    if op == "prefill":
        gate = torch.sigmoid(s["x"].double() @ s["w_g"].double())
        kg = torch.einsum("nhc,hcj->nhj", k, s["A_k"].double())
        vg = v * s["s_v"].double() + s["b_v"].double()
        qg = torch.einsum("nhc,hcj->nhj", q, s["A_q"].double())
        res.update(p=gate, k_g=kg, v_g=vg)
    z, thr = _select64(case, s, gate, lens)
    gate = gate.double()
    idx = torch.nonzero(z).flatten()
    n_sel = int(idx.numel())
    tok2sel = torch.full((N,), -1, dtype=torch.int32, device=dev)
    tok2sel[idx] = torch.arange(n_sel, dtype=torch.int32, device=dev)
    counts = [int(z[offs[b]:offs[b] + lens[b]].sum()) for b in range(B)]
    c0 = [sum(counts[:b]) for b in range(B + 1)]
    cu_sel = torch.tensor(c0, dtype=torch.int32, device=dev)
    # the global branch of the selected rows
    og = torch.zeros((n_sel, Hq, d), dtype=q.dtype, device=dev)
    lg = torch.zeros((Hq, n_sel), dtype=q.dtype, device=dev)
    for b in range(B):
        a0, a1, i = offs[b], offs[b] + lens[b], idx[c0[b]:c0[b + 1]]
        if i.numel():
            og[c0[b]:c0[b + 1]], lg[:, c0[b]:c0[b + 1]] = _attn64(
                qg[i], kg[a0:a1], vg[a0:a1], i - a0, lens[b], scale)
    if op == "sparse":
        do = s["dout"].double()[:n_sel]
        dq, dk, dv = torch.zeros_like(q), torch.zeros_like(k), torch.zeros_like(v)
        for b in range(B):
            a0, a1, i = offs[b], offs[b] + lens[b], idx[c0[b]:c0[b + 1]]
            if i.numel():
                e = slice(c0[b], c0[b + 1])
                dq[i], dk[a0:a1], dv[a0:a1] = _attn64(q[i], k[a0:a1], v[a0:a1], i - a0, lens[b],
                                                     scale, do[e], og[e], lg[:, e])
        whole = n_sel == s["cap"]          # (ties leave rows that no one writes)
        return dict(o=og if whole else None, lse=lg if whole else None, tok2sel=tok2sel, dq=dq,
                    dk=dk, dv=dv)
    ol, ll = torch.zeros_like(q), torch.zeros((Hq, N), dtype=q.dtype, device=dev)
    for b in range(B):
        a0, a1 = offs[b], offs[b] + lens[b]
        pos = torch.arange(lens[b], device=dev)
        ol[a0:a1], ll[:, a0:a1] = _attn64(q[a0:a1], k[a0:a1], v[a0:a1], pos, w, scale)
    out = _norm64(ol, gl)
    p = gate[idx][:, None, None]
    nl, ng = out[idx], _norm64(og, gg)
    out[idx] = (1 - p) * nl + p * ng
    if op == "prefill":
        return dict(res, out=out, cu_sel=cu_sel)
    if op == "layer":
        si = torch.full((s["cap"],), -1, dtype=torch.int32, device=dev)
        si[:n_sel] = idx.to(torch.int32)
        return dict(out=out, sel_idx=si, cu_sel=cu_sel, tok2sel=tok2sel, thr=thr)
    # training: the backward pass with the selection held fixed
    dout = s["dout"].double()
    dn = dout.clone()
    dn[idx] *= 1 - p
    dol, dgain_l = _norm_bwd64(ol, gl, dn)
    dog, dgain_g = _norm_bwd64(og, gg, dout[idx] * p)
    dgate = torch.zeros(N, dtype=q.dtype, device=dev)
    dgate[idx] = (dout[idx] * (ng - nl)).sum((1, 2))
    dq, dk, dv = torch.zeros_like(q), torch.zeros_like(k), torch.zeros_like(v)
    dqg, dkg, dvg = torch.zeros_like(q), torch.zeros_like(k), torch.zeros_like(v)
    for b in range(B):
        a0, a1, i = offs[b], offs[b] + lens[b], idx[c0[b]:c0[b + 1]]
        pos = torch.arange(lens[b], device=dev)
        dq[a0:a1], dk[a0:a1], dv[a0:a1] = _attn64(q[a0:a1], k[a0:a1], v[a0:a1], pos, w, scale,
                                                 dol[a0:a1], ol[a0:a1], ll[:, a0:a1])
        if i.numel():
            e = slice(c0[b], c0[b + 1])
            dqg[i], dkg[a0:a1], dvg[a0:a1] = _attn64(qg[i], kg[a0:a1], vg[a0:a1], i - a0, lens[b],
                                                    scale, dog[e], og[e], lg[:, e])
    grads = dict(dq=dq, dk=dk, dv=dv, dgate=dgate, dgain_local=dgain_l, dgain_global=dgain_g)
    if case["distinct"]:
        grads.update(dq_g=dqg, dk_g=dkg, dv_g=dvg)
    else:
        grads.update(dq=dq + dqg, dk=dk + dkg, dv=dv + dvg)
    return dict(out=out, tok2sel=tok2sel, **grads)
