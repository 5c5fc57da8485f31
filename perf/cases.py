"""The work this library is timed on: one pass through its public entry points
(the plans of `hstu.py`, the lookups of `embedding.py`) over the range a user
of a sequence recommender meets, from a handful of short sequences served in
fp32 to a training step on a thousand sequences of up to 8192 tokens.

Four kinds of case:

* "attn":  jagged HSTU attention, forward alone (serving) or forward and
  backward (training); bf16 or fp32, either bias or both, plain or
  deterministic table gradients, plain or scaled scores;
* "layer": the HSTU layer around it (both GEMMs), forward alone or a step;
* "emb":   the jagged multi-table embedding lookup, forward alone or with its
  sparse backward;
* "rab":   the standalone relative attention bias and its backward.

A case names its batch by numbers alone.  `lens` seeds the sequence lengths,
which belong to the case (they set the work); the values of the tensors follow
the seed that `prepare` is given.  Inputs are drawn on the GPU with the
distributions of `inputs.py` and `emb_inputs.py`.
"""
import math

import numpy as np
import torch

from paper_2605_13433_amd import embedding, hstu

DEV = "cuda"
LN_EPS = 1e-6
TS_GAP_MEAN = 600.0
RAB_STD = 0.1
EMB_ALPHA = 1.05
HASH_MUL = 2654435761


# ------------------------------------------------------------------- cases
def _attn(name, dtype, B, kind, lo, hi, H, d, pos, time, bwd, N=None, alpha=1.0, det=False,
          nb=128, lens=1, p=0.0):
    return dict(name=name, kind="attn", dtype=dtype, B=B, dist=kind, p=p, lo=lo, hi=hi,
                N=N or hi, H=H, d=d, pos=pos, time=time, nb=nb, alpha=alpha, det=det, bwd=bwd,
                lens=lens)


def listed():
    return [
        # the smallest call: four short sequences in fp32, forward only
        # (launches and latency are all of it)
        _attn("serve_tiny_f32", "f32", 4, "uniform", 1, 64, 2, 32, True, False, False, lens=1),
        # online scoring of a few users in bf16, odd lengths, both biases
        _attn("serve_small", "bf16", 8, "uniform", 3, 250, 4, 64, True, True, False, N=256,
              lens=2),
        # prefill of a few long histories at the wide head
        _attn("serve_long", "bf16", 6, "uniform", 700, 8192, 4, 128, True, True, False, lens=3),
        # training step on many short users (power law, at most 512 tokens)
        _attn("train_powerlaw", "bf16", 128, "powerlaw", 16, 512, 4, 64, True, True, True,
              p=1.2, lens=2),
        # training step on a short/long mix at 8 heads of 128
        _attn("train_longtail", "bf16", 64, "mix", 32, 2048, 8, 128, True, True, True, p=0.2,
              lens=3),
        # the largest training step: a thousand users, Zipf lengths to 8192
        _attn("train_zipf", "bf16", 1024, "powerlaw", 1, 8192, 4, 64, True, False, True,
              p=1.05, lens=5),
        # training step in fp32 (the precision the models are checked at)
        _attn("train_f32", "f32", 48, "powerlaw", 16, 512, 4, 64, True, True, True, p=1.2,
              lens=7),
        # a whole layer's training step: both GEMMs and the attention
        dict(name="layer_train", kind="layer", B=32, dist="powerlaw", p=1.1, lo=64, hi=4096,
             N=4096, H=4, d=128, D=512, pos=True, time=True, nb=128, bwd=True, lens=4),
        # a layer's forward on a small ragged batch
        dict(name="layer_serve", kind="layer", B=12, dist="uniform", p=0.0, lo=5, hi=500,
             N=512, H=4, d=64, D=256, pos=True, time=True, nb=128, bwd=False, lens=9),
        # embedding of a training batch: 8 tables, hot to cold, fp32, the
        # token layout a sequence model reads, with the sparse backward
        dict(name="emb_train", kind="emb", dtype="f32", tables=8, top=22, step=2, T=77971, D=128,
             layout="token", bwd=True),
        # lookup of a serving batch from bf16 tables
        dict(name="emb_serve", kind="emb", dtype="bf16", tables=6, top=20, step=2, T=5003, D=64,
             layout="flat", bwd=False),
        # the bias tensor on its own, all three encodings, with its backward
        dict(name="rab_train", kind="rab", B=64, dist="mix", p=0.2, lo=32, hi=2048, N=2048, H=8,
             pos=True, time=True, fn=True, nb=128, bwd=True, lens=3),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["attn", "attn", "attn", "f32", "layer", "emb", "rab"])
    bias = rng.choice([(True, True), (True, True), (True, False), (False, True), (False, False)])
    dist, p = rng.choice([("uniform", 0.0), ("powerlaw", rng.uniform(1.0, 1.3)),
                          ("mix", rng.uniform(0.1, 0.4))])
    lens = rng.randrange(1 << 20)
    nb = rng.choice([32, 64, 128])
    if kind in ("attn", "f32", "layer"):
        d = rng.choice([32, 64, 128] if kind == "f32" else [64, 128])
        c = dict(kind="attn" if kind == "f32" else kind, B=_log_int(rng, 1, 1024),
                 dist=dist, p=round(p, 3), lo=_log_int(rng, 1, 60),
                 hi=_log_int(rng, 64, 700 if kind == "f32" else 8192), H=rng.choice([1, 2, 4, 8]),
                 d=d, pos=bias[0], time=bias[1], nb=nb, bwd=rng.random() < 0.6, lens=lens)
        c["N"] = c["hi"] + rng.choice([0, 0, 1, 13])
        if kind == "layer":
            c["D"] = rng.choice([128, 200, 256, 512])
        else:
            c.update(dtype="f32" if kind == "f32" else "bf16",
                     alpha=rng.choice([1.0, 1.0, round(d ** -0.5, 4)]),
                     det=bool(c["bwd"] and rng.random() < 0.25))
        cap = {"attn": 2.2e12, "layer": 1.5e12, "f32": 4e9}[kind]
        while c["B"] > 1 and (work(c)["flops"] > cap or work(c)["bytes"] > 2e10):
            c["B"] //= 2
        while work(c)["flops"] > cap:
            c["hi"] = c["N"] = max(c["lo"] + 1, c["hi"] // 2)
        return c
    if kind == "emb":
        F = rng.randrange(1, 13)
        return dict(kind="emb", dtype=rng.choice(["f32", "bf16"]), tables=F,
                    top=rng.randrange(10, 23), step=rng.choice([1, 2, 3]),
                    T=max(1, min(_log_int(rng, 40, 150000), 600000 // F)),
                    D=rng.choice([8, 24, 64, 128, 256]), layout=rng.choice(["flat", "token"]),
                    bwd=rng.random() < 0.6)
    enc = rng.choice([(True, True, True), (True, True, False), (True, False, False),
                      (False, True, False), (False, False, True)])
    c = dict(kind="rab", B=_log_int(rng, 1, 128), dist=dist, p=round(p, 3),
             lo=_log_int(rng, 1, 60), hi=_log_int(rng, 64, 2048), H=rng.choice([1, 2, 4, 8]),
             pos=enc[0], time=enc[1], fn=enc[2], nb=nb, bwd=rng.random() < 0.6, lens=lens)
    c["N"] = c["hi"] + rng.choice([0, 0, 1, 13])
    while c["B"] > 1 and work(c)["bytes"] > 8e8:
        c["B"] //= 2
    return c


def _lengths(case):
    """Sequence lengths of the batch (host, from the case alone)."""
    rng = np.random.default_rng(case["lens"])
    B, lo, hi = case["B"], case["lo"], case["hi"]
    if case["dist"] == "uniform":
        return rng.integers(lo, hi + 1, size=B).astype(np.int64)
    if case["dist"] == "powerlaw":
        support = np.arange(lo, hi + 1, dtype=np.float64)
        w = support ** -case["p"]
        return rng.choice(np.arange(lo, hi + 1), size=B, p=w / w.sum()).astype(np.int64)
    cut = max(lo + 1, hi // 8)                        # "mix": many short, some long
    return np.where(rng.random(B) < case["p"], rng.integers(cut, hi + 1, size=B),
                    rng.integers(lo, cut + 1, size=B)).astype(np.int64)


def _offsets(lengths):
    off = np.zeros(len(lengths) + 1, dtype=np.int64)
    np.cumsum(lengths, out=off[1:])
    return off


# ------------------------------------------------------------------ inputs
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _normal(g, shape, dtype=torch.float32, std=1.0):
    x = torch.randn(shape, generator=g, device=DEV, dtype=torch.float32)
    if std != 1.0:
        x *= std
    return x.to(dtype)


def _timestamps(g, off):
    """Per sequence a Poisson clock: ts_0 = 0, gaps 1 + floor(Exp(600 s))."""
    T = int(off[-1])
    if T == 0:
        return torch.zeros(0, dtype=torch.int64, device=DEV)
    gaps = 1 + torch.empty(T, device=DEV, dtype=torch.float64).exponential_(
        1.0 / TS_GAP_MEAN, generator=g).floor().to(torch.int64)
    c = torch.cumsum(gaps, 0)
    first = torch.from_numpy(np.repeat(off[:-1], np.diff(off))).to(DEV)
    return c - c[first]


def _bias_inputs(case, g, off):
    H, N = case["H"], case["N"]
    pos = _normal(g, (H, 2 * N - 1), std=RAB_STD) if case["pos"] else None
    time = _normal(g, (H, case["nb"]), std=RAB_STD) if case["time"] else None
    ts = _timestamps(g, off) if case["time"] or case.get("fn") else None
    return pos, time, ts


def _inputs(case, seed):
    g = _gen(seed)
    if case["kind"] == "emb":
        rows = [1 << max(7, case["top"] - case["step"] * t) for t in range(case["tables"])]
        ro = _offsets(np.asarray(rows, dtype=np.int64))
        T, D = case["T"], case["D"]
        dt = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
        ids = []
        for R in rows:
            # rank r with probability ~ (r + 1)^-alpha, by the inverse of the
            # continuous power law on [1, R + 1), hashed onto scattered rows
            u = torch.rand(T, generator=g, device=DEV, dtype=torch.float64)
            e = 1.0 - EMB_ALPHA
            r = (1.0 + u * ((R + 1.0) ** e - 1.0)) ** (1.0 / e)
            r = r.floor().to(torch.int64).clamp_(1, R) - 1
            ids.append((r * HASH_MUL) % R)
        x = dict(weights=_normal(g, (int(ro[-1]), D), dt), ids=torch.cat(ids),
                 ro=torch.from_numpy(ro).to(DEV),
                 io=torch.arange(len(rows) + 1, device=DEV, dtype=torch.int64) * T,
                 total_rows=int(ro[-1]))
        shape = (T * len(rows), D) if case["layout"] == "flat" else (T, len(rows) * D)
        x["dout"] = _normal(g, shape, dt) if case["bwd"] else None
        return x
    L = _lengths(case)
    off = _offsets(L)
    x = dict(lengths=L, off_np=off, off=torch.from_numpy(off).to(DEV))
    x["pos"], x["time"], x["ts"] = _bias_inputs(case, g, off)
    T, H = int(off[-1]), case["H"]
    if case["kind"] == "rab":
        x["fn"] = None
        if case["fn"]:                                # amplitude, exponent
            x["fn"] = torch.stack([_normal(g, (H,), std=0.2),
                                   0.1 + 0.5 * torch.rand(H, generator=g, device=DEV)], 1)
            x["fn"] = x["fn"].contiguous()
        x["square"] = int((L * L).sum())
        x["d_rab"] = _normal(g, (H, x["square"])) if case["bwd"] else None
        return x
    d = case["d"]
    if case["kind"] == "layer":
        D, bf = case["D"], torch.bfloat16
        x["x"] = _normal(g, (T, D), bf)
        x["w1"] = _normal(g, (D, 4 * H * d), bf, D ** -0.5)
        x["w2"] = _normal(g, (H * d, D), bf, (H * d) ** -0.5)
        x["dout"] = _normal(g, (T, D), bf) if case["bwd"] else None
        return x
    dt = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    for n in "qkvu":
        x[n] = _normal(g, (T, H, d), dt)
    x["dy"] = _normal(g, (T, H * d), dt) if case["bwd"] else None
    return x


def prepare(case, seed):
    """Inputs on the GPU and the plan (outputs and workspace) a program keeps."""
    x = _inputs(case, seed)
    s = dict(case=case, x=x)
    if case["kind"] == "emb":
        s["plan"] = embedding.plan(x["weights"], x["ro"], x["io"], x["total_rows"],
                                   x["ids"].numel(), case["layout"], with_bwd=case["bwd"])
        s["out"] = torch.empty(s["plan"].out_shape, dtype=x["weights"].dtype, device=DEV)
        if case["bwd"]:
            s["grad"] = torch.zeros(x["total_rows"], case["D"], device=DEV)
            s["rows"] = torch.full((x["ids"].numel(),), -1, dtype=torch.int64, device=DEV)
            s["count"] = torch.zeros(1, dtype=torch.int32, device=DEV)
    elif case["kind"] == "rab":
        s["plan"] = hstu.RabPlan(x["off"], case["N"], case["H"], int(x["off_np"][-1]),
                                 x["square"], x["pos"], x["time"], x["fn"], x["ts"], case["nb"])
    elif case["kind"] == "layer":
        s["plan"] = hstu.LayerPlan(x["x"], x["off"], case["N"], case["H"], case["d"], x["pos"],
                                   x["time"], x["ts"], case["nb"], backward=case["bwd"])
    else:
        s["plan"] = hstu.Plan(x["q"], x["off"], case["N"], x["pos"], x["time"], x["ts"],
                              case["nb"], backward=case["bwd"], alpha=case["alpha"],
                              deterministic=case["det"])
    return s


# --------------------------------------------------------------------- run
def run(state):
    case, x, plan = state["case"], state["x"], state["plan"]
    if case["kind"] == "emb":
        out = dict(out=embedding.lookup(plan, x["weights"], x["ids"], state["out"]))
        if case["bwd"]:
            embedding.lookup_backward(plan, x["ids"], x["dout"], state["grad"], state["rows"],
                                      state["count"])
            out.update(grad=state["grad"], rows=state["rows"], count=state["count"])
        return out
    if case["kind"] == "rab":
        out = dict(rab=plan.forward())
        if case["bwd"]:
            g = plan.backward(x["d_rab"])
            out.update({k: v for k, v in zip(("d_pos", "d_time", "d_fn"), g) if v is not None})
        return out
    if case["kind"] == "layer":
        f = plan.forward(x["x"], x["w1"], x["w2"], x["off"])
        out = dict(out=f.out, h=f.h, z=f.z, y=f.y, o=f.o, mean=f.ln_mean, rstd=f.ln_rstd)
        if case["bwd"]:
            g = plan.backward(x["x"], x["w1"], x["w2"], x["off"], x["dout"])
            out.update(dx=g.dx, dw1=g.dw1, dw2=g.dw2)
    else:
        f = plan.forward(x["q"], x["k"], x["v"], x["u"], x["off"])
        out = dict(y=f.y, o=f.o, mean=f.ln_mean, rstd=f.ln_rstd)
        if case["bwd"]:
            g = plan.backward(x["q"], x["k"], x["v"], x["u"], x["off"], x["dy"])
            out.update(dq=g.dq, dk=g.dk, dv=g.dv, du=g.du)
    if case["bwd"] and case["pos"]:
        out["d_pos"] = g.d_pos_w
    if case["bwd"] and case["time"]:
        out["d_time"] = g.d_time_w
    return out


# -------------------------------------------------------------------- work
def work(case):
    """Bytes: every input and output of the pass once.  Flops: the products
    over causal pairs (4 d forward, 8 d backward per head and pair; the
    recomputed scores are not counted) and the layer's GEMMs; for the bias
    tensor one add per encoding and element, for the lookup one add per
    gathered gradient value."""
    if case["kind"] == "emb":
        n, e = case["T"] * case["tables"], 4 if case["dtype"] == "f32" else 2
        by = n * (8 + 2 * case["D"] * e)
        if case["bwd"]:
            by += n * (8 + case["D"] * e + 4 * case["D"] + 8)
        return dict(bytes=by, flops=n * case["D"] if case["bwd"] else 0)
    L = _lengths(case).astype(np.float64)
    T, H, N = float(L.sum()), case["H"], case["N"]
    tab = 4.0 * H * ((2 * N - 1 if case["pos"] else 0) + (case["nb"] if case["time"] else 0))
    ts = 8.0 * T if case["time"] or case.get("fn") else 0.0
    if case["kind"] == "rab":
        sq = float((L * L).sum()) * H
        enc = int(case["pos"]) + int(case["time"]) + int(case["fn"])
        k = 2 if case["bwd"] else 1
        return dict(bytes=k * (4 * sq + tab + ts), flops=k * enc * sq)
    pairs, d = float((L * (L + 1) / 2).sum()), case["d"]
    C = H * d
    if case["kind"] == "layer":
        D = case["D"]
        fl = 4 * d * H * pairs + 2 * T * D * 4 * C + 2 * T * C * D
        w = 2.0 * (D * 4 * C + C * D)
        by = w + tab + ts + T * (2 * (D + 4 * C + 4 * C + C + C + D) + 8)
        if case["bwd"]:
            fl += 8 * d * H * pairs + 2 * (2 * T * D * 4 * C + 2 * T * C * D)
            by += 2 * w + 2 * tab + ts + T * (2 * (D + D + 4 * C + 4 * C + C + C + D) + 8)
        return dict(bytes=by, flops=fl)
    e = 4 if case["dtype"] == "f32" else 2
    by = 6 * T * C * e + 8 * T + tab + ts
    fl = 4 * d * H * pairs
    if case["bwd"]:
        by += 10 * T * C * e + 8 * T + 2 * tab + ts
        fl += 8 * d * H * pairs
    return dict(bytes=by, flops=fl)


def tolerance(case):
    """bf16: operands and probabilities are rounded to 8 bits on the way, in
    another order where tiles are summed differently (3e-3 from 64 bits; 9e-3
    through a layer's chain).  fp32: sums over up to a few thousand terms and
    hardware exp2 / reciprocal (4e-7 from 64 bits, with more terms 1e-6).  The bias tensor: the
    power law's log2 / exp2 at gaps of 1e6 s.  The lookup's forward copies
    rows; its gradients are fp32 sums over up to thousands of rows."""
    if case["kind"] == "emb":
        return {"rel": 2e-6, "max": 4e-4} if case["bwd"] else "exact"
    if case["kind"] == "rab":
        return {"rel": 2e-6, "max": 1e-4}
    if case["kind"] == "attn" and case["dtype"] == "f32":
        return {"rel": 4e-6, "max": 1e-3}
    return {"rel": 2e-2 if case["kind"] == "layer" else 1e-2, "max": 0.5}


# ------------------------------------------------------------------- exact
def _bucket64(dt, nb):
    """|x| < 4 -> |x|, else 4 (e - 1) + the two bits under the leading one,
    e = floor(log2 |x|), at most nb - 1."""
    x = dt.abs()
    e = torch.floor(torch.log2(x.clamp(min=1).double())).to(torch.int64)
    e = torch.where((x >> e) > 1, e + 1, torch.where((x >> e) < 1, e - 1, e))
    b = torch.where(x < 4, x, 4 * (e - 1) + ((x >> (e - 2).clamp(min=0)) & 3))
    return b.clamp(max=nb - 1)


def _rows_scatter(idx, val, n):
    """Sum val [H, L, L] by idx [L, L] into n bins, row by row first."""
    H, L, _ = val.shape
    out = torch.zeros(H, n, dtype=val.dtype, device=val.device)
    for h in range(H):
        r = torch.zeros(L, n, dtype=val.dtype, device=val.device)
        out[h] = r.scatter_add_(1, idx, val[h]).sum(0)
    return out


def _attn64(case, x, q, k, v, u, dy, alpha):
    """o, mean, rstd, y and the gradients of sum(y dy) in float64, sequence
    by sequence as dense masked products."""
    H, d, N = case["H"], case["d"], case["N"]
    T, off = q.shape[0], x["off_np"]
    f8 = dict(dtype=torch.float64, device=DEV)
    o = torch.zeros(T, H, d, **f8)
    pos = x["pos"].double() if x["pos"] is not None else None
    tim = x["time"].double() if x["time"] is not None else None

    def scores(a, b):
        L = b - a
        qq, kk = (t[a:b].permute(1, 0, 2).contiguous() for t in (q, k))
        s = alpha * torch.bmm(qq, kk.transpose(1, 2).contiguous())
        i = torch.arange(L, device=DEV)
        buk = None
        if pos is not None:
            # pos[h, j - i + N - 1] as a sliding window over the reversed rows
            w = pos[:, N - L:N + L - 1].unfold(1, L, 1)          # [H, L, L], row x: i = L-1-x
            s += w.flip(1)
        if tim is not None:
            buk = _bucket64(x["ts"][a:b, None] - x["ts"][None, a:b], case["nb"])
            s += tim[:, buk]
        return s, i[None, :] <= i[:, None], buk

    for n in range(case["B"]):
        a, b = int(off[n]), int(off[n + 1])
        if b == a:
            continue
        s, mask, _ = scores(a, b)
        p = (s * torch.sigmoid(s) / N).masked_fill_(~mask, 0.0)
        del s
        o[a:b] = torch.bmm(p, v[a:b].permute(1, 0, 2).contiguous()).permute(1, 0, 2)
    of = o.reshape(T, H * d)
    mean = of.mean(1)
    rstd = (of.var(1, unbiased=False) + LN_EPS).rsqrt()
    nrm = (of - mean[:, None]) * rstd[:, None]
    uf = u.reshape(T, H * d)
    f = dict(y=nrm * uf, o=o, mean=mean, rstd=rstd)
    if dy is None:
        return f, None
    gy = dy * uf
    dO = rstd[:, None] * (gy - gy.mean(1, keepdim=True) - nrm * (gy * nrm).mean(1, keepdim=True))
    dO = dO.reshape(T, H, d)
    g = dict(du=nrm * dy)
    dq, dk, dv = (torch.zeros(T, H, d, **f8) for _ in range(3))
    d_pos = torch.zeros(H, 2 * N - 1, **f8) if pos is not None else None
    d_time = torch.zeros(H, case["nb"], **f8) if tim is not None else None
    for n in range(case["B"]):
        a, b = int(off[n]), int(off[n + 1])
        if b == a:
            continue
        L = b - a
        qq, kk, vv, oo = (t[a:b].permute(1, 0, 2).contiguous() for t in (q, k, v, dO))
        s, mask, buk = scores(a, b)
        sg = torch.sigmoid(s)
        p = (s * sg / N).masked_fill_(~mask, 0.0)
        dv[a:b] = torch.bmm(p.transpose(1, 2).contiguous(), oo).permute(1, 0, 2)
        del p
        ds = torch.bmm(oo, vv.transpose(1, 2).contiguous())
        ds *= (sg * (1 + s * (1 - sg)) / N).masked_fill_(~mask, 0.0)
        del s, sg
        dq[a:b] = alpha * torch.bmm(ds, kk).permute(1, 0, 2)
        dk[a:b] = alpha * torch.bmm(ds.transpose(1, 2).contiguous(), qq).permute(1, 0, 2)
        if d_pos is not None:
            # diagonals: rows of L + 1 of the shifted flat array line up m = i - j
            z = torch.cat([torch.zeros(H, L, **f8), ds.reshape(H, L * L)], 1)
            z = z.view(H, L, L + 1).sum(1)                        # column L - m
            d_pos[:, N - L:N] += z[:, 1:]
        if d_time is not None:
            d_time += _rows_scatter(buk, ds, case["nb"])
        del ds
    g.update(dq=dq, dk=dk, dv=dv)
    if d_pos is not None:
        g["d_pos"] = d_pos
    if d_time is not None:
        g["d_time"] = d_time
    return f, g


def _exact_attn(case, seed):
    x = _inputs(case, seed)
    q, k, v, u = (x[n].double() for n in "qkvu")
    dy = x["dy"].double() if case["bwd"] else None
    f, g = _attn64(case, x, q, k, v, u, dy, case["alpha"])
    if g is not None:
        g["du"] = g["du"].reshape(q.shape[0], -1)
        f.update(g)
    return f


def _exact_layer(case, seed):
    x = _inputs(case, seed)
    H, d = case["H"], case["d"]
    C = H * d
    xx, w1, w2 = x["x"].double(), x["w1"].double(), x["w2"].double()
    T = xx.shape[0]
    h = xx @ w1
    sg = torch.sigmoid(h)
    z = h * sg
    u, v, q, k = (z[:, n * C:(n + 1) * C].reshape(T, H, d) for n in range(4))
    dout = x["dout"].double() if case["bwd"] else None
    dy = dout @ w2.t().contiguous() if case["bwd"] else None
    f, g = _attn64(case, x, q, k, v, u, dy, 1.0)
    out = dict(f, out=f["y"] @ w2, h=h, z=torch.stack([u, v, q, k]))
    if case["bwd"]:
        dz = torch.cat([g[n].reshape(T, C) for n in ("du", "dv", "dq", "dk")], 1)
        dh = dz * sg * (1 + h * (1 - sg))
        out.update(dx=dh @ w1.t().contiguous(), dw1=xx.t().contiguous() @ dh,
                   dw2=f["y"].t().contiguous() @ dout)
        out.update({n: g[n] for n in ("d_pos", "d_time") if n in g})
    return out


def _exact_emb(case, seed):
    x = _inputs(case, seed)
    F, T, D = case["tables"], case["T"], case["D"]
    rows = x["ids"] + x["ro"][:-1].repeat_interleave(T)

    def place(t):                                     # flat [F T, D] -> the case's layout
        return t if case["layout"] == "flat" else \
            t.reshape(F, T, D).permute(1, 0, 2).reshape(T, F * D)

    out = dict(out=place(x["weights"][rows].double()))
    if case["bwd"]:
        dout = x["dout"].double()
        if case["layout"] == "token":
            dout = dout.reshape(T, F, D).permute(1, 0, 2).reshape(F * T, D)
        uniq, inv = torch.unique(rows, return_inverse=True)
        sums = torch.zeros(len(uniq), D, dtype=torch.float64, device=DEV)
        sums.index_add_(0, inv, dout)
        grad = torch.zeros(x["total_rows"], D, dtype=torch.float64, device=DEV)
        grad[uniq] = sums
        ids = torch.full((F * T,), -1, dtype=torch.int64, device=DEV)
        ids[:len(uniq)] = uniq
        out.update(grad=grad, rows=ids,
                   count=torch.tensor([len(uniq)], dtype=torch.int32, device=DEV))
    return out


def _exact_rab(case, seed):
    x = _inputs(case, seed)
    H, N, off = case["H"], case["N"], x["off_np"]
    f8 = dict(dtype=torch.float64, device=DEV)
    rab = torch.zeros(H, x["square"], **f8)
    d_pos = torch.zeros(H, 2 * N - 1, **f8)
    d_time = torch.zeros(H, case["nb"], **f8)
    d_fn = torch.zeros(H, 2, **f8)
    at = 0
    for n in range(case["B"]):
        a, b = int(off[n]), int(off[n + 1])
        L = b - a
        blk = torch.zeros(H, L, L, **f8)
        dr = x["d_rab"][:, at:at + L * L].double().reshape(H, L, L) if case["bwd"] else None
        i = torch.arange(L, device=DEV)
        if case["pos"]:
            idx = i[None, :] - i[:, None] + N - 1
            blk += x["pos"].double()[:, idx]
            if dr is not None:
                # rows of 2L - 1 read as rows of 2L: entry (i, j) in column j - i + L - 1
                z = torch.cat([dr, torch.zeros(H, L, L - 1, **f8)], 2).reshape(H, -1)
                z = torch.cat([torch.zeros(H, L - 1, **f8), z, torch.zeros(H, 1, **f8)], 1)
                d_pos[:, N - L:N + L - 1] += z.reshape(H, L, 2 * L).sum(1)[:, :-1]
        dt = x["ts"][a:b, None] - x["ts"][None, a:b] if x["ts"] is not None else None
        if case["time"]:
            buk = _bucket64(dt, case["nb"])
            blk += x["time"].double()[:, buk]
            if dr is not None:
                d_time += _rows_scatter(buk, dr, case["nb"])
        if case["fn"]:
            amp, beta = (x["fn"].double()[:, c, None, None] for c in (0, 1))
            lg = torch.log1p(dt.abs().double())[None]
            e = torch.exp(-beta * lg)
            blk += amp * e
            if dr is not None:
                d_fn[:, 0] += (dr * e).sum((1, 2))
                d_fn[:, 1] += (dr * (-amp * e * lg)).sum((1, 2))
        rab[:, at:at + L * L] = blk.reshape(H, L * L)
        at += L * L
    out = dict(rab=rab)
    if case["bwd"]:
        out.update({n: t for n, t, on in (("d_pos", d_pos, case["pos"]),
                                          ("d_time", d_time, case["time"]),
                                          ("d_fn", d_fn, case["fn"])) if on})
    return out


def exact(case, seed):
    return {"attn": _exact_attn, "layer": _exact_layer, "emb": _exact_emb,
            "rab": _exact_rab}[case["kind"]](case, seed)
