"""Workloads that stand for what a user runs through the public entry points
(`paper_2512_09200_amd.api`): whole training steps and serving forwards, and
the single layers a program can call on their own -- pooled lookups with their
sparse gradient, the interactions, MLPs with objective heads, FP8 linear
layers -- from latency-bound calls to chip-filling ones, in both storage
types, forward and backward.

A case is a dict of plain values.  `listed()` names the fixed ones, `draw(rng)`
gives one more of the same ranges, `prepare(case, seed)` makes a call's inputs
on the GPU, `run(state)` is one pass, `work(case)` its compulsory bytes and
operations, `tolerance(case)` how far two correct evaluations may differ, and
`exact(case, seed)` the same outputs from plain torch in 64 bits.
"""
import math

import numpy as np
import torch

from paper_2512_09200_amd import api

DEV = "cuda"
BF16, F32 = torch.bfloat16, torch.float32
LR = 0.01           # row-sparse SGD step of the tables
LN_EPS = 1e-5


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------
def listed():
    return [
        # The smallest training step (fp32 tables and layers, DOT): every stage
        # is a launch or two, so it stands for latency-bound use.
        dict(name="step-tiny-f32", kind="step", dtype="f32", B=128, F=8, rows=4096, d=32, zipf=0.0,
             bag=4.5, bag_hi=8, dense=13, bottom="64,32", inter="dot", k=0, top="64,4"),
        # A mid-size DLRM-like training step in bf16.
        dict(name="step-mid-dot-bf16", kind="step", dtype="bf16", B=2048, F=26, rows=100_000, d=64,
             zipf=1.1, bag=10.0, bag_hi=64, dense=13, bottom="256,64", inter="dot", k=0, top="512,256,8"),
        # The large-embedding training step: 33 GB of tables, FM interaction.
        dict(name="step-large-fm-bf16", kind="step", dtype="bf16", B=8192, F=64, rows=2_000_000, d=128,
             zipf=1.05, bag=20.0, bag_hi=128, dense=64, bottom="512,128", inter="fm", k=32, top="1024,512,16"),
        # Serving: the forward alone on a request batch of that model.
        dict(name="forward-serve-fm-bf16", kind="forward", dtype="bf16", B=512, F=64, rows=500_000, d=128,
             zipf=1.05, bag=20.0, bag_hi=128, dense=64, bottom="512,128", inter="fm", k=32, top="1024,512,16"),
        # Multi-domain embedding traffic: most bags of a sample are empty
        # (forward, sparse gradient and SGD).
        dict(name="lookup-multidomain-bf16", kind="lookup", dtype="bf16", B=8192, F=96, rows=250_000, d=128,
             zipf=1.1, bag=15.0, bag_hi=128, active=40, pool="sum", sgd=True),
        # fp32 embeddings, mean pooling, row gradients handed to an optimizer.
        dict(name="lookup-mid-f32", kind="lookup", dtype="f32", B=2048, F=26, rows=100_000, d=64, zipf=1.1,
             bag=10.0, bag_hi=64, active=26, pool="mean", sgd=False),
        # The DOT interaction of the multi-domain model, forward and backward.
        dict(name="dot-multidomain-bf16", kind="inter", dtype="bf16", B=8192, n=97, d=128, inter="dot", k=0),
        # The FM interaction in fp32 (a quarter of the large model's batch).
        dict(name="fm-f32", kind="inter", dtype="f32", B=2048, n=65, d=128, inter="fm", k=32),
        # Two layers of the deep model's fusion blocks, forward and backward:
        # the largest products of the framework.
        dict(name="stack-deep-bf16", kind="stack", dtype="bf16", B=4096, n=256, nv=64, d=128, k=64, layers=2, lcb=0),
        # The multi-domain model's task MLP with heads and loss, forward and backward.
        dict(name="mlp-top-bf16", kind="mlp", dtype="bf16", B=8192, k_in=4784, widths="1024,512,32", act="relu"),
        # The mid model's task MLP in fp32.
        dict(name="mlp-mid-f32", kind="mlp", dtype="f32", B=2048, k_in=415, widths="512,256,8", act="relu"),
        # An FP8 linear layer as training runs it: activations and weights
        # quantised row-wise every call, accumulation in fp32.
        dict(name="fp8-linear", kind="fp8", dtype="bf16", M=8192, N=1024, K=2208, fast=False),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _model(rng, dtype, Bmax):
    d = rng.choice([32, 64, 128] if dtype == "f32" else [64, 128])
    inter = rng.choice(["dot", "fm"])
    F = _log(rng, 6, 80)
    k = rng.choice([16, 32]) if inter == "fm" else 0
    w0 = 64 * rng.randint(1, 16)
    return dict(dtype=dtype, B=_log(rng, 100, Bmax), F=F, rows=_log(rng, 3000, 800_000), d=d,
                zipf=rng.choice([0.0, 1.05, 1.1]), bag=float(rng.randint(3, 20)), bag_hi=64,
                dense=rng.choice([13, 40, 64]), bottom="%d,%d" % (32 * rng.randint(2, 16), d), inter=inter, k=k,
                top="%d,%d,%d" % (w0, max(32, w0 // 2), rng.randint(2, 32)))


def draw(rng):
    kind = rng.choice(["step", "forward", "lookup", "inter", "stack", "mlp", "fp8"])
    dtype = rng.choice(["bf16", "bf16", "f32"])
    if kind == "step":
        return dict(kind="step", **_model(rng, dtype, 512 if dtype == "f32" else 8192))
    if kind == "forward":
        return dict(kind="forward", **_model(rng, dtype, 512 if dtype == "f32" else 2048))
    if kind == "lookup":
        F, d = _log(rng, 4, 96), rng.choice([32, 64, 96, 128, 256])
        return dict(kind="lookup", dtype=dtype, B=_log(rng, 200, 8192), F=F,
                    rows=_log(rng, 2000, min(400_000, 2_000_000_000 // (F * d))), d=d, zipf=rng.choice([0.0, 1.05, 1.1]),
                    bag=float(rng.randint(3, 15)), bag_hi=128, active=max(1, int(F * rng.choice([0.4, 1.0, 1.0]))),
                    pool=rng.choice(["sum", "mean"]), sgd=rng.choice([True, False]))
    if kind == "inter":
        inter = rng.choice(["dot", "fm"])
        return dict(kind="inter", dtype=dtype, B=_log(rng, 64, 8192 if dtype == "bf16" else 4096),
                    n=rng.randint(9, 97), d=rng.choice([64, 128] if dtype == "bf16" else [32, 64, 128]),
                    inter=inter, k=rng.choice([16, 32]) if inter == "fm" else 0)
    if kind == "stack":
        nv = 2 * rng.randint(8, 32)
        return dict(kind="stack", dtype="bf16", B=_log(rng, 256, 4096), n=2 * rng.randint(16, 128), nv=nv,
                    d=rng.choice([64, 128]), k=rng.choice([32, 64]), layers=rng.randint(1, 2),
                    lcb=rng.choice([0, nv // 4]))
    if kind == "mlp":
        w0 = 64 * rng.randint(2, 16) if dtype == "bf16" else 32 * rng.randint(2, 16)
        return dict(kind="mlp", dtype=dtype, B=_log(rng, 100, 8192 if dtype == "bf16" else 2048),
                    k_in=rng.randint(60, 4800) if dtype == "bf16" else rng.randint(60, 1000),
                    widths="%d,%d,%d" % (w0, w0 // 2, rng.randint(2, 64)),
                    act=rng.choice(["relu", "relu", "swishrn", "hardswishrn"]) if dtype == "bf16" else "relu")
    return dict(kind="fp8", dtype="bf16", M=_log(rng, 256, 16384), N=64 * rng.randint(2, 32),
                K=16 * rng.randint(8, 300), fast=rng.choice([True, False]))


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _dt(case):
    return BF16 if case["dtype"] == "bf16" else F32


def _widths(text):
    return [int(w) for w in text.split(",")]


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 7919 + 17)
    return g


def _randn(g, shape, scale=1.0, dtype=F32):
    return (torch.randn(shape, generator=g, device=DEV, dtype=F32) * scale).to(dtype)


def _table(g, rows, d, dtype):
    """N(0, 0.01^2) table rows, drawn in pieces (the large tables are tens of GB)."""
    E = torch.empty((rows, d), dtype=dtype, device=DEV)
    step = max(1, (1 << 29) // d)
    for r in range(0, rows, step):
        E[r:r + step].normal_(0.0, 0.01, generator=g)
    return E


def _capacity(case):
    """Lookups that buffers are sized for, whatever the seed."""
    bags = case["B"] * case.get("active", case["F"])
    return int(1.05 * bags * case["bag"] + 6.0 * math.sqrt(bags) * case["bag"]) + 64


def _bags(case, g, seed):
    """Feature-major jagged batch on the GPU: offsets, indices, domain activity
    (a sample carries `active` of the features; the others' bags are empty)."""
    B, F, N = case["B"], case["F"], case["rows"]
    if case["zipf"] == 0.0:
        lens = torch.randint(1, max(2, int(2 * case["bag"])), (F, B), generator=g, device=DEV)
    else:
        lens = torch.poisson(torch.full((F, B), case["bag"], device=DEV), generator=g).long()
    lens = lens.clamp(1, case["bag_hi"])
    active = case.get("active", F)
    rng = np.random.default_rng([int(seed), 5])
    if active < F:
        on = np.zeros((4, F), dtype=np.int64)
        for q in range(4):
            on[q, rng.choice(F, size=active, replace=False)] = 1
        dom = torch.multinomial(torch.tensor([0.4, 0.3, 0.2, 0.1], device=DEV), B, replacement=True, generator=g)
        lens = lens * torch.from_numpy(on).to(DEV)[dom].t()
    offsets = torch.zeros(F * B + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(lens.reshape(-1), 0, out=offsets[1:])
    nnz = int(offsets[-1])
    feat = torch.repeat_interleave(torch.arange(F, device=DEV), lens.sum(1), output_size=nnz)
    u = torch.rand(nnz, generator=g, device=DEV, dtype=torch.float64)
    if case["zipf"] == 0.0:
        idx = (u * N).long().clamp_(max=N - 1)
    else:
        # bounded power law by inverse CDF; ranks scattered over each table's rows
        a = 1.0 - case["zipf"]
        rank = ((u * ((N + 1.0) ** a - 1.0) + 1.0) ** (1.0 / a)).long().clamp_(1, N) - 1
        A, C = [], []
        for _ in range(F):
            m = int(rng.integers(1, N))
            while math.gcd(m, N) != 1:
                m = int(rng.integers(1, N))
            A.append(m)
            C.append(int(rng.integers(0, N)))
        idx = (rank * torch.tensor(A, device=DEV)[feat] + torch.tensor(C, device=DEV)[feat]) % N
    return dict(offsets=offsets.to(torch.int32), indices=idx.to(torch.int32), nnz=nnz,
                row_base=torch.arange(F + 1, dtype=torch.int64, device=DEV) * N)


def _linears(g, dims, dtype, act="relu", B=0):
    out = []
    for i in range(len(dims) - 1):
        o, n = dims[i + 1], dims[i]
        L = dict(W=_randn(g, (o, n), math.sqrt(2.0 / (o + n)), dtype), b=_randn(g, (o,), 0.01),
                 dW=torch.zeros((o, n), device=DEV), db=torch.zeros(o, device=DEV))
        if act != "relu" and i < len(dims) - 2:
            L["gain"] = 1.0 + _randn(g, (2, o), 0.2)
            L["dgain"] = torch.zeros((2, o), device=DEV)
            L["pre"] = torch.zeros((B, o), dtype=dtype, device=DEV)
            L["rinv"] = torch.zeros((B, -(-o // 128)), device=DEV)
        out.append(L)
    return out


def _inter_width(inter, n, k):
    return n * (n - 1) // 2 if inter == "dot" else n * k


def _labels(g, B, T):
    labels = (torch.rand((B, T), generator=g, device=DEV) < 0.15).float()
    mask = (torch.rand((B, T), generator=g, device=DEV) < 0.5).to(torch.uint8)
    return labels, mask


def prepare(case, seed):
    g, dt = _gen(seed), _dt(case)
    s = dict(case=case)
    kind = case["kind"]
    if kind in ("step", "forward"):
        B, F, d = case["B"], case["F"], case["d"]
        n = F + 1
        bot, top = _widths(case["bottom"]), _widths(case["top"])
        s["table"] = _table(g, F * case["rows"], d, dt)
        s.update(_bags(case, g, seed))
        s["dense"] = _randn(g, (B, case["dense"]), 1.0, dt)
        s["labels"], s["mask"] = _labels(g, B, top[-1])
        s["bottom"] = _linears(g, [case["dense"]] + bot, dt)
        s["top"] = _linears(g, [d + _inter_width(case["inter"], n, case["k"])] + top, dt)
        s["fm_W"] = _randn(g, (n, case["k"]), 1.0 / math.sqrt(n), dt) if case["inter"] == "fm" else None
        s["fm_dW"] = torch.zeros((n, case["k"]), device=DEV) if case["inter"] == "fm" else None
        s["model"] = api.StepModel(tables=s["table"], row_base=s["row_base"], num_features=F, dense_in=case["dense"],
                                   bottom=s["bottom"], top=s["top"], interact=case["inter"], fm_W=s["fm_W"],
                                   fm_dW=s["fm_dW"], max_rows=case["rows"])
        s["cap"] = _capacity(case)
        lay = api.lattice_step_plan(s["model"], B, s["cap"], LR)
        s["ws"] = torch.zeros(lay.total_bytes, dtype=torch.uint8, device=DEV)
        s["views"] = api.step_views(s["model"], s["ws"], lay, B, top[-1], s["cap"])
        s["side"] = api.SideStream()
    elif kind == "lookup":
        B, F, d = case["B"], case["F"], case["d"]
        s["table"] = _table(g, F * case["rows"], d, dt)
        s.update(_bags(case, g, seed))
        s["X"] = torch.zeros((B, F, d), dtype=dt, device=DEV)
        s["dX"] = _randn(g, (B, F, d), 1.0 / B, dt)
        cap = _capacity(case)
        s["sparse"] = dict(unique_rows=torch.zeros(cap, dtype=torch.int32, device=DEV),
                           seg_offsets=torch.zeros(cap + 1, dtype=torch.int32, device=DEV),
                           sorted_bags=torch.zeros(cap, dtype=torch.int32, device=DEV),
                           num_unique=torch.zeros(1, dtype=torch.int32, device=DEV),
                           grad_rows=None if case["sgd"] else torch.zeros((cap, d), device=DEV))
    elif kind == "inter":
        B, n, d, k = case["B"], case["n"], case["d"], case["k"]
        w = d + _inter_width(case["inter"], n, k)
        s["X"] = _randn(g, (B, n, d), 0.3, dt)
        s["W"] = _randn(g, (n, k), 1.0 / math.sqrt(n), dt) if k else None
        s["dW"] = torch.zeros((n, k), device=DEV) if k else None
        s["out"] = torch.zeros((B, (w + 7) // 8 * 8), dtype=dt, device=DEV)
        s["d_out"] = _randn(g, (B, (w + 7) // 8 * 8), 0.1, dt)
        s["dX"] = torch.zeros((B, n, d), dtype=dt, device=DEV)
    elif kind == "stack":
        B, n, nv, d, k = case["B"], case["n"], case["nv"], case["d"], case["k"]
        s["X"] = _randn(g, (B, n, d), 0.3, dt)
        s["layers"] = []
        for l in range(case["layers"]):
            nl, nF = (n if l == 0 else nv), nv - case["lcb"]
            L = dict(W=_randn(g, (nl, k), 1.0 / math.sqrt(nl), dt),
                     A=_randn(g, (nF * d, nl * k), math.sqrt(2.0 / (nF * d + nl * k)), dt),
                     gamma=1.0 + _randn(g, (d,), 0.1),
                     C=_randn(g, (nv, nl), math.sqrt(2.0 / (nv + nl)), dt) if nl != nv else None)
            if case["lcb"]:
                L["L"] = _randn(g, (case["lcb"], nl), math.sqrt(2.0 / (case["lcb"] + nl)), dt)
            for name in ("W", "A", "gamma", "C", "L"):
                if L.get(name) is not None:
                    L["d" + name] = torch.zeros(L[name].shape, device=DEV)
            s["layers"].append(L)
        s["out"] = torch.zeros((B, nv * d), dtype=dt, device=DEV)
        s["d_out"] = _randn(g, (B, nv * d), 0.1, dt)
        s["dX"] = torch.zeros((B, n, d), dtype=dt, device=DEV)
    elif kind == "mlp":
        B, w = case["B"], _widths(case["widths"])
        kp = (case["k_in"] + 7) // 8 * 8       # rows padded as the step's top input is
        s["x"] = _randn(g, (B, kp), 1.0, dt)[:, :case["k_in"]]
        s["layers"] = _linears(g, [case["k_in"]] + w, dt, case["act"], B)
        s["acts"] = [torch.zeros((B, o), dtype=dt if i < len(w) - 1 else F32, device=DEV) for i, o in enumerate(w)]
        s["labels"], s["mask"] = _labels(g, B, w[-1])
        s["loss"] = dict(labels=s["labels"], mask=s["mask"], loss=torch.zeros(1, device=DEV),
                         d_logits=torch.zeros((B, w[-1]), device=DEV),
                         d_logits_op=torch.zeros((B, w[-1]), dtype=dt, device=DEV))
        s["d_in"] = torch.zeros((B, kp), dtype=dt, device=DEV)[:, :case["k_in"]]
    else:
        s["x"] = _randn(g, (case["M"], case["K"]), 1.0, dt)
        s["w"] = _randn(g, (case["N"], case["K"]), math.sqrt(2.0 / (case["N"] + case["K"])), dt)
        s["b"] = _randn(g, (case["N"],), 0.01)
    return s


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
def _grads(layers):
    return [{k: L[k] for k in ("dW", "db", "dgain") if k in L} for L in layers]


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "step":
        api.lattice_step(s["model"], s["offsets"], s["indices"], s["dense"], s["labels"], s["mask"], s["ws"], LR,
                         nnz_capacity=s["cap"], side=s["side"])
        v = s["views"]
        out = dict(loss=v["loss"], logits=v["logits"], bottom=_grads(s["bottom"]), top=_grads(s["top"]),
                   tables=s["table"], rows=v["unique_rows"], bags=v["sorted_bags"], count=v["num_unique"])
        if s["fm_dW"] is not None:
            out["fm_dW"] = s["fm_dW"]
        return out
    if kind == "forward":
        api.lattice_forward(s["model"], s["offsets"], s["indices"], s["dense"], case["B"], s["ws"],
                            nnz_capacity=s["cap"], side=s["side"])
        return dict(logits=s["views"]["logits"])
    if kind == "lookup":
        F, B = case["F"], case["B"]
        api.lattice_embbag_fwd(s["table"], s["row_base"], s["offsets"], s["indices"], F, B, s["X"], pool=case["pool"])
        r = s["sparse"]
        api.lattice_embbag_bwd_noalloc(s["table"], s["row_base"], s["offsets"], s["indices"], F, B, s["dX"], r,
                                       lr=LR if case["sgd"] else 0.0, pool=case["pool"], max_rows=case["rows"])
        out = dict(X=s["X"], rows=r["unique_rows"], starts=r["seg_offsets"], bags=r["sorted_bags"],
                   count=r["num_unique"])
        out["table" if case["sgd"] else "grad"] = s["table"] if case["sgd"] else r["grad_rows"]
        return out
    if kind == "inter":
        ws = api.lattice_interact_fwd(case["inter"], s["X"], s["out"], True, fm_W=s["W"])
        api.lattice_interact_bwd(case["inter"], s["X"], s["d_out"], s["dX"], True, fm_W=s["W"], fm_dW=s["dW"],
                                 ws=ws if s["W"] is not None else None)
        w = case["d"] + _inter_width(case["inter"], case["n"], case["k"])
        out = dict(out=s["out"][:, :w], dX=s["dX"])
        if s["dW"] is not None:
            out["dW"] = s["dW"]
        return out
    if kind == "stack":
        ws = api.lattice_interact_fwd("stack", s["X"], s["out"], stack=s["layers"], stack_n=case["nv"], ln_eps=LN_EPS)
        api.lattice_interact_bwd("stack", s["X"], s["d_out"], s["dX"], stack=s["layers"], stack_n=case["nv"],
                                 ln_eps=LN_EPS, ws=ws)
        return dict(out=s["out"], dX=s["dX"],
                    grads=[{k: L[k] for k in ("dW", "dA", "dC", "dgamma", "dL") if k in L} for L in s["layers"]])
    if kind == "mlp":
        act = case["act"]
        api.lattice_mlp_heads_fwd(s["layers"], s["x"], s["acts"], False, loss=s["loss"], act=act)
        api.lattice_mlp_heads_bwd(s["layers"], s["x"], s["acts"], s["loss"]["d_logits_op"], False, d_in=s["d_in"],
                                  act=act)
        return dict(loss=s["loss"]["loss"], logits=s["acts"][-1], d_in=s["d_in"], grads=_grads(s["layers"]))
    qa, sa = api.lattice_fp8_quantize(s["x"])
    qw, sw = api.lattice_fp8_quantize(s["w"])
    y = api.lattice_linear_fp8_fwd(qa, sa, qw, sw, case["K"], bias=s["b"], relu=True, fast_accum=case["fast"])
    return dict(y=y, codes=qa, scales=sa, w_codes=qw, w_scales=sw)


# ---------------------------------------------------------------------------
# compulsory work
# ---------------------------------------------------------------------------
def _distinct(case):
    """Expected (lookups, distinct rows) of a batch."""
    bags = case["B"] * case.get("active", case["F"])
    nnz = bags * case["bag"]
    N, m = case["rows"], case["bag"] * bags / case["F"]
    if case["zipf"] == 0.0:
        p = np.full(1, 1.0 / N)
        return nnz, case["F"] * N * float(-np.expm1(m * np.log1p(-p[0])))
    a = 1.0 - case["zipf"]
    edge = np.arange(1, N + 2, dtype=np.float64) ** a
    p = np.diff(edge) / ((N + 1.0) ** a - 1.0)
    return nnz, case["F"] * float(-np.expm1(m * np.log1p(-np.minimum(p, 1 - 1e-12))).sum())


def _mlp_work(dims, B, es, backward, need_dx0):
    macs = [dims[i] * dims[i + 1] for i in range(len(dims) - 1)]
    w = sum(macs)
    if not backward:
        return w * es, 2.0 * B * w
    return w * (es + 4), 2.0 * B * (3 * w - (0 if need_dx0 else macs[0]))


def _inter_flops(inter, B, n, d, k):
    """(forward, backward)"""
    if inter == "dot":
        p = n * (n - 1) // 2
        return 2.0 * B * p * d, 4.0 * B * p * d
    return 4.0 * B * n * d * k, 8.0 * B * n * d * k


def work(case):
    kind = case["kind"]
    es = 2 if case["dtype"] == "bf16" else 4
    if kind in ("step", "forward"):
        B, F, d, n = case["B"], case["F"], case["d"], case["F"] + 1
        nnz, rows = _distinct(case)
        step = kind == "step"
        bot, top = _widths(case["bottom"]), _widths(case["top"])
        b1, f1 = _mlp_work([case["dense"]] + bot, B, es, step, False)
        b2, f2 = _mlp_work([d + _inter_width(case["inter"], n, case["k"])] + top, B, es, step, True)
        fi, bi = _inter_flops(case["inter"], B, n, d, case["k"])
        nbytes = rows * d * es * (2 if step else 1) + nnz * 4 + F * B * 4 + B * case["dense"] * es + b1 + b2 + B * top[-1] * 4
        if step:
            nbytes += nnz * 4 + rows * 4 + B * top[-1] * 5
        return dict(bytes=nbytes, flops=f1 + f2 + fi + (bi if step else 0.0) + nnz * d * (2 if step else 1))
    if kind == "lookup":
        B, F, d = case["B"], case["F"], case["d"]
        nnz, rows = _distinct(case)
        nbytes = nnz * 8 + F * B * 4 + rows * (d * es + 8) + 2 * B * F * d * es + rows * d * (es if case["sgd"] else 4)
        return dict(bytes=nbytes, flops=2.0 * nnz * d)
    if kind == "inter":
        B, n, d, k = case["B"], case["n"], case["d"], case["k"]
        f, b = _inter_flops(case["inter"], B, n, d, k)
        return dict(bytes=2 * B * (n * d + d + _inter_width(case["inter"], n, k)) * es + n * k * (es + 4), flops=f + b)
    if kind == "stack":
        B, d, k, nv, lcb = case["B"], case["d"], case["k"], case["nv"], case["lcb"]
        nbytes, flops = 2.0 * B * (case["n"] + nv) * d * es, 0.0
        for l in range(case["layers"]):
            n = case["n"] if l == 0 else nv
            A = (nv - lcb) * d * n * k
            nbytes += (A + n * k + lcb * n) * (es + 4)
            flops += 6.0 * B * (A + lcb * n * d) + 12.0 * B * n * d * k
            if n != nv:
                nbytes += nv * n * (es + 4)
                flops += 6.0 * B * nv * n * d
        return dict(bytes=nbytes, flops=flops)
    if kind == "mlp":
        B, w = case["B"], _widths(case["widths"])
        b, f = _mlp_work([case["k_in"]] + w, B, es, True, True)
        return dict(bytes=b + 2 * B * case["k_in"] * es + B * w[-1] * 9, flops=f)
    M, N, K = case["M"], case["N"], case["K"]
    return dict(bytes=(M + N) * K * 3 + M * N * 2, flops=2.0 * M * N * K)


def tolerance(case):
    kind, f32 = case["kind"], case["dtype"] == "f32"
    if kind in ("step", "mlp") and f32:
        # fp32 sums give about 1e-6; a ReLU whose pre-activation is within that
        # of zero may go either way, which moves one unit's gradient
        return {"rel": 2e-3, "max": 0.2}
    if f32:
        return {"rel": 1e-5}
    if kind == "lookup":
        # bf16 results of fp32 sums: a last-bit rounding of few elements
        return {"rel": 1e-3, "max": 0.02}
    if kind == "inter":
        return {"rel": 2e-3, "max": 0.05}
    return {"rel": 1e-2}


# ---------------------------------------------------------------------------
# the same in 64 bits, plain torch
# ---------------------------------------------------------------------------
def _f64(t):
    return t.detach().double().requires_grad_(True)


def _pool64(case, s):
    """Pooled rows [B, F, d] and each lookup's weight, bag and global row."""
    B, F = case["B"], case["F"]
    off = s["offsets"].long()
    lens = off[1:] - off[:-1]
    bag = torch.repeat_interleave(torch.arange(F * B, device=DEV), lens, output_size=s["nnz"])
    row = s["row_base"][bag // B] + s["indices"].long()
    wt = 1.0 / lens[bag].double() if case.get("pool") == "mean" else None
    X = torch.zeros((F * B, case["d"]), dtype=torch.float64, device=DEV)
    for i in range(0, s["nnz"], 1 << 23):
        e = s["table"][row[i:i + (1 << 23)]].double()
        X.index_add_(0, bag[i:i + (1 << 23)], e if wt is None else e * wt[i:i + (1 << 23), None])
    return X.view(F, B, -1).transpose(0, 1).contiguous(), wt, bag, row


def _inter64(inter, X, W, emit0=True):
    B, n, _ = X.shape
    if inter == "dot":
        G = X @ X.transpose(1, 2).contiguous()
        i, j = torch.triu_indices(n, n, 1, device=DEV)
        o = G[:, i, j]
    else:
        o = (X @ (X.transpose(1, 2).contiguous() @ W)).reshape(B, -1)
    return torch.cat([X[:, 0], o], 1) if emit0 else o


def _swish64(h, gain, hard):
    n = torch.cat([c * torch.rsqrt(c.square().mean(1, keepdim=True) + 1e-6) for c in h.split(128, 1)], 1)
    z = gain[1] * n
    return gain[0] * n * (torch.clamp(z / 6 + 0.5, 0, 1) if hard else torch.sigmoid(z))


def _mlp64(P, x, relu_last, act="relu"):
    for i, L in enumerate(P):
        x = x @ L["W"].t() + L["b"]
        if relu_last or i < len(P) - 1:
            x = torch.relu(x) if act == "relu" else _swish64(x, L["gain"], act == "hardswishrn")
    return x


def _params64(layers):
    return [{k: _f64(L[k]) for k in ("W", "b", "gain") if k in L} for L in layers]


def _pgrads(P):
    return [{"d" + k if k != "gain" else "dgain": v.grad for k, v in L.items()} for L in P]


def _loss64(z, labels, mask):
    m = mask.double()
    y = labels.double()
    return (m * (z.clamp(min=0) - z * y + torch.log1p(torch.exp(-z.abs())))).sum() / m.sum().clamp(min=1)


def exact(case, seed):
    s = prepare(case, seed)
    kind = case["kind"]
    if kind in ("step", "forward"):
        X, _, _, _ = _pool64(case, s)
        bot, top = _params64(s["bottom"]), _params64(s["top"])
        W = _f64(s["fm_W"]) if s["fm_W"] is not None else None
        h = _mlp64(bot, s["dense"].double(), True)
        z = _mlp64(top, _inter64(case["inter"], torch.cat([h[:, None], X], 1), W), False)
        if kind == "forward":
            return dict(logits=z.detach())
        loss = _loss64(z, s["labels"], s["mask"])
        loss.backward()
        out = dict(loss=loss.detach().reshape(1), logits=z.detach(), bottom=_pgrads(bot), top=_pgrads(top),
                   tables=None, rows=None, bags=None, count=None)
        if W is not None:
            out["fm_dW"] = W.grad
        return out
    if kind == "lookup":
        X, wt, bag, row = _pool64(case, s)
        rows, inv = torch.unique(row, return_inverse=True)
        G = torch.zeros((rows.numel(), case["d"]), dtype=torch.float64, device=DEV)
        dX = s["dX"].transpose(0, 1).reshape(-1, case["d"])
        for i in range(0, s["nnz"], 1 << 23):
            e = dX[bag[i:i + (1 << 23)]].double()
            G.index_add_(0, inv[i:i + (1 << 23)], e if wt is None else e * wt[i:i + (1 << 23), None])
        out = dict(X=X, rows=None, starts=None, bags=None, count=None)
        if not case["sgd"]:
            full = torch.zeros((_capacity(case), case["d"]), dtype=torch.float64, device=DEV)
            full[:rows.numel()] = G
            return dict(out, grad=full)
        E = s["table"].double()
        E[rows] -= LR * G
        return dict(out, table=E)
    if kind == "inter":
        X = _f64(s["X"])
        W = _f64(s["W"]) if s["W"] is not None else None
        o = _inter64(case["inter"], X, W)
        o.backward(s["d_out"][:, :o.shape[1]].double())
        out = dict(out=o.detach(), dX=X.grad)
        if W is not None:
            out["dW"] = W.grad
        return out
    if kind == "stack":
        X = _f64(s["X"])
        P = [{k: _f64(L[k]) for k in ("W", "A", "C", "gamma", "L") if L.get(k) is not None} for L in s["layers"]]
        x = X
        for L in P:
            B, n, d = x.shape
            Fm = x @ (x.transpose(1, 2).contiguous() @ L["W"])
            H = (Fm.reshape(B, -1) @ L["A"].t()).view(B, -1, d)
            if "L" in L:
                H = torch.cat([H, L["L"] @ x], 1)
            u = H + (L["C"] @ x if "C" in L else x)
            u = u - u.mean(2, keepdim=True)
            x = L["gamma"] * u * torch.rsqrt(u.square().mean(2, keepdim=True) + LN_EPS)
        o = x.reshape(x.shape[0], -1)
        o.backward(s["d_out"].double())
        return dict(out=o.detach(), dX=X.grad, grads=[{"d" + k: v.grad for k, v in L.items()} for L in P])
    if kind == "mlp":
        P = _params64(s["layers"])
        x = _f64(s["x"])
        z = _mlp64(P, x, False, case["act"])
        loss = _loss64(z, s["labels"], s["mask"])
        loss.backward()
        return dict(loss=loss.detach().reshape(1), logits=z.detach(), d_in=x.grad, grads=_pgrads(P))
    x, w = s["x"].double(), s["w"].double()
    return dict(y=torch.relu(x @ w.t() + s["b"].double()), codes=None, scales=x.abs().amax(1) / 448,
                w_codes=None, w_scales=w.abs().amax(1) / 448)
