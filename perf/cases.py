"""The work a user of the attribution library has it do, as timed cases.

Each case is one pass through the public entry points of
``paper_2606_11660_amd``, on inputs with the shapes and distributions of the
repository's workloads (``synth``, ``bench.py``): GPT-2-shaped and 1B-shaped
token rows for the projection, low-rank-plus-noise rows for the second
moments and the preconditioner, unit rows with planted near-duplicates for
the store scan.  A case is a dict with a ``kind``:

project     attr_project of a batch (one example: a query; many: the store
            build), or attr_project_tokens (per-token attribution)
step        one step of the on-the-fly store build: project, unit-normalise
            into the fp16 store slot, merge into the running top-k
tiny        project and unit-normalise a small store and its queries, score
diag        the diagonal preconditioner over a store: accumulate, finalize,
            apply with unit norm
accumulate  the full second moment of a store
kfac        the K-FAC factors of one layer over a batch's token rows
apply       the full preconditioner on store rows or on a handful of queries
score       exact top-k of queries against a store
"""
import math
import random

import torch

import paper_2606_11660_amd as P
from paper_2606_11660_amd import finalize

F32, F16, BF16 = torch.float32, torch.float16, torch.bfloat16
DT = {"f32": F32, "f16": F16, "bf16": BF16}
BYTES = {"f32": 4, "f16": 2, "bf16": 2}
N_QUERIES, TOPK = 64, 10    # the resident queries of the on-the-fly step

# d_in, d_out and the input rows a module shares (same tag in one layer: same rows)
GPT2_LAYER = ((768, 2304, "x"), (768, 768, "o"), (768, 3072, "m"), (3072, 768, "d"))
LLAMA1B_LAYER = ((2048, 2048, "x"), (2048, 2048, "x"), (2048, 2048, "x"), (2048, 2048, "o"),
                 (2048, 8192, "m"), (2048, 8192, "m"), (8192, 2048, "d"))
LAYERS = {"gpt2": GPT2_LAYER, "llama1b": LLAMA1B_LAYER}


# ----------------------------------------------------------------------------
# the cases
# ----------------------------------------------------------------------------
def listed():
    return [
        # the smallest calls: a 256-example toy store and 8 queries, all the way to the top-5
        {"name": "tiny", "kind": "tiny", "n": 256, "T": 32, "d": 64, "nq": 8, "topk": 5},
        # one query's gradient through all of GPT-2's modules: interactive attribution
        {"name": "project_query", "kind": "project", "shape": "gpt2", "layers": 12, "n": 1, "T": 389,
         "ragged": False, "dtype": "bf16", "k": 16, "norm": False, "tokens": False},
        # a store batch of a model trained in 32 bits, with the wider projection
        {"name": "project_f32", "kind": "project", "shape": "gpt2", "layers": 12, "n": 16, "T": 512,
         "ragged": True, "dtype": "f32", "k": 32, "norm": False, "tokens": False},
        # the store build with on-the-fly scoring, 1B-shaped, ragged packed batch
        {"name": "step_1b", "kind": "step", "shape": "llama1b", "layers": 16, "n": 16, "T": 2048,
         "ragged": True, "dtype": "bf16", "k": 16, "norm": False},
        # per-token attribution of a small batch
        {"name": "project_tokens", "kind": "project", "shape": "gpt2", "layers": 12, "n": 16, "T": 512,
         "ragged": True, "dtype": "bf16", "k": 16, "norm": False, "tokens": True},
        # K-FAC factors of one 1B-shaped layer over a batch's valid tokens
        {"name": "kfac_layer", "kind": "kfac", "width": 2048, "mlp": 8192, "n": 21900},
        # the second moment of the whole 10^6-row store
        {"name": "accumulate_full", "kind": "accumulate", "n": 1000000, "D": 8192, "dtype": "f16"},
        # the preconditioner on a session's queries
        {"name": "apply_queries", "kind": "apply", "n": 256, "D": 8192, "out": "f16"},
        # the preconditioner on a slab of store rows
        {"name": "apply_store", "kind": "apply", "n": 131072, "D": 8192, "out": "f16"},
        # the diagonal preconditioner over a GPT-2 store
        {"name": "diag_store", "kind": "diag", "n": 200000, "D": 12288, "dtype": "f16"},
        # a few queries against a large store: bound by reading it
        {"name": "score_few", "kind": "score", "nq": 16, "n": 1000000, "D": 8192, "k": 100,
         "dtype": "f16", "merge": False},
        # a query set against a large store: bound by the products
        {"name": "score_many", "kind": "score", "nq": 1024, "n": 500000, "D": 8192, "k": 100,
         "dtype": "f16", "merge": False},
    ]


def _log(rng, lo, hi, step=1):
    """lo..hi, even over the logarithm, a multiple of step."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(lo, min(hi, int(round(v / step)) * step))


def draw(rng):
    kind = rng.choice(["project", "project", "tokens", "step", "tiny", "diag", "accumulate", "kfac",
                       "apply", "apply", "score", "score", "score"])
    if kind == "tiny":
        return {"kind": kind, "n": _log(rng, 33, 1500), "T": rng.randint(8, 96),
                "d": 32 * rng.randint(2, 12), "nq": rng.randint(1, 16), "topk": rng.randint(1, 10)}
    if kind in ("project", "tokens", "step"):
        shape = rng.choice(["gpt2", "gpt2", "llama1b"])
        layers = rng.randint(2, 12 if shape == "gpt2" else 6)
        T = _log(rng, 33, 2048)
        most = 16000 if shape == "gpt2" else 12000  # tokens of a batch
        n = _log(rng, 1, max(1, min(64, (most if kind != "tokens" else most // 2) // T)))
        case = {"kind": "step" if kind == "step" else "project", "shape": shape, "layers": layers,
                "n": n, "T": T, "ragged": rng.random() < 0.6,
                "dtype": rng.choice(["bf16", "bf16", "f32"]), "k": rng.choice([16, 16, 32, 64]),
                "norm": rng.random() < 0.25}
        if kind == "tokens":
            case["k"] = rng.choice([16, 16, 32])
            if case["k"] == 32:
                case["layers"] = min(layers, 4)
        if kind != "step":
            case["tokens"] = kind == "tokens"
        return case
    if kind == "diag":
        D = 8 * _log(rng, 128, 3584)
        dtype = rng.choice(["f16", "f16", "f32"])
        return {"kind": kind, "n": _log(rng, 1000, int(2.4e9 / D / (BYTES[dtype] // 2))), "D": D, "dtype": dtype}
    if kind == "accumulate":
        D = 64 * _log(rng, 8, 192)
        return {"kind": kind, "n": _log(rng, 2000, min(600000, int(4e13 / D / D))), "D": D,
                "dtype": rng.choice(["f16", "bf16"])}
    if kind == "kfac":
        w = 64 * rng.randint(12, 40)
        return {"kind": kind, "width": w, "mlp": w * rng.choice([3, 4]), "n": _log(rng, 1000, 30000)}
    if kind == "apply":
        D = 64 * _log(rng, 16, 160)
        n = _log(rng, 1, 1024) if rng.random() < 0.5 else _log(rng, 1024, int(1.2e13 / D / D))
        return {"kind": kind, "n": n, "D": D, "out": rng.choice(["f16", "f16", "f32"])}
    # score: one query to a few hundred, a new batch of rows to a large store
    dtype = rng.choice(["f16", "f16", "f16", "f32"])
    D = 64 * _log(rng, 16, 448)
    nq = _log(rng, 1, 1024)
    most = min(int((6e9 if dtype == "f16" else 2e9) / D),
               int((1e13 if dtype == "f16" else 6e11) / D / nq))
    return {"kind": "score", "nq": nq, "n": _log(rng, 100, max(200, most)), "D": D,
            "k": rng.choice([5, 10, 100]), "dtype": dtype, "merge": rng.random() < 0.3}


# ----------------------------------------------------------------------------
# inputs
# ----------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _randn(gen, *shape, dtype=F32):
    return torch.randn(shape, generator=gen, device="cuda", dtype=dtype)


def _lengths(case):
    """Token counts of a batch's examples: part of the case, the same for every seed."""
    n, T = case["n"], case["T"]
    if not case["ragged"]:
        return [T] * n
    r = random.Random("%d %d" % (n, T))
    return [r.randint(max(1, T // 8), T) for _ in range(n)]


def _student_t4(gen, rows, d, dtype):
    z = _randn(gen, rows, d)
    u = torch.rand((rows, d), generator=gen, device="cuda").clamp_(min=1e-7).log_()
    u += torch.rand((rows, d), generator=gen, device="cuda").clamp_(min=1e-7).log_()
    return (z / u.mul_(-0.5).sqrt_()).to(dtype)


def _modules(case, gen, rows):
    dtype, k, mods = DT[case["dtype"]], case["k"], []
    heavy = case["shape"] == "llama1b"
    for _ in range(case["layers"]):
        seen = {}
        for d_in, d_out, tag in LAYERS[case["shape"]]:
            if tag not in seen:
                seen[tag] = _student_t4(gen, rows, d_in, dtype) if heavy else _randn(gen, rows, d_in, dtype=dtype)
            g = _randn(gen, rows, d_out, dtype=dtype).mul_(1e-2)
            R = (_randn(gen, d_out, k) / k ** 0.5).to(dtype)
            S = (_randn(gen, d_in, k) / k ** 0.5).to(dtype)
            vo = vi = None
            if case["norm"]:
                vo = torch.rand(d_out, generator=gen, device="cuda") + 0.5
                vi = torch.rand(d_in, generator=gen, device="cuda") + 0.5
            mods.append(P.Module(seen[tag], g, R, S, len(mods) * k * k, v_out=vo, v_in=vi))
    return mods


def _batch(case, seed):
    """A packed batch: modules, offsets, lengths, the output rows."""
    gen, lens = _gen(seed), _lengths(case)
    rows = sum(lens)
    mods = _modules(case, gen, rows)
    D = len(mods) * case["k"] ** 2
    offs = [0]
    for x in lens[:-1]:
        offs.append(offs[-1] + x)
    st = {"case": case, "mods": mods, "gen": gen, "D": D, "rows": rows,
          "offs": torch.tensor(offs, dtype=torch.int64, device="cuda") if case["ragged"] else None,
          "lens": torch.tensor(lens, dtype=torch.int32, device="cuda") if case["ragged"] else None}
    n_out = rows if case.get("tokens") else case["n"]
    st["out"] = torch.zeros((n_out, D), dtype=F32, device="cuda")
    return st


def _unit(x):
    return x / x.norm(dim=1, keepdim=True)


def _unit_rows(gen, n, D, dtype):
    out = torch.empty((n, D), dtype=dtype, device="cuda")
    for i in range(0, n, 65536):
        m = min(65536, n - i)
        out[i:i + m] = _unit(_randn(gen, m, D)).to(dtype)
    return out


def _factor(seed, D):
    g = torch.Generator()
    g.manual_seed(seed)
    return torch.randn((D, 64), generator=g, dtype=torch.float64)


def _lowrank_rows(gen, F, n, dtype):
    D, Ft = F.shape[0], F.float().cuda().T.contiguous()
    out = torch.empty((n, D), dtype=dtype, device="cuda")
    for i in range(0, n, 65536):
        m = min(65536, n - i)
        out[i:i + m] = torch.addmm(_randn(gen, m, D), _randn(gen, m, 64), Ft, beta=0.1).to(dtype)
    return out


def _running(gen, nq, k, D, seen):
    """The sorted top-k of `seen` earlier rows."""
    s, i = torch.topk(_randn(gen, nq, seen) * D ** -0.5, k, dim=1)
    return s.contiguous(), i.contiguous()


def prepare(case, seed):
    kind = case["kind"]
    if kind == "project":
        st = _batch(case, seed)
    elif kind == "step":
        st = _batch(case, seed)
        st["Q"] = _unit_rows(st["gen"], N_QUERIES, st["D"], F16)
        st["store"] = torch.zeros((case["n"], st["D"]), dtype=F16, device="cuda")
        st["base"] = 4096
        st["ts"], st["ti"] = _running(st["gen"], N_QUERIES, TOPK, st["D"], st["base"])
    elif kind == "tiny":
        gen, d, T = _gen(seed), case["d"], case["T"]
        R, S = _randn(gen, d, 16) / 4, _randn(gen, d, 16) / 4
        st = {"case": case}
        for tag, n in (("g", case["n"]), ("q", case["nq"])):
            mod = P.Module(_randn(gen, n * T, d), _randn(gen, n * T, d), R, S, 0)
            st[tag] = (mod, n, torch.empty((n, 256), dtype=F32, device="cuda"),
                       torch.empty((n, 256), dtype=F32, device="cuda"))
        st["ts"] = torch.empty((case["nq"], case["topk"]), dtype=F32, device="cuda")
        st["ti"] = torch.empty((case["nq"], case["topk"]), dtype=torch.int64, device="cuda")
    elif kind == "diag":
        st = {"case": case, "X": _lowrank_rows(_gen(seed), _factor(seed, case["D"]), case["n"], DT[case["dtype"]])}
        st["Y"] = torch.empty((case["n"], case["D"]), dtype=F16, device="cuda")
    elif kind == "accumulate":
        st = {"case": case, "X": _lowrank_rows(_gen(seed), _factor(seed, case["D"]), case["n"], DT[case["dtype"]])}
        st["H"] = torch.zeros((case["D"], case["D"]), dtype=F32, device="cuda")
    elif kind == "kfac":
        gen, w, m = _gen(seed), case["width"], case["mlp"]
        # inputs of q/k/v, of o, of gate/up and of down; then the seven output gradients
        widths = [w, w, w, m, w, w, w, w, m, m, w]
        st = {"case": case, "X": [], "H": []}
        for j, d in enumerate(widths):
            x = _student_t4(gen, case["n"], d, BF16) if j < 4 else _randn(gen, case["n"], d, dtype=BF16).mul_(1e-2)
            st["X"].append(x)
            st["H"].append(torch.zeros((d, d), dtype=F32, device="cuda"))
    elif kind == "apply":
        F = _factor(seed, case["D"])
        U, s, _ = torch.linalg.svd(F, full_matrices=False)
        U, s = U.cuda(), s.cuda()
        # H^{-1/2} of H = F F^T + 0.01 I
        M = (U * ((s * s + 0.01).rsqrt() - 10.0)) @ U.T
        M.diagonal().add_(10.0)
        st = {"case": case, "M": M.float().contiguous(),
              "X": _lowrank_rows(_gen(seed), F, case["n"], F16),
              "Y": torch.empty((case["n"], case["D"]), dtype=DT[case["out"]], device="cuda")}
    else:
        gen, nq, D, dtype = _gen(seed), case["nq"], case["D"], DT[case["dtype"]]
        G = _unit_rows(gen, case["n"], D, dtype)
        q = _unit(_randn(gen, nq, D))
        p = min(16, nq)  # queries with a near-duplicate in the store
        g = _unit(G[torch.randint(0, case["n"], (p,), generator=gen, device="cuda")].float())
        u = _unit(q[:p] - (q[:p] * g).sum(1, keepdim=True) * g)
        q[:p] = 0.9 * g + 0.19 ** 0.5 * u
        st = {"case": case, "G": G, "Q": q.to(dtype).contiguous()}
        if case["merge"]:
            st["base"] = 100000
            st["ts"], st["ti"] = _running(gen, nq, case["k"], D, st["base"])
        else:
            st["base"] = 0
            st["ts"] = torch.empty((nq, case["k"]), dtype=F32, device="cuda")
            st["ti"] = torch.empty((nq, case["k"]), dtype=torch.int64, device="cuda")
    return st


# ----------------------------------------------------------------------------
# one pass
# ----------------------------------------------------------------------------
def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "project":
        call = P.attr_project_tokens if case["tokens"] else P.attr_project
        return call(st["mods"], case["k"], case["n"], case["T"], st["out"], row_offset=st["offs"], length=st["lens"])
    if kind == "step":
        P.attr_project(st["mods"], case["k"], case["n"], case["T"], st["out"], row_offset=st["offs"], length=st["lens"])
        P.attr_precond_apply(st["out"], P.PRECOND_NONE, None, True, st["store"])
        P.attr_score_topk(st["Q"], st["store"], TOPK, st["ts"], st["ti"], index_base=st["base"], merge=True)
        st["base"] += case["n"]
        return {"rows": st["out"], "store": st["store"], "scores": st["ts"], "index": st["ti"]}
    if kind == "tiny":
        for tag in ("g", "q"):
            mod, n, raw, unit = st[tag]
            P.attr_project([mod], 16, n, case["T"], raw)
            P.attr_precond_apply(raw, P.PRECOND_NONE, None, True, unit)
        P.attr_score_topk(st["q"][3], st["g"][3], case["topk"], st["ts"], st["ti"])
        return {"rows": st["g"][3], "scores": st["ts"], "index": st["ti"]}
    if kind == "diag":
        h = torch.zeros(case["D"], dtype=F32, device="cuda")
        P.attr_precond_accumulate(st["X"], P.PRECOND_DIAG, h)
        m = finalize.finalize_diag(h, case["n"])
        P.attr_precond_apply(st["X"], P.PRECOND_DIAG, m, True, st["Y"])
        return {"h": h, "m": m, "rows": st["Y"]}
    if kind == "accumulate":
        return P.attr_precond_accumulate(st["X"], P.PRECOND_FULL, st["H"])
    if kind == "kfac":
        for x, h in zip(st["X"], st["H"]):
            P.attr_precond_accumulate(x, P.PRECOND_FULL, h)
        return list(st["H"])
    if kind == "apply":
        return P.attr_precond_apply(st["X"], P.PRECOND_FULL, st["M"], True, st["Y"])
    ts, ti = P.attr_score_topk(st["Q"], st["G"], case["k"], st["ts"], st["ti"], index_base=st["base"],
                               merge=case["merge"])
    if case["merge"]:
        st["base"] += case["n"]
    return {"scores": ts, "index": ti}


# ----------------------------------------------------------------------------
# what a pass cannot do without
# ----------------------------------------------------------------------------
def _project_work(case):
    tokens, k, eb = sum(_lengths(case)), case["k"], BYTES[case["dtype"]]
    rows = pairs = 0
    for d_in, d_out, tag in LAYERS[case["shape"]]:
        rows += d_out
        pairs += d_in + d_out
    rows += sum({tag: d_in for d_in, d_out, tag in LAYERS[case["shape"]]}.values())
    n_mods = len(LAYERS[case["shape"]]) * case["layers"]
    out = (tokens if case.get("tokens") else case["n"]) * n_mods * k * k * 4
    return {"bytes": case["layers"] * (rows * tokens + pairs * k) * eb + out,
            "flops": 2 * tokens * (case["layers"] * pairs * k + n_mods * k * k)}


def work(case):
    kind = case["kind"]
    if kind == "project":
        return _project_work(case)
    if kind == "step":
        w, D = _project_work(case), len(LAYERS[case["shape"]]) * case["layers"] * case["k"] ** 2
        w["bytes"] += case["n"] * D * 2 + N_QUERIES * (D * 2 + 2 * TOPK * 12)
        w["flops"] += 2 * N_QUERIES * case["n"] * D
        return w
    if kind == "tiny":
        n, d, T = case["n"] + case["nq"], case["d"], case["T"]
        return {"bytes": n * (2 * T * d + 512) * 4 + 2 * d * 64 + case["nq"] * case["topk"] * 12,
                "flops": n * T * (4 * d * 16 + 512) + 2 * case["n"] * case["nq"] * 256}
    if kind == "diag":  # the scale needs the whole store's moment first: its rows are read twice
        x = case["n"] * case["D"]
        return {"bytes": x * (2 * BYTES[case["dtype"]] + 2), "flops": 6 * x}
    if kind == "accumulate":
        n, D = case["n"], case["D"]
        return {"bytes": n * D * 2 + D * (D + 1) * 4, "flops": n * D * (D + 1)}
    if kind == "kfac":
        n, w, m = case["n"], case["width"], case["mlp"]
        return {"bytes": sum(c * (n * d * 2 + d * (d + 1) * 4) for c, d in ((8, w), (3, m))),
                "flops": sum(c * n * d * (d + 1) for c, d in ((8, w), (3, m)))}
    if kind == "apply":
        n, D = case["n"], case["D"]
        return {"bytes": n * D * (2 + BYTES[case["out"]]) + D * D * 4, "flops": 2 * n * D * D}
    nq, n, D, eb = case["nq"], case["n"], case["D"], BYTES[case["dtype"]]
    return {"bytes": (nq + n) * D * eb + nq * case["k"] * (24 if case["merge"] else 12), "flops": 2 * nq * n * D}


def tolerance(case):
    """About four times what another order of the 32-bit sums shows, and one
    rounding step of the outputs held in 16 bits.  Neighbours in a top-k list
    may change places where their scores differ by less than that."""
    kind = case["kind"]
    if kind == "project":
        return {"rel": 1e-5}
    if kind == "step":
        return {"rel": 2e-4, "max": 4e-3, "differ": 0.01}
    if kind == "tiny":
        return {"rel": 1e-5, "differ": 0.01}
    if kind == "diag":
        return {"rel": 1e-4, "max": 4e-3}
    if kind in ("accumulate", "kfac"):
        return {"rel": 1e-5}
    if kind == "apply":
        return {"rel": 4e-4 if case["out"] == "f16" else 1e-4, "max": 1e-2}
    return {"rel": 1e-5, "differ": 0.01}


# ----------------------------------------------------------------------------
# the same in 64 bits
# ----------------------------------------------------------------------------
def _exact_rows(st):
    case, lens, k = st["case"], _lengths(st["case"]), st["case"]["k"]
    out = torch.zeros(st["out"].shape, dtype=torch.float64, device="cuda")
    for m in st["mods"]:
        R, S = m.R.double(), m.S.double()
        if m.v_out is not None:
            R = R * (m.v_out.double().sum() / m.v_out.double()).sqrt()[:, None]
            S = S * m.v_in.double().rsqrt()[:, None]
        t0 = 0
        for i, n in enumerate(lens):
            x, y = m.g[t0:t0 + n].double() @ R, m.a[t0:t0 + n].double() @ S
            cols = slice(m.out_col, m.out_col + k * k)
            if case.get("tokens"):
                out[t0:t0 + n, cols] = (x[:, :, None] * y[:, None, :]).reshape(n, k * k)
            else:
                out[i, cols] = (x.T @ y).reshape(-1)
            t0 += n
    return out


def _exact_scores(Q, G, k, old=None):
    best = old.double() if old is not None else None
    Qd = Q.double()
    for i in range(0, G.shape[0], 65536):
        s = Qd @ G[i:i + 65536].double().T
        s = s if best is None else torch.cat([best, s], 1)
        best = torch.topk(s, min(k, s.shape[1]), dim=1).values
    pad = torch.full((Q.shape[0], k - best.shape[1]), -math.inf, dtype=torch.float64, device="cuda")
    return torch.cat([best, pad], 1)


def _exact_moment(X):
    H = torch.zeros((X.shape[1],) * 2, dtype=torch.float64, device="cuda")
    for i in range(0, X.shape[0], 65536):
        x = X[i:i + 65536].double()
        H.addmm_(x.T, x)
    return H.triu_()


def exact(case, seed):
    kind, st = case["kind"], prepare(case, seed)
    if kind == "project":
        return _exact_rows(st)
    if kind == "step":
        rows = _exact_rows(st)
        store = _unit(rows)
        return {"rows": rows, "store": store, "scores": _exact_scores(st["Q"], store, TOPK, st["ts"]), "index": None}
    if kind == "tiny":
        unit = {}
        for tag in ("g", "q"):
            mod, n, _, _ = st[tag]
            x = (mod.g.double() @ mod.R.double()).reshape(n, case["T"], 16)
            y = (mod.a.double() @ mod.S.double()).reshape(n, case["T"], 16)
            unit[tag] = _unit((x[:, :, :, None] * y[:, :, None, :]).sum(1).reshape(n, 256))
        return {"rows": unit["g"], "scores": _exact_scores(unit["q"], unit["g"], case["topk"]), "index": None}
    if kind == "diag":
        X = st["X"]
        h = sum(X[i:i + 65536].double().square().sum(0) for i in range(0, X.shape[0], 65536))
        m = (h / case["n"]).rsqrt()
        rows = torch.empty(X.shape, dtype=F32, device="cuda")
        for i in range(0, X.shape[0], 65536):
            rows[i:i + 65536] = _unit(X[i:i + 65536].double() * m).float()
        return {"h": h, "m": m, "rows": rows}
    if kind == "accumulate":
        return _exact_moment(st["X"])
    if kind == "kfac":
        return [_exact_moment(x) for x in st["X"]]
    if kind == "apply":
        M, X = st["M"].double(), st["X"]
        rows = torch.empty(X.shape, dtype=F32, device="cuda")
        for i in range(0, X.shape[0], 65536):
            rows[i:i + 65536] = _unit(X[i:i + 65536].double() @ M.T).float()
        return rows
    return {"scores": _exact_scores(st["Q"], st["G"], case["k"], st["ts"] if case["merge"] else None), "index": None}
