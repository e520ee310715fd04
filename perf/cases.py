"""The work a serving program (and the offline compressor before it) has this
framework do, as measurable cases.

A case is a dict of plain values; "kind" names the public entry point:
  layer        apply                 y = W x + U_k Sigma_i V_k^T x
  diag         apply_diag            diagonal Sigma_i
  ranked       apply_ranked          a rank per cluster
  lora         apply_uncompressed    y = W x + B_i A_i x
  lora_ranked  apply_uncompressed_ranked
  qkv          apply_multi_packed    several projections of one input, from the ids
  block        sort_by_cluster once, then every projection of a decoder layer
               through apply_multi_packed / apply_multi_sorted
  jd_full, jd_diag   the offline compressor
Tensors are drawn on the GPU from the seed: x ~ N(0, 1), weights with variance
1 / fan-in, bases with columns of unit norm, Sigma_i ~ N(0, 1/r), and LoRAs
whose adapter term is about 1/8 of the base term.
"""
import math
import random

import torch

import paper_2407_00066_amd as cts
from paper_2407_00066_amd import compress as jd

BF16, F32, F64 = torch.bfloat16, torch.float32, torch.float64
DTYPES = {"bf16": BF16, "f32": F32}
SINGLE = ("layer", "diag", "ranked", "lora", "lora_ranked")


def _case(name, kind, T, d_in, d_out, r, n, K, ids="uniform", dtype="bf16"):
    return {"name": name, "kind": kind, "T": T, "d_in": d_in, "d_out": d_out, "r": r, "n": n, "K": K,
            "ids": ids, "dtype": dtype}


def listed():
    return [
        # one request decoding alone: a single token through q_proj
        _case("decode_1", "layer", 1, 4096, 4096, 64, 1000, 25),
        # a decode batch of 64 requests on a 7B-shaped q_proj, 100 LoRAs in one cluster
        _case("decode_q", "layer", 64, 4096, 4096, 64, 100, 1),
        # the fused q/k/v projection of a decode batch of 33 requests, 1000 LoRAs in 50 clusters
        {"name": "decode_qkv", "kind": "qkv", "T": 33, "d_in": 4096, "d_out": 4096, "d_kv": 1024, "M": 3, "r": 64,
         "n": 1000, "K": 50, "ids": "uniform", "dtype": "bf16"},
        # the same decode batch through uncompressed rank-16 LoRAs
        _case("lora_decode", "lora", 64, 4096, 4096, 16, 100, 100),
        # MLP up-projection of 256 requests with a few popular LoRAs, at the largest rank
        _case("mlp_up", "layer", 256, 4096, 14336, 128, 1000, 50, "zipf"),
        # every projection of one decoder layer for 512 requests, tokens bucketed once
        {"name": "block_512", "kind": "block", "T": 512, "d_in": 4096, "d_kv": 1024, "d_ff": 14336, "r": 64,
         "n": 1000, "K": 50, "ids": "uniform", "dtype": "bf16"},
        # prefill of 32 prompts, 1000 LoRAs in 25 clusters (the paper's serving setting)
        _case("prefill_mix", "layer", 4096, 4096, 4096, 64, 1000, 25, "prefill"),
        # prefill with diagonal cores at sizes that are no multiple of any tile
        _case("prefill_diag_ragged", "diag", 2777, 3000, 5000, 48, 500, 16, "prefill"),
        # prefill through uncompressed LoRAs of ranks 8 to 32
        _case("lora_prefill", "lora_ranked", 4096, 4096, 4096, 32, 1000, 1000, "prefill"),
        # fp32 weights throughout
        _case("fp32_layer", "layer", 500, 1024, 2816, 32, 200, 8, "zipf", "f32"),
        # offline: 1000 rank-16 LoRAs of a 4096 x 4096 projection compressed to rank 64
        {"name": "jd_full", "kind": "jd_full", "n": 1000, "d_in": 4096, "d_out": 4096, "r_l": 16, "r": 64,
         "iters": 10, "normalize": True},
        # offline: the diagonal compressor on a smaller, ragged collection
        {"name": "jd_diag", "kind": "jd_diag", "n": 300, "d_in": 2048, "d_out": 5632, "r_l": 16, "r": 64,
         "iters": 5, "normalize": False},
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _dim(rng, lo, hi):
    """A feature count: usually a multiple of 128, sometimes only of 8."""
    v = _log_int(rng, lo, hi)
    q = 8 if rng.random() < 0.3 else 128
    return max(lo, v // q * q)


def draw(rng):
    pick = rng.random()
    if pick < 0.12:
        kind = rng.choice(("jd_full", "jd_diag"))
        r_l = rng.choice((8, 16, 32))
        return {"kind": kind, "n": _log_int(rng, 64, 800 * 16 // max(r_l, 16)), "d_in": _dim(rng, 512, 4096),
                "d_out": _dim(rng, 512, 4096), "r_l": r_l, "r": rng.choice((16, 32, 64, 96)),
                "iters": rng.randint(3, 8), "normalize": rng.random() < 0.5}
    n = _log_int(rng, 8, 1000)
    K = _log_int(rng, 1, min(50, n))
    r = rng.choice((16, 32, 48, 64, 64, 64, 128))
    if pick < 0.24:
        return {"kind": "block", "T": _log_int(rng, 8, 2048), "d_in": _dim(rng, 1024, 4096),
                "d_kv": 128 * rng.randint(2, 8), "d_ff": _dim(rng, 2816, 11008), "r": rng.choice((32, 64)),
                "n": n, "K": K, "ids": rng.choice(("uniform", "zipf", "prefill")), "dtype": "bf16"}
    if pick < 0.36:
        M = rng.choice((2, 3))
        d = _dim(rng, 1024, 6144)
        return {"kind": "qkv", "T": _log_int(rng, 1, 1024), "d_in": _dim(rng, 1024, 6144), "d_out": d,
                "d_kv": 128 * rng.randint(2, 8) if M == 3 else d, "M": M, "r": rng.choice((32, 64)), "n": n, "K": K,
                "ids": rng.choice(("uniform", "zipf")), "dtype": "bf16"}
    kind = rng.choice(("layer", "layer", "layer", "layer", "diag", "ranked", "lora", "lora_ranked"))
    if kind.startswith("lora"):
        r, K = rng.choice((8, 16, 32)), n
    band = rng.random()
    if band < 0.45:                                     # decode
        T, ids = _log_int(rng, 1, 128), rng.choice(("uniform", "zipf"))
    elif band < 0.7:                                    # larger decode batches, mixed batches
        T, ids = _log_int(rng, 129, 2047), rng.choice(("uniform", "zipf", "prefill"))
    else:                                               # prefill, past one bucketing's 8192 tokens too
        T, ids = _log_int(rng, 2048, 10000), "prefill"
    f32 = rng.random() < 0.12
    hi = 2048 if f32 else 8192 if T < 2048 else 6144
    return {"kind": kind, "T": min(T, 1500) if f32 else T, "d_in": _dim(rng, 256 if f32 else 1024, hi),
            "d_out": _dim(rng, 256 if f32 else 1024, hi if f32 or T >= 2048 else 14336), "r": r, "n": n, "K": K,
            "ids": ids, "dtype": "f32" if f32 else "bf16"}


# ---------------------------------------------------------------- inputs
def _ids(c, seed):
    """(adapter_id[T], cluster_of[n]) as lists: requests pick LoRAs uniformly
    or by a Zipf law; in a prefill all tokens of a prompt name one LoRA; the
    clusters hold equally many LoRAs."""
    rng = random.Random(seed * 7 + 1)
    n, K, T = c["n"], c["K"], c["T"]
    order = list(range(n))
    rng.shuffle(order)
    cof = [0] * n
    for p, i in enumerate(order):
        cof[i] = p * K // n if K < n else i
    zipf = [1.0 / (k + 1) ** 1.1 for k in range(n)]
    if c["ids"] == "uniform":
        aid = [rng.randrange(n) for _ in range(T)]
    elif c["ids"] == "zipf":
        aid = rng.choices(range(n), zipf, k=T)
    else:
        aid = []
        while len(aid) < T:
            aid += [rng.choices(range(n), zipf)[0]] * min(T - len(aid), rng.randint(32, 256))
    return aid, cof


def _ranks(c, seed):
    rng = random.Random(seed * 7 + 2)
    return [8 * rng.randint(1, c["r"] // 8) for _ in range(c["K"])]


class _Draw:
    def __init__(self, seed, dtype):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(seed)
        self.dtype = dtype

    def __call__(self, shape, var):
        return torch.randn(shape, generator=self.g, device="cuda").mul_(math.sqrt(var)).to(self.dtype)


def _i32(v):
    return torch.tensor(v, dtype=torch.int32, device="cuda")


def _groups(c):
    """The projections of a case, in groups that share an input: (d_in, [d_out])."""
    if c["kind"] == "block":
        d, f = c["d_in"], c["d_ff"]
        return [(d, [d, c["d_kv"], c["d_kv"]]), (d, [d]), (d, [f, f]), (f, [d])]
    if c["kind"] == "qkv":
        return [(c["d_in"], [c["d_out"]] + [c["d_kv"]] * (c["M"] - 1))]
    return [(c["d_in"], [c["d_out"]])]


def _inputs(c, seed):
    if c["kind"] in ("jd_full", "jd_diag"):
        # LoRAs that share directions of falling weight, each with a part of its own
        dr = _Draw(seed, F32)
        n, r_l, r, di, do = c["n"], c["r_l"], c["r"], c["d_in"], c["d_out"]
        fall = torch.linspace(1.0, 0.1, 2 * r, device="cuda")
        A = dr((n * r_l, 2 * r), 1.0 / r).mul_(fall) @ dr((2 * r, di), 1.0 / di)
        A = A.add_(dr((n * r_l, di), 0.25 / di)).view(n, r_l, di)
        M = dr((2 * r, n * r_l), 1.0 / r).mul_(fall[:, None])
        B = (dr((do, 2 * r), 1.0 / (64 * r_l)) @ M).view(do, n, r_l).transpose(0, 1).contiguous()
        B.add_(dr((n, do, r_l), 0.25 / (64 * r_l)))
        U0, V0 = dr((do, r), 1.0 / do), dr((di, r), 1.0 / di)
        if c["kind"] == "jd_full":
            U0, V0 = (torch.linalg.qr(m.cpu().double())[0].float().cuda() for m in (U0, V0))
        return {"A": A, "B": B, "U0": U0.contiguous(), "Vt0": V0.t().contiguous()}
    dr = _Draw(seed, DTYPES[c["dtype"]])
    aid, cof = _ids(c, seed)
    s = {"adapter_id": _i32(aid), "cluster_of": _i32(cof), "groups": []}
    T, r, n, K = c["T"], c["r"], c["n"], c["K"]
    for d_in, d_outs in _groups(c):
        g = {"x": dr((T, d_in), 1.0), "W": [dr((d, d_in), 1.0 / d_in) for d in d_outs]}
        if c["kind"].startswith("lora"):
            g["A"], g["B"] = dr((n, r, d_in), 1.0 / d_in), dr((n, d_outs[0], r), 1.0 / (64 * r))
        else:
            g["Vt"] = dr((K, len(d_outs) * r, d_in), 1.0 / d_in)
            g["U"] = [dr((K, d, r), 1.0 / d) for d in d_outs]
            g["Sigma"] = [dr((n, r) if c["kind"] == "diag" else (n, r, r), 1.0 if c["kind"] == "diag" else 1.0 / r)
                          for _ in d_outs]
        s["groups"].append(g)
    if c["kind"].endswith("ranked"):
        s["ranks"] = _i32(_ranks(c, seed))
    return s


def prepare(case, seed):
    """Weights, inputs and the caller's output and workspace buffers."""
    s = _inputs(case, seed)
    s["case"] = case
    if case["kind"] in ("jd_full", "jd_diag"):
        s["ws"] = torch.empty(jd.workspace_size(s["A"], s["B"], case["r"]), dtype=torch.uint8, device="cuda")
        return s
    T, dt = case["T"], DTYPES[case["dtype"]]
    code = cts.CTS_BF16 if dt == BF16 else cts.CTS_F32
    need = 1
    for g in s["groups"]:
        d_outs = [w.shape[0] for w in g["W"]]
        g["out"] = torch.empty((T, sum(d_outs)), dtype=dt, device="cuda")
        lora = case["kind"].startswith("lora")
        p = cts.make_problem(T, g["x"].shape[1], d_outs[0], r=0 if lora else case["r"], n_adapters=case["n"],
                             n_clusters=1 if lora else case["K"], r_lora=case["r"] if lora else 0, dtype=code)
        need = max(need, cts.workspace_size_multi(p, d_outs) if case["kind"] in ("qkv", "block")
                   else cts.workspace_size(p, not lora))
    s["ws"] = torch.empty(need, dtype=torch.uint8, device="cuda")
    if case["kind"] == "block":
        s["perm"] = torch.empty(T, dtype=torch.int32, device="cuda")
        s["offs"] = torch.empty(case["K"] + 1, dtype=torch.int32, device="cuda")
        s["bucketing"] = torch.empty(cts.bucketing_size(T, case["n"], case["K"]), dtype=torch.uint8, device="cuda")
    return s


def run(s):
    c = s["case"]
    kind, ws = c["kind"], s["ws"]
    if kind == "jd_full":
        return jd.jd_full(s["A"], s["B"], s["U0"], s["Vt0"], iters=c["iters"], normalize=c["normalize"],
                          workspace=ws)[:4]
    if kind == "jd_diag":
        return jd.jd_diag(s["A"], s["B"], s["U0"], s["Vt0"], sweeps=c["iters"], normalize=c["normalize"], workspace=ws)
    aid, cof = s["adapter_id"], s["cluster_of"]
    if kind == "block":
        perm, _, buck = cts.sort_by_cluster(aid, cof, c["n"], c["K"], s["perm"], s["offs"], s["bucketing"])
        outs = []
        for g in s["groups"]:
            if len(g["W"]) == 1:
                outs += cts.apply_multi_sorted(perm, buck, g["x"], g["W"], g["U"], g["Vt"], g["Sigma"],
                                               outs=[g["out"]], workspace=ws)
            else:
                outs.append(cts.apply_multi_packed(g["x"], g["W"], g["U"], g["Vt"], g["Sigma"], perm=perm,
                                                   bucketing=buck, out=g["out"], workspace=ws))
        return outs
    g = s["groups"][0]
    x, W, out = g["x"], g["W"][0], g["out"]
    if kind == "qkv":
        return cts.apply_multi_packed(x, g["W"], g["U"], g["Vt"], g["Sigma"], adapter_id=aid, cluster_of=cof, out=out,
                                      workspace=ws)
    if kind == "layer":
        return cts.apply(x, aid, cof, W, g["U"][0], g["Vt"], g["Sigma"][0], out=out, workspace=ws)
    if kind == "diag":
        return cts.apply_diag(x, aid, cof, W, g["U"][0], g["Vt"], g["Sigma"][0], out=out, workspace=ws)
    if kind == "ranked":
        return cts.apply_ranked(x, aid, cof, W, g["U"][0], g["Vt"], g["Sigma"][0], s["ranks"], out=out, workspace=ws)
    if kind == "lora":
        return cts.apply_uncompressed(x, aid, W, g["A"], g["B"], out=out, workspace=ws)
    return cts.apply_uncompressed_ranked(x, aid, W, g["A"], g["B"], s["ranks"], out=out, workspace=ws)


# ---------------------------------------------------------------- work, tolerance
def work(case):
    """Each weight, each touched basis and core, every input and output once."""
    c = case
    if c["kind"] in ("jd_full", "jd_diag"):
        n, r_l, r, di, do, it = c["n"], c["r_l"], c["r"], c["d_in"], c["d_out"], c["iters"]
        N = n * r_l
        if c["kind"] == "jd_full":
            # per iteration P, Q, sum B C, sum A D, the r_l x r_l products; then the cores
            flops = it * (4.0 * N * r * (di + do) + 8.0 * N * r_l * r) + 2.0 * N * r * (di + do) + 2.0 * N * r * r
            passes, out = 2 * it + 1, n * r * r
        else:
            # per sweep P, Q and the two sums; the first diagonals need one P and Q
            flops = (it + 1) * 2.0 * N * r * (di + do) + it * 2.0 * N * r * (di + do)
            passes, out = 2 * it + 1, n * r
        return {"bytes": 4.0 * (passes * N * (di + do) + 2 * r * (di + do) + out), "flops": flops}
    T, r, n = c["T"], c["r"], c["n"]
    aid, cof = _ids(c, 0)
    e = 2.0 if c["dtype"] == "bf16" else 4.0
    nad, ncl = len(set(aid)), len({cof[i] for i in aid})
    nbytes = flops = 0.0
    for d_in, d_outs in _groups(c):
        nbytes += e * T * d_in
        for d in d_outs:
            nbytes += e * (d * d_in + T * d)
            if c["kind"].startswith("lora"):
                nbytes += e * nad * r * (d_in + d)
                flops += 2.0 * T * (d_in * d + r * (d_in + d))
            else:
                diag = c["kind"] == "diag"
                nbytes += e * (ncl * r * (d_in + d) + nad * r * (1 if diag else r))
                flops += 2.0 * T * (d_in * d + r * (d_in + (0 if diag else r) + d))
    return {"bytes": nbytes + 4.0 * (T + n), "flops": flops}


def tolerance(case):
    """bf16 outputs round once to 8 bits (2-norm about 1.7e-3); fp32 layers sum
    up to a few thousand products (6e-7 seen); the compressor's iterations carry
    fp32 rounding from step to step (up to 1.9e-6, single values 1.2e-5)."""
    if case["kind"] in ("jd_full", "jd_diag"):
        return {"rel": 1e-5, "max": 1e-4}
    if case["dtype"] == "f32":
        return {"rel": 3e-6, "max": 3e-5}
    return {"rel": 6e-3, "max": 4e-2}


# ---------------------------------------------------------------- 64-bit results
def _exact_jd_full(c, s):
    A, B = s["A"].double(), s["B"].double()
    n, r_l, di = A.shape
    do, r = B.shape[1], c["r"]
    A2, B2 = A.reshape(n * r_l, di), B.transpose(0, 1).reshape(do, n * r_l)
    w = torch.ones(n, dtype=F64, device="cuda")
    if c["normalize"]:
        gb = torch.stack([b.t() @ b for b in B])
        ga = torch.stack([a @ a.t() for a in A])
        w = 1.0 / (gb * ga).sum((1, 2))
    U, V = s["U0"].double(), s["Vt0"].double().t().contiguous()

    def qr(X):
        q, t = torch.linalg.qr(X.cpu())
        return (q * torch.sign(torch.diagonal(t))).cuda()

    def small(X, Y):                                     # X_i (Y_i^T Z_i) per LoRA, without batched products
        return (X[:, :, :, None] * Y[:, None, :, :]).sum(2)

    crit = []
    for _ in range(c["iters"]):
        P = (A2 @ V).view(n, r_l, r)
        Q = (B2.t() @ U).view(n, r_l, r)
        G = (P[:, :, None, :] * P[:, None, :, :]).sum(3)
        H = (Q[:, :, None, :] * Q[:, None, :, :]).sum(3)
        C = small(G, Q) * w[:, None, None]
        D = small(H, P) * w[:, None, None]
        Un, Vn = qr(B2 @ C.reshape(n * r_l, r)), qr(A2.t() @ D.reshape(n * r_l, r))
        crit.append(max(((X1 - X0 @ (X0.t() @ X1)).norm() / X1.norm()).item() for X0, X1 in ((U, Un), (V, Vn))))
        U, V = Un, Vn
    P = (A2 @ V).view(n, r_l, r)
    Q = (B2.t() @ U).view(n, r_l, r)
    S = torch.stack([q.t() @ p for q, p in zip(Q, P)])
    return [U, V.t().contiguous(), S, torch.tensor(crit, dtype=F64)]


def _exact_jd_diag(c, s):
    A, B = s["A"].double(), s["B"].double()
    n, r_l, di = A.shape
    do, r = B.shape[1], c["r"]
    A2, B2 = A.reshape(n * r_l, di), B.transpose(0, 1).reshape(do, n * r_l)
    U, V = s["U0"].double(), s["Vt0"].double().t().contiguous()

    def solve_right(X, M):                               # X M^-1 for a symmetric M
        return torch.linalg.solve(M.cpu(), X.t().cpu()).t().contiguous().cuda()

    def diagonals():
        P, Q = (A2 @ V).view(n, r_l, r), (B2.t() @ U).view(n, r_l, r)
        return solve_right((P * Q).sum(1), (U.t() @ U) * (V.t() @ V))

    sg = diagonals()
    for _ in range(c["iters"]):
        ss = sg.t() @ sg
        U = solve_right(B2 @ ((A2 @ V).view(n, r_l, r) * sg[:, None, :]).reshape(n * r_l, r), (V.t() @ V) * ss)
        V = solve_right(A2.t() @ ((B2.t() @ U).view(n, r_l, r) * sg[:, None, :]).reshape(n * r_l, r), (U.t() @ U) * ss)
        sg = diagonals()
        if c["normalize"]:
            nu = sg.norm()
            sg, U, V = sg / nu, U * nu.sqrt(), V * nu.sqrt()
    return [U, V.t().contiguous(), sg]


def exact(case, seed):
    c, s = case, _inputs(case, seed)
    if c["kind"] == "jd_full":
        return _exact_jd_full(c, s)
    if c["kind"] == "jd_diag":
        return _exact_jd_diag(c, s)
    lora = c["kind"].startswith("lora")
    aid = s["adapter_id"].long()
    seg = aid if lora else s["cluster_of"].long()[aid]
    ranks = s["ranks"].tolist() if "ranks" in s else None
    r, outs = c["r"], []
    for g in s["groups"]:
        x, ys = g["x"].double(), []
        for m, W in enumerate(g["W"]):
            y = x @ W.double().t()
            if not lora:
                core = g["Sigma"][m]
            for k in sorted(set(seg.tolist())):
                rows = torch.nonzero(seg == k).flatten()
                rk = ranks[k] if ranks else r
                down, up = (g["A"][k], g["B"][k]) if lora else (g["Vt"][k, m * r:(m + 1) * r], g["U"][m][k])
                z = x[rows] @ down[:rk].double().t()
                if not lora:
                    if c["kind"] == "diag":
                        z = z * core[aid[rows]].double()
                    else:
                        for i in sorted(set(aid[rows].tolist())):
                            at = torch.nonzero(aid[rows] == i).flatten()
                            z[at] = z[at] @ core[i][:rk, :rk].double().t()
                y[rows] += z @ up[:, :rk].double().t()
            ys.append(y)
        outs.append(torch.cat(ys, 1))
    return outs if c["kind"] == "block" else outs[0]
