"""The work this library is measured on, as a program that uses it would call it.

A case is a dict of plain values.  `op` names the entry point:

  reduce   Reducer.reduce (entry "context"), Reducer.reduce_given_s ("given_s")
           or reduce_noalloc ("noalloc"): score, select and gather a packed batch
  project  Reducer.reduce_project: the same with the kept tokens projected
  select   Reducer.select: Algorithm 1 on scores the caller holds
  mlp      Reducer.mlp_out_cos: the encoder MLP's second layer with its cosine
  gemm     Reducer.gemm: the projector on tokens already gathered

`images` images of n_lo .. n_hi tokens (their sizes are drawn from `pick`, part
of the case), rows of `d` elements of X and `dc` of the pre- and post-MLP
states, `keep` the kept share of an image's tokens or `kept` their number.
"""
import math
import random

import torch

import paper_2607_13500_amd as tr

DEV = "cuda"
THIRD = 1.0 / 3.0


def reduce_case(name, images, n_lo, n_hi, d, dc, dtype, kept=0, keep=0.0, entry="context", lam=THIRD, shannon=False,
                stride_real=False, scores=False, pick=1, op="reduce", nout=0):
    return {"name": name, "op": op, "images": images, "n_lo": n_lo, "n_hi": n_hi, "d": d, "dc": dc, "dtype": dtype,
            "kept": kept, "keep": keep, "entry": entry, "lam": lam, "shannon": shannon, "stride_real": stride_real,
            "scores": scores, "pick": pick, "nout": nout}


def matrix_case(name, op, m, n, k):
    return {"name": name, "op": op, "m": m, "n": n, "k": k}


def listed():
    return [
        # one request of a server: a single 24 x 24 fp32 image, bound by latency
        reduce_case("one_image_fp32", 1, 576, 576, 1024, 1024, "fp32", kept=64),
        # the benchmark's batch: LLaVA-1.5 tokens to 64 each
        reduce_case("batch_64x576", 64, 576, 576, 4096, 4096, "bf16", kept=64),
        # high-resolution images of five tiles each (LLaVA-NeXT)
        reduce_case("tiles_16x2880", 16, 2880, 2880, 4096, 4096, "bf16", kept=320),
        # a batch of dynamic-resolution images, kept by ratio: the largest call
        reduce_case("ragged_32x16384", 32, 256, 16384, 3584, 3584, "bf16", keep=0.11),
        # four clips of 32 frames, near the selection's largest image
        reduce_case("video_4x18432", 4, 18432, 18432, 4096, 4096, "bf16", kept=1152),
        # small ragged batch of odd row widths (no 16-byte alignment), scores wanted too
        reduce_case("odd_7x1500", 7, 50, 1500, 1025, 333, "bf16", keep=0.2, scores=True),
        # the entry for callers that cannot allocate, with a class token in each
        # image and both variants of the method (Shannon entropy, real interval)
        reduce_case("noalloc_16x577", 16, 577, 577, 1024, 1024, "fp32", kept=192, entry="noalloc", shannon=True,
                    stride_real=True, scores=True),
        # selection from scores that the caller computed itself, sizes over the whole range
        reduce_case("select_24x18000", 24, 64, 18000, 1, 1, "fp32", keep=0.15, op="select", pick=3),
        # the module with the projector applied to the kept tokens, a batch and one image
        reduce_case("project_64x576", 64, 576, 576, 4096, 4096, "bf16", kept=64, op="project", nout=4096),
        reduce_case("project_one", 1, 576, 576, 1024, 1024, "bf16", kept=64, op="project", nout=4096),
        # the last MLP's second layer for the benchmark's batch (states of 1024)
        matrix_case("mlp_36864x1024", "mlp", 36864, 1024, 4096),
        # a projector whose sizes are multiples of the smallest tile only
        matrix_case("gemm_3001x1664", "gemm", 3001, 1664, 4160),
    ]


def spread(rng, lo, hi):
    """A whole number in [lo, hi], its logarithm uniform."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    op = rng.choice(["reduce", "reduce", "reduce", "project", "select", "mlp", "gemm"])
    if op in ("mlp", "gemm"):
        while True:
            c = {"op": op, "m": spread(rng, 16, 36864), "n": 128 * spread(rng, 1, 32), "k": 64 * spread(rng, 1, 64)}
            if c["m"] * c["n"] * c["k"] <= 36864 * 1024 * 4096:
                return c
    while True:
        images, n_hi = spread(rng, 1, 64), spread(rng, 16, 18432)
        n_lo = rng.choice([n_hi, n_hi, max(1, n_hi // 4), max(1, n_hi // 40)])
        c = {"op": op, "images": images, "n_lo": n_lo, "n_hi": n_hi, "d": 1, "dc": 1, "dtype": "fp32", "kept": 0,
             "keep": spread(rng, 20, 600) / 1000.0, "entry": "context", "lam": rng.choice([THIRD, THIRD, 0.5, 1.0, 0.0]),
             "shannon": False, "stride_real": rng.random() < 0.25, "scores": False, "pick": rng.randrange(1 << 20),
             "nout": 0}
        if op == "select":
            return c
        c["shannon"] = rng.random() < 0.2
        if op == "project":
            c.update(d=64 * spread(rng, 4, 64), dtype="bf16", nout=128 * spread(rng, 2, 32))
            c["dc"] = rng.choice([c["d"], 1024])
        else:
            c.update(d=spread(rng, 64, 4096), dtype=rng.choice(["bf16", "bf16", "fp32"]),
                     entry=rng.choice(["context", "context", "noalloc", "given_s"]))
            if rng.random() < 0.75:
                c["d"] = (c["d"] + 7) // 8 * 8      # encoders' widths are multiples of 8, mostly
            c["dc"] = rng.choice([c["d"], c["d"], 1024])
            # tr_reduce reads the states for scores or where Stage II ranks; a supplied key has no scores to return
            c["scores"] = c["entry"] != "given_s" and rng.random() < 0.3
        w = work(c)
        if w["bytes"] <= 3e9 and w["flops"] <= 3e11 and images * n_hi <= 1 << 19:
            return c


# ---- what a case means -------------------------------------------------------
def sizes(case):
    rng = random.Random(case["pick"])
    N = [rng.randint(case["n_lo"], case["n_hi"]) for _ in range(case["images"])]
    K = [case["kept"] or max(1, min(n, math.floor(case["keep"] * n))) for n in N]
    return N, K


def torch_type(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def ranked(case, N, K):
    """Whether Stage I (by entropy) and Stage II (by cosine) order any image's tokens."""
    one = two = False
    for n, k in zip(N, K):
        k1 = math.floor(case["lam"] * k)
        one = one or 0 < k1 < n
        two = two or 0 < k - k1 < n - k1
    return one, two


def work(case):
    if case["op"] in ("mlp", "gemm"):
        m, n, k = case["m"], case["n"], case["k"]
        more = 2 * m * n + 4 * m if case["op"] == "mlp" else 0      # X_pre read, s written
        return {"bytes": 2 * (m * k + n * k + m * n) + more, "flops": 2 * m * n * k}
    N, K = sizes(case)
    rows, kept = sum(N), sum(K)
    if case["op"] == "select":
        return {"bytes": 8 * rows + 5 * kept, "flops": 0}
    e = 2 if case["dtype"] == "bf16" else 4
    one, two = ranked(case, N, K)
    one, two = one or case["scores"], two or case["scores"]
    given = case["entry"] == "given_s"
    read = (rows if one else kept) * case["d"] * e
    if two:
        read += 4 * rows if given else 2 * rows * case["dc"] * e
    flops = (4 * rows * case["d"] if one else 0) + (6 * rows * case["dc"] if two and not given else 0)
    bytes_ = read + 5 * kept + (8 * rows if case["scores"] else 0)
    if case["op"] == "project":
        return {"bytes": bytes_ + 2 * case["nout"] * (case["d"] + kept), "flops": flops + 2 * kept * case["d"] * case["nout"]}
    return {"bytes": bytes_ + e * kept * case["d"], "flops": flops}


def tolerance(case):
    if case["op"] == "select":
        return "exact"
    if case["op"] in ("mlp", "gemm", "project"):
        # fp32 sums rounded to bf16: another order of the sums moves a few of
        # them to the neighbouring bf16 value (2^-8 of it)
        return {"rel": 1e-3, "max": 2e-2}
    # h2 and s are fp32 sums.  A row's sums have one order in this library,
    # whatever path reads the row, so the kept tokens and their copies stay.
    return {"rel": 1e-5}


# ---- inputs --------------------------------------------------------------------
def generator(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def randn(g, *shape):
    return torch.randn(*shape, generator=g, device=DEV)


def tokens(case, seed):
    """X, Xpre, Xpost of a batch: clustered tokens of varying magnitude, one in
    ten of low variance (smooth background), one in twenty a repetition of
    another token of its image; the states' agreement varies per token."""
    g = generator(seed)
    N, _ = sizes(case)
    d, dc, dt = case["d"], case["dc"], torch_type(case)
    rows = sum(N)
    X = torch.empty(rows, d, dtype=dt, device=DEV)
    P, Q = (torch.empty(rows, dc, dtype=dt, device=DEV) for _ in range(2))
    gamma = torch.exp(0.25 * randn(g, dc))
    r0 = 0
    for n in N:
        label = torch.randint(0, 16, (n,), generator=g, device=DEV)
        x = (randn(g, 16, d)[label] + randn(g, n, d)) / math.sqrt(2.0) * torch.exp(0.5 * randn(g, n, 1))
        order = torch.randperm(n, generator=g, device=DEV)
        low, rep = order[: n // 10], order[n // 10: n // 10 + n // 20]
        x[low] = 1.0 + 0.05 * torch.exp(0.3 * randn(g, low.numel(), 1)) * randn(g, low.numel(), d)
        p = gamma * randn(g, n, dc)
        q = (0.3 + 0.1 * randn(g, n, 1)) * p + randn(g, n, dc)
        source = order[n // 10 + n // 20:][: rep.numel()]
        for t in (x, p, q):
            t[rep] = t[source]
        X[r0:r0 + n], P[r0:r0 + n], Q[r0:r0 + n] = x.to(dt), p.to(dt), q.to(dt)
        r0 += n
    return X, P, Q


def given_scores(rows, seed):
    """Scores as a program has them: entropy-like keys, cosines, a few repeated."""
    g = generator(seed)
    key = torch.exp(0.5 * randn(g, rows))
    s = 0.3 + 0.1 * randn(g, rows)
    order = torch.randperm(rows, generator=g, device=DEV)
    same, source = order[: rows // 50], order[rows // 50:][: rows // 50]
    key[same], s[same] = key[source], s[source]
    return key, s


def matrices(case, seed):
    g = generator(seed)
    m, n, k = case["m"], case["n"], case["k"]
    A = randn(g, m, k)
    if case["op"] == "mlp":
        A = torch.nn.functional.gelu(A)     # hidden activations
    W = randn(g, n, k) / math.sqrt(k)
    P = randn(g, m, n) if case["op"] == "mlp" else None
    return [None if t is None else t.to(torch.bfloat16) for t in (A, W, P)]


def prepare(case, seed):
    op = case["op"]
    if op in ("mlp", "gemm"):
        A, W, P = matrices(case, seed)
        r = tr.Reducer(case["n"], case["n"], torch.bfloat16, max_images=1, max_tokens=case["m"], max_N=1)
        return {"case": case, "A": A, "W": W, "P": P, "reducer": r}
    N, K = sizes(case)
    st = {"case": case, "N": N, "K": K if case["kept"] else None}
    rows, kept, dt = sum(N), sum(K), torch_type(case)
    if op == "select":
        st["key"], st["s"] = given_scores(rows, seed)
    else:
        st["X"], st["P"], st["Q"] = tokens(case, seed)
    if case["entry"] == "given_s":
        st["s"] = given_scores(rows, seed)[1]
    if op == "project":
        st["W"] = (randn(generator(seed + 1), case["nout"], case["d"]) / math.sqrt(case["d"])).to(dt)
    if case["entry"] == "noalloc":
        st["out"] = {"out": torch.empty(kept, case["d"], dtype=dt, device=DEV),
                     "out_idx": torch.empty(kept, dtype=torch.int32, device=DEV),
                     "out_src": torch.empty(kept, dtype=torch.uint8, device=DEV)}
        if case["scores"]:
            st["out"].update(out_h2=torch.empty(rows, device=DEV), out_s=torch.empty(rows, device=DEV))
    else:
        st["reducer"] = tr.Reducer(case["d"], case["dc"], dt, lam=case["lam"], keep_ratio=case["keep"] or None,
                                   max_images=len(N), max_tokens=rows, max_N=max(N), stride_real=case["stride_real"],
                                   shannon=case["shannon"])
    return st


def run(st):
    case, r = st["case"], st.get("reducer")
    if case["op"] == "mlp":
        post, s = r.mlp_out_cos(st["A"], st["W"], st["P"])
        return {"post": post, "s": s}
    if case["op"] == "gemm":
        return {"out": r.gemm(st["A"], st["W"])}
    N, K = st["N"], st["K"]
    if case["op"] == "select":
        idx, src = r.select(st["key"], st["s"], N, K)
        return {"idx": idx, "src": src}
    if case["op"] == "project":
        res = r.reduce_project(st["X"], st["P"], st["Q"], N, K, st["W"])
    elif case["entry"] == "given_s":
        res = r.reduce_given_s(st["X"], st["s"], N, K)
    elif case["entry"] == "noalloc":
        res = tr.reduce_noalloc(st["X"], st["P"], st["Q"], N, K, lam=case["lam"], keep_ratio=case["keep"] or None,
                                stride_real=case["stride_real"], shannon=case["shannon"], **st["out"])
    else:
        res = r.reduce(st["X"], st["P"], st["Q"], N, K, want_scores=case["scores"])
    got = {"out": res.out, "idx": res.idx, "src": res.src}
    if case["scores"]:
        got.update(h2=res.h2, s=res.s)
    return got


# ---- the same in 64 bits, in plain torch ----------------------------------------
def scores64(case, X, P, Q, chunk=4096):
    """(Stage I key, entropy, cosine) of every row."""
    key, h, s = [], [], []
    for r0 in range(0, X.shape[0], chunk):
        x = X[r0:r0 + chunk].double().abs()
        p = x / x.sum(1, keepdim=True)
        v = -torch.special.xlogy(p, p).sum(1) if case["shannon"] else -torch.log((p * p).sum(1))
        a, b = P[r0:r0 + chunk].double(), Q[r0:r0 + chunk].double()
        h.append(v)
        key.append(math.log(X.shape[1]) - v)
        s.append((a * b).sum(1) / (a.norm(dim=1) * b.norm(dim=1)))
    # repeated tokens tie exactly, whatever order torch sums each of them in
    return torch.cat(key).round(decimals=12), torch.cat(h), torch.cat(s).round(decimals=12)


def select64(case, key, s, N, K):
    """Kept token indices of each image, or None where 32-bit scores may choose otherwise."""
    idx, src, r0 = [], [], 0
    for n, k in zip(N, K):
        a, b = key[r0:r0 + n], s[r0:r0 + n]
        r0 += n
        k1 = math.floor(case["lam"] * k)
        k2 = k - k1
        order = torch.argsort(a, stable=True)
        va = a[order]
        if 0 < k1 < n and 1e-12 < va[k1] - va[k1 - 1] < 1e-5 * va[k1]:
            return None
        imp = torch.zeros(n, dtype=torch.bool, device=a.device)
        imp[order[:k1]] = True
        rem = torch.nonzero(~imp).flatten()
        rem = rem[torch.argsort(b[rem], stable=True)]
        R = n - k1
        t = max(1, R // k2) if k2 else 1
        at = torch.tensor([j * R // k2 if case["stride_real"] else j * t for j in range(k2)], dtype=torch.long, device=a.device)
        vb = b[rem]
        if 0 < k2 < R:
            gap = vb[1:] - vb[:-1]
            close = (gap > 1e-12) & (gap < 1e-7)
            near = torch.zeros(R, dtype=torch.bool, device=a.device)
            near[1:] |= close
            near[:-1] |= close
            if bool(near[at].any()):
                return None
        keep = torch.cat([torch.nonzero(imp).flatten(), rem[at]])
        keep, order = torch.sort(keep)
        idx.append(keep)
        src.append((order >= k1).to(torch.uint8))
    return idx, src


def exact(case, seed):
    if case["op"] in ("mlp", "gemm"):
        A, W, P = matrices(case, seed)
        Wt = W.double().t().contiguous()
        post = torch.cat([a.double() @ Wt for a in A.split(4096)])
        if case["op"] == "gemm":
            return {"out": post}
        P, Q = P.double(), post.to(torch.bfloat16).double()     # the cosine is of the states as stored
        return {"post": post, "s": (P * Q).sum(1) / (P.norm(dim=1) * Q.norm(dim=1))}
    N, K = sizes(case)
    if case["op"] == "select":
        key, s = (t.double() for t in given_scores(sum(N), seed))
        idx, src = select64_given(case, key, s, N, K)
        return {"idx": idx, "src": src}
    if sum(N) > 100000 and not case["scores"]:
        return None
    X, P, Q = tokens(case, seed)
    key, h, s = scores64(case, X, P, Q)
    got = {"out": None, "idx": None, "src": None}
    if case["scores"]:
        got.update(h2=h, s=s)
    if case["entry"] == "given_s":
        s = given_scores(sum(N), seed)[1].double()
    picked = select64(case, key, s, N, K)
    if picked is not None:
        starts = [sum(N[:b]) for b in range(len(N))]
        out = X[torch.cat([i + r0 for i, r0 in zip(picked[0], starts)])].double()
        if case["op"] == "project":
            W = (randn(generator(seed + 1), case["nout"], case["d"]) / math.sqrt(case["d"])).to(X.dtype)
            out = out @ W.double().t().contiguous()
        got.update(out=out, idx=torch.cat(picked[0]).to(torch.int32), src=torch.cat(picked[1]))
    return got if picked is not None or case["scores"] else None


def select64_given(case, key, s, N, K):
    """select64 on keys that both sides hold exactly: no tie is uncertain."""
    idx, src, r0 = [], [], 0
    for n, k in zip(N, K):
        one = select64(case, *(torch.unique(t[r0:r0 + n], return_inverse=True)[1].double() for t in (key, s)), [n], [k])
        idx += one[0]
        src += one[1]
        r0 += n
    return torch.cat(idx).to(torch.int32), torch.cat(src)
