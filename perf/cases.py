"""The work a program that uses this library has it do, as measurable cases.

A case is one call sequence through the public binding on one problem:

  step     one training iteration: ``ep_step`` on the next batch of an epoch's
           permutation, then ``ep_get_alpha`` (the updated model)
  predict  ``ep_predict`` on n_z held-out rows
  serve    ``ep_predict_noalloc`` on n_z rows, the entry point of serving loops
  setup    ``ep_setup`` + ``ep_get_preconditioner``, once per trained model

Shapes are those of ``synth/configs.py`` (the sizes of the paper's data sets),
of the studies and the share of a centre split in ``bench.py``, and of the
small ragged problems of the tests. Data follow the same laws as the synthetic
workloads, so that typical kernel values are 0.1 to 0.4 as in those. All
inputs are float32, the only type the interface takes.
"""

import math

import torch

import paper_1806_06144_amd as ep

KERNELS = ("gaussian", "laplacian")


def _case(name, do, n, d, l, law, kernel, bw, s, k, m):
    """m: batch rows of a step, rows predicted otherwise."""
    return dict(name=name, do=do, n=n, d=d, l=l, law=law, kernel=kernel, bw=bw, s=s, k=k, m=m)


def listed():
    return [
        # a toy problem, as in a notebook or a test: launches and latency
        _case("step tiny", "step", 2000, 64, 4, "normal_scaled", "gaussian", 1.0, 500, 20, 256),
        # digits, Gaussian kernel, at the analytic batch size
        _case("step mnist", "step", 60000, 784, 10, "sparse80", "gaussian", 5.0, 4000, 160, 1310),
        # colour images, Laplacian kernel: long rows, few labels
        _case("step cifar", "step", 50000, 3072, 10, "uniform", "laplacian", 10.0, 4000, 200, 3039),
        # speech frames: many centres, short rows, 144 labels
        _case("step timit", "step", 1100000, 440, 144, "normal", "gaussian", 15.0, 12000, 160, 1257),
        # the headline workload: 1000 labels, the largest problem
        _case("step imagenet", "step", 1280000, 2048, 1000, "halfnormal50", "gaussian", 20.0,
              20000, 200, 3561),
        # an epoch's short last batch on one GPU's share of an 8-way centre split
        _case("step imagenet share, last batch", "step", 160000, 2048, 1000, "halfnormal50",
              "gaussian", 20.0, 12000, 200, 1601),
        # plain kernel SGD (rank 0) with the small batch it needs
        _case("step sgd 64", "step", 100000, 440, 144, "normal", "gaussian", 15.0, 4000, 0, 64),
        # features with a constant column appended: odd rows, nothing divides anything
        _case("step odd", "step", 50001, 785, 11, "sparse80", "laplacian", 4.0, 1999, 61, 1001),
        # a held-out set after training
        _case("predict mnist test set", "predict", 60000, 784, 10, "sparse80", "gaussian", 5.0,
              4000, 160, 10000),
        # a served request: one row, and a small group of rows
        _case("serve 1 mnist", "serve", 60000, 784, 10, "sparse80", "gaussian", 5.0, 4000, 160, 1),
        _case("serve 48 timit", "serve", 1100000, 440, 144, "normal", "gaussian", 15.0, 4000, 40, 48),
        # the once-per-model preparation at the digits' size
        _case("setup mnist", "setup", 60000, 784, 10, "sparse80", "gaussian", 5.0, 4000, 160, 0),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the listed ranges: n 2000 .. 1.28 M, d 16 .. 3072, l 1 .. 1000,
    batches of 16 .. 4096 rows, single rows to 10000 for prediction."""
    while True:
        do = rng.choice(["step"] * 4 + ["predict"] * 2 + ["serve"] * 2 + ["setup"])
        n = _log_int(rng, 2000, 1280000)
        d = _log_int(rng, 16, 3072)
        l = rng.choice([1, 2, 10, 100]) if rng.random() < 0.3 else _log_int(rng, 1, 1000)
        if rng.random() < 0.6:            # most feature sets have rows of a multiple of 4
            d = max(16, d // 4 * 4)
        law = rng.choice(["normal", "normal_scaled", "uniform", "sparse80", "halfnormal50"])
        kernel = rng.choice(KERNELS)
        s = min(n // 2, _log_int(rng, 200, 8000))
        k = 0 if rng.random() < 0.15 else _log_int(rng, 4, max(5, min(200, s // 8)))
        m = {"step": _log_int(rng, 16, 4096), "predict": _log_int(rng, 100, 10000),
             "serve": _log_int(rng, 1, 256), "setup": 0}[do]
        m = min(m, n)
        if 2.0 * m * n * (d + l) > 1.0e13 or n * (d + 2 * l) > 2.5e9:
            continue
        d2 = 2.0 * d * {"normal": 1.0, "normal_scaled": 1.0 / d, "uniform": 1.0 / 12,
                        "sparse80": 0.0567, "halfnormal50": 0.341}[law]
        bw = math.sqrt(d2 / 3.5) if kernel == "gaussian" else math.sqrt(d2) / 2.2
        bw = float(torch.tensor(round(bw, 4), dtype=torch.float32))
        return dict(do=do, n=n, d=d, l=l, law=law, kernel=kernel, bw=bw, s=s, k=k, m=m)


def _features(rows, d, law, gen):
    x = torch.empty((rows, d), dtype=torch.float32, device="cuda")
    step = max(1, (1 << 28) // d)
    for i in range(0, rows, step):        # by pieces, so that masks stay small
        p = x[i:i + step]
        if law in ("normal", "normal_scaled", "halfnormal50"):
            p.normal_(generator=gen)
            if law == "normal_scaled":
                p.mul_(1.0 / math.sqrt(d))
        else:
            p.uniform_(generator=gen)
        if law == "halfnormal50":
            p.abs_()
        if law in ("halfnormal50", "sparse80"):
            keep = 0.5 if law == "halfnormal50" else 0.2
            p.mul_(torch.rand(p.shape, device="cuda", generator=gen) < keep)
    return x


BATCHES = 4          # batches of the epoch's permutation that a state holds


def _inputs(case, seed):
    """Everything a program has in hand, from the seed alone."""
    n, d, l, s, m = (case[x] for x in ("n", "d", "l", "s", "m"))
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    u = {"X": _features(n, d, case["law"], gen)}
    perm = torch.randperm(n, device="cuda", generator=gen)
    u["r"] = perm[torch.randperm(n, device="cuda", generator=gen)[:s]].cpu().numpy()
    if case["do"] == "setup":
        return u
    u["alpha"] = torch.randn((n, l), device="cuda", generator=gen).mul_(1.0 / math.sqrt(n))
    if case["do"] == "step":
        nb = max(1, min(BATCHES, n // m))
        u["t"] = [perm[i * m:(i + 1) * m].contiguous() for i in range(nb)]
        u["y"] = []
        for _ in range(nb):               # one-hot labels
            y = torch.zeros((m, l), device="cuda")
            y[torch.arange(m, device="cuda"),
              torch.randint(0, l, (m,), device="cuda", generator=gen)] = 1.0
            u["y"].append(y)
    else:
        u["Z"] = _features(m, d, case["law"], gen)
    return u


class _Model:
    """A context that lives as long as the state that holds it."""

    def __init__(self, X, case, r):
        self.X = X                        # borrowed by the context
        self.ctx, self.info = ep.ep_setup(X, case["n"], case["d"], case["l"], case["kernel"],
                                          case["bw"], case["s"], case["k"], sub_idx=r)

    def __del__(self):
        ctx, self.ctx = getattr(self, "ctx", None), None
        if ctx is not None:
            ep.ep_destroy(ctx)


def prepare(case, seed):
    u = _inputs(case, seed)
    st = {"case": case}
    if case["do"] == "setup":
        st.update(X=u["X"], r=u["r"])
        return st
    st["model"] = _Model(u["X"], case, u["r"])
    ep.ep_set_alpha(st["model"].ctx, u["alpha"])
    ep.ep_sync(st["model"].ctx)
    out_rows = case["m"]
    st["out"] = torch.empty((out_rows, case["l"]), dtype=torch.float32, device="cuda")
    if case["do"] == "step":
        st.update(t=u["t"], y=u["y"], at=0)
        st["alpha"] = torch.empty((case["n"], case["l"]), dtype=torch.float32, device="cuda")
    else:
        st["Z"] = u["Z"]
    return st


def run(st):
    case = st["case"]
    if case["do"] == "setup":
        model = _Model(st["X"], case, st["r"])
        sigma, D, _, r = ep.ep_get_preconditioner(model.ctx, model.info)
        # (eigenvectors are determined up to sign and, in clusters, rotation;
        # beta is formed from them, and the steps' outputs depend on them)
        return {"sigma": sigma, "D": D, "r": r, "beta": model.info.beta,
                "m_star": model.info.m_star}
    ctx = st["model"].ctx
    if case["do"] == "step":
        i = st["at"]
        st["at"] = (i + 1) % len(st["t"])
        ep.ep_step(ctx, st["t"][i], case["m"], st["y"][i], st["out"])
        ep.ep_get_alpha(ctx, st["alpha"])
        return {"f": st["out"], "alpha": st["alpha"]}
    call = ep.ep_predict if case["do"] == "predict" else ep.ep_predict_noalloc
    call(ctx, st["Z"], case["m"], st["out"])
    return st["out"]


def work(case):
    """Each input read once and each output written once: X, alpha, the rows
    and labels of the call, the results; for a step also the eigenvectors and
    the updated model. Kernel entries cost 2 d flops, their contraction 2 l;
    the correction its cheaper order of products."""
    n, d, l, s, k, m = (case[x] for x in ("n", "d", "l", "s", "k", "m"))
    if case["do"] == "setup":
        # K_s (symmetric: half its entries) and a rank k+1 iteration's least:
        # one product of K_s with a block of k+1 columns
        return {"bytes": 4.0 * (n * d + s * d + s * k) + 8.0 * s * s,
                "flops": 1.0 * s * s * d + 2.0 * s * s * (k + 1)}
    b = 4.0 * (n * d + n * l + m * d + m * l)
    f = 2.0 * m * n * (d + l)
    if case["do"] == "step":
        b += 4.0 * (n * l + m * l + s * k) + 8.0 * (m + s)
        if k:
            f += 2.0 * min(s * m * l + k * s * l, k * s * m + k * m * l) + 2.0 * k * s * l
    return {"bytes": b, "flops": f}


def tolerance(case):
    """Float32 storage and accumulation: distances from |x|^2 + |z|^2 - 2 x.z,
    sums of n terms in any order. Setup is float64."""
    if case["do"] == "setup":
        return {"rel": 1e-9, "max": 1e-6}
    return {"rel": 4e-5}


def _kernel64(A, B, case):
    """k(a, b) in float64; |a|^2 + |b|^2 - 2 a.b, clamped at 0."""
    d2 = torch.matmul(A, B.T).mul_(-2.0)
    d2 += (A * A).sum(1)[:, None]
    d2 += (B * B).sum(1)[None, :]
    d2.clamp_(min=0.0)
    bw = float(torch.tensor(case["bw"], dtype=torch.float32))
    if case["kernel"] == "gaussian":
        return d2.mul_(-1.0 / (2.0 * bw * bw)).exp_()
    return d2.sqrt_().mul_(-1.0 / bw).exp_()


def _predict64(X, alpha, Q, case, ids=None):
    """sum_j k(q_i, x_j) alpha_j; k = 1 where row i is centre ids[i]."""
    f = torch.zeros((Q.shape[0], alpha.shape[1]), dtype=torch.float64, device="cuda")
    Qd = Q.double()
    step = max(256, (1 << 28) // max(Q.shape[0], X.shape[1], alpha.shape[1]))
    for c in range(0, X.shape[0], step):
        K = _kernel64(Qd, X[c:c + step].double(), case)
        if ids is not None:
            here = (ids >= c) & (ids < c + K.shape[1])
            K[here.nonzero()[:, 0], ids[here] - c] = 1.0
        f += torch.matmul(K, alpha[c:c + step].double())
    return f


def _eigen64(X, r, case):
    """sigma_1 .. sigma_{k+1}, the k eigenvectors and D of the subsample."""
    k = case["k"]
    K = _kernel64(X[r].double(), X[r].double(), case)
    K.fill_diagonal_(1.0)
    w, V = torch.linalg.eigh(K)
    w, V = w.flip(0)[:k + 1], V.flip(1)[:, :k]
    D = (1.0 - w[k] / w[:k]) / w[:k]
    beta = float((1.0 - (V * V) @ (w[:k] - w[k])).max()) if k else 1.0
    return w, V, D, beta


def exact(case, seed):
    u = _inputs(case, seed)
    X = u["X"]
    if case["do"] in ("predict", "serve"):
        return _predict64(X, u["alpha"], u["Z"], case)
    if case["s"] > 12000:
        return None                       # the eigensolve alone would take too long
    r = torch.from_numpy(u["r"]).cuda()
    w, V, D, beta = _eigen64(X, r, case)
    lam = float(w[case["k"]]) / case["s"]
    if case["do"] == "setup":
        return {"sigma": w.cpu().numpy(), "D": D.cpu().numpy(), "r": u["r"], "beta": beta,
                "m_star": beta / lam}
    t, y, m = u["t"][0], u["y"][0].double(), case["m"]
    f = _predict64(X, u["alpha"], X[t], case, ids=t)
    R = f - y
    c = 1.0 / (beta + (m - 1) * lam)
    alpha = u["alpha"].double()
    alpha[t] -= c * R
    if case["k"]:
        K = _kernel64(X[r].double(), X[t].double(), case)
        K[r[:, None] == t[None, :]] = 1.0
        alpha[r] += c * torch.matmul(V, D[:, None] * torch.matmul(V.T.contiguous(), torch.matmul(K, R)))
    return {"f": f, "alpha": alpha}
