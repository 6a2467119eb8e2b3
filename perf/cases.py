"""The work that a program has this library do, as cases that can be timed and compared.

A case is one call of one of the library's public entry points (the k-means + affine fit, the PCA front-end, the
inference with and without it, the sweep of the blending coefficient) on synthetic rows of a stated shape.  The shapes
are those of the workloads in ``paper_2509_26277_amd/workloads.py`` and of the paper's set-up (logits of 1000 classes,
50 principal components, ten blending coefficients, up to 256 clusters), a serving batch, and row lengths that are not
whole 16-byte groups.  The inputs follow the recipes of ``workloads.py`` and are drawn on the GPU; the parameters of an
inference case come from a short k-means on a sample of its rows, as a deployment's do (``stream``: drawn with the rows).
"""
import math

import torch

from paper_2509_26277_amd import binding

ALPHAS = [0.1 * k for k in range(1, 11)]  # the paper's grid of blending coefficients


def listed():
    return [
        # a tiny fit: nothing but launches and dependent steps
        dict(name="fit_small", kind="fit", data="mixture", dtype="f32", N=4096, D=64, K=4, iters=20),
        # calibration logits of a 1000-class network
        dict(name="fit_logits", kind="fit", data="logits", dtype="f32", N=65536, D=1000, K=16, iters=30),
        # a feature map: many short rows
        dict(name="fit_features", kind="fit", data="features", dtype="f32", N=1048576, D=256, K=32, iters=15),
        # wide bfloat16 rows, clusters of very different sizes
        dict(name="fit_wide_bf16", kind="fit", data="zipf", dtype="bf16", N=262144, D=2048, K=64, iters=20),
        # an odd row length and many clusters (the upper end of the paper's cluster counts)
        dict(name="fit_ragged", kind="fit", data="logits", dtype="f32", N=50021, D=1001, K=200, iters=20),
        # PCA of the calibration logits and their scores (first step of the paper's Algorithm 1)
        dict(name="pca_logits", kind="pca", data="logits", dtype="f32", N=65536, D=1000, p=50),
        # one batch at serving time
        dict(name="apply_batch", kind="apply", data="logits", dtype="f32", N=256, D=1000, K=50),
        # inference over wide bfloat16 rows
        dict(name="apply_wide_bf16", kind="apply", data="zipf", dtype="bf16", N=262144, D=2048, K=64),
        # inference over a long stream of rows
        dict(name="apply_stream", kind="apply", data="stream", dtype="f32", N=4194304, D=512, K=128),
        # inference over rows of an odd length
        dict(name="apply_ragged", kind="apply", data="logits", dtype="f32", N=50021, D=1001, K=50),
        # inference with the PCA front-end (the paper's Algorithm 2)
        dict(name="apply_pca_logits", kind="apply_pca", data="logits", dtype="f32", N=65536, D=1000, K=50, p=50),
        # one fitted transformation over the whole grid of blending coefficients
        dict(name="sweep_logits", kind="sweep", data="logits", dtype="f32", N=65536, D=1000, K=16),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the same ranges: any of the calls, rows of 24 .. 2048 entries, up to 2^27 entries in all (PCA: 2^26 and
    rows of up to 1024), 1 .. 256 clusters."""
    kind = rng.choice(["fit", "fit", "apply", "apply", "pca", "apply_pca", "sweep"])
    dtype = "bf16" if rng.random() < 0.25 else "f32"
    data = rng.choice(["mixture", "logits", "features", "zipf"] + (["stream"] if kind == "apply" else []))
    D = _log_int(rng, 24, 1024 if kind == "pca" else 2048)
    if rng.random() < 0.5:  # half of the row lengths as they come, half in whole 16-byte groups
        D = (D + 7) // 8 * 8
    if dtype == "bf16":
        D += D % 2
    N = _log_int(rng, 256 if kind in ("apply", "apply_pca") else 2048, min(1 << 20, (1 << (26 if kind == "pca" else 27)) // D))
    case = dict(kind=kind, data=data, dtype=dtype, N=N, D=D)
    if kind != "pca":
        case["K"] = _log_int(rng, 1, 256 if kind != "sweep" else 64)
    if kind == "fit":
        case["iters"] = rng.randint(5, 30)
    if kind in ("pca", "apply_pca"):
        case["p"] = min(D, _log_int(rng, 4, 64))
    return case


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
class _Draws:
    def __init__(self, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(int(seed) * 7919 + 12345)

    def normal(self, *shape):
        return torch.randn(*shape, generator=self.g, device="cuda")

    def uniform(self, lo, hi, *shape):
        return torch.rand(*shape, generator=self.g, device="cuda") * (hi - lo) + lo

    def exponential(self, *shape):
        return -torch.log1p(-torch.rand(*shape, generator=self.g, device="cuda").clamp_(max=1.0 - 2.0 ** -24))

    def labels(self, N, K, zipf):
        w = torch.arange(1, K + 1, device="cuda", dtype=torch.float64) ** (-1.1 if zipf else 0.0)
        edges = torch.cumsum(w / w.sum(), 0)
        u = torch.rand(N, generator=self.g, device="cuda", dtype=torch.float64)
        return torch.searchsorted(edges, u).clamp_(max=K - 1)


def _rows(d, case, components):
    """(lq, fp) of the case's shape and type; fp is None for ``stream``; the third value is what ``stream`` drew."""
    N, D, C = case["N"], case["D"], components
    data = case["data"]
    labels = d.labels(N, C, data == "zipf")
    if data == "stream":
        cent = d.normal(C, D)
        gamma, beta = d.uniform(0.8, 1.2, C, D), d.normal(C, D) * math.sqrt(0.1)
        lq = d.normal(N, D)
        lq += cent[labels]
        return lq.to(_torch_dtype(case)), None, (cent, gamma, beta)
    g, b = d.uniform(0.5, 1.5, C, D), d.normal(C, D) * math.sqrt(0.5)
    if data == "logits":  # Student-t noise with four degrees of freedom, LQ coarsely rounded
        mu = d.normal(C, D) * 3.0
        fp = d.normal(N, D)
        fp *= torch.rsqrt((d.exponential(N, D) + d.exponential(N, D)) * 0.5)
        fp += mu[labels]
        lq = g[labels] * fp + b[labels] + d.uniform(-0.5, 0.5, N, D)
    elif data == "features":  # after a ReLU, LQ on four levels
        mu = d.normal(C, D) * 2.0 - 1.0
        fp = (mu[labels] + d.normal(N, D)).clamp_(min=0.0)
        lq = g[labels] * (torch.round(fp.clamp(max=9.0) / 3.0) * 3.0) + b[labels]
    else:  # planted mixture, even or skewed component sizes
        mu = d.normal(C, D) * 2.0
        fp = mu[labels] + d.normal(N, D)
        lq = g[labels] * fp + b[labels] + 0.05 * d.normal(N, D)
    return lq.to(_torch_dtype(case)), fp.to(_torch_dtype(case)), None


def _torch_dtype(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def _one_hot(a, K):
    return torch.nn.functional.one_hot(a, K).to(torch.float64)


def _nearest(x, cent):
    """Nearest centroid per row and its squared distance, in double; the lowest index on ties."""
    s = (cent * cent).sum(1)[None, :] - 2.0 * (x @ cent.t())
    best, a = s.min(1)
    return a, (best + (x * x).sum(1)).clamp_(min=0.0)


def _means(x, a, cent):
    """Mean of every cluster's rows as the float32 values a centroid is held in; a cluster without rows keeps its own."""
    h = _one_hot(a, cent.shape[0])
    n = h.sum(0)
    m = (h.t() @ x) / n.clamp(min=1.0)[:, None]
    return torch.where(n[:, None] > 0, m, cent).float().double()


def _affine(x, y, a, K):
    h = _one_hot(a, K)
    n = h.sum(0).clamp(min=1.0)[:, None]
    mx, my = (h.t() @ x) / n, (h.t() @ y) / n
    dx, dy = x - mx[a], y - my[a]
    var, cov = (h.t() @ (dx * dx)) / n, (h.t() @ (dx * dy)) / n
    g = cov / var.clamp(min=1e-8)
    b = my - g * mx
    empty = (h.sum(0) == 0)[:, None]
    return torch.where(empty, torch.ones_like(g), g), torch.where(empty, torch.zeros_like(b), b)


def _fitted(lq, fp, K, space=None):
    """Centroids, gamma and beta of a short k-means on the first rows (``space``: their coordinates for the k-means)."""
    S = min(lq.shape[0], max(8192, 16 * K))
    x, y = lq[:S].double(), fp[:S].double()
    z = x if space is None else space[:S].double()
    cent = z[torch.arange(K, device="cuda") * S // K].float().double()
    for _ in range(6):
        cent = _means(z, _nearest(z, cent)[0], cent)
    g, b = _affine(x, y, _nearest(z, cent)[0], K)
    return cent.float().contiguous(), g.float().contiguous(), b.float().contiguous()


def _covariance(x):
    mean = x.mean(0)
    x = x - mean
    return mean, (x.t() @ x) / x.shape[0]


def _principal(cov, p):
    """Leading eigenvalues and unit directions (rows), the entry of largest magnitude positive."""
    w, v = torch.linalg.eigh(cov.cpu())
    w, v = w.flip(0)[:p], v.flip(1)[:, :p].t().contiguous()
    at = v.abs().argmax(1, keepdim=True)
    return w, v * torch.sign(torch.gather(v, 1, at))


def _leading(cov, p):
    """Nearly the leading directions of a covariance, by a few subspace iterations: what an inference case projects on."""
    cov = cov.cpu()
    q = torch.linalg.qr(cov[:, :p] + torch.eye(cov.shape[0], p, dtype=cov.dtype))[0]
    for _ in range(6):
        q = torch.linalg.qr(cov @ q)[0]
    v = torch.linalg.eigh(q.t() @ cov @ q)[1].flip(1)
    return (q @ v).t().contiguous()


def _components_of(case):
    return case.get("K", 16) if case["kind"] != "apply_pca" else 16


def prepare(case, seed):
    d = _Draws(seed)
    kind, N, D, K = case["kind"], case["N"], case["D"], case.get("K", 0)
    dt = binding.CAT_BF16 if case["dtype"] == "bf16" else binding.CAT_F32
    lq, fp, drawn = _rows(d, case, _components_of(case))
    lq = lq.contiguous()
    s = dict(kind=kind, lq=lq, seed=int(seed))
    if kind == "fit":
        s.update(fp=fp, K=K, iters=case["iters"])
        s["workspace"] = torch.empty(binding.cat_fit_workspace_bytes(N, D, K, dt), dtype=torch.uint8, device="cuda")
    elif kind == "pca":
        s["p"] = case["p"]
        need = binding.load_library().cat_pca_workspace_bytes(N, D, case["p"], dt)
        s["workspace"] = torch.empty(max(256, need), dtype=torch.uint8, device="cuda")
    elif kind == "apply":
        s["params"] = drawn if drawn is not None else _fitted(lq, fp, min(K, N))
        s["out"] = torch.empty_like(lq)
        need = binding.cat_apply_workspace_bytes(N, D, s["params"][0].shape[0], dt)
        s["workspace"] = torch.empty(max(256, need), dtype=torch.uint8, device="cuda")
    elif kind == "apply_pca":
        sample = lq[:16384].double()
        mean, cov = _covariance(sample)
        comps = _leading(cov, case["p"]).cuda()
        mean, comps = mean.float(), comps.float().contiguous()
        z = (sample - mean.double()) @ comps.double().t()
        cz, g, b = _fitted(lq[:16384], fp[:16384], min(K, N), z)
        s["params"] = (mean, comps, cz, g, b)
        s["out"] = torch.empty_like(lq)
        need = binding.load_library().cat_apply_pca_workspace_bytes(N, D, cz.shape[0], case["p"], dt)
        s["workspace"] = torch.empty(max(256, need), dtype=torch.uint8, device="cuda")
    else:
        cent, g, b = _fitted(lq, fp, min(K, N))
        a = torch.cat([_nearest(c.double(), cent.double())[0] for c in lq.split(65536)]).int()
        s.update(fp=fp, gamma=g, beta=b, assignments=a, labels=fp.float().argmax(1).int())
    return s


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
def run(s):
    kind = s["kind"]
    if kind == "fit":
        r = binding.cat_fit(s["lq"], s["fp"], s["K"], s["iters"], seed=s["seed"], workspace=s["workspace"])
        return {k: r[k] for k in ("centroids", "gamma", "beta", "assignments", "counts", "inertia")}
    if kind == "pca":
        mean, comps, evals = binding.cat_pca_fit(s["lq"], s["p"], workspace=s["workspace"])
        return dict(mean=mean, components=comps, eigenvalues=evals, scores=binding.cat_pca_project(s["lq"], mean, comps))
    if kind == "apply":
        out, a = binding.cat_apply(s["lq"], *s["params"], alpha=0.6, out=s["out"], workspace=s["workspace"])
        return dict(corrected=out, assignments=a)
    if kind == "apply_pca":
        out, a = binding.cat_apply_pca(s["lq"], *s["params"], alpha=0.6, out=s["out"], workspace=s["workspace"])
        return dict(corrected=out, assignments=a)
    r = binding.cat_alpha_sweep(s["lq"], s["assignments"], s["gamma"], s["beta"], ALPHAS, fp=s["fp"], labels=s["labels"])
    return dict(hits=r["hits"], sq_err=r["sq_err"], moments=r["moments"])


def work(case):
    """Rows read once and results written once; the products of the contractions (each assignment pass of a fit is one)."""
    kind, N, D, K, p = case["kind"], case["N"], case["D"], case.get("K", 0), case.get("p", 0)
    e = 2 if case["dtype"] == "bf16" else 4
    rows = N * D * e
    if kind == "fit":
        return dict(bytes=2 * rows + 4 * N + 12 * K * D, flops=2.0 * N * D * K * (case["iters"] + 1) + 12.0 * N * D)
    if kind == "pca":
        return dict(bytes=rows + 4 * N * p + 4 * (p + 1) * D, flops=1.0 * N * D * (D + 1) + 2.0 * N * D * p + 4.0 * D ** 3 / 3)
    if kind == "apply":
        return dict(bytes=2 * rows + 4 * N + 12 * K * D, flops=2.0 * N * D * K + 2.0 * N * D)
    if kind == "apply_pca":
        return dict(bytes=2 * rows + 4 * N + 4 * (2 * K + p) * D, flops=2.0 * N * (D * p + p * K + D))
    return dict(bytes=2 * rows + 8 * N + 8 * K * D, flops=2.0 * N * D * (len(ALPHAS) + 3))


def tolerance(case):
    """Rows, parameters and results are float32 (bfloat16 rows: the corrected rows are rounded to bfloat16 once), sums
    are in double.  Against exact() every float32 output measures 2e-8 .. 5e-8, the objective of a fit 4e-8 .. 2e-6 (the
    sum of |x|^2 + score, both float32), the PCA scores 5e-7 (float32 accumulation over a row)."""
    if case["kind"] == "fit":
        return dict(rel=1e-5, max=1e-3, differ=1e-4)
    if case["kind"] in ("apply", "apply_pca"):
        # one fused multiply-add per entry; a row whose two nearest centroids are equidistant to rounding may go either way
        return dict(rel=4e-3, max=0.02, differ=1e-4) if case["dtype"] == "bf16" else dict(rel=1e-6, max=1e-4, differ=1e-4)
    if case["kind"] == "pca":
        return dict(rel=2e-6, max=1e-3)
    return dict(rel=1e-6, max=1e-5)


# ---------------------------------------------------------------------------
# the same in 64 bits
# ---------------------------------------------------------------------------
_GOLDEN, _MASK = 0x9E3779B97F4A7C15, (1 << 64) - 1


def _seeded_rows(N, K, seed):
    """The distinct rows a fit starts from: SplitMix64 outputs modulo N, those already taken skipped."""
    taken, t = [], 0
    while len(taken) < K:
        z = (seed + (t + 1) * _GOLDEN) & _MASK
        z = ((z ^ (z >> 30)) * 0xBF58476D1CE4E5B9) & _MASK
        z = ((z ^ (z >> 27)) * 0x94D049BB133111EB) & _MASK
        i = (z ^ (z >> 31)) % N
        t += 1
        if i not in taken:
            taken.append(i)
    return taken


def exact(case, seed):
    s = prepare(case, seed)
    kind, x = s["kind"], s["lq"].double() if case["kind"] != "apply" else None
    if kind == "fit":
        K = s["K"]
        cent = x[torch.tensor(_seeded_rows(x.shape[0], K, s["seed"]), device="cuda")]
        inertia = []
        for _ in range(s["iters"]):
            a, d2 = _nearest(x, cent)
            inertia.append(d2.sum())
            cent = _means(x, a, cent)
        a, d2 = _nearest(x, cent)
        inertia.append(d2.sum())
        g, b = _affine(x, s["fp"].double(), a, K)
        return dict(centroids=cent, gamma=g, beta=b, assignments=a.int(), counts=torch.bincount(a, minlength=K).int(),
                    inertia=torch.stack(inertia))
    if kind == "pca":
        mean, cov = _covariance(x)
        w, v = _principal(cov, s["p"])
        v = v.cuda()
        return dict(mean=mean, components=v, eigenvalues=w.cuda(), scores=(x - mean) @ v.t())
    if kind == "apply":
        cent, g, b = (t.double() for t in s["params"])
        out = torch.empty(s["lq"].shape, dtype=torch.float64, device="cuda")
        labels = []
        for lo in range(0, out.shape[0], 262144):
            c = s["lq"][lo:lo + 262144].double()
            a = _nearest(c, cent)[0]
            out[lo:lo + 262144] = c + 0.6 * (g[a] * c + b[a] - c)
            labels.append(a.int())
        return dict(corrected=out, assignments=torch.cat(labels))
    if kind == "apply_pca":
        mean, comps, cz, g, b = (t.double() for t in s["params"])
        a = _nearest((x - mean) @ comps.t(), cz)[0]
        return dict(corrected=x + 0.6 * (g[a] * x + b[a] - x), assignments=a.int())
    fp, a = s["fp"].double(), s["assignments"].long()
    t = (s["gamma"].double() - 1.0)[a] * x + s["beta"].double()[a]
    hits = [((x + al * t).argmax(1) == s["labels"]).sum() for al in ALPHAS]
    r = x - fp
    m = torch.stack([(r * r).sum(), (r * t).sum(), (t * t).sum()])
    al = torch.tensor(ALPHAS, dtype=torch.float64, device="cuda")
    return dict(hits=torch.stack(hits), sq_err=m[0] + 2 * al * m[1] + al * al * m[2], moments=m)
