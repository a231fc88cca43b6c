"""The calls that a reconstruction program makes, at the sizes it makes them, for timing.

Each case is one pass through the public binding (paper_1307_5824_amd.firm):

  kernel       plan.kernel_precompute: gridding of the sample points, FFTs, circulant spectrum
  backproject  plan.backproject: A*b of complex slices
  project      plan.forward_project: slices of a volume
  images       plan.images_to_slices: step 1 on real-space images
  apply        plan.apply_AtA / apply_AtA_f64: one Toeplitz product
  cg           plan.cg_solve for a fixed number of iterations (the paper regularizes by stopping early)
  learned_pcg  features, network, Chan's spectrum, diagonal, then preconditioned CG
  train        one batch of the preconditioner's training: unrolled PCG gradients, then the network's
  reconstruct  kernel, back-projection and CG of a small volume, end to end

Views, shifts and CTFs are drawn by paper_1307_5824_amd.synth (the workloads' own recipes); slices,
images, volumes and kernels are drawn here with torch.  `exact` gives the same results in 64 bits
with plain torch.
"""
import math

import numpy as np
import torch

DEV = "cuda"
LAM = 1e-2            # lambda relative to Ker(0), as the workloads take it (a case may give its own)
EXACT_FLOPS = 1.5e14  # the most that a 64-bit direct sum may cost


def listed():
    return [
        # a first look at a small particle: the latency of every launch and host wait of the chain
        {"name": "reconstruct_16", "op": "reconstruct", "N": 16, "M": 200, "views": "haar", "groups": 0, "shifts": False,
         "W": 7, "iters": 4},
        # the kernel of the mid workload; the preconditioner's training builds thousands of these
        {"name": "kernel_64", "op": "kernel", "N": 64, "M": 10000, "views": "haar", "groups": 10, "W": 7},
        # the kernel of the headline workload: once per reconstruction, its largest part with A*b
        {"name": "kernel_256", "op": "kernel", "N": 256, "M": 100000, "views": "vmf", "groups": 50, "W": 7},
        # A*b at the mid size, with a ragged number of views
        {"name": "backproject_64", "op": "backproject", "N": 64, "M": 9973, "views": "haar", "groups": 10, "shifts": True,
         "W": 7},
        # A*b at the headline size, half its views (20 GB of slices)
        {"name": "backproject_256", "op": "backproject", "N": 256, "M": 50000, "views": "vmf", "groups": 50,
         "shifts": True, "W": 7},
        # the data residual of a reconstruction: a conical tilt series at the headline size
        {"name": "project_256", "op": "project", "N": 256, "M": 20000, "views": "rct", "groups": 3, "shifts": True,
         "W": 7},
        # step 1 on recorded images of the uneven workload's size
        {"name": "images_128", "op": "images", "N": 128, "M": 10007},
        # one product of a small volume: launches and drains
        {"name": "apply_32", "op": "apply", "N": 32, "dtype": "f32"},
        # one product at the headline size: the step that CG repeats
        {"name": "apply_256", "op": "apply", "N": 256, "dtype": "f32"},
        # CG of the uneven workload's size, stopped early (before FP32 iterates lose orthogonality and
        # with it their distance to the 64-bit ones)
        {"name": "cg_128", "op": "cg", "N": 128, "precision": 0, "iters": 10},
        # inference of the preconditioner and PCG at the headline size
        {"name": "learned_pcg_256", "op": "learned_pcg", "N": 256, "iters": 25},
        # one batch of the preconditioner's training
        {"name": "train_64", "op": "train", "N": 64, "batch": 8, "k": 32},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _lam(rng):
    return round(math.exp(rng.uniform(math.log(3e-3), math.log(1e-1))), 6)


def draw(rng):
    op = rng.choice(["kernel", "kernel", "backproject", "backproject", "project", "project", "images", "apply", "cg",
                     "learned_pcg", "train", "reconstruct"])
    if op in ("kernel", "backproject", "project"):
        N = rng.choice([16, 32, 64, 128, 256])
        # N = 256 up to the listed cases' sizes, smaller volumes up to the workloads' view counts
        most = {16: 20000, 32: 50000, 64: 50000, 128: 50000,
                256: {"kernel": 100000, "backproject": 50000, "project": 20000}[op]}[N]
        c = {"op": op, "N": N, "M": _log_int(rng, 30, most), "views": rng.choice(["haar", "vmf", "rct"]),
             "groups": rng.choice([0, 1, 3, 10, 50]), "W": rng.choice([7, 7, 7, 7, 6, 8])}
        if op != "kernel":
            c["shifts"] = rng.random() < 0.7
        return c
    if op == "images":
        N = rng.choice([16, 32, 64, 128, 256])
        return {"op": op, "N": N, "M": _log_int(rng, 30, min(50000, 10007 * 128 * 128 // (N * N)))}
    if op == "apply":
        return {"op": op, "N": rng.choice([8, 16, 32, 64, 128, 256]), "dtype": rng.choice(["f32", "f32", "f64"]),
                "lam": _lam(rng)}
    if op == "cg":
        return {"op": op, "N": rng.choice([16, 32, 64, 128, 256]), "precision": rng.choice([0, 0, 2]),
                "iters": rng.randint(3, 10), "lam": _lam(rng)}
    if op == "learned_pcg":
        return {"op": op, "N": rng.choice([64, 128, 256]), "iters": rng.randint(5, 25), "lam": _lam(rng)}
    if op == "train":
        return {"op": op, "N": 64, "batch": rng.randint(1, 8), "k": rng.randint(8, 32)}
    return {"op": op, "N": rng.choice([8, 16, 32]), "M": _log_int(rng, 50, 2000), "views": rng.choice(["haar", "vmf"]),
            "groups": rng.choice([0, 3]), "shifts": rng.random() < 0.5, "W": 7, "iters": rng.randint(2, 4)}


# ------------------------------------------------------------------ inputs --

def _seeds(seed):
    return np.random.SeedSequence([13075824, int(seed)]).spawn(3)


def _gen(seed, what=0):
    return torch.Generator(device=DEV).manual_seed(int(seed) * 16 + what)


def geometry(case, seed):
    """(rotations, shifts, groups, table) of a case, as the workloads draw them."""
    from paper_1307_5824_amd import synth
    N, M = case["N"], case["M"]
    rr, rs, rc = (np.random.default_rng(s) for s in _seeds(seed))
    if case["views"] == "rct":
        R = synth.rct_rotations(M, 60.0, rr)
    else:
        R = synth.mixed_rotations(M, 10.0 if case["views"] == "vmf" else 0.0, 0.0, rr)
    shifts = rs.uniform(-2.0, 2.0, size=(M, 2)) if case.get("shifts") else None
    groups = table = None
    if case["groups"]:
        table = synth.ctf_table(N, synth.defoci(case["groups"], rc))
        groups = rc.integers(0, case["groups"], size=M).astype(np.int32)
    return R, shifts, groups, table


def disk(N):
    """k1, k2 of the disk points in the canonical order (k1, then k2, ascending)."""
    k = np.arange(-(N // 2), N // 2 + 1)
    k1, k2 = (a.ravel() for a in np.meshgrid(k, k, indexing="ij"))
    keep = 4 * (k1 * k1 + k2 * k2) <= N * N
    return k1[keep], k2[keep]


def slices(N, M, seed):
    """Noisy slices of real images: strong at low frequencies, white noise everywhere, b(-k) = conj b(k)."""
    k1, k2 = disk(N)
    q = torch.as_tensor(k1 * k1 + k2 * k2, dtype=torch.float32, device=DEV)
    env = 1.0 + 20.0 * torch.exp(-q / (2 * (0.08 * N) ** 2))
    g = _gen(seed, 1)
    b = torch.empty((M, k1.size), dtype=torch.complex64, device=DEV)
    step = max(1, (1 << 27) // k1.size)
    for a in range(0, M, step):
        z = torch.randn((min(M, a + step) - a, k1.size), dtype=torch.complex64, device=DEV, generator=g)
        b[a:a + step] = (z + z.flip(1).conj()) * env
    return b


def blobs(N, seed, dtype=torch.float32):
    """A volume of Gaussian blobs plus a little white noise."""
    g = _gen(seed, 2)
    n = torch.arange(N, device=DEV, dtype=torch.float32) - N // 2
    V = 0.02 * torch.randn((N, N, N), device=DEV, generator=g)
    c = (torch.rand((12, 3), device=DEV, generator=g) - 0.5) * (0.5 * N)
    s = (0.05 + 0.1 * torch.rand((12,), device=DEV, generator=g)) * N
    for i in range(12):
        e = [torch.exp(-(n - c[i, d]) ** 2 / (2 * s[i] ** 2)) for d in range(3)]
        V += e[0][:, None, None] * e[1][None, :, None] * e[2][None, None, :]
    return V.to(dtype)


def kernel(N, seed):
    """A kernel of the shape that uneven views give, in centred order: the sampling density falls as
    1 / |q|, is low along one axis, and carries a CTF's rings; positive spectrum, Ker(0) near 1e4 N^2."""
    g = torch.Generator().manual_seed(int(seed))
    a, f, w = (float(v) for v in torch.rand(3, generator=g))
    q = torch.fft.fftfreq(2 * N, d=1.0 / (2 * N), device=DEV, dtype=torch.float64)
    r2 = q[:, None, None] ** 2 + q[None, :, None] ** 2 + q[None, None, :] ** 2
    r = r2.sqrt().clamp_(min=1.0)
    u2 = q[None, None, :] ** 2 / r2.clamp(min=1.0)
    S = (0.05 + torch.exp(-(2 + 4 * a) * u2)) / r
    S *= 1.02 - torch.cos((4 + 6 * f) * math.pi * r2 / (N * N) + w)
    S *= 1.0 / (1.0 + torch.exp((r - N) / 2.0))  # nothing beyond the disk
    k = torch.fft.ifftn(S).real
    k *= 1e4 * N * N / float(k[0, 0, 0])
    k = torch.fft.fftshift(k)
    k[0] = 0
    k[:, 0] = 0
    k[:, :, 0] = 0
    return k.float().contiguous()


def _few_views(firm, N, **kw):
    """A plan whose kernel is set from outside: its views do not matter."""
    return firm.Plan(N, np.eye(3)[None], lambda_relative=1, **kw)


def prepare(case, seed):
    from paper_1307_5824_amd import firm
    op, N = case["op"], case["N"]
    s = {"case": case}
    if op in ("kernel", "backproject", "project", "reconstruct"):
        R, shifts, groups, table = geometry(case, seed)
        s["plan"] = firm.Plan(N, R, shifts, groups, table, kb_width=case["W"], lambda_relative=1)
        if op in ("backproject", "reconstruct"):
            s["b"] = slices(N, case["M"], seed)
        if op == "project":
            s["V"] = blobs(N, seed)
    elif op == "images":
        s["plan"] = firm.Plan(N, np.broadcast_to(np.eye(3), (case["M"], 3, 3)))
        s["images"] = images(case, seed)
    elif op == "train":
        from paper_1307_5824_amd import train_precond
        s["plan"] = _few_views(firm, N)
        s["net"] = firm.PCNet(max_batch=8)
        s["net"].set_params(train_precond.load_weights())
        s["ker"] = [kernel(N, seed * 64 + j) for j in range(case["batch"])]
        s["ker0"] = np.array([float(k[N, N, N]) for k in s["ker"]])
        feats, ts = [], []
        for k in s["ker"]:
            s["plan"].kernel_set(k)
            feats.append(s["plan"].kernel_features(LAM))
            ts.append(s["plan"].chan_spectrum(LAM))
        s["feat"], s["t"] = torch.stack(feats), torch.stack(ts)
        s["probes"] = torch.randn((case["batch"], 1, N, N, N), device=DEV, generator=_gen(seed))
    else:
        dtype = torch.float64 if case.get("dtype") == "f64" else torch.float32
        s["plan"] = _few_views(firm, N, precision=case.get("precision", 0))
        s["plan"].kernel_set(kernel(N, seed))
        if op == "apply":
            s["x"] = blobs(N, seed, dtype)
        else:
            s["atb"] = torch.randn((N, N, N), device=DEV, generator=_gen(seed))
        if op == "learned_pcg":
            from paper_1307_5824_amd import train_precond
            s["net"] = firm.PCNet(max_batch=1)
            s["net"].set_params(train_precond.load_weights())
    return s


def images(case, seed):
    N, M = case["N"], case["M"]
    x = torch.arange(N, device=DEV) - N // 2
    soft = 4 * torch.exp(-(x[:, None] ** 2 + x[None, :] ** 2) / (2 * (0.15 * N) ** 2))
    return torch.randn((M, N, N), device=DEV, generator=_gen(seed)) + soft


# -------------------------------------------------------------------- runs --

def run(s):
    from paper_1307_5824_amd import firm
    case, plan = s["case"], s["plan"]
    op, N, lam = case["op"], case["N"], case.get("lam", LAM)
    if op == "kernel":
        plan.kernel_precompute()
        return plan.kernel_get()
    if op == "backproject":
        return plan.backproject(s["b"])
    if op == "project":
        return plan.forward_project(s["V"])
    if op == "images":
        return plan.images_to_slices(s["images"])
    if op == "apply":
        return plan.apply_AtA_f64(s["x"], lam) if case["dtype"] == "f64" else plan.apply_AtA(s["x"], lam)
    if op == "cg":
        return plan.cg_solve(s["atb"], lam, 1e-12, case["iters"])[0]
    if op == "learned_pcg":
        feat = plan.kernel_features(lam, res=firm.inference_res(N))
        t = plan.chan_spectrum(lam)
        d = plan.precond_from_output(s["net"].forward(feat[None])[0], t)
        x, _ = plan.cg_solve(s["atb"], lam, 1e-12, case["iters"], precond=d)
        return {"x": x, "d": d, "t": t}
    if op == "train":
        net, loss, G = s["net"], [], []
        for j, ker in enumerate(s["ker"]):
            plan.kernel_set(ker)
            d = plan.precond_from_output(net.forward(s["feat"][j][None])[0], s["t"][j])
            v, g = plan.pcg_unrolled(d, s["probes"][j], case["k"], lam)
            loss.append(v)
            G.append(g)
        G = torch.stack(G)
        _, grad = net.loss_grad(s["feat"], N, s["t"], G, ker0=s["ker0"], objective="logd")
        return {"loss": np.array(loss), "G": G, "grad": grad}
    plan.kernel_precompute()
    atb = plan.backproject(s["b"])
    x, _ = plan.cg_solve(atb, lam, 1e-12, case["iters"])
    return {"ker": plan.kernel_get(), "atb": atb, "x": x}


# ------------------------------------------------------------- what it needs --

def points(N):
    """Disk points of a slice."""
    k1, _ = disk(N)
    return k1.size


def _fft(n, real=True):
    """Operations of one transform of n points."""
    return (2.5 if real else 5.0) * n * math.log2(n)


def _solve_work(N, iters):
    n3 = N ** 3
    return {"bytes": iters * (4 * n3 * 2 + 4 * (2 * N) ** 2 * (N + 1)), "flops": iters * 2 * _fft((2 * N) ** 3)}


def work(case):
    op, N, W = case["op"], case["N"], case.get("W", 7)
    n3 = N ** 3
    if op in ("kernel", "backproject", "project", "reconstruct"):
        M = case["M"]
        half = M * (points(N) - 1) / 2
        ker = {"bytes": 72 * M + 4 * 8 * n3, "flops": half * 2 * W ** 3 + _fft((4 * N) ** 3) + _fft((2 * N) ** 3)}
        atb = {"bytes": 8 * M * points(N) + 72 * M + 4 * n3, "flops": half * 4 * W ** 3 + _fft((2 * N) ** 3)}
        if op == "kernel":
            return ker
        if op != "reconstruct":
            return atb
        cg = _solve_work(N, case["iters"])
        return {k: ker[k] + atb[k] + cg[k] for k in ker}
    if op == "images":
        return {"bytes": case["M"] * (4 * N * N + 8 * points(N)), "flops": case["M"] * _fft(N * N)}
    if op == "apply":
        e = 8 if case["dtype"] == "f64" else 4
        return {"bytes": e * (2 * n3 + (2 * N) ** 2 * (N + 1)), "flops": 2 * _fft((2 * N) ** 3)}
    if op == "cg":
        return _solve_work(N, case["iters"])
    if op == "learned_pcg":
        w = _solve_work(N, case["iters"])
        return {"bytes": w["bytes"] + 4 * n3 * case["iters"], "flops": w["flops"] + case["iters"] * 2 * _fft(n3)}
    w = _solve_work(N, 2 * case["k"] * case["batch"])
    net = 3 * 2 * 57000 * 32 ** 3 * case["batch"]
    return {"bytes": w["bytes"], "flops": w["flops"] + net}


# ------------------------------------------------------------ 64-bit results --

def _half_points(case, R, shifts, groups, table, a, e):
    """xi (views a..e, half-disk points, 3), h and the disk indices of the points, in 64 bits."""
    N = case["N"]
    k1, k2 = disk(N)
    idx = np.arange((k1.size + 1) // 2, k1.size)  # the half after the origin
    k = torch.as_tensor(np.stack([k1[idx], k2[idx]], 1) * (2 * math.pi / N), dtype=torch.float64, device=DEV)
    Rt = torch.as_tensor(R[a:e, :2], dtype=torch.float64, device=DEV)
    xi = (k[None, :, :1] * Rt[:, None, 0] + k[None, :, 1:] * Rt[:, None, 1])
    h = torch.ones(xi.shape[:2], dtype=torch.float64, device=DEV)
    if table is not None:
        q = torch.as_tensor(k1[idx] ** 2 + k2[idx] ** 2, device=DEV)
        h = torch.as_tensor(table, dtype=torch.float64, device=DEV)[torch.as_tensor(groups[a:e], device=DEV).long()][:, q]
    ph = torch.zeros(xi.shape[:2], dtype=torch.float64, device=DEV)
    if shifts is not None:
        ph = torch.as_tensor(shifts[a:e], dtype=torch.float64, device=DEV) @ k.T
    return xi, h, ph, idx


def _sum_re(xi, c, n1, n2, n3):
    """Re sum_j c_j exp(i <n, xi_j>) over the box n1 x n2 x n3 (c complex or real)."""
    def cs(x, n):
        t = x[:, None] * n[None, :]
        return torch.complex(torch.cos(t), torch.sin(t))
    e = cs(xi[:, 0], n1) * c[:, None]
    e = (e[:, :, None] * cs(xi[:, 1], n2)[:, None, :]).reshape(xi.shape[0], -1)
    f = cs(xi[:, 2], n3)
    return (e.real.T.contiguous() @ f.real.contiguous() - e.imag.T.contiguous() @ f.imag.contiguous()).reshape(
        n1.numel(), n2.numel(), n3.numel())


def _chunks(case, cells):
    """Ranges of views whose half-disk points by `cells` fit in about a gigabyte."""
    per = max(1, int((1 << 26) / cells / ((points(case["N"]) + 1) // 2)))
    return [(a, min(case["M"], a + per)) for a in range(0, case["M"], per)]


def _exact_kernel(case, seed):
    N = case["N"]
    geo = geometry(case, seed)
    n = torch.arange(-N + 1, N, dtype=torch.float64, device=DEV)
    half = torch.zeros((2 * N - 1, 2 * N - 1, N), dtype=torch.float64, device=DEV)  # n3 >= 0
    k0 = 0.0
    for a, e in _chunks(case, (2 * N - 1) ** 2):
        xi, h, _, _ = _half_points(case, *geo, a, e)
        x, w = xi.reshape(-1, 3), 2 * (h * h).reshape(-1)
        for j in range(0, x.shape[0], max(1, (1 << 26) // (2 * N - 1) ** 2)):
            k = slice(j, j + max(1, (1 << 26) // (2 * N - 1) ** 2))
            half += _sum_re(x[k], w[k], n, n, n[N - 1:])
    table, groups = geo[3], geo[2]
    k0 = float(case["M"]) if table is None else float((table[groups, 0].astype(np.float64) ** 2).sum())
    out = torch.zeros((2 * N,) * 3, dtype=torch.float64, device=DEV)
    half += k0
    out[1:, 1:, N:] = half
    out[1:, 1:, 1:N] = half[:, :, 1:].flip(0, 1, 2)
    return out


def _exact_atb(case, seed):
    N = case["N"]
    geo = geometry(case, seed)
    b = slices(N, case["M"], seed)
    n = torch.arange(N, dtype=torch.float64, device=DEV) - N // 2
    out = torch.zeros((N, N, N), dtype=torch.float64, device=DEV)
    P = b.shape[1]
    for a, e in _chunks(case, N * N):
        xi, h, ph, idx = _half_points(case, *geo, a, e)
        i = torch.as_tensor(idx, device=DEV)
        bb = b[a:e].to(torch.complex128)
        c = (bb[:, i] + bb[:, P - 1 - i].conj()) * torch.polar(h, ph)
        x, c = xi.reshape(-1, 3), c.reshape(-1)
        for j in range(0, x.shape[0], max(1, (1 << 26) // (N * N))):
            k = slice(j, j + max(1, (1 << 26) // (N * N)))
            out += _sum_re(x[k], c[k], n, n, n)
    table, groups = geo[3], geo[2]
    h0 = np.ones(case["M"]) if table is None else table[groups, 0].astype(np.float64)
    out += float((torch.as_tensor(h0, device=DEV) * b[:, (P - 1) // 2].real.double()).sum())
    return out


def _exact_project(case, seed):
    N = case["N"]
    geo = geometry(case, seed)
    V = blobs(N, seed).double()
    n = torch.arange(N, dtype=torch.float64, device=DEV) - N // 2
    P = points(N)
    out = torch.empty((case["M"], P), dtype=torch.complex128, device=DEV)
    for a, e in _chunks(case, N * N):
        xi, h, ph, idx = _half_points(case, *geo, a, e)
        x = xi.reshape(-1, 3)
        v = torch.empty(x.shape[0], dtype=torch.complex128, device=DEV)
        for j in range(0, x.shape[0], max(1, (1 << 25) // (N * N))):
            k = slice(j, j + max(1, (1 << 25) // (N * N)))
            t = x[k, 2][None, :] * n[:, None]
            W = V.reshape(N * N, N)
            f = torch.complex(W @ torch.cos(t), -(W @ torch.sin(t))).reshape(N, N, -1)
            for d in (1, 0):  # the axes left, last first
                t = x[k, d][None, :] * n[:, None]
                f = (f * torch.complex(torch.cos(t), -torch.sin(t))).sum(-2)
            v[k] = f
        v = v.reshape(h.shape) * torch.polar(h, -ph)
        i = torch.as_tensor(idx, device=DEV)
        out[a:e, i] = v
        out[a:e, P - 1 - i] = v.conj()
    table, groups = geo[3], geo[2]
    h0 = np.ones(case["M"]) if table is None else table[groups, 0].astype(np.float64)
    out[:, (P - 1) // 2] = torch.as_tensor(h0, device=DEV).to(torch.complex128) * V.sum()
    return out


def _exact_images(case, seed):
    N = case["N"]
    k1, k2 = disk(N)
    at = torch.as_tensor((k1 % N) * N + k2 % N, device=DEV)
    sign = torch.as_tensor(1.0 - 2.0 * ((k1 + k2) % 2), dtype=torch.float64, device=DEV)
    J = images(case, seed)
    out = torch.empty((case["M"], k1.size), dtype=torch.complex128, device=DEV)
    step = max(1, (1 << 26) // (N * N))
    for a in range(0, case["M"], step):
        out[a:a + step] = torch.fft.fft2(J[a:a + step].double()).reshape(-1, N * N)[:, at] * sign
    return out


def _product(ker, lam_rel):
    """x -> Ker * x + lambda Ker(0) x in 64 bits, for a kernel in centred order."""
    N = ker.shape[0] // 2
    K = ker.double()
    lam = lam_rel * float(K[N, N, N])
    S = torch.fft.rfftn(torch.fft.ifftshift(K)).real.contiguous()

    def apply(x):
        return torch.fft.irfftn(S * torch.fft.rfftn(x, s=(2 * N,) * 3), s=(2 * N,) * 3)[:N, :N, :N] + lam * x
    return apply


def _cg(apply, b, iters):
    x, r = torch.zeros_like(b), b.clone()
    p, rr = r.clone(), float((b * b).sum())
    for _ in range(iters):
        q = apply(p)
        a = rr / float((p * q).sum())
        x += a * p
        r -= a * q
        new = float((r * r).sum())
        p = r + (new / rr) * p
        rr = new
    return x


def exact(case, seed):
    op, N, lam = case["op"], case["N"], case.get("lam", LAM)
    if op in ("kernel", "backproject", "project", "reconstruct"):
        pts = case["M"] * (points(N) - 1) / 2
        cells = {"kernel": (2 * N - 1) ** 2 * N}.get(op, N ** 3)
        if 4 * pts * cells > EXACT_FLOPS:
            return None
    if op == "kernel":
        return _exact_kernel(case, seed)
    if op == "backproject":
        return _exact_atb(case, seed)
    if op == "project":
        return _exact_project(case, seed)
    if op == "images":
        return _exact_images(case, seed)
    if op == "apply":
        x = blobs(N, seed, torch.float64 if case["dtype"] == "f64" else torch.float32)
        return _product(kernel(N, seed), lam)(x.double())
    if op == "cg":
        return _cg(_product(kernel(N, seed), lam), torch.randn((N, N, N), device=DEV, generator=_gen(seed)).double(),
                   case["iters"])
    if op == "reconstruct":
        ker, atb = _exact_kernel(case, seed), _exact_atb(case, seed)
        return {"ker": ker, "atb": atb, "x": _cg(_product(ker, lam), atb, case["iters"])}
    return None  # through the BF16 network
