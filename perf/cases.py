"""Performance cases: the calls a user of the library makes, over the range of sizes it serves.

Each case is a dict of plain values.  `kind` names the use:

  labels  a training step of a label-space loss: B histograms over d classes, one shared cost of squared
          distances between class embeddings ("line": classes on a line), gradients of both histograms
  images  a training step on histograms over an h x w pixel grid with one shared cost, squared ("sq") or
          plain ("l2") grid distance, optionally with the per-sample early stop (tol > 0) or the gradient of
          the sharp loss
  costs   a training step with one cost matrix per sample (point clouds whose distances the program already
          holds), the gradient reaching the cost too; a share of the masses can be exactly zero
  points  a training step on per-sample point clouds given by coordinates, gradients of the coordinates
  warm    a forward continued from the previous step's potentials

The shapes come from the repository's workloads (tiny, label, image, grid, clouds, clouds from points), the
early-stop and sharp-gradient measurements on the image workload, and generic larger and ragged sizes.
"""
import math

import torch

import paper_1907_01729_amd as sk


def listed():
    return [
        # the smallest call: four histograms over ten bins; launches and latency are all of it
        {"name": "tiny", "kind": "labels", "B": 4, "d": 10, "cost": "line", "lam": 0.1, "n_iter": 100},
        # the paper's own setting: label losses over 100 classes, a full training batch
        {"name": "label", "kind": "labels", "B": 1024, "d": 100, "cost": "plane", "lam": 0.05, "n_iter": 200},
        # label losses over a large class vocabulary
        {"name": "vocabulary", "kind": "labels", "B": 256, "d": 1000, "cost": "plane", "lam": 0.05, "n_iter": 200},
        # a batch of 28 x 28 images
        {"name": "image", "kind": "images", "B": 256, "h": 28, "w": 28, "cost": "sq", "lam": 0.01, "n_iter": 300,
         "tol": 0.0, "sharp": False},
        # the same images stopped one by one: counts per image spread over most of the range
        {"name": "image_stop", "kind": "images", "B": 1024, "h": 28, "w": 28, "cost": "sq", "lam": 0.01,
         "n_iter": 300, "tol": 2e-4, "sharp": False},
        # images with the gradient of the sharp loss
        {"name": "image_sharp", "kind": "images", "B": 64, "h": 28, "w": 28, "cost": "sq", "lam": 0.01,
         "n_iter": 100, "tol": 0.0, "sharp": True},
        # the largest: 64 x 64 grids at small lambda
        {"name": "grid", "kind": "images", "B": 64, "h": 64, "w": 64, "cost": "sq", "lam": 1e-3, "n_iter": 500,
         "tol": 1e-6, "sharp": False},
        # small per-sample costs, ragged, with zero masses (graph or set matching in a batch)
        {"name": "pairs", "kind": "costs", "B": 500, "d1": 90, "d2": 77, "lam": 0.1, "n_iter": 100, "zeros": 0.1},
        # large per-sample costs: bandwidth
        {"name": "clouds", "kind": "costs", "B": 32, "d1": 1024, "d2": 2048, "lam": 0.05, "n_iter": 100,
         "zeros": 0.0},
        # the same clouds by their coordinates
        {"name": "points", "kind": "points", "B": 32, "d1": 1024, "d2": 2048, "D": 3, "lam": 0.05, "n_iter": 100},
        # a few small ragged clouds: a call of many short launches
        {"name": "points_small", "kind": "points", "B": 6, "d1": 300, "d2": 257, "D": 3, "lam": 0.05, "n_iter": 50},
        # a label batch resumed from the previous step's potentials for a few iterations
        {"name": "label_warm", "kind": "warm", "B": 512, "d": 100, "cost": "plane", "lam": 0.02, "n_iter": 20},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


#: Cell updates (B * d1 * d2 * n_iter) and per-sample cost cells (B * d1 * d2) that a drawn case may have.
CELLS, COSTS = 2.0e11, 6.4e7


def draw(rng):
    kind = rng.choice(["labels", "labels", "images", "images", "images", "costs", "points", "warm"])
    n_iter = _log(rng, 20, 500)
    if kind in ("labels", "warm"):
        d = _log(rng, 8, 128) if rng.random() < 0.5 else _log(rng, 129, 2500)
        most = max(1, min(2048, int(CELLS / (d * d * n_iter))))
        c = {"kind": kind, "B": _log(rng, 1, most), "d": d, "cost": rng.choice(["plane", "plane", "line"]),
             "lam": round(math.exp(rng.uniform(math.log(0.02), math.log(0.2))), 4), "n_iter": n_iter}
        return c
    if kind == "images":
        h, w = _log(rng, 8, 64), _log(rng, 8, 64)
        most = max(1, min(512, int(CELLS / ((h * w) ** 2 * n_iter))))
        return {"kind": kind, "B": _log(rng, 1, most), "h": h, "w": w, "cost": rng.choice(["sq", "sq", "l2"]),
                "lam": round(math.exp(rng.uniform(math.log(2e-3), math.log(0.1))), 5), "n_iter": n_iter, "tol": 0.0,
                "sharp": False}
    d1, d2 = _log(rng, 24, 2048), _log(rng, 24, 2048)
    most = max(1, min(1024, int(min(COSTS, CELLS / n_iter) / (d1 * d2))))
    c = {"kind": kind, "B": _log(rng, 1, most), "d1": d1, "d2": d2,
         "lam": round(math.exp(rng.uniform(math.log(0.05), math.log(0.5))), 4), "n_iter": n_iter}
    if kind == "costs":
        c["zeros"] = rng.choice([0.0, 0.1])
    else:
        c["D"] = rng.choice([2, 3])
    return c


def _sizes(case):
    if case["kind"] == "images":
        d = case["h"] * case["w"]
        return case["B"], d, d
    if case["kind"] in ("labels", "warm"):
        return case["B"], case["d"], case["d"]
    return case["B"], case["d1"], case["d2"]


def _blobs(g, B, h, w):
    """Histograms over the pixels of an h x w grid: three Gaussian blobs each, on a small floor."""
    dev = g.device
    n = 3
    cr = h * torch.rand(B, n, 1, 1, generator=g, device=dev)
    cc = w * torch.rand(B, n, 1, 1, generator=g, device=dev)
    sig = 1.0 + 3.0 * torch.rand(B, n, 1, 1, generator=g, device=dev)
    r = torch.arange(h, device=dev).view(1, 1, h, 1)
    c = torch.arange(w, device=dev).view(1, 1, 1, w)
    e = torch.exp(-((r - cr) ** 2 + (c - cc) ** 2) / (2 * sig**2)) / sig**2
    p = e.sum(1).reshape(B, h * w).double() + 1e-30
    p = p / p.sum(1, keepdim=True) + 1e-6
    return (p / p.sum(1, keepdim=True)).float()


def _uniform_histograms(g, B, d, zeros):
    p = 0.05 + torch.rand(B, d, generator=g, device=g.device, dtype=torch.float64)
    if zeros:
        off = torch.rand(B, d, generator=g, device=g.device) < zeros
        off[:, 0] = False
        p[off] = 0.0
    return (p / p.sum(1, keepdim=True)).float()


def _softmax_histograms(g, B, d):
    return torch.softmax(2.0 * torch.randn(B, d, generator=g, device=g.device, dtype=torch.float64), 1).float()


def _sq_dists(x, y):
    return ((x.unsqueeze(-2) - y.unsqueeze(-3)) ** 2).sum(-1)


def _inputs(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    dev = g.device
    B, d1, d2 = _sizes(case)
    kind = case["kind"]
    s = {}
    if kind in ("labels", "warm"):
        s["mu"], s["nu"] = _softmax_histograms(g, B, d1), _softmax_histograms(g, B, d2)
        if case["cost"] == "line":
            e = torch.arange(d1, device=dev, dtype=torch.float64).view(-1, 1) / (d1 - 1)
        else:
            e = torch.rand(d1, 2, generator=g, device=dev, dtype=torch.float64)
        s["C"] = _sq_dists(e, e).float()
        if kind == "warm":  # the potentials that some earlier iterations left
            s["alpha0"] = _solve(s["mu"], s["nu"], s["C"], case["lam"], 10)["alpha"].float()
    elif kind == "images":
        h, w = case["h"], case["w"]
        s["mu"], s["nu"] = _blobs(g, B, h, w), _blobs(g, B, h, w)
        r, c = torch.meshgrid(torch.arange(h, device=dev), torch.arange(w, device=dev), indexing="ij")
        pts = torch.stack([r.flatten(), c.flatten()], 1).double()
        C = _sq_dists(pts, pts) / float(max(h, w) - 1) ** 2
        s["C"] = (C if case["cost"] == "sq" else C.sqrt()).float()
    else:
        D = case.get("D", 3)
        zeros = case.get("zeros", 0.0)
        if zeros:
            s["mu"], s["nu"] = _uniform_histograms(g, B, d1, zeros), _uniform_histograms(g, B, d2, zeros)
        else:
            s["mu"] = torch.full((B, d1), 1.0 / d1, device=dev)
            s["nu"] = torch.full((B, d2), 1.0 / d2, device=dev)
        x = torch.randn(B, d1, D, generator=g, device=dev, dtype=torch.float64)
        y = torch.randn(B, d2, D, generator=g, device=dev, dtype=torch.float64)
        y = y + torch.randn(B, 1, D, generator=g, device=dev, dtype=torch.float64)
        if kind == "points":
            s["X"], s["Y"] = x.float(), y.float()
        else:
            s["C"] = torch.empty(B, d1, d2, device=dev)
            for b in range(B):
                s["C"][b] = _sq_dists(x[b], y[b])
    return s


def prepare(case, seed):
    state = _inputs(case, seed)
    state["case"] = dict(case)
    grad = {"labels": ("mu", "nu"), "images": ("mu", "nu"), "costs": ("mu", "nu", "C"),
            "points": ("mu", "nu", "X", "Y"), "warm": ()}[case["kind"]]
    for k in grad:
        state[k].requires_grad_()
    return state


def run(state):
    c = state["case"]
    kind = c["kind"]
    if kind == "points":
        loss = sk.sinkhorn_loss_points(state["mu"], state["nu"], state["X"], state["Y"], c["lam"], c["n_iter"])
        g = torch.autograd.grad(loss.sum(), [state["mu"], state["nu"], state["X"], state["Y"]])
        return {"loss": loss, "grad_mu": g[0], "grad_nu": g[1], "grad_X": g[2], "grad_Y": g[3]}
    if kind == "costs":
        loss = sk.sinkhorn_loss(state["mu"], state["nu"], state["C"], c["lam"], c["n_iter"])
        g = torch.autograd.grad(loss.sum(), [state["mu"], state["nu"], state["C"]])
        return {"loss": loss, "grad_mu": g[0], "grad_nu": g[1], "grad_C": g[2]}
    if kind == "warm":
        out = sk.sinkhorn_forward(state["mu"], state["nu"], state["C"], c["lam"], c["n_iter"],
                                  alpha0=state["alpha0"])
        return {k: out[k] for k in ("loss", "alpha", "beta", "iters")}
    if kind == "labels":
        loss = sk.sinkhorn_loss(state["mu"], state["nu"], state["C"], c["lam"], c["n_iter"])
        g = torch.autograd.grad(loss.sum(), [state["mu"], state["nu"]])
        return {"loss": loss, "grad_mu": g[0], "grad_nu": g[1]}
    loss = sk.sinkhorn_loss(state["mu"], state["nu"], state["C"], c["lam"], c["n_iter"], tol=c["tol"],
                            sharp=c["sharp"])
    g = torch.autograd.grad(loss.sum(), [state["mu"], state["nu"]])
    return {"loss": loss, "grad_mu": g[0], "grad_nu": g[1]}


def work(case):
    """Inputs read once, outputs written once; two products of the plan per iteration (a multiply and an add per cell
    each) and one of the plan and the cost for the loss."""
    B, d1, d2 = _sizes(case)
    kind = case["kind"]
    cells = float(B) * d1 * d2
    flops = (4.0 * case["n_iter"] + 4.0) * cells
    values = 2.0 * B * (d1 + d2) + B  # histograms, their gradients (or the potentials), the loss
    if kind == "costs":
        values += 2.0 * cells
        flops += cells
    elif kind == "points":
        values += 2.0 * B * (d1 + d2) * case["D"]
        flops += 4.0 * case["D"] * cells
    else:
        values += float(d1) * d2
        if kind == "warm":
            values += B * d1
    return {"bytes": 4.0 * values, "flops": flops}


def tolerance(case):
    """About four times the largest difference from exact() over the listed and drawn cases of a kind: sums of up to
    thousands of 32-bit terms, plan entries whose exponents are differences of potentials of up to thousands of units
    (gradients of costs and coordinates are made of those), the linear solve of the sharp loss stopped at a residual
    of 1e-6, and under an early stop the few per cent of samples whose count a rounding moves by one."""
    rel = {"labels": 2e-5, "warm": 2e-5, "images": 2e-5, "costs": 3e-5, "points": 6e-5}[case["kind"]]
    if case.get("sharp"):
        rel = 5e-4
    return {"rel": rel, "max": max(1e-3, 40 * rel)}


# ---- the same results in 64 bits, in plain torch ----


def _safe_log(x):
    return torch.log(x)  # log 0 = -inf: a zero mass has the log-scaling -inf


def _lse_rows(x, C, lam, over_rows):
    """log sum over one index of exp(x - C / lam), for every problem; C [1 or B, d1, d2]."""
    out = []
    for b in range(x.shape[0]):
        Cb = C[b if C.shape[0] > 1 else 0]
        t = x[b].unsqueeze(1) - Cb / lam if over_rows else x[b].unsqueeze(0) - Cb / lam
        out.append(torch.logsumexp(t, 0 if over_rows else 1))
    return torch.stack(out)


def _solve(mu, nu, C, lam, n_iter, tol=0.0, alpha0=None):
    """Sinkhorn iterations (v-update, then u-update) in 64 bits: log-scalings, loss and counts.  The plan is kept as
    diag(u) K diag(v) with the potentials' logarithms absorbed into K whenever the scalings grow."""
    mu, nu, C = mu.detach().double(), nu.detach().double(), C.detach().double()
    lam = float(torch.tensor(lam, dtype=torch.float32))
    C = C.unsqueeze(0) if C.dim() == 2 else C
    B, d1 = mu.shape
    logmu, lognu = _safe_log(mu), _safe_log(nu)
    on1, on2 = mu > 0, nu > 0
    z = torch.zeros((), dtype=torch.float64, device=mu.device)
    a = torch.where(on1, z if alpha0 is None else alpha0.double(), -z.new_tensor(math.inf))
    its = torch.full((B,), n_iter, dtype=torch.int32, device=mu.device)
    span = float(C.max() - C.min()) / lam
    alpha, beta = torch.empty_like(mu), torch.empty_like(nu)

    if span < 300.0 and (alpha0 is None or float(a[on1].abs().max()) < 150.0):
        # the plain form: 64 bits hold every scaling
        low = float(C.min())
        K = torch.exp(-(C - low) / lam)
        shared = K.shape[0] == 1
        if shared:
            K0, Kt = K[0], K[0].t().contiguous()
            rows = lambda v: v @ Kt  # noqa: E731
            cols = lambda u: u @ K0  # noqa: E731
        else:
            Kt = K.transpose(1, 2).contiguous()
            rows = lambda v: torch.bmm(K, v.unsqueeze(2)).squeeze(2)  # noqa: E731
            cols = lambda u: torch.bmm(Kt, u.unsqueeze(2)).squeeze(2)  # noqa: E731
        u = torch.exp(a)
        S = cols(u)
        v = nu / S
        live = torch.ones(B, dtype=torch.bool, device=mu.device)
        for k in range(1, n_iter + 1):
            un = mu / rows(v)
            u = torch.where(live.unsqueeze(1), un, u)
            if k == n_iter:
                break
            S = cols(u)
            if tol > 0:
                err = (u * rows(v) - mu).abs().sum(1) + (v * S - nu).abs().sum(1)
                stop = live & (err <= tol)
                its[stop] = k
                live = live & ~stop
                if not bool(live.any()):
                    break
            v = torch.where(live.unsqueeze(1), nu / S, v)
        alpha, beta = torch.log(u), torch.log(v) - low / lam
        loss = torch.empty(B, dtype=torch.float64, device=mu.device)
        for b in range(B):
            i = 0 if shared else b
            loss[b] = u[b] @ ((K[i] * C[i]) @ v[b])
        return {"alpha": alpha, "beta": beta, "loss": loss, "iters": its}

    b_ = lognu - _lse_rows(a, C, lam, True)
    loss = torch.empty(B, dtype=torch.float64, device=mu.device)
    chunk = max(1, int(8e9 / (8.0 * C.shape[1] * C.shape[2])))
    for lo in range(0, B, chunk):
        sl = slice(lo, min(B, lo + chunk))
        Cc = C if C.shape[0] == 1 else C[sl]
        m, n, ac, bc = mu[sl], nu[sl], a[sl], b_[sl]
        ac = logmu[sl] - _lse_rows(bc, Cc, lam, False)  # the first u-update
        live = torch.ones(m.shape[0], dtype=torch.bool, device=mu.device)

        def absorb():
            P = ac.unsqueeze(2) + bc.unsqueeze(1)
            P -= Cc / lam
            P.exp_()
            return P, torch.zeros_like(m) + on1[sl], torch.zeros_like(n) + on2[sl]

        P, u, v = absorb()
        ac = torch.where(on1[sl], ac, z)
        bc = torch.where(on2[sl], bc, z)
        for k in range(2, n_iter + 1):
            S = torch.bmm(u.unsqueeze(1), P).squeeze(1)
            if tol > 0:  # the rows fit after the u-update, up to 64-bit rounding
                stop = live & ((v * S - n).abs().sum(1) <= tol)
                its[sl][stop] = k - 1
                live = live & ~stop
            on = live.unsqueeze(1)
            v = torch.where(on & on2[sl], n / S.clamp_min(1e-300), v)
            R = torch.bmm(P, v.unsqueeze(2)).squeeze(2)
            u = torch.where(on & on1[sl], m / R.clamp_min(1e-300), u)
            if k < 4 or k % 5 == 0:
                far = max(float(u[on1[sl]].log().abs().max()), float(v[on2[sl]].log().abs().max()))
                if k < 4 or far > 60.0:
                    ac = ac + torch.where(on1[sl], u, z + 1).log()
                    bc = bc + torch.where(on2[sl], v, z + 1).log()
                    ac = torch.where(on1[sl], ac, -z.new_tensor(math.inf))
                    bc = torch.where(on2[sl], bc, -z.new_tensor(math.inf))
                    del P
                    P, u, v = absorb()
                    ac, bc = torch.where(on1[sl], ac, z), torch.where(on2[sl], bc, z)
        alpha[sl], beta[sl] = ac + u.log(), bc + v.log()
        for i in range(m.shape[0]):
            loss[lo + i] = u[i] @ ((P[i] * Cc[i if Cc.shape[0] > 1 else 0]) @ v[i])
        del P
    return {"alpha": alpha, "beta": beta, "loss": loss, "iters": its}


def _centred(x, on, lam):
    x = torch.where(on, x, torch.zeros_like(x))
    mean = x.sum(1, keepdim=True) / on.sum(1, keepdim=True)
    return torch.where(on, lam * (x - mean), torch.zeros_like(x))


def _plan(r, C, lam):
    lam = float(torch.tensor(lam, dtype=torch.float32))
    return torch.exp(r["alpha"].unsqueeze(2) + r["beta"].unsqueeze(1) - C / lam)


def _sharp(mu, nu, C, r, lam):
    """Gradient of the sharp loss: [diag(r) P; P^T diag(c)] z = (a, b) by conjugate gradients in 64 bits."""
    P = _plan(r, C, lam)
    Pt = P.transpose(1, 2).contiguous()
    rows, cols = P.sum(2), P.sum(1)
    a, b = (P * C).sum(2), (P * C).sum(1)
    mv = lambda M, x: torch.bmm(M, x.unsqueeze(2)).squeeze(2)  # noqa: E731
    d1 = a.shape[1]
    H = lambda x: torch.cat([rows * x[:, :d1] + mv(P, x[:, d1:]), mv(Pt, x[:, :d1]) + cols * x[:, d1:]], 1)  # noqa: E731
    rhs, M = torch.cat([a, b], 1), torch.cat([rows, cols], 1)
    n = torch.cat([torch.ones_like(a), -torch.ones_like(b)], 1)
    rhs = rhs - n * (rhs * n).sum(1, keepdim=True) / n.shape[1]
    x = torch.zeros_like(rhs)
    res = rhs.clone()
    zed = res / M
    p, rz = zed.clone(), (res * zed).sum(1, keepdim=True)
    for _ in range(400):
        q = H(p)
        t = rz / (p * q).sum(1, keepdim=True).clamp_min(1e-300)
        x, res = x + t * p, res - t * q
        zed = res / M
        new = (res * zed).sum(1, keepdim=True)
        p, rz = zed + (new / rz.clamp_min(1e-300)) * p, new
        if float(new.max()) < 1e-28 * 1e-4:
            break
    return _centred(x[:, :d1], mu > 0, 1.0), _centred(x[:, d1:], nu > 0, 1.0)


def exact(case, seed):
    s = _inputs(case, seed)
    kind, lam = case["kind"], case["lam"]
    lam32 = float(torch.tensor(lam, dtype=torch.float32))
    mu, nu = s["mu"].double(), s["nu"].double()
    if kind == "points":
        C = torch.empty(mu.shape[0], mu.shape[1], nu.shape[1], dtype=torch.float64, device=mu.device)
        for b in range(C.shape[0]):
            C[b] = _sq_dists(s["X"][b].double(), s["Y"][b].double())
    else:
        C = s["C"].double()
    r = _solve(mu, nu, C, lam, case["n_iter"], case.get("tol", 0.0), s.get("alpha0"))
    if kind == "warm":
        return {"loss": r["loss"], "alpha": r["alpha"], "beta": r["beta"], "iters": None}
    out = {"loss": r["loss"]}
    if kind == "images" and case["sharp"]:
        out["grad_mu"], out["grad_nu"] = _sharp(mu, nu, C, r, lam)
    else:
        out["grad_mu"], out["grad_nu"] = _centred(r["alpha"], mu > 0, lam32), _centred(r["beta"], nu > 0, lam32)
    if kind == "costs":
        out["grad_C"] = _plan(r, C, lam)
    elif kind == "points":
        P = _plan(r, C, lam)
        X, Y = s["X"].double(), s["Y"].double()
        out["grad_X"] = 2 * (P.sum(2).unsqueeze(2) * X - torch.bmm(P, Y))
        out["grad_Y"] = 2 * (P.sum(1).unsqueeze(2) * Y - torch.bmm(P.transpose(1, 2).contiguous(), X))
    return out
