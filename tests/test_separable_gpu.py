"""GPU parity of the solve of a shared cost that splits over two axes
(sk_sep_solve) with the oracle: line lengths at the edges of its buckets (16,
32, 64 lanes), different grids on the two sides, tables that are neither
symmetric nor distances, zero masses up to whole lines, the early stop, the
warm start, block sizes 16 and 4 of the line sums, and costs that miss the
test of the cost by one entry or by their spread (left to the sweeps)."""
import sys

import numpy as np
import pytest
import torch

import oracle
import paper_1907_01729_amd as sk
import workloads
from parity_util import gauge_fixed_errors, loss_rel_err

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def _t(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to(DEV)


def make(seed, B, g1, g2, kind, zero=0.0):
    rng = np.random.default_rng(seed)
    (h1, w1), (h2, w2) = g1, g2
    mu = rng.uniform(0.05, 1.0, size=(B, h1, w1))
    nu = rng.uniform(0.05, 1.0, size=(B, h2, w2))
    if zero:
        for m in (mu, nu):
            m[rng.random(m.shape) < zero] = 0.0
            m[0, 1, :] = 0.0  # a whole row, and a whole column
            m[0, :, 2] = 0.0
            m[:, 0, 0] = 0.5
    mu, nu = mu.reshape(B, -1), nu.reshape(B, -1)
    mu, nu = mu / mu.sum(1, keepdims=True), nu / nu.sum(1, keepdims=True)
    if kind == "sq":
        a = np.subtract.outer(np.arange(h1) / (h1 - 1), np.arange(h2) / (h2 - 1)) ** 2
        b = np.subtract.outer(np.arange(w1) / (w1 - 1), np.arange(w2) / (w2 - 1)) ** 2
    elif kind == "abs":
        a = np.abs(np.subtract.outer(np.arange(h1) / (h1 - 1), np.arange(h2) / (h2 - 1)))
        b = np.abs(np.subtract.outer(np.arange(w1) / (w1 - 1), np.arange(w2) / (w2 - 1)))
    else:  # any two tables, negative entries too
        a = rng.uniform(-0.3, 1.0, size=(h1, h2))
        b = rng.uniform(-0.3, 1.0, size=(w1, w2))
    C = a[:, None, :, None] + b[None, :, None, :]
    return mu.astype(np.float32), nu.astype(np.float32), C.reshape(h1 * w1, h2 * w2).astype(np.float32)


def check(mu, nu, C, lam, n_iter, tol=0.0, alpha0=None, splits=True):
    B, d1, d2 = mu.shape[0], mu.shape[1], nu.shape[1]
    print(f"[split] B={B} d1={d1} d2={d2} lam={lam} n_iter={n_iter} tol={tol}", file=sys.stderr, flush=True)
    assert ("sk_sep_solve" in sk.sinkhorn_describe(B, d1, d2, 0, lam, n_iter, tol)) == splits
    out = sk.sinkhorn_forward(_t(mu), _t(nu), _t(C), lam, n_iter, tol, alpha0=None if alpha0 is None else _t(alpha0))
    torch.cuda.synchronize()
    g = {k: v.cpu().numpy() for k, v in out.items()}
    if tol > 0:
        free = oracle.forward(mu, nu, C[None], lam, n_iter, tol=tol)
        assert np.all(np.abs(free["iters"] - g["iters"]) <= 1)
        ref = oracle.forward(mu, nu, C[None], lam, n_iter, n_iter_b=g["iters"])
    else:
        assert np.all(g["iters"] == n_iter)
        ref = oracle.forward(mu, nu, C[None], lam, n_iter, alpha0=alpha0)
    el = loss_rel_err(g["loss"], ref["loss"])
    ea, eb = gauge_fixed_errors(mu, nu, g["alpha"], g["beta"], ref["alpha"], ref["beta"])
    top = max(np.max(np.abs(x[np.isfinite(x)])) for x in (ref["alpha"], ref["beta"]))
    print(f"   loss rel {el:.2e}  alpha {ea:.2e}  beta {eb:.2e}  potentials to {top:.0f}", file=sys.stderr, flush=True)
    # The cost may differ from the tables' sum by two fp32 roundings of either
    # part (2^-22 of it), which moves potentials by at most that over lambda
    # and the loss by the like; the potentials are rounded to fp32.
    cost = 2.0 ** -22 * 2.0 * np.max(np.abs(C))
    assert ea <= 2 * cost / lam + 2.0 ** -22 * top and eb <= 2 * cost / lam + 2.0 ** -22 * top
    assert el <= 5e-6
    assert np.all(np.abs(g["marg_err"] - ref["marg_err"]) <= 2e-6 + 1e-3 * ref["marg_err"])
    return g


@pytest.mark.parametrize("g1, g2, kind, lam", [
    ((12, 12), (12, 12), "sq", 0.02),   # 16 lanes
    ((16, 9), (16, 9), "any", 0.05),    # a full and a partly filled line
    ((17, 16), (17, 16), "sq", 0.01),   # 32 and 16 lanes
    ((28, 28), (28, 28), "sq", 0.004),  # spread above 150 within 16: blocks of 4
    ((32, 12), (32, 12), "abs", 0.02),
    ((33, 8), (33, 8), "sq", 0.01),     # 64 and 16 lanes
    ((20, 12), (10, 16), "any", 0.05),  # different grids
    ((12, 20), (33, 5), "sq", 0.03),
])
def test_split_cost(g1, g2, kind, lam):
    mu, nu, C = make(11, 8, g1, g2, kind)
    check(mu, nu, C, lam, 170)


@pytest.mark.parametrize("g, kind", [((14, 14), "sq"), ((35, 10), "any")])
def test_split_zero_masses(g, kind):
    mu, nu, C = make(12, 4, g, g, kind, zero=0.3)
    check(mu, nu, C, 0.03, 170)


def test_split_warm_start():
    mu, nu, C = make(13, 3, (18, 15), (18, 15), "sq", zero=0.1)
    a0 = oracle.forward(mu, nu, C[None], 0.02, 20)["alpha"]
    check(mu, nu, C, 0.02, 170, alpha0=np.where(mu > 0, a0, 7.0).astype(np.float32))


@pytest.mark.parametrize("g, B", [((20, 18), 9), ((40, 9), 9)])
def test_split_early_stop(g, B):
    mu, nu, C = make(14, B, g, g, "sq", zero=0.05)
    out = check(mu, nu, C, 0.02, 400, tol=1e-3)
    assert out["iters"].min() < out["iters"].max() and out["iters"].min() < 400


def test_widest_lines():
    """64 x 64 (4096 columns), small lambda: the smallest batch that takes the
    solve, against the same problems in a batch below it (the sweeps)."""
    mu, nu, C = make(15, 8, (64, 64), (64, 64), "sq")
    out = sk.sinkhorn_forward(_t(mu), _t(nu), _t(C), 2e-3, 100)
    few = sk.sinkhorn_forward(_t(mu[:2]), _t(nu[:2]), _t(C), 2e-3, 100)
    assert "sk_sep_solve" in sk.sinkhorn_describe(8, 4096, 4096, 0, 2e-3, 100)
    assert "sk_sep_solve" not in sk.sinkhorn_describe(2, 4096, 4096, 0, 2e-3, 100)
    for k in ("alpha", "beta", "loss"):
        x, y = out[k][:2].double(), few[k].double()
        # the sweeps' own exponents are rounded at the size of the potentials (2^-24 of ~1000, a few sums deep)
        assert float((x - y).norm() / y.norm()) <= 5e-6, k


# One entry moved by 1, where plan has mass: rows and columns in the first work-groups of the cost's test, in late ones,
# and the last entry.
ENTRIES = [(0, 1), (77, 101), (130, 127), (195, 195)]


@pytest.mark.parametrize("case", ENTRIES + ["spread", "nan"])
def test_cost_left_to_the_sweeps(case):
    mu, nu, C = make(16, 3, (14, 14), (14, 14), "sq")
    lam, split = 0.03, C.copy()
    if case == "nan":
        C[77, 101] = np.nan
        out = sk.sinkhorn_forward(_t(mu), _t(nu), _t(C), lam, 170)
        assert torch.isnan(out["loss"]).all()
        return
    if case == "spread":
        lam = 3e-4  # 4 neighbours span more than 150 bits
    else:
        C[case] -= 1.0
    out = {k: v.cpu().numpy() for k, v in sk.sinkhorn_forward(_t(mu), _t(nu), _t(C), lam, 170).items()}
    log = {k: v.cpu().numpy() for k, v in sk.sinkhorn_forward_select("log", _t(mu), _t(nu), _t(C), lam, 170).items()}
    ref = oracle.forward(mu, nu, C[None], lam, 170)
    if case != "spread":  # dropping the entry would show in every result
        other = oracle.forward(mu, nu, split[None], lam, 170)
        assert loss_rel_err(other["loss"], ref["loss"]) > 1e-2
        assert max(gauge_fixed_errors(mu, nu, other["alpha"], other["beta"], ref["alpha"], ref["beta"])) > 1e-1
    assert loss_rel_err(out["loss"], ref["loss"]) <= 1e-4
    ea, eb = gauge_fixed_errors(mu, nu, out["alpha"], out["beta"], ref["alpha"], ref["beta"])
    assert max(ea, eb) <= 1e-3 * max(1.0, 0.03 / lam)
    for k in out:
        np.testing.assert_array_equal(out[k], log[k])  # the sweeps


@pytest.mark.parametrize("d, at", [(4096, (4095, 4095)), (4096, (4094, 63)), (1600, (1, 1599))])
def test_every_entry_of_a_large_cost_counts(d, at):
    """Rows beyond the first pass of the cost's test (1024 work-groups of four)."""
    h = int(d ** 0.5)
    mu, nu, C = make(17, 8, (h, h), (h, h), "sq")
    C[at] += 1e-3
    out = sk.sinkhorn_forward(_t(mu), _t(nu), _t(C), 0.05, 150)
    log = sk.sinkhorn_forward_select("log", _t(mu), _t(nu), _t(C), 0.05, 150)
    assert "sk_sep_solve" in sk.sinkhorn_describe(8, d, d, 0, 0.05, 150)
    for k in out:
        assert torch.equal(out[k], log[k]), k


def returned_error(g, mu, nu, C, lam, side):
    """||P 1 - mu||_1 + ||P^T 1 - nu||_1 of the returned potentials, in 64 bits, with the library's fp32 scale of the
    cost, log2(e) / lam, and the cost that splits: the sum of the entries of its first rows and columns."""
    s = np.float64(np.float32(1.4426950408889634) / np.float32(lam)) * np.log(2.0)
    D = C.astype(np.float64).reshape(side, side, side, side)
    D = D[:, :1, :, :1] + D[:1, :, :1, :] - D[0, 0, 0, 0]
    D = D.reshape(C.shape)
    out = []
    for b in range(mu.shape[0]):
        P = np.exp(g["alpha"][b].astype(np.float64)[:, None] + g["beta"][b].astype(np.float64)[None, :] - s * D)
        out.append(np.abs(P.sum(1) - mu[b]).sum() + np.abs(P.sum(0) - nu[b]).sum())
    return np.array(out)


@pytest.mark.parametrize("side, lam, tol, n_iter", [
    (28, 0.01, 0.0, 300),     # converged below the rounding of the potentials
    (32, 0.002, 2e-6, 2000),  # a tolerance below that rounding
    (28, 0.02, 2e-5, 2000),   # and above it
    (40, 0.004, 2e-6, 2000),  # lines of up to 64 entries: one plane of v
    (40, 0.004, 0.0, 700),
])
def test_split_marginal_error_is_the_returned_iterates(side, lam, tol, n_iter):
    """marg_err speaks of the returned fp32 potentials, their rounding included; the early stop of the iterate, as the
    oracle's does."""
    p = workloads.image(seed=21, B=8, side=side, n_iter=n_iter, lam=lam)
    mu, nu, C = p.mu, p.nu, p.C[0]
    assert "sk_sep_solve" in sk.sinkhorn_describe(8, side ** 2, side ** 2, 0, lam, n_iter, tol)
    g = {k: v.cpu().numpy() for k, v in sk.sinkhorn_forward(_t(mu), _t(nu), _t(C), lam, n_iter, tol).items()}
    true = returned_error(g, mu, nu, C, lam, side)
    print(f"[split] side={side} lam={lam} tol={tol} iters {g['iters']} reported {g['marg_err']} true {true}",
          file=sys.stderr, flush=True)
    # the line sums' own rounding: a few 2^-24 of a unit mass on either side
    assert np.all(np.abs(g["marg_err"] - true) <= 2e-7 + 1e-3 * true)
    if tol == 2e-5:
        free = oracle.forward(mu, nu, C[None], lam, n_iter, tol=tol)
        assert np.all(np.abs(free["iters"] - g["iters"]) <= 1)


@pytest.mark.parametrize("value", [np.nan, -0.25])
def test_split_bad_mass_reaches_the_marginal_error(value):
    """A NaN in nu makes the sample's marginal error NaN, a negative mass counts as missed (as in the sweeps); neither
    lets the sample stop."""
    mu, nu, C = make(22, 4, (18, 17), (18, 17), "sq")
    bad = nu.copy()
    bad[1, 40] = value
    run = lambda n, select: {k: v.cpu().numpy() for k, v in
                             sk.sinkhorn_forward_select(select, _t(mu), _t(n), _t(C), 0.05, 200, 1e-3).items()}
    good, out = run(nu, "default"), run(bad, "default")
    assert np.all(good["iters"] < 200) and out["iters"][1] == 200
    if np.isnan(value):
        assert np.isnan(out["marg_err"][1])
    else:
        assert out["marg_err"][1] >= 0.25
    rest = [0, 2, 3]
    for k in good:
        np.testing.assert_array_equal(out[k][rest], good[k][rest])


def test_log_selector_reaches_the_sweeps():
    mu, nu, C = make(23, 8, (14, 14), (14, 14), "sq")
    assert "sk_sep_solve" in sk.sinkhorn_describe(8, 196, 196, 0, 0.03, 170)
    line = sk.sinkhorn_describe(8, 196, 196, 0, 0.03, 170, select="log")
    assert "sk_sep_solve" not in line and "matrix products" not in line
    solve = sk.sinkhorn_forward(_t(mu), _t(nu), _t(C), 0.03, 170)
    sweeps = sk.sinkhorn_forward_select("log", _t(mu), _t(nu), _t(C), 0.03, 170)
    ref = oracle.forward(mu, nu, C[None], 0.03, 170)
    for out in (solve, sweeps):
        g = {k: v.cpu().numpy() for k, v in out.items()}
        assert loss_rel_err(g["loss"], ref["loss"]) <= 1e-5
    assert not torch.equal(solve["alpha"], sweeps["alpha"])  # other arithmetic: it was the sweeps that ran
