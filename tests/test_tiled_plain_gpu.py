"""GPU parity of the plain form of the tiled regime (a shared cost that spans at
most 64 bits, products on the matrix cores): sizes around the 32 x 32 tiles,
zero masses, a cost just outside the range (the sweeps), and a problem whose
sums leave fp32's guarded range (solved again in the log domain)."""
import time

import numpy as np
import pytest
import torch

import oracle
import paper_1907_01729_amd as sk
import workloads
from parity_util import GRAD_RTOL, LOSS_RTOL, POT_ATOL, gauge_fixed_errors, loss_rel_err, rel_err_rows

pytestmark = pytest.mark.gpu


def _t(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to("cuda:0")


def run(mu, nu, C, lam, n_iter, sample):
    assert "matrix products" in sk.sinkhorn_describe(mu.shape[0], mu.shape[1], nu.shape[1], 0, lam, n_iter)
    out = {k: v.cpu().numpy() for k, v in sk.sinkhorn_forward(_t(mu), _t(nu), _t(C), lam, n_iter).items()}
    ref = oracle.forward(mu[sample], nu[sample], C, lam, n_iter)
    ea, eb = gauge_fixed_errors(mu[sample], nu[sample], out["alpha"][sample], out["beta"][sample], ref["alpha"],
                                ref["beta"])
    assert np.all(out["iters"] == n_iter)
    return out, ref, loss_rel_err(out["loss"][sample], ref["loss"]), max(ea, eb)


# Sums of d positive fp32 products: relative error of a potential <= (d + few) 2^-24 in the worst case, a few 2^-24
# in practice; the potentials (tens of units) are rounded to fp32 at the end.
LOSS, POT = 2e-6, 2e-5


@pytest.mark.parametrize("B, d1, d2, lam, zero", [
    (224, 640, 640, 0.05, 0.0),    # whole tiles
    (225, 641, 672, 0.05, 0.1),    # one row, one problem past a tile
    (255, 607, 801, 0.04, 0.1),    # one short of a tile
    (100, 1100, 1030, 0.023, 0.0),  # 62.7 bits
])
def test_plain_tiled(B, d1, d2, lam, zero):
    p = workloads.random_problem(41, B, d1, d2, lam, 120, zero_frac=zero)
    sample = [0, 1, 31, 32, B - 1]
    _, _, el, ep = run(p.mu, p.nu, p.C, lam, 120, sample)
    assert el <= LOSS and ep <= POT


@pytest.mark.parametrize("B, n_iter", [(38000, 1), (19000, 2)])
def test_plain_tiled_few_iterations(B, n_iter):
    """The last products are the first ones."""
    rng = np.random.default_rng(50)
    C = rng.random((640, 640), dtype=np.float32)
    mu, nu = (0.05 + rng.random((64, 640)) for _ in range(2))
    mu, nu = (np.tile((h / h.sum(1, keepdims=True)).astype(np.float32), (B // 64 + 1, 1))[:B] for h in (mu, nu))
    _, _, el, ep = run(mu, nu, C, 0.05, n_iter, [0, 63, 64, B - 1])
    assert el <= LOSS and ep <= POT


def test_cost_out_of_range():
    p = workloads.random_problem(42, 224, 640, 640, 0.0222, 120)  # 65 bits
    _, _, el, ep = run(p.mu, p.nu, p.C, p.lam, 120, [0, 223])
    assert el <= 1e-4 and ep <= 1e-3


def test_problem_out_of_range():
    p = workloads.random_problem(43, 224, 640, 640, 0.05, 120)
    mu, nu = p.mu.copy(), p.nu.copy()
    mu[7] *= np.float32(2.0 ** 112)  # not a histogram: as they are, these masses make sums of 2^103
    nu[7] *= np.float32(2.0 ** 112)
    out, ref, el, ep = run(mu, nu, p.C, p.lam, 120, [0, 6, 8, 223])
    assert el <= LOSS and ep <= POT
    one = oracle.forward(mu[7:8], nu[7:8], p.C, p.lam, 120)
    ea, eb = gauge_fixed_errors(mu[7:8], nu[7:8], out["alpha"][7:8], out["beta"][7:8], one["alpha"], one["beta"])
    assert max(ea, eb) <= 1e-3 and loss_rel_err(out["loss"][7:8], one["loss"]) <= 1e-4


def test_small_masses():
    """Masses down to fp32's smallest subnormal: a scaling may underflow, the potentials of the returned iterate may
    not, and the gradient of the sample (centred over the support) stays finite."""
    p = workloads.random_problem(44, 224, 640, 640, 0.05, 120)
    tiny = np.array([1e-30, 1e-38, 1e-43, 1.5e-45], np.float32)
    mu, nu = p.mu.copy(), p.nu.copy()
    mu[5, [3, 99, 400, 639]] = tiny
    nu[6, [3, 99, 400, 639]] = tiny
    mu[7, 100:104] = nu[7, 300:304] = tiny
    z = 15.0 * np.random.default_rng(45).standard_normal((2, 640))  # confident classifiers
    mu[9], nu[9] = (np.exp(z - z.max(1, keepdims=True)) / np.exp(z - z.max(1, keepdims=True)).sum(1, keepdims=True))
    sample = [4, 5, 6, 7, 9]
    assert (mu[9] < 1e-37).any() and (nu[9] < 1e-37).any()
    out, ref, el, ep = run(mu, nu, p.C, p.lam, 120, sample)  # finite on the supports
    # masses below 2^-126 have as few as one significant bit, the same for the oracle: the bounds stand
    assert el <= LOSS and ep <= 10 * POT, (el, ep)
    g = sk.sinkhorn_backward(torch.ones(224, device="cuda:0"), _t(mu), _t(nu), _t(p.C), p.lam, _t(out["alpha"]),
                             _t(out["beta"]))
    r = oracle.backward(np.ones(len(sample)), mu[sample], nu[sample], p.C, p.lam, ref["alpha"], ref["beta"])
    for k in ("grad_mu", "grad_nu"):
        assert rel_err_rows(g[k].cpu().numpy()[sample], r[k]) <= GRAD_RTOL


def test_masses_that_do_not_sum_to_one():
    """Masses of 64, 1 / 5 or 1.01 against 1 move the scalings by their ratio in every iteration, the first two out of
    fp32; as in the log domain, the potentials follow."""
    p = workloads.random_problem(49, 224, 640, 640, 0.05, 120, zero_frac=0.1)
    mu, nu = p.mu.copy(), p.nu.copy()
    mu[5] *= np.float32(64.0)
    mu[6] *= np.float32(0.2)
    mu[7] *= np.float32(1.01)
    nu[8] *= np.float32(1e-20)
    _, ref, el, ep = run(mu, nu, p.C, p.lam, 120, [4, 5, 6, 7, 8])
    # potentials of 120 log 64 = 500 and 119 log 1e20 = 5480, rounded to fp32 (2^-25 of them) and from base 2, and the
    # exponents of the plan with them
    top = 5500.0
    assert ep <= 2.0 ** -23 * top and el <= 2.0 ** -22 * top


@pytest.mark.parametrize("B, d1, d2", [(1024, 500, 400), (768, 400, 1000), (384, 500, 1030), (384, 300, 2100)])
def test_problem_solved_again(B, d1, d2):
    """The log-domain solve of a problem out of range, here by masses whose sum fp32 does not hold, at each of its
    column widths."""
    p = workloads.random_problem(46, B, d1, d2, 0.05, 60, zero_frac=0.1)
    mu, nu = p.mu.copy(), p.nu.copy()
    mu[7, :3] = nu[7, :3] = 1.2e38
    out, _, el, _ = run(mu, nu, p.C, p.lam, 60, [6])
    assert el <= LOSS
    one = oracle.forward(mu[7:8], nu[7:8], p.C, p.lam, 60)
    ea, eb = gauge_fixed_errors(mu[7:8], nu[7:8], out["alpha"][7:8], out["beta"][7:8], one["alpha"], one["beta"])
    assert max(ea, eb) <= POT_ATOL


def test_problem_without_mass():
    """Padded samples (no mass on one side, or on both) leave the other problems alone; without a row mass they come
    back as the sweeps give them."""
    p = workloads.random_problem(47, 224, 640, 640, 0.05, 120)
    mu, nu = p.mu.copy(), p.nu.copy()
    mu[7] = 0.0
    mu[8] = nu[8] = 0.0
    nu[9] = 0.0
    whole, out = ({k: v.cpu().numpy() for k, v in sk.sinkhorn_forward(_t(m), _t(n), _t(p.C), p.lam, 120).items()}
                  for m, n in ((p.mu, p.nu), (mu, nu)))
    log = {k: v.cpu().numpy() for k, v in
           sk.sinkhorn_forward_select("log", _t(mu), _t(nu), _t(p.C), p.lam, 120).items()}
    rest = [b for b in range(224) if b not in (7, 8, 9)]
    for k in out:
        np.testing.assert_array_equal(out[k][7:9], log[k][7:9], err_msg=k)
        np.testing.assert_array_equal(out[k][rest], whole[k][rest], err_msg=k)
    assert np.isneginf(out["alpha"][7]).all() and np.isneginf(out["beta"][8]).all() and out["loss"][8] == 0.0


@pytest.mark.parametrize("what", ["no mass", "sum 64", "sum above fp32"])
def test_time_with_a_problem_out_of_range(what):
    """A batch with such a problem costs no more than it does in the log-domain sweeps."""
    p = workloads.random_problem(48, 256, 1000, 1000, 0.05, 100)
    mu, nu = p.mu.copy(), p.nu.copy()
    if what == "no mass":
        mu[7] = 0.0
    elif what == "sum 64":
        mu[7] *= np.float32(64.0)
    else:
        mu[7, :3] = nu[7, :3] = 1.2e38
    m, n, C = _t(mu), _t(nu), _t(p.C)

    def best(f):
        ts = []
        for _ in range(4):
            torch.cuda.synchronize()
            t = time.perf_counter()
            f()
            torch.cuda.synchronize()
            ts.append(time.perf_counter() - t)
        return min(ts)

    sweeps = best(lambda: sk.sinkhorn_forward_select("log", m, n, C, 0.05, 100))
    plain = best(lambda: sk.sinkhorn_forward(m, n, C, 0.05, 100))
    print(f"{what}: {1e3 * plain:.2f} ms, in the sweeps {1e3 * sweeps:.2f} ms", flush=True)
    assert plain <= 1.1 * sweeps
