"""GPU parity across the accepted hyperparameter range.

The posterior's triangular product scales both of its operands by powers of
two before their fp16 hi/lo split (the candidates' kernel values per
candidate, L^{-1} per 16-row block), so its error is that of fp32 arithmetic
whatever the output scale or the noise. These cases hold the HIP path to the
parity bar at output scales 1e-3 and 1e3 and at noise 1e-6 and 0 (away from
the data, and near it through the variance bound), check the fp32 error
model at hyperparameters learned by maximising the marginal likelihood
(implementation section), the conditioning limit (BO_ERR_ILL_CONDITIONED),
and that a NaN candidate yields NaN and never wins the argmax.
"""
import math

import numpy as np
import pytest

import bo_inputs as bi
import oracle as O
from gpu_util import (TOL_MU, TOL_SIGMA, TOL_EHVI, gpu_run, oracle_fit, oracle_score,
                      assert_close, check_argmax, log_ratio, near_var_tol, oracle_ehvi_given,
                      to_dev)

pytestmark = pytest.mark.gpu

# (config, M, seed): sizes the oracle finishes in seconds, ragged against the
# 64-point posterior tiles and the 256-candidate EHVI blocks
CASES = [(0, 4096, 0), (2, 2003, 1)]


def _announce(*a):
    print("[case]", *a, flush=True)


def _full_parity(wl, g, o, what):
    assert_close(g["mu"], o["mu"], TOL_MU, f"mu {what}")
    assert_close(g["sigma"], o["sigma"], TOL_SIGMA, f"sigma {what}")
    assert_close(g["ehvi"], o["ehvi"], TOL_EHVI, f"ehvi {what}")
    check_argmax(g["idx"], o["ehvi"])


def _near_data(wl, what, count=384):
    """Candidates within ~0.01 of observations and the observations
    themselves: mu at the bar, the variance through the near-data bound.
    At the observations sigma is near zero (exactly zero without noise) and
    resolved by fp32 only to the square root of that bound, which the
    acquisition inherits; so the EHVI stage is held to the bar on the GPU's own
    posterior (the oracle's EHVI of the GPU's mu and sigma), and to the
    oracle's EHVI directly wherever sigma^2 is resolved to better than 1e-3
    relative."""
    near = bi.near_data_candidates(wl, count, scale=0.01)
    at = wl.X[: min(wl.n, 128)][:, None, :].astype(np.float32)
    cand = np.concatenate([near, at], axis=0)
    g = gpu_run(wl, cand=cand)
    o = oracle_score(oracle_fit(wl), wl, cand=cand)
    assert_close(g["mu"], o["mu"], TOL_MU, f"mu near data {what}")
    vt = near_var_tol(float(np.max(wl.outputscale)))
    assert_close(g["sigma"] ** 2, o["sigma"] ** 2, vt, f"variance near data {what}")
    assert_close(g["ehvi"], oracle_ehvi_given(g["mu"], g["sigma"], wl.Z, o), TOL_EHVI,
                 f"ehvi of the GPU posterior near data {what}")
    resolved = np.all(o["sigma"][:, 0, :] ** 2 >= 1e3 * vt[1], axis=1)
    assert resolved.sum() >= count // 2
    assert_close(g["ehvi"][resolved], o["ehvi"][resolved], TOL_EHVI,
                 f"ehvi near data (sigma resolved) {what}")


@pytest.mark.parametrize("s", [1e-3, 1e3])
@pytest.mark.parametrize("cfg,M,seed", CASES)
def test_outputscale_parity(cfg, M, seed, s):
    _announce("outputscale", cfg, M, seed, s)
    wl = bi.make_config(cfg, seed=seed, M=M)
    wl.outputscale = np.full(wl.m, s, dtype=np.float32)
    g = gpu_run(wl)
    o = oracle_score(oracle_fit(wl), wl)
    _full_parity(wl, g, o, f"cfg{cfg} s={s:g}")
    _near_data(wl, f"cfg{cfg} s={s:g}")


@pytest.mark.parametrize("eta", [1e-6, 0.0])
@pytest.mark.parametrize("cfg,M,seed", CASES)
def test_small_and_zero_noise_parity(cfg, M, seed, eta):
    """Noise 1e-6 and exactly 0: the training inputs are well separated at
    these lengthscales (the Gram matrices' smallest eigenvalues are near 0.5),
    so the model stays well conditioned while the posterior variance at the
    data drops to (almost) zero."""
    _announce("noise", cfg, M, seed, eta)
    wl = bi.make_config(cfg, seed=seed, M=M)
    wl.noise = np.full(wl.m, eta, dtype=np.float32)
    g = gpu_run(wl)
    o = oracle_score(oracle_fit(wl), wl)
    _full_parity(wl, g, o, f"cfg{cfg} eta={eta:g}")
    _near_data(wl, f"cfg{cfg} eta={eta:g}")


def _learn_hyperparameters(wl):
    """Maximise each objective's exact marginal likelihood over
    (log l, log s, log eta) with L-BFGS on bo_mll (the GPU likelihood)."""
    import paper_2602_10729_amd as bo
    from scipy.optimize import minimize
    d = wl.d
    X = to_dev(wl.X)
    ls = np.empty((wl.m, d), np.float32)
    s = np.empty(wl.m, np.float32)
    eta = np.empty(wl.m, np.float32)
    for k in range(wl.m):
        Yk = to_dev(np.ascontiguousarray(np.repeat(wl.Y[:, k:k + 1], 2, axis=1)))

        def unpack(th):
            th = np.clip(th, [-6.0] * d + [-6.0, -16.0], [4.0] * d + [6.0, 2.0])
            return (np.repeat(np.exp(th[:d]).astype(np.float32)[None], 2, 0),
                    np.full(2, np.exp(th[d]), np.float32), np.full(2, np.exp(th[d + 1]), np.float32))

        def f(th):
            v, gr = bo.mll(X, Yk, *unpack(th))
            return -v[0], -gr[0]
        th0 = np.concatenate([np.log(wl.lengthscale[k].astype(np.float64)), [0.0, math.log(1e-4)]])
        r = minimize(f, th0, jac=True, method="L-BFGS-B", options=dict(maxiter=80))
        a, b, c = unpack(r.x)
        ls[k], s[k], eta[k] = a[0], b[0], c[0]
    return ls, s, eta


def test_learned_hyperparameters_fp32_error_model():
    """At the marginal-likelihood optimum of config 0 (lengthscales ~3,
    output scales ~20-40, noise ~1e-6: cond(K) ~ 1e5) every posterior sits
    far below its prior, where fp32 arithmetic bounds the error absolutely:
      |mu_g - mu_o| <= 1e-4 |mu_o| + 1e-5 + 2^-18 sum_i |k_i alpha_i|
      |sigma_g^2 - sigma_o^2| <= 1e-4 sigma_o^2 + 64 2^-24 k(x, x)
    (the second is the near-data bound with 64 units of 2^-24 instead of 24:
    the conditioning roughly doubles the error). The relative error of sigma
    itself is logged: this is the regime where the scores need more than
    fp32."""
    _announce("learned hyperparameters")
    wl = bi.make_config(0, seed=0, M=2048)
    wl.lengthscale, wl.outputscale, wl.noise = _learn_hyperparameters(wl)
    print("[learned]", wl.lengthscale.min(), wl.lengthscale.max(), wl.outputscale, wl.noise,
          flush=True)
    near = bi.near_data_candidates(wl, 256, scale=0.01)
    cand = np.concatenate([wl.cand, near], axis=0)
    g = gpu_run(wl, cand=cand)
    model = oracle_fit(wl)
    o = oracle_score(model, wl, cand=cand)
    P = cand[:, 0, :].astype(np.float64)
    for k in range(wl.m):
        Ks = model.cov(k, P, model.X)
        sabs = np.abs(Ks) @ np.abs(model.alpha[k])
        mu_tol = TOL_MU[0] * np.abs(o["mu"][:, 0, k]) + TOL_MU[1] + 2.0 ** -18 * sabs
        assert_close(g["mu"][:, 0, k], o["mu"][:, 0, k], (0.0, mu_tol), f"mu learned k={k}")
        var_tol = near_var_tol(float(wl.outputscale[k]), ulps=64)
        assert_close(g["sigma"][:, 0, k] ** 2, o["sigma"][:, 0, k] ** 2, var_tol,
                     f"variance learned k={k}")
        rel = np.abs(g["sigma"][:, 0, k] - o["sigma"][:, 0, k]) / o["sigma"][:, 0, k]
        log_ratio(f"sigma relative error learned k={k} (informational)", float(rel.max()))


def _near_duplicate_workload():
    wl = bi.make_config(0, seed=0, M=8)
    X = wl.X.copy()
    X[5] = X[3]
    X[5, 0] += 1e-5            # 1e-5 apart (3.3e-5 in scaled units)
    wl.X = X
    return wl


def test_near_duplicates_without_noise_are_refused():
    """Two observations 1e-5 apart and zero noise: max K_ii max|L^-1|^2 is far
    beyond 2^24 (L^-1 reaches ~1e5), so bo_fit refuses the model."""
    import paper_2602_10729_amd as bo
    _announce("ill-conditioned fit")
    wl = _near_duplicate_workload()
    wl.noise = np.zeros(wl.m, np.float32)
    with pytest.raises(bo.BoError) as ei:
        bo.fit(to_dev(wl.X), to_dev(wl.Y), wl.lengthscale, wl.outputscale, wl.noise)
    assert ei.value.name == "BO_ERR_ILL_CONDITIONED", str(ei.value)


def test_noisy_acquisition_refuses_a_singular_noise_free_factor():
    """With noise 1e-4 the same observations fit (the noise regularises K),
    but the noisy acquisition conditions on the noise-free K_XX, which the
    near-duplicates make singular: bo_nehvi_prepare refuses it."""
    import paper_2602_10729_amd as bo
    _announce("ill-conditioned noise-free factor")
    wl = _near_duplicate_workload()
    model = bo.fit(to_dev(wl.X), to_dev(wl.Y), wl.lengthscale, wl.outputscale, wl.noise)
    ZX = to_dev(np.random.default_rng(0).standard_normal((16, wl.n, wl.m)).astype(np.float32))
    with pytest.raises(bo.BoError) as ei:
        bo.nehvi_prepare(model, ZX, wl.ref)
    assert ei.value.name == "BO_ERR_ILL_CONDITIONED", str(ei.value)


@pytest.mark.parametrize("q", [1, 2])
def test_nan_candidate_gives_nan_and_never_wins(q):
    """A candidate with a NaN coordinate gets NaN mu, sigma and acquisition
    (no clamp turns its variance into 0), the others are unaffected, and the
    argmax skips it."""
    _announce("nan candidate", q)
    wl = bi.make_config(0, seed=0, M=300)
    rng = np.random.default_rng(3)
    cand = rng.random((300, q, wl.d)).astype(np.float32)
    Z = rng.standard_normal((wl.S, q, wl.m)).astype(np.float32)
    bad = [17, 250]
    cand[17, q - 1, 2] = np.nan
    cand[250, 0, :] = np.nan
    g = gpu_run(wl, cand=cand, Z=Z)
    for b in bad:
        assert np.isnan(g["ehvi"][b])
        assert np.isnan(g["mu"][b]).any() and np.isnan(g["sigma"][b]).any()
    ok = np.setdiff1d(np.arange(300), bad)
    assert np.isfinite(g["ehvi"][ok]).all()
    o = oracle_score(oracle_fit(wl), wl, cand=cand[ok], Z=Z)
    assert_close(g["mu"][ok], o["mu"], TOL_MU, f"mu beside NaN q={q}")
    assert_close(g["ehvi"][ok], o["ehvi"], TOL_EHVI, f"ehvi beside NaN q={q}")
    assert g["idx"] not in bad
    check_argmax(g["idx"], o["ehvi"], idx_pool=ok)


def _far_pair_error(X, ls, cand):
    """Relative error of mu where one observation alone carries it: the error
    of its kernel value, for candidates far from it (no exact differences)."""
    M = len(cand)
    wl = bi.make_config(0, seed=0, M=M)
    wl.X, wl.n, wl.d = X, 2, X.shape[1]
    wl.Y = np.array([[1, 1], [0, 0]], np.float32)
    wl.lengthscale = np.stack([ls, ls]).astype(np.float32)
    wl.outputscale, wl.noise = np.ones(2, np.float32), np.full(2, 1e-4, np.float32)
    wl.cand = np.ascontiguousarray(cand.reshape(M, 1, -1), dtype=np.float32)
    wl.Z = wl.Z[:4].copy()
    wl.ref = np.array([-1, -1], np.float32)
    g, o = gpu_run(wl), oracle_score(oracle_fit(wl), wl)
    return (g["mu"][:, 0, 0] - o["mu"][:, 0, 0]) / o["mu"][:, 0, 0]


def test_small_cross_terms_count():
    """The products of a large coordinate's low half with a small one reach r^2.
    x = +-(1 + 2^-11) in each of 32 dimensions, candidates c in [0, 2^-12]: those
    products add up to 32 * 2^-11 * 2^-13 = 1.9e-6, half an fp32 ulp of the norms
    (33), so an accumulator that already holds the norms loses them. Then r^2 is
    off by +-3.8e-6 for c and -c and the kernel values (r = 5.7: |d ln k / d r^2|
    = 0.17) by 1.3e-6 against each other. The roundings of r^2 and k, 5e-7 a
    value, are another for every candidate: the mean difference over 8192 of
    each sign is 8e-9 by their spread, and below 4e-8 where c or x have other
    sizes (the errors of the hardware's sqrt and exp2 are no pure noise)."""
    r = np.random.default_rng(3)
    x = np.full((1, 32), 1 + 0.499 * 2.0 ** -10, np.float32)
    c = (2.0 ** -12 * r.random((8192, 32))).astype(np.float32)
    _announce("small cross terms")
    e = _far_pair_error(np.concatenate([x, -x]), np.ones(32), np.concatenate([c, -c]))
    diff = float(np.mean(e[:8192] - e[8192:]))
    log_ratio("small cross terms, mean difference", abs(diff) / 2e-7)
    assert abs(diff) < 2e-7, diff


def test_kernel_values_carry_no_common_error():
    """A rounded constant in the exponent moves every kernel value the same
    way: 3.4e-8 of the exponent sqrt5 r is 2.3e-7 of k at r = 3. Candidates at
    r = 2.5 .. 3.5 of one observation (the other far away: its norm asks for
    exact differences everywhere), 16 different lengthscales. The fp32 rates of
    the coordinates are each within 2^-24, in rms below 2^-24 / sqrt3 and
    independent, so r within 2^-24 / sqrt3 / sqrt16 = 8.6e-9 and k (|d ln k / d ln
    r| = 5.1 at r = 3) within 4.4e-8: twice that, and 1e-8 for the constants of
    the polynomial (ln2, ln2^2 / 3 and their products with the scale)."""
    r = np.random.default_rng(4)
    ls = (0.5 + r.random(16)).astype(np.float32)
    u = r.standard_normal((8192, 16))
    u *= (2.5 + r.random((8192, 1))) / np.linalg.norm(u, axis=1, keepdims=True)
    x = (0.2 * r.standard_normal(16)).astype(np.float32)
    far = (x + 20.0 * ls).astype(np.float32)
    _announce("common error")
    e = _far_pair_error(np.stack([x, far]), ls, x + u * ls)
    mean = float(np.mean(e))
    log_ratio("kernel values, mean relative error", abs(mean) / 1e-7)
    assert abs(mean) < 1e-7, mean
