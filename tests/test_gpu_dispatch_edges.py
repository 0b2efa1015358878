"""GPU tests of the launch rules' edges: sizes either side of each line."""
import numpy as np
import pytest

import bo_inputs as bi
import oracle as O
from gpu_util import TOL_EHVI, gpu_run, oracle_ehvi_given, to_dev

pytestmark = pytest.mark.gpu


def _announce(*a):
    print("[case]", *a, flush=True)


@pytest.mark.parametrize("m,S", [(2, 1), (2, 15), (2, 17), (2, 255), (3, 257), (2, 4096)])
def test_single_point_ehvi_sample_groups(m, S):
    """q = 1: the samples' groups (remainders, empty groups) and the waves that
    share them. A candidate's value depends neither on the batch it is in nor
    on how many waves share its samples: the prefixes take 16, 8, 4, 2 and 1
    waves per 64 candidates. The first rows are checked against the oracle's
    boxes on the GPU's own posterior: sums of at most 4096 fp32 products whose
    factors carry a few units of 2^-24, far inside the parity bar."""
    wl = bi.make_config(0, seed=3, M=262145)
    if m == 3:
        y3 = (-np.sum(wl.X.astype(np.float64) ** 2, axis=1) / wl.d).astype(np.float32)
        wl.Y = np.concatenate([wl.Y, y3[:, None]], axis=1)
        wl.m = 3
        for f in ("lengthscale", "outputscale", "noise"):
            v = getattr(wl, f)
            setattr(wl, f, np.concatenate([v, v[:1]]))
        wl.ref = np.append(wl.ref, wl.Y[:, 2].min() - np.float32(0.1)).astype(np.float32)
    wl.Z = np.random.default_rng(S).standard_normal((S, 1, m)).astype(np.float32)
    full = gpu_run(wl)["ehvi"]
    for M in (1, 63, 65, 16384, 16385, 32769, 65537, 131073):
        _announce("ehvi groups", m, S, M)
        part = gpu_run(wl, cand=wl.cand[:M], want_musd=False)["ehvi"]
        np.testing.assert_array_equal(part, full[:M])
    g = gpu_run(wl, cand=wl.cand[:200])
    front = O.pareto_front(wl.Y.astype(np.float64), wl.ref.astype(np.float64))
    lo, hi = O.box_decomposition(wl.Y[front].astype(np.float64), wl.ref.astype(np.float64))
    want = oracle_ehvi_given(g["mu"], g["sigma"], wl.Z, {"lo": lo, "hi": hi})
    np.testing.assert_allclose(g["ehvi"], want, rtol=TOL_EHVI[0], atol=TOL_EHVI[1])


@pytest.mark.parametrize("cfg,n", [(2, n) for n in (1, 17, 129, 160, 161, 192, 256, 257, 511, 513, 545,
                                                    639, 641, 1024)] +
                         [(4, n) for n in (1025, 1057, 1537, 2047)])
def test_posterior_block_counts(cfg, n):
    """Observation counts either side of the posterior's chunk, pass and ring
    lines (32-row blocks: 5 are made before the first step, chunks of 4, passes
    of 16, two 128-row slots up to 256 rows), two tiles and a remainder."""
    from gpu_util import TOL_MU, TOL_SIGMA, oracle_fit, oracle_score
    wl = bi.make_config(cfg, seed=5, M=130 if cfg == 2 else 33)
    wl.X, wl.Y, wl.n = wl.X[:n].copy(), wl.Y[:n].copy(), n
    wl.Z = wl.Z[:16].copy()
    for comp in (None, bi.composite_hyperparameters(wl)):
        _announce("posterior blocks", cfg, n, comp is not None)
        g = gpu_run(wl, comp=comp)
        o = oracle_score(oracle_fit(wl, comp), wl)
        np.testing.assert_allclose(g["mu"], o["mu"], rtol=TOL_MU[0], atol=TOL_MU[1])
        np.testing.assert_allclose(g["sigma"], o["sigma"], rtol=TOL_SIGMA[0], atol=TOL_SIGMA[1])
        np.testing.assert_allclose(g["ehvi"], o["ehvi"], rtol=TOL_EHVI[0], atol=TOL_EHVI[1])


@pytest.mark.parametrize("n", [1, 15, 16, 17, 33, 47, 48, 64, 65, 127, 129, 200])
def test_diagonal_block_factor(n):
    """The 16-column panels of the 64x64 diagonal blocks: every panel and block
    remainder, against LAPACK in fp64 (inputs and results rounded to fp32 once:
    2^-24 relative; rows grow by at most the condition number, below 100), and
    an indefinite pivot in each panel of the first and second block."""
    import torch
    import paper_2602_10729_amd as bo
    _announce("diagonal factor", n)
    r = np.random.default_rng(n)
    B = r.standard_normal((n, n))
    A = (B @ B.T / n + np.eye(n)).astype(np.float32)
    up = np.triu(np.full((n, n), np.float32(7.0)), 1)            # above: not read
    L = bo.cholesky_test(torch.from_numpy(np.tril(A) + up).cuda()).cpu().numpy()
    np.testing.assert_allclose(L, np.linalg.cholesky(A.astype(np.float64)), rtol=2e-7, atol=2e-7)
    for j in range(0, n, 16):
        bad = A.copy()
        bad[j, j] = -1.0
        with pytest.raises(bo.BoError) as e:
            bo.cholesky_test(torch.from_numpy(bad).cuda())
        assert e.value.name == "BO_ERR_NOT_POSITIVE_DEFINITE"
