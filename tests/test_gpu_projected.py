"""The float64 projected solve (k_solve) by itself: the coefficients of a
solve against the oracle's projected Tikhonov problem on the GPU's own
Hessenberg matrix (rtg_arnoldi takes the same steps as rtg_solve), at the
edges of the kernel's row tiers and at odd and even column counts.

Both sides solve the same float64 problem.  mu is a root of a function whose
float64 evaluations differ by a few hundred eps (1e-13); its slope in log(mu)
is at least about 1e-4 of its value on these problems, so mu agrees to 1e-8
(bar 1e-6).  X is assembled in float32 from m + 1 terms: rounding of the
coefficients and of the sums, at most (m + 1) 2^-24 of sum |y_j| ||V_j||."""
import sys

import numpy as np
import pytest

from paper_2603_00839_amd import synth
from oracle.projected import projected_tikhonov, solve_14
import _util as U

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [1, 2, 3, 16, 17, 32, 33, 64, 65, 80, 81, 96])
@pytest.mark.parametrize("rule", ["discrepancy", "fixed", "unreachable"])
def test_projected_solve_matches_float64(m, rule):
    from paper_2603_00839_amd import rtg
    p = synth.small_problem(7, 48, 56, 3, 4, 3, 1, 24, 20, 3, m, nu=1e-2)
    op, sk = U.gpu_pair(p)
    C, delta = U.observation(p)
    Cd = U.to_dev(C)
    d = rtg.arnoldi(op, sk, Cd, m)
    k = int(d["m_done"].item())
    H, beta = d["H"].cpu().numpy()[:k + 1, :k], float(d["beta"].item())
    # a noise level between the least-squares residual and beta
    ls = projected_tikhonov(H, beta, mu=0.0)["res_proj"]
    target = {"discrepancy": np.sqrt(ls * beta), "unreachable": 0.5 * ls, "fixed": 0.0}[rule]
    mu = 1e-3 if rule == "fixed" else None
    ref = projected_tikhonov(H, beta, mu=mu, delta=target, eta=1.0)
    prm = rtg.make_params(m, rtg.F32, mu=-1.0 if mu is None else mu, delta=target, eta=1.0)
    X, ib = rtg.solve(op, sk, Cd, None, prm)
    info = rtg.read_info(ib)
    V = d["V"].cpu().numpy().reshape(m + 1, -1)[:k].astype(np.float64)
    want, got = ref["y"] @ V, X.cpu().numpy().astype(np.float64).ravel()
    scale = float(np.sum(np.abs(ref["y"]) * np.linalg.norm(V, axis=1)))
    err = float(np.linalg.norm(got - want))
    print(f"m {m} k {k} {rule}: mu {info.mu:.10e} ({ref['mu']:.10e}) res {info.res_proj:.10e} "
          f"({ref['res_proj']:.10e}) X err {err / scale:.2e}", file=sys.stderr, flush=True)
    assert info.iters == k and info.flags & ref["flags"] == ref["flags"]
    np.testing.assert_allclose(info.mu, ref["mu"], rtol=1e-6)
    np.testing.assert_allclose(info.res_proj, ref["res_proj"], rtol=1e-7)
    assert err <= (m + 1) * 2.0 ** -24 * scale


@pytest.mark.parametrize("m", [10, 40, 96])
@pytest.mark.parametrize("bits", [26, 24, 20])
def test_projected_solve_with_clustered_singular_values(m, bits):
    """Singular values within a few eps = 2^-bits of 1, where the SVD's
    rotations turn by large angles at cosines of eps and put back what earlier
    ones rotated away.  Phi shifts an image by one pixel and adds eps times the
    pixel and its other neighbour; from a single pixel and with Frobenius
    products every tensor and product is exact, and H is tridiagonal with ones
    below the diagonal and eps on and above it.

    y is read where the solve leaves it, in the caller's workspace (the only
    256-byte aligned run of float64 values close to the reference's), since X
    takes it rounded to float32.  Columns orthogonal to 1e-13 in every pair
    leave a relative error of at most (k - 1) 1e-13 s_max^2 / (s_min^2 + mu)
    in y; the bar is twice that for the roundings of the rotations."""
    import torch
    from paper_2603_00839_amd import rtg
    I1, I2, J, eps = 104, 40, 3, 2.0 ** -bits

    def band(n, taps):
        b = np.repeat(np.array([taps], np.float32), n, axis=0)
        b[0, 0] = b[-1, 2] = 0.0
        return b

    one = (0.0, 1.0, 0.0)
    op = rtg.setup_operator(I1, I2, J, band(I1, (1.0, eps, eps)), band(I2, one), band(J, one))
    sk = rtg.setup_sketch(I1, I2, J, None, None, None)
    C = np.zeros((I1, I2, J), np.float32)
    C[0, 5, 1] = 1.0
    Cd = U.to_dev(C)
    H = rtg.arnoldi(op, sk, Cd, m, bd_tol=0.0)["H"].cpu().numpy()
    want = np.eye(m + 1, m, k=-1) + eps * (np.eye(m + 1, m) + np.eye(m + 1, m, k=1))
    np.testing.assert_allclose(H, want, rtol=1e-15 + 4 * eps ** 2)    # (float32 sums of squares: 1 + eps^2)
    mu = 0.25
    # (the normal equations: H^T e_1 is of size eps and exact, unlike the SVD's U^T e_1)
    ref = solve_14(H, 1.0, mu)
    ws = torch.zeros(rtg.workspace_bytes(op, sk, m), dtype=torch.uint8, device="cuda")
    rtg.solve(op, sk, Cd, None, rtg.make_params(m, rtg.F32, mu=mu, bd_tol=0.0), ws=ws)
    words = ws[:ws.numel() // 256 * 256].view(torch.float64).cpu().numpy()
    rows = np.lib.stride_tricks.sliding_window_view(words, m)[::32]
    with np.errstate(all="ignore"):
        err = np.linalg.norm(rows - ref, axis=1) / np.linalg.norm(ref)
    err = np.sort(np.where(np.isfinite(err), err, np.inf))
    s = np.linalg.svd(H, compute_uv=False)
    print(f"m {m} eps 2^-{bits}: y err {err[0]:.2e} (next {err[1]:.1e})", file=sys.stderr, flush=True)
    assert err[1] > 1e-3
    assert err[0] <= 2 * (m - 1) * 1e-13 * s[0] ** 2 / (s[-1] ** 2 + mu)
