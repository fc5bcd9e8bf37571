"""GPU parity of the offline construction where its kernels change route: the
one-workgroup solve up to 128 features and the launch-per-product solve past
it, iterations long enough to restart their scaling, products on and off the
16-byte tile path, and covariance tiles at their edges.  Tolerances as in
test_gpu_recolor: 4 k eps for products and moments, 1e-8 for the solve."""

import numpy as np
import pytest

from oracle import recolor as rc

pytestmark = pytest.mark.gpu

EPS = np.finfo(np.float64).eps


@pytest.fixture(scope="module")
def hf():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_32259_amd import heterofold
    heterofold.lib()
    return heterofold


def _dev(a):
    import torch
    return torch.as_tensor(np.ascontiguousarray(a, np.float64), device="cuda")


def _np(t):
    import torch
    torch.cuda.synchronize()
    return t.cpu().numpy()


@pytest.mark.parametrize("p,q", [(128, 128), (129, 20), (20, 129), (33, 32), (16, 17), (260, 130)])
def test_solve_on_both_sides_of_the_one_workgroup_limit(hf, p, q):
    from paper_2609_32259_amd import synth
    cfg = synth.CalibConfig("route", n=3000, p=p, q=q)
    x, y, w = synth.make_calibration(cfg, seed=5, device="cuda")
    print(f"[gpu-recolor] route p={p} q={q}", flush=True)
    r, mu, cov = hf.hf_recolor_moments(x, y, w)
    A, b, info = hf.hf_recolor_solve(mu, cov, p, ridge=1e-6)
    inf = hf.recolor_info(info)
    assert inf["converged"] == [1, 1, 1], inf
    M, c = _np(mu), _np(cov)
    A_ref, b_ref = rc.recolor(M[:p], M[p:], c[:p, :p], c[:p, p:], c[p:, p:], 1e-6)
    A_ref = rc.abi_orientation(A_ref)
    assert np.linalg.norm(_np(A) - A_ref) <= 1e-8 * np.linalg.norm(A_ref)
    assert np.linalg.norm(_np(b) - b_ref) <= 1e-8 * (np.linalg.norm(b_ref) + np.linalg.norm(A_ref))


@pytest.mark.parametrize("p,q", [(40, 8), (150, 20)])
def test_solve_restarts_the_scaling_on_ill_conditioned_roots(hf, p, q):
    # eigenvalues 1 .. 1e-12 of S_Z: plain steps need about 40 iterations, scaled
    # ones go past their first schedule.  A S_Z A^T = S_Y holds to kappa eps.
    rng = np.random.default_rng(6)
    U, _ = np.linalg.qr(rng.standard_normal((p, p)))
    e = np.logspace(0, -12, p)
    Sz = (U * e) @ U.T
    Sz = 0.5 * (Sz + Sz.T)
    G = (U * np.sqrt(e)) @ np.linalg.qr(rng.standard_normal((p, q)))[0]  # S_ZY of y = Q^T whitened z
    cov = np.block([[Sz, G], [G.T, np.eye(q)]])
    A, b, info = hf.hf_recolor_solve(_dev(np.zeros(p + q)), _dev(cov), p)
    inf = hf.recolor_info(info)
    print(f"[gpu-recolor] ill-conditioned p={p}: {inf}", flush=True)
    assert inf["converged"][0] == 1 and inf["iterations"][0] > 20, inf
    Am = _np(A)
    assert np.linalg.norm(Am @ Sz @ Am.T - np.eye(q)) <= 1e12 * EPS * 100


@pytest.mark.parametrize("ak,bk", [(False, True), (True, True), (False, False), (True, False)])
@pytest.mark.parametrize("m,n,k", [(256, 128, 64), (129, 65, 48), (127, 63, 15), (300, 200, 33)])
def test_gemm_tile_edges(hf, ak, bk, m, n, k):
    rng = np.random.default_rng(m + n + k)
    opA, opB = rng.standard_normal((m, k)), rng.standard_normal((k, n))
    D = hf.hf_gemm_f64(_dev(opA.T if ak else opA), _dev(opB if bk else opB.T), a_kmajor=ak, b_kmajor=bk)
    ref = opA @ opB
    assert np.all(np.abs(_np(D) - ref) <= 4 * k * EPS * (np.abs(opA) @ np.abs(opB)) + 1e-300)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n,p,q", [(47, 60, 68), (2000, 132, 4), (513, 126, 6), (33, 61, 66)])
def test_moments_at_tile_edges(hf, dtype, n, p, q):
    # 128 columns exactly, 4 columns past a tile (groups of 4 whole in x or y), and
    # groups that straddle x and y (read one by one); a few zero weights
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    x = torch.randn((n, p), generator=g, device="cuda").to(dt)
    y = (torch.randn((n, q), generator=g, device="cuda") + 0.5).to(dt)
    w = torch.rand(n, generator=g, device="cuda")
    w[::7] = 0.0
    r, mu, cov = hf.hf_recolor_moments(x, y, w)
    X, Y, W = (t.double().cpu().numpy() for t in (x, y, w))
    rr = rc.sender_rms(X, W)
    V = np.concatenate([X / rr, Y], axis=1)
    m = W @ V / W.sum()
    D = V - m
    ref = (D * W[:, None]).T @ D / W.sum()
    bound = 16 * n * EPS * ((np.abs(D) * W[:, None]).T @ np.abs(D) / W.sum()) + 1e-14
    got = _np(cov)
    assert np.all(np.abs(got - ref) <= bound)
    np.testing.assert_array_equal(got, got.T)
