"""Kernels at the sizes where their work split can go wrong (chunk and tile remainders, the smallest
sizes), each against the oracle with the tolerance of its family's parity tests."""
import numpy as np
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2506_14792_amd as sps  # noqa: E402
from test_gpu_closure import test_closure_net_forward_and_vjp as check_closure_net  # noqa: E402

dev = lambda a: torch.from_numpy(np.ascontiguousarray(a).view(np.float64).ravel().copy()).cuda()


# a chunk of 64 pixels cut by the image's end, rows of one and of three 32-pixel segments, images whose
# chunks of 512 pixels end inside a wave's quarter
@pytest.mark.parametrize("shape", [(1, 3, 32), (3, 5, 32), (2, 9, 96)], ids=["3x32", "5x32x3", "9x96x2"])
def test_closure_net_ragged_chunks(shape):
    check_closure_net(shape)


# one step, one more step than the summing block has threads
@pytest.mark.parametrize("nsteps", [1, 257])
def test_rollout_loss_steps(nsteps):
    from oracle.kolmo import Kolmogorov, rollout_loss_and_gradients
    N, dt = 16, 1e-3
    print(f"rollout loss, {nsteps} steps", flush=True)
    P = Kolmogorov(N, Re=1000.0, drag=0.1)
    v = [wl.kolmo_vorticity(seed=s, N=N)[0] for s in range(4)]
    tg = [v[1 + k % 3] for k in range(nsteps)]
    G = sps.Kolmogorov(2, N, Re=1000.0, dt=dt, max_steps=nsteps, drag=0.1)
    X0 = torch.cat([dev(v[0].T), dev(v[1].T)])
    T = torch.cat([torch.cat([dev(t.T), dev(t.T)]) for t in tg])
    J = torch.zeros(2, dtype=torch.float64, device="cuda")
    G.rollout(X0, T, nsteps, J=J)
    G.sync()
    for i in range(2):
        Jo = rollout_loss_and_gradients(P, v[i].reshape(-1, 1), [t.reshape(-1, 1) for t in tg], dt, nsteps)[0]
        assert abs(J[i].item() - Jo) < 1e-11 * Jo


# inverse iteration from the library's fixed start vector, iteration by iteration, on the smallest
# Chebyshev size, a size whose last block of eight rows is partial, and the largest; the solves' relative
# error is about eps times the condition number of sigma M + L_s (1e5 to 1e6 here)
@pytest.mark.parametrize("nx,nz,iters", [(8, 8, 1), (8, 10, 3), (24, 64, 2)])
def test_inverse_iteration_steps(nx, nz, iters):
    from oracle.rbc import RBC
    print(f"inverse iteration {nx}x{nz}, {iters}", flush=True)
    sigma, P = 0.3, RBC(Nx=nx, Nz=nz, Lx=4.0, Ra=1e5, Pr=1.0)
    G = sps.Problem(sps.RBC2D, nx, nz, 4.0, 1e5, 1.0, 1.5, 1e-3, 1, 1)
    lam, X, Y, _ = G.stability(sigma, iters)
    G.sync()
    s = np.arange(P.S)
    start = np.where(s < 3 * nz, 1.0 / (1 + s % nz) + 0.5j / (1 + s // nz), 0.0)
    Ls = P.stability_operator()
    for k in range(P.K):
        A, M = sigma * P.M[k] + Ls[k], P.M[k]
        x, y = start, start
        for _ in range(iters):
            z = np.linalg.solve(A, M @ x)
            mu, x = np.vdot(x, z), z / np.linalg.norm(z)
            z = np.linalg.solve(A.conj().T, M.conj().T @ y)
            y = z / np.linalg.norm(z)
        assert abs(lam[k].item() - (sigma - 1.0 / mu)) <= 1e-9 * abs(1.0 / mu)
        assert np.linalg.norm(X[k].cpu().numpy() - x) <= 1e-9
        assert np.linalg.norm(Y[k].cpu().numpy() - y) <= 1e-9
