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
from test_couette_host import ROW_SIZES  # noqa: E402
from test_gpu_closure import test_closure_net_forward_and_vjp as check_closure_net  # noqa: E402
from test_gpu_couette import test_couette_explicit_term_and_solve as check_couette_F  # noqa: E402
from test_gpu_rbc import test_explicit_term_and_vjp as check_rbc_F  # noqa: E402
from test_gpu_rbc_batch import test_batch_against_oracle as check_rbc_batch  # noqa: E402
from test_gpu_ks import test_ks_F_vjp_and_solve as check_ks_F  # noqa: E402
from test_gpu_ks import test_ks_forward_and_gradient as check_ks_gradient  # noqa: E402
from test_gpu_ks import test_ks_rk_forward_and_gradient as check_ks_rk_gradient  # noqa: E402

dev = lambda a: torch.from_numpy(np.ascontiguousarray(a).view(np.float64).ravel().copy()).cuda()


# a chunk of 64 pixels cut by the image's end, rows of one and of three 32-pixel segments, images whose
# chunks of 512 pixels end inside a wave's quarter
@pytest.mark.parametrize("shape", [(1, 3, 32), (3, 5, 32), (2, 9, 96)], ids=["3x32", "5x32x3", "9x96x2"])
def test_closure_net_ragged_chunks(shape):
    check_closure_net(shape)


# numbers of blocks that are no multiple of the eight parts an image is dealt out in (9 and 17 blocks of tiles, 27 and
# 45 of weights), chunks that leave one and two waves of a block without work
@pytest.mark.parametrize("shape", [(5, 7, 32), (1, 33, 64)], ids=["7x32x5", "33x64"])
def test_closure_net_block_parts(shape):
    check_closure_net(shape)


# the input cotangent written over the output's, and half over it: the same bits as in a buffer of its own
@pytest.mark.parametrize("shift", [0, 1])
def test_closure_net_cotangent_in_place(shift):
    from oracle import closure as cl
    from test_gpu_closure import params
    print(f"closure net, cotangent in place, {shift}", flush=True)
    B, H, W = 4, 64, 64
    net, n = sps.ClosureNet(B, H, W), B * H * W
    theta = torch.from_numpy(cl.flatten(params(7))).cuda()
    net.set_params(theta)
    rng = np.random.default_rng(9)
    x, yb = (torch.from_numpy(rng.standard_normal(n)).cuda() for _ in range(2))
    xb, tb, tb2 = torch.zeros_like(x), torch.zeros_like(theta), torch.zeros_like(theta)
    net.vjp(x, yb, xb, tb)
    buf = torch.zeros(n + shift * n // 2, dtype=torch.float64, device="cuda")
    buf[:n] = yb
    out = buf[shift * n // 2:]
    net.vjp(x, buf[:n], out, tb2)
    torch.cuda.synchronize()
    assert torch.equal(out, xb) and torch.equal(tb, tb2)


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


# more steps than the loss's launch has blocks (4096): from the run's own states, the squared differences summed in
# numpy.  At most 4096 terms a lane and tree, all positive: 1e-12 and less
def test_rollout_loss_many_steps():
    from oracle.kolmo import Kolmogorov
    N, B, dt, n = 8, 2, 1e-4, 4099
    print(f"rollout loss, {n} steps", flush=True)
    P = Kolmogorov(N, Re=1000.0, drag=0.1)
    G = sps.Kolmogorov(B, N, Re=1000.0, dt=dt, max_steps=n, drag=0.1)
    X0 = torch.cat([dev(wl.kolmo_vorticity(seed=s, N=N)[0].T) for s in range(B)])
    rng = np.random.default_rng(3)
    T = torch.from_numpy(rng.standard_normal((n, X0.numel()))).cuda()
    J = torch.zeros(B, dtype=torch.float64, device="cuda")
    snap = torch.zeros(n * B * N * N, dtype=torch.float64, device="cuda")
    G.rollout(X0, T.reshape(-1), n, J=J)
    G.forward(X0, n, snap=snap, every=1, nc=N)
    G.sync()
    view = lambda t: t.cpu().numpy().view(np.complex128).reshape(n, B, N // 2, N).transpose(0, 1, 3, 2)
    e = view(snap) - view(T)
    e[:, :, N // 2] = 0.0
    for b in range(B):
        ref = np.mean([np.mean(P.T.to_grid(c, N) ** 2) for c in e[:, b]])
        assert abs(J[b].item() - ref) <= 1e-11 * ref


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


# plane Poiseuille flow: inverse iteration from the library's fixed start vector, iteration by iteration,
# in the band's coordinates, at sizes whose last block of eight rows holds 5 (the smallest, S = 29), 8, 1
# and 5 (the largest, S = 773) of them, several systems at once.  Each solve's backward error is at most
# S u |A| on both sides, so its result is within S u cond(A) of the exact one.
@pytest.mark.parametrize("nz,iters", [(8, 1), (9, 3), (220, 2), (256, 1)])
def test_poiseuille_inverse_iteration_steps(nz, iters):
    print(f"Poiseuille inverse iteration {nz}, {iters}", flush=True)
    prm = [(1.0, 5000.0, 0.01 - 0.23j), (1.02, 6000.0, -0.02 - 0.28j), (0.8, 900.0, 0.05 - 0.3j)]
    G = sps.PoiseuilleStability(nz, len(prm))
    n, S = len(prm), 3 * nz + 5
    lam, dlam, info, X, Y = (torch.zeros(q * n, dtype=torch.float64, device="cuda") for q in (2, 4, 3, 2 * S, 2 * S))
    G.solve(prm, lam, dlam, info, iters=iters, X=X, Y=Y)
    G.sync()
    lam, X, Y = (t.cpu().numpy().view(complex).reshape(n, -1) for t in (lam, X, Y))
    dense = lambda h: sum(np.diag(h["band"][max(0, -o):S - max(0, o), o + h["kl"]], o) for o in range(-h["kl"], h["ku"] + 1))
    i = np.arange(S)
    start = 1.0 / (1 + i % 7) + 0.5j / (1 + i % 5)
    for q, (alpha, Re, sigma) in enumerate(prm):
        h = sps.poiseuille_host_band(nz, alpha, Re, sigma)
        A = dense(h)
        M = dense(sps.poiseuille_host_band(nz, alpha, Re, sigma + 1.0)) - A
        x = y = start / np.linalg.norm(start)
        for _ in range(iters):
            z = np.linalg.solve(A, M @ x)
            mu, size, x = np.vdot(x, z), np.linalg.norm(z), z / np.linalg.norm(z)
            z = np.linalg.solve(A.conj().T, M.conj().T @ y)
            y = z / np.linalg.norm(z)
        tol = 2 * iters * S * 2.0 ** -53 * np.linalg.cond(A)
        c = np.zeros(S, complex)
        c[h["colmap"]] = x
        c[:-2] += h["rho"][:-2] * c[2:]
        r = np.zeros(S, complex)
        r[h["rowmap"]] = y
        print(f"  tolerance {tol:.1e}", flush=True)
        assert abs(lam[q, 0] - (sigma - 1.0 / mu)) <= tol * size / abs(mu) ** 2
        assert np.linalg.norm(X[q] - c / np.linalg.norm(c)) <= tol
        assert np.linalg.norm(Y[q] - r) <= tol


# folded sums: the smallest grids (6 and 9 points), the last size of every form (K = 32, 31, 64, 63: 96, 93,
# 192 and 189 points; with the table of twiddles K = 128, 127, 256, 169), the first past each (K = 33, 66, 65, 129),
# a grid of 4 n + 2 points (K = 6), and the direct sums (K = 171, 255).  Sums of at most 768 terms of size one:
# 768 u = 1e-13, within the checks' 1e-11.
@pytest.mark.parametrize("nx", [4, 6, 12, 62, 64, 66, 126, 128, 130, 132, 254, 256, 258, 338, 342, 510, 512])
def test_ks_sizes(nx):
    cfg = (nx, 32.0, 0.01)
    check_ks_F(cfg)
    check_ks_gradient(cfg, 5)
    check_ks_rk_gradient(cfg, 2, "rk222")


# the padded grid lengths with a plan of their own (48 to 768), the first and last of them in tiles of one and
# two row pairs and of four and eight columns; forcing, Nyquist row and snapshots in the fused step.  Same bound as
# test_gpu_kolmo.py: 1e-11 of the largest magnitude, FP64 on both sides.
@pytest.mark.parametrize("N", [32, 64, 96, 128, 192, 256, 384, 512])
def test_kolmo_grid_lengths(N):
    from oracle import imex
    from oracle.kolmo import Kolmogorov
    from test_gpu_kolmo import from_dev, rel, to_dev
    print(f"Kolmogorov grid length, N = {N}", flush=True)
    B, dt, n, Nc = (3 if N <= 128 else 1), 1e-3 * 64 / N, 3, 16
    c0 = wl.kolmo_vorticity(seed=N, N=N, batch=B)
    P = Kolmogorov(N, Re=1000.0, drag=0.1)
    G = sps.Kolmogorov(B, N, Re=1000.0, dt=dt, max_steps=1, keep_history=False, drag=0.1)
    X0 = to_dev(list(c0))
    XN, F = torch.zeros_like(X0), torch.zeros_like(X0)
    snap = torch.full((n * B * Nc * Nc,), 7.0, dtype=torch.float64, device="cuda")
    G.eval_F(X0, F)
    G.forward(X0, n, XN=XN, snap=snap, every=1, nc=Nc)
    G.sync()
    s = snap.cpu().numpy().view(np.complex128).reshape(n, B, Nc // 2, Nc)
    iy = np.arange(Nc)
    rows = np.where(iy < Nc // 2, iy, iy - Nc + N)
    for b in range(B):
        X = c0[b].reshape(-1, 1)
        _, states = imex.sbdf_forward(P, X, dt, n)
        assert rel(from_dev(F, B, N)[b], P.F(X).reshape(N, N // 2)) <= 1e-11
        assert rel(from_dev(XN, B, N)[b], states[-1].reshape(N, N // 2)) <= 1e-11
        assert np.all(from_dev(XN, B, N)[b][N // 2] == 0.0)
        for k in range(n):
            ref = states[k + 1].reshape(N, N // 2)[rows, : Nc // 2].copy()
            ref[Nc // 2, :] = 0.0
            assert rel(s[k, b].T, ref) <= 1e-11


# The reverse steps at the same lengths, with and without the closure (whose grids N = 32 to 96 are in
# test_gpu_kolmo.py): gradient of a rollout of two steps, so one with and one without a target's term.  Bounds of
# test_gpu_kolmo.py: 1e-11 without the closure; with it (activations rounded to bfloat16) 2^-7 of the largest at
# most and 2^-13 in the median.
@pytest.mark.parametrize("N,closure", [(N, False) for N in (32, 64, 96, 128, 192, 256, 384, 512)]
                         + [(N, True) for N in (128, 192, 256, 384, 512)])
def test_kolmo_gradient_grid_lengths(N, closure):
    from oracle import closure as cl
    from oracle.kolmo import Kolmogorov, rollout_loss_and_gradients
    from test_gpu_kolmo import from_dev, params, rel, to_dev
    print(f"Kolmogorov gradient, N = {N}, closure {closure}", flush=True)
    B, dt, n = (2 if N <= 128 else 1), 1e-3 * 64 / N, 2
    p = params(11) if closure else None
    c0 = wl.kolmo_vorticity(seed=2, N=N, batch=B)
    tg = [wl.kolmo_vorticity(seed=20 + k, N=N, batch=B) for k in range(n)]
    P = Kolmogorov(N, Re=1000.0, params=p, bf=True, drag=0.1)
    G = sps.Kolmogorov(B, N, Re=1000.0, dt=dt, max_steps=n, closure=closure, keep_history=True, drag=0.1)
    X0, gth = to_dev(list(c0)), None
    if closure:
        theta = torch.from_numpy(cl.flatten(p)).cuda()
        G.set_params(theta)
        gth = torch.zeros_like(theta)
    J, g0 = torch.zeros(B, dtype=torch.float64, device="cuda"), torch.zeros_like(X0)
    G.rollout(X0, torch.cat([to_dev(list(t)) for t in tg]), n, J=J, dJdX0=g0, dJdtheta=gth)
    G.sync()
    g0, J, tr = from_dev(g0, B, N), J.cpu().numpy(), 0.0
    for b in range(B):
        Jo, go, gp, _ = rollout_loss_and_gradients(P, c0[b].reshape(-1, 1), [t[b].reshape(-1, 1) for t in tg], dt, n)
        e = np.abs(g0[b] - go.reshape(N, N // 2)) / np.max(np.abs(go))
        if not closure:
            assert e.max() <= 1e-11 and abs(J[b] - Jo) <= 1e-11 * abs(Jo)
            continue
        assert e.max() <= 2.0 ** -7 and np.median(e) <= 2.0 ** -13
        tr = tr + gp
    if closure:
        tp, to = cl.unflatten(gth.cpu().numpy()), cl.unflatten(tr)
        for k in cl.PARAM_ORDER:
            e = np.abs(tp[k] - to[k]) / np.max(np.abs(to[k]))
            assert e.max() <= 2.0 ** -7 and np.median(e) <= 2.0 ** -13, k


# Swift-Hohenberg grid lengths with a plan of their own (48 to 384 points, so N = 24 to 192), one of them with a
# partial column tile (N = 72), together with lengths that have none; sizes above the largest plan.  Same checks as
# test_gpu_sh.py; and an instance alone gives the same bits as in the mixed batch.
def test_sh_grid_lengths(monkeypatch):
    import test_gpu_sh as ts
    sizes = [24, 32, 48, 54, 64, 72, 96, 128, 144, 162, 192, 216]
    monkeypatch.setattr(ts, "SMALL_N", sizes)
    monkeypatch.setattr(ts, "SMALL_R", [0.2 + 0.02 * i for i in range(len(sizes))])
    ts.test_sh_gradient_mixed_batch(2)
    print("SH grid lengths, batch independence", flush=True)
    rng = np.random.default_rng(7)
    X = [torch.from_numpy(rng.standard_normal(N * N)).cuda() for N in sizes]

    def run(idx):
        G = sps.ShBatch([sizes[i] for i in idx], [0.3] * len(idx), ts.L, 0.05, max_steps=2)
        out = torch.zeros(G.n, dtype=torch.float64, device="cuda")
        g = torch.zeros_like(out)
        J = torch.zeros(len(idx), dtype=torch.float64, device="cuda")
        G.gradient(torch.cat([X[i] for i in idx]), 2, out, g, J)
        G.sync()
        cut = np.cumsum([0] + [X[i].numel() for i in idx])
        return [(out[a:b], g[a:b], J[k]) for k, (a, b) in enumerate(zip(cut[:-1], cut[1:]))]

    every = run(range(len(sizes)))
    for i in (3, 4, 10):
        assert all(torch.equal(a, b) for a, b in zip(run([i])[0], every[i]))


# Lengths without a plan, alone (in blocks of as many threads as the build's tuner found fastest: 128 or 256 for
# N = 36 and 54, which varies from build to build) and next to a planned length (in blocks of 256): state, gradient,
# cost and its derivative, each the same bits.  Several builds and states, as the order in which a cost is summed
# shows in the last bit of some states only.
def test_sh_general_lengths_alone():
    import test_gpu_sh as ts
    sizes = [8, 18, 36, 54, 162, 24]
    rng = np.random.default_rng(17)
    X = [[torch.from_numpy(rng.standard_normal(N * N)).cuda() for N in sizes] for _ in range(16)]

    def run(idx):
        G = sps.ShBatch([sizes[i] for i in idx], [0.3] * len(idx), ts.L, 0.05, max_steps=2)
        cut = np.cumsum([0] + [sizes[i] ** 2 for i in idx])
        res = []
        for Xs in X:
            x = torch.cat([Xs[i] for i in idx])
            out, g, dJ = (torch.zeros_like(x) for _ in range(3))
            J, J0 = (torch.zeros(len(idx), dtype=torch.float64, device="cuda") for _ in range(2))
            G.gradient(x, 2, out, g, J)
            G.cost(x, J0, dJ)
            G.sync()
            res.append([dict(state=out[a:b], gradient=g[a:b], J=J[k], cost=J0[k], dJ=dJ[a:b])
                        for k, (a, b) in enumerate(zip(cut[:-1], cut[1:]))])
        return G.tuning()["threads"], res

    every = run(range(len(sizes)))[1]
    bad = []
    for i, N in enumerate(sizes):
        for build in range(6):
            threads, alone = run([i])
            print(f"SH alone, N = {N}, build {build}, {threads} threads", flush=True)
            bad += [(N, threads, s, what) for s in range(len(X)) for what, v in alone[s][0].items()
                    if not torch.equal(v, every[s][i][what])]
    assert not bad, f"(N, threads alone, which input, array): {bad}"


# plane Couette flow: the padded z lengths with a plan of their own (24 to 192), tiles of modes that are not full (Kx =
# 12, 36), and lengths with a plan next to one without; of the x lengths only 192 has blocks enough for its row kernels
@pytest.mark.parametrize("nx,nz", [(16, 16), (24, 24), (32, 8), (12, 32), (48, 48), (64, 64), (72, 72), (96, 96), (128, 128)])
def test_couette_grid_lengths(nx, nz):
    check_couette_F(dict(Nx=nx, Ny=8, Nz=nz, Lx=3.0, Lz=2.5))


# The row kernels of every x length that has them, their last tiles not full: F and its VJP against the oracle (whose
# transforms need none of its dense matrices)
@pytest.mark.parametrize("nx,ny,nz", ROW_SIZES)
def test_couette_row_kernels(nx, ny, nz, monkeypatch):
    import test_gpu_couette as tc

    class Planes(tc.Couette):
        def _build_matrices(self):
            return None, None

    assert sps.couette_plane_kernels(nx, ny, nz)[0]
    monkeypatch.setattr(tc, "Couette", Planes)
    check_couette_F(dict(Nx=nx, Ny=ny, Nz=nz, Lx=3.0, Lz=2.5))


# 2D convection: the padded row lengths with kernels of their own (24 to 288 points), an odd number of rows (15:
# two rows a block up to 72 points), a length without (54); and three instances at once
@pytest.mark.parametrize("nx", [16, 24, 32, 36, 48, 64, 72, 96, 144, 192])
def test_rbc_row_lengths(nx):
    check_rbc_F((nx, 10, 3.0, 1e5, 0.7, 2e-3))


def test_rbc_row_lengths_batch():
    check_rbc_batch(64, 10, 3.0, 0.7, 2e-3, [1e4, 1e5, 3e5], 4, 2, [0, 1, 2])
