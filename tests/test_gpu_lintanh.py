"""Linear-tanh family (dense d, matrix-core path) and its reverse mode.

Forward: GPU values and trajectories after K fixed iterations against the FP64
oracle run for the same K (FP32 bar: 1e-4 relative, |a-b| <= 1e-4 max(|b|,1)).
Reverse: d phi/d x, d phi/d A, d phi/d Q and d phi/d eps from hjpd_value_grad
against FP64 central differences of the oracle's fixed-K value, taken as
directional derivatives (phi(b + hV) - phi(b - hV)) / 2h along random unit
directions V, h = 1e-6 max(1, |b|).
"""
import numpy as np
import pytest

import workloads as W
from helpers import rel_err, traj_err

pytestmark = pytest.mark.gpu


def _small_workload(d=16, n=6, N=12, K=100, seed=5):
    r = np.random.default_rng(seed)
    A = r.standard_normal((d, d)) / np.sqrt(d)
    Mq = r.standard_normal((d, d))
    Q = Mq @ Mq.T / d + 0.5 * np.eye(d)
    w = W.lintanh100(8)
    w.d, w.n, w.N_max, w.max_iter = d, n, N, K
    w.x = r.standard_normal((n, d))
    w.t = np.full(n, 1.0)
    w.N = np.full(n, N, np.int32)
    w.hp = np.concatenate([[0.1], A.ravel()])
    w.gp = Q.ravel().copy()
    w.extra = {"A": A, "Q": Q, "ids": np.arange(n)}
    return w


def _f32(a):
    return np.asarray(a, np.float64).astype(np.float32).astype(np.float64)


def _gpu_lt(w, K, E, grad_phi, traj=False):
    import torch

    from paper_1803_01215_amd.autograd import LinearTanhValue
    lt = LinearTanhValue(w.d, w.N_max, w.sigma, w.tau, K, ckpt_every=E, seed=w.init_seed)
    dev = "cuda"
    x = torch.tensor(w.x, dtype=torch.float32, device=dev)
    t = torch.tensor(w.t, dtype=torch.float32, device=dev)
    N = torch.tensor(w.N, dtype=torch.int32, device=dev)
    hp = torch.tensor(w.hp, dtype=torch.float32, device=dev)
    Q = torch.tensor(w.gp, dtype=torch.float32, device=dev)
    gphi = torch.tensor(grad_phi, dtype=torch.float32, device=dev)
    out = lt.solver.solve(x, t, N, hp, Q, traj=traj)
    phi, dx, dh, dg = lt.value_grad(x, t, N, hp, Q, gphi)
    torch.cuda.synchronize()
    res = dict(phi_solve=out.phi.cpu().numpy().astype(np.float64), status=out.status.cpu().numpy(),
               iters=out.iters.cpu().numpy(), phi=phi.cpu().numpy().astype(np.float64),
               dx=dx.cpu().numpy().astype(np.float64), dh=dh.cpu().numpy().astype(np.float64),
               dg=dg.cpu().numpy().astype(np.float64))
    if traj:
        res["x_traj"] = out.x_traj.cpu().numpy().astype(np.float64)
        res["p_traj"] = out.p_traj.cpu().numpy().astype(np.float64)
    lt.close()
    return res


def _oracle_phi(O, w, K, x=None, hp=None, gp=None, idx=None, traj=False):
    idx = np.arange(w.n) if idx is None else np.asarray(idx)
    x = _f32(w.x) if x is None else x
    hp = _f32(w.hp) if hp is None else hp
    gp = _f32(w.gp) if gp is None else gp
    pb = O.Problem(w.H, w.g, w.d, 0, hp, gp)
    return O.solve(pb, x[idx], _f32(w.t)[idx], w.N[idx], sigma=float(_f32(w.sigma)), tau=float(_f32(w.tau)),
                   tol=1e-30, max_iter=K, fixed_iters=True, seed=w.init_seed, N_max=w.N_max, ids=idx, traj=traj)


def test_lintanh100_forward_matches_oracle(oracle_mod):
    w = W.lintanh100().subset(np.arange(20))
    K = w.max_iter
    g = _gpu_lt(w, K, 50, np.ones(w.n), traj=True)
    assert np.all(g["iters"] == K)
    o = _oracle_phi(oracle_mod, w, K, traj=True)
    e = rel_err(g["phi_solve"], o.phi)
    print("lintanh100 phi rel err max %.3g" % e.max())
    assert e.max() <= 1e-4
    assert rel_err(g["phi"], o.phi).max() <= 1e-4  # value returned by value_grad
    ex = traj_err(g["x_traj"], o.x_traj, w.N)
    ep = traj_err(g["p_traj"], o.p_traj, w.N)
    print("traj rel err x %.3g p %.3g" % (ex.max(), ep.max()))
    assert ex.max() <= 1e-4 and ep.max() <= 1e-4


def _fd_dir(O, w, K, which, V, wts, h_rel=1e-6):
    """Central difference of sum_i wts_i phi_i along V for x (per point), A, Q or eps."""
    base = {"x": _f32(w.x), "hp": _f32(w.hp), "gp": _f32(w.gp)}
    if which == "x":
        h = h_rel * max(1.0, np.abs(base["x"]).max())
        vals = []
        for s in (1, -1):
            vals.append(_oracle_phi(O, w, K, x=base["x"] + s * h * V).phi)
        return (vals[0] - vals[1]) / (2 * h)
    key = "gp" if which == "Q" else "hp"
    vec = np.zeros_like(base[key])
    if which == "A":
        vec[1:] = V.ravel()
    elif which == "eps":
        vec[0] = 1.0
    else:
        vec[:] = V.ravel()
    h = h_rel * max(1.0, np.abs(base[key]).max())
    vals = []
    for s in (1, -1):
        kw = {key: base[key] + s * h * vec}
        vals.append(np.dot(wts, _oracle_phi(O, w, K, **kw).phi))
    return (vals[0] - vals[1]) / (2 * h)


def _check_grads(O, w, K, E, n_dirs=2, seed=0):
    rng = np.random.default_rng(seed)
    wts = rng.uniform(0.5, 1.5, w.n)
    g = _gpu_lt(w, K, E, wts)
    d = w.d
    # d phi / d x per point, along random unit directions
    errs = []
    for _ in range(n_dirs):
        V = rng.standard_normal((w.n, d))
        V /= np.linalg.norm(V, axis=1, keepdims=True)
        fd = _fd_dir(O, w, K, "x", V, wts)  # per point, unweighted
        an = np.sum(g["dx"] * V, axis=1) / wts
        errs.append(np.max(np.abs(an - fd) / np.maximum(np.abs(fd), 1)))
    for which in ("A", "Q"):
        for _ in range(n_dirs):
            V = rng.standard_normal((d, d))
            V /= np.linalg.norm(V)
            fd = _fd_dir(O, w, K, which, V, wts)
            an = np.sum((g["dh"][1:] if which == "A" else g["dg"]) * V.ravel())
            errs.append(abs(an - fd) / max(abs(fd), 1))
    fd = _fd_dir(O, w, K, "eps", None, wts)
    errs.append(abs(g["dh"][0] - fd) / max(abs(fd), 1))
    print("gradient rel errors:", np.array(errs))
    return np.array(errs), g


def test_lintanh_small_gradients_match_central_differences(oracle_mod):
    w = _small_workload()
    errs, _ = _check_grads(oracle_mod, w, K=100, E=25)
    assert errs.max() <= 1e-4


@pytest.mark.parametrize("d", [32, 128])
def test_lintanh_other_sizes_values_and_gradients(oracle_mod, d):
    """d = 32 leaves six waves without a row tile of their own, and the reverse
    step forms node 0's adjoint product on them; d = 128 leaves none, and every
    wave sums a quarter of each row's terms."""
    w = _small_workload(d=d, n=3, N=12, K=60, seed=11)
    errs, g = _check_grads(oracle_mod, w, K=60, E=20, n_dirs=1)
    assert errs.max() <= 1e-4
    o = _oracle_phi(oracle_mod, w, 60)
    assert rel_err(g["phi"], o.phi).max() <= 1e-4


def test_lintanh100_gradients_match_central_differences(oracle_mod):
    w = W.lintanh100().subset(np.arange(3))
    errs, _ = _check_grads(oracle_mod, w, K=w.max_iter, E=50, n_dirs=1)
    assert errs.max() <= 1e-4


def test_checkpoint_interval_does_not_change_gradients():
    w = _small_workload(n=4, K=60)
    wts = np.ones(w.n)
    a = _gpu_lt(w, 60, 60, wts)
    b = _gpu_lt(w, 60, 7, wts)
    for k in ("dx", "dh", "dg", "phi"):
        assert np.allclose(a[k], b[k], rtol=1e-6, atol=1e-7), k


def test_envelope_identity_on_gpu_gradient():
    """At a converged iterate d phi/d x = p_N - delta grad_x H(x, p_N)
    (the value is the Lagrangian at a stationary point; x enters as x_N)."""
    w = _small_workload(n=4, K=400, N=10)
    g = _gpu_lt(w, 400, 50, np.ones(w.n), traj=True)
    A = w.extra["A"]
    delta = w.t[0] / w.N[0]
    for i in range(w.n):
        x = w.x[i]
        pN = g["p_traj"][i, w.N[i]]
        th = np.tanh(x)
        env = pN + delta * (A.T @ pN + 0.1 * (1 - th * th) * pN)
        assert np.max(np.abs(env - g["dx"][i])) < 1e-3 * max(1, np.abs(env).max())


def test_autograd_function_matches_value_grad():
    import torch

    from paper_1803_01215_amd.autograd import LinearTanhValue, hj_value
    w = _small_workload(n=5, K=80)
    lt = LinearTanhValue(w.d, w.N_max, w.sigma, w.tau, 80, ckpt_every=20, seed=w.init_seed)
    dev = "cuda"
    x = torch.tensor(w.x, dtype=torch.float32, device=dev, requires_grad=True)
    t = torch.tensor(w.t, dtype=torch.float32, device=dev)
    N = torch.tensor(w.N, dtype=torch.int32, device=dev)
    eps = torch.tensor(0.1, dtype=torch.float32, device=dev, requires_grad=True)
    A = torch.tensor(w.extra["A"], dtype=torch.float32, device=dev, requires_grad=True)
    Q = torch.tensor(w.extra["Q"], dtype=torch.float32, device=dev, requires_grad=True)
    wts = torch.linspace(0.5, 1.5, w.n, device=dev)
    phi = hj_value(x, t, N, eps, A, Q, lt)
    (phi * wts).sum().backward()
    hp = torch.cat([eps.detach().reshape(1), A.detach().reshape(-1)])
    _, dx, dh, dg = lt.value_grad(x.detach(), t, N, hp, Q.detach().reshape(-1), wts)
    torch.cuda.synchronize()
    assert torch.allclose(x.grad, dx)
    assert torch.allclose(A.grad.reshape(-1), dh[1:])
    assert torch.allclose(eps.grad.reshape(1), dh[:1])
    assert torch.allclose(Q.grad.reshape(-1), dg)
    lt.close()


@pytest.mark.parametrize("d", [16, 32, 100, 128])
def test_node0_matrix_with_row_exchanges(d):
    """x_0 <- (I + tau Q_s)^{-1} (x_0 + tau p_1) for an indefinite Q whose
    I + tau Q_s has a zero diagonal, so every elimination step has to take its
    pivot from another row.  One step is read off the trajectories of two
    solves of one and two iterations; the bound is the FP32 dot product's,
    (d + 3) 2^-24 sum |M_ij| |v_j|."""
    w = _small_workload(d=d, n=2, N=4, K=2)
    rng = np.random.default_rng(d)
    B = rng.standard_normal((d, d))
    B = (B + B.T) / 2
    np.fill_diagonal(B, 0.0)
    w.gp = ((B - np.eye(d)) / w.tau).ravel()
    Q = _f32(w.gp).reshape(d, d)
    M = np.linalg.inv(np.eye(d) + w.tau * 0.5 * (Q + Q.T))
    one, two = (_gpu_lt(w, K, 1, np.ones(w.n), traj=True) for K in (1, 2))
    for i in range(w.n):
        v = one["x_traj"][i, 0] + w.tau * two["p_traj"][i, 1]
        bound = (d + 3) * 2.0 ** -24 * (np.abs(M) @ np.abs(v))
        assert np.all(np.abs(two["x_traj"][i, 0] - M @ v) <= bound)


def _edge_cases():
    out = []
    for d in (16, 32, 100, 128):
        for N in (1, 2, 15, 16, 17, 32, 33, 48, 49, 64):
            if d < 128 or N <= 48:  # d = 128 is built for N up to 48
                out.append((d, N))
    return out


@pytest.mark.parametrize("d,N_max", _edge_cases())
def test_column_tile_edges_match_oracle(oracle_mod, d, N_max):
    """Step counts on both sides of the 16-node column tiles, each batch with
    every step count from N_max down, inputs at an address that is only 4-byte
    aligned.  FP32 bar 1e-4 against the oracle, values and trajectories."""
    import torch

    from paper_1803_01215_amd.autograd import LinearTanhValue
    K, n = 30, min(9, N_max)
    w = _small_workload(d=d, n=n, N=N_max, K=K, seed=100 + N_max)
    w.N = np.arange(N_max, N_max - n, -1).astype(np.int32)
    w.t = np.random.default_rng(N_max).uniform(0.3, 1.2, n)
    lt = LinearTanhValue(d, N_max, w.sigma, w.tau, K, seed=w.init_seed)

    def odd(a):
        a = np.asarray(a, np.float32).ravel()
        buf = torch.empty(a.size + 1, dtype=torch.float32, device="cuda")
        buf[1:] = torch.tensor(a, device="cuda")
        return buf[1:]

    out = lt.solver.solve(odd(w.x), odd(w.t), torch.tensor(w.N, device="cuda"), odd(w.hp), odd(w.gp), traj=True)
    torch.cuda.synchronize()
    o = _oracle_phi(oracle_mod, w, K, traj=True)
    assert rel_err(out.phi.cpu().numpy().astype(np.float64), o.phi).max() <= 1e-4
    for got, want in ((out.x_traj, o.x_traj), (out.p_traj, o.p_traj)):
        assert traj_err(got.cpu().numpy().astype(np.float64), want, w.N).max() <= 1e-4
    lt.close()


def _torch_phi(x, t, N, eps, A, Q, x0_all, p0_all, K, sigma, tau):
    """phi of every point after K iterations, binary64 torch on the CPU; x0_all, p0_all: the random start."""
    import torch
    out = []
    for i in range(len(N)):
        n, d = int(N[i]), x.shape[1]
        delta = t[i] / n
        lam = sigma * delta
        Qs = 0.5 * (Q + Q.T)
        M = torch.linalg.inv(torch.eye(d, dtype=torch.float64) + tau * Qs)
        # x_j starts at x + noise (j < N), x_N = x
        X = torch.cat([x[i] + x0_all[i][:n], x[i][None]])
        P = torch.cat([torch.zeros(1, d, dtype=torch.float64), p0_all[i][1:n + 1]])
        Z = X
        for _ in range(K):
            th = torch.tanh(X[1:])
            Pn = (P[1:] + sigma * (Z[1:] - Z[:-1]) + lam * (X[1:] @ A.T + eps * th)) / (1 + lam)
            x0 = M @ (X[0] + tau * Pn[0])
            mid = (X[1:n] - tau * (Pn[:-1] - Pn[1:])
                   - tau * delta * (Pn[:-1] @ A + eps * (1 - th[:-1] ** 2) * Pn[:-1]))
            Xn = torch.cat([x0[None], mid, X[n:]])
            Z = 2 * Xn - X
            X, P = Xn, torch.cat([P[:1], Pn])
        f = X[1:] @ A.T + eps * torch.tanh(X[1:])
        p = P[1:]
        out.append(0.5 * X[0] @ Qs @ X[0] + (p * (X[1:] - X[:-1]) - delta * (0.5 * p * p - p * f)).sum())
    return torch.stack(out)


@pytest.mark.parametrize("d,N_max", _edge_cases())
def test_column_tile_edges_gradients(oracle_mod, d, N_max):
    """Gradients on both sides of the 16-node column tiles against binary64
    autograd through the unrolled iterations (checkpoints that do not divide
    the count, one output weight zero).  FP32 bar 1e-4."""
    import torch
    K, E, n = 20, 7, min(4, N_max)
    w = _small_workload(d=d, n=n, N=N_max, K=K, seed=200 + N_max)
    w.N = np.arange(N_max, N_max - n, -1).astype(np.int32)
    wts = np.linspace(0.5, 1.5, n)
    if n > 2:
        wts[1] = 0.0
    g = _gpu_lt(w, K, E, wts)
    noise = [np.zeros((n, N_max + 1, d)) for _ in range(2)]
    for i in range(n):
        for j in range(N_max + 1):
            for c in range(d):
                noise[0][i, j, c] = oracle_mod.init_noise(w.init_seed, i, 0, j, c)
                noise[1][i, j, c] = oracle_mod.init_noise(w.init_seed, i, 1, j, c)
    T = lambda a: torch.tensor(a, dtype=torch.float64)
    x, A, Q = T(_f32(w.x)).requires_grad_(), T(_f32(w.hp[1:])).reshape(d, d).requires_grad_(), \
        T(_f32(w.gp)).reshape(d, d).requires_grad_()
    eps = T(_f32(w.hp[0])).requires_grad_()
    phi = _torch_phi(x, T(_f32(w.t)), w.N, eps, A, Q, T(noise[0]), T(noise[1]), K, float(w.sigma), float(w.tau))
    dx, de, dA, dQ = torch.autograd.grad((phi * T(_f32(wts))).sum(), [x, eps, A, Q])
    bar = lambda got, want: np.max(np.abs(got - want.numpy().ravel())) / max(1.0, float(want.abs().max()))
    assert rel_err(g["phi"], phi.detach().numpy()).max() <= 1e-4
    assert bar(g["dx"].ravel(), dx) <= 1e-4
    assert bar(g["dh"][:1], de.reshape(1)) <= 1e-4
    assert bar(g["dh"][1:], dA) <= 1e-4
    assert bar(g["dg"], dQ) <= 1e-4


def _reference_gradients(O, w, K, wts):
    """(phi, d/dx, d/deps, d/dA, d/dQ) in binary64 by autograd through the unrolled iterations, on the
    inputs as the GPU gets them."""
    import torch
    n, d = w.n, w.d
    noise = [np.zeros((n, w.N_max + 1, d)) for _ in range(2)]
    for i in range(n):
        for j in range(w.N_max + 1):
            for c in range(d):
                noise[0][i, j, c] = O.init_noise(w.init_seed, int(w.ids[i]), 0, j, c)
                noise[1][i, j, c] = O.init_noise(w.init_seed, int(w.ids[i]), 1, j, c)
    T = lambda a: torch.tensor(a, dtype=torch.float64)
    x, A, Q = T(_f32(w.x)).requires_grad_(), T(_f32(w.hp[1:])).reshape(d, d).requires_grad_(), \
        T(_f32(w.gp)).reshape(d, d).requires_grad_()
    eps = T(_f32(w.hp[0])).requires_grad_()
    phi = _torch_phi(x, T(_f32(w.t)), w.N, eps, A, Q, T(noise[0]), T(noise[1]), K, float(w.sigma), float(w.tau))
    g = torch.autograd.grad((phi * T(_f32(wts))).sum(), [x, eps, A, Q])
    return (phi.detach().numpy(),) + tuple(v.numpy() for v in g)


@pytest.mark.parametrize("d", [16, 32, 100, 128])
def test_rounding_of_the_query_point_gradient(oracle_mod, d):
    """dphi/dx gathers small terms over every iteration on a sum far larger
    than they are.  A float32 model of the sweep (N = 24, 100 iterations) is
    2.6e-7 to 2.7e-7 from binary64 in the root mean square where a step rounds
    once at the sum's size, and 5.6e-7 to 5.9e-7 where it adds the terms one by
    one; the bound lies between."""
    w = _small_workload(d=d, n=8, N=24, K=100, seed=40 + d)
    wts = np.random.default_rng(d).uniform(0.5, 1.5, w.n)
    g = _gpu_lt(w, 100, 25, wts)
    want = _reference_gradients(oracle_mod, w, 100, wts)[1]
    err = np.linalg.norm(g["dx"] - want) / np.linalg.norm(want)
    print("d = %d: rms error of dphi/dx %.3g" % (d, err))
    assert err <= 4e-7


@pytest.mark.parametrize("N,K", [(32, 300), (48, 150)])
@pytest.mark.parametrize("d", [100, 128])
def test_rounding_of_the_matrix_gradient(oracle_mod, d, N, K):
    """dphi/dA sums outer products over every iteration.  On FP32 products it
    is 1.9e-6 to 2.1e-6 from binary64 in the root mean square (N = 48, 150
    iterations), with the six piece products added one by one to the sum 3.1e-6
    to 3.4e-6 over 200 points: the bound is below the former."""
    w = _small_workload(d=d, n=3, N=N, K=K, seed=60 + d)
    wts = np.random.default_rng(d).uniform(0.5, 1.5, w.n)
    g = _gpu_lt(w, K, K, wts)
    want = _reference_gradients(oracle_mod, w, K, wts)[3].ravel()
    err = np.linalg.norm(g["dh"][1:] - want) / np.linalg.norm(want)
    print("d = %d, N = %d: rms error of dphi/dA %.3g" % (d, N, err))
    assert err <= 1.5e-6


@pytest.mark.parametrize("power", [-116, 100])
@pytest.mark.parametrize("d", [16, 32, 100, 128])
def test_gradients_scale_with_the_output_weights(d, power):
    """Gradients are linear in grad_phi, and a power of two is exact: very small
    and very large weights give the same digits, for all points or for some
    beside others of ordinary weight.  What FP32 cannot hold is below 2^-149,
    1e-9 of the largest entry here."""
    w = _small_workload(d=d, n=6, N=20, K=60, seed=80 + d)
    wts = _f32(np.random.default_rng(d).uniform(0.5, 1.5, w.n))
    one = _gpu_lt(w, 60, 25, wts)
    f = 2.0 ** power
    g = _gpu_lt(w, 60, 25, wts * f)
    for k in ("dx", "dh", "dg"):
        assert np.max(np.abs(g[k] / f - one[k])) <= 1e-7 * np.max(np.abs(one[k])), k
    s = np.where(np.arange(w.n) % 2, f, 1.0)
    g = _gpu_lt(w, 60, 25, wts * s)
    for i in range(w.n):
        assert np.max(np.abs(g["dx"][i] / s[i] - one["dx"][i])) <= 1e-7 * np.max(np.abs(one["dx"][i])), i
    # the parameters' gradients are those of the points whose weights count
    big = s == s.max()
    alone = _gpu_lt(w, 60, 25, wts * big * s)
    for k in ("dh", "dg"):
        assert np.max(np.abs(g[k] - alone[k])) <= 1e-7 * np.max(np.abs(alone[k])), k


def test_value_and_gradient_refuse_capture():
    """The reverse sweep's buffers grow with the largest call and are replaced
    then, so a captured call, which keeps their addresses, is refused."""
    import torch

    from paper_1803_01215_amd.autograd import LinearTanhValue
    w = _small_workload(n=3, K=10)
    lt = LinearTanhValue(w.d, w.N_max, w.sigma, w.tau, 10, ckpt_every=5, seed=w.init_seed)
    T = lambda a: torch.tensor(a, dtype=torch.float32, device="cuda")
    args = (T(w.x), T(w.t), torch.tensor(w.N, device="cuda"), T(w.hp), T(w.gp), torch.ones(3, device="cuda"))
    want = lt.value_grad(*args)
    torch.cuda.synchronize()
    graph, stream = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    with torch.cuda.stream(stream):
        graph.capture_begin()
        try:
            with pytest.raises(Exception, match="captured"):
                lt.value_grad(*args, stream=stream)
        finally:
            graph.capture_end()
    got = lt.value_grad(*args)
    torch.cuda.synchronize()
    for a, b in zip(got, want):
        assert torch.equal(a, b)
    lt.close()


def test_segment_buffers_that_do_not_fit_take_fewer_workgroups():
    """One segment of 4,000 iterations at d = 100 takes 64 MB per workgroup,
    16 GB for a workgroup on each of 256 CUs; with 8 GB free the call runs on
    fewer, and only the order of the sums over points changes."""
    import torch

    from paper_1803_01215_amd.autograd import LinearTanhValue
    K, n = 4000, 260
    w = _small_workload(d=100, n=n, N=4, K=K)
    T = lambda a: torch.tensor(a, dtype=torch.float32, device="cuda")
    args = (T(w.x), T(w.t), torch.tensor(w.N, device="cuda"), T(w.hp), T(w.gp), torch.ones(n, device="cuda"))
    res, held = [], None
    for E, short in ((100, False), (K, True)):
        lt = LinearTanhValue(w.d, w.N_max, w.sigma, w.tau, K, ckpt_every=E, seed=w.init_seed)
        if short:
            torch.cuda.empty_cache()
            held = torch.empty(torch.cuda.mem_get_info()[0] - (8 << 30), dtype=torch.uint8, device="cuda")
        res.append([v.cpu().numpy() for v in lt.value_grad(*args)])
        torch.cuda.synchronize()
        lt.close()
    del held
    torch.cuda.empty_cache()
    for a, b in zip(*res):
        assert np.max(np.abs(a - b)) <= 1e-5 * np.max(np.abs(b))


@pytest.mark.parametrize("d,n", [(16, 9001), (32, 9001), (100, 601), (128, 601)])
def test_workgroups_that_take_several_points(oracle_mod, d, n):
    """More points than the persistent grids hold (a workgroup takes its second
    and third), segments longer than the 32 steps that dM's staging holds.
    Sampled points against the oracle and binary64 autograd, FP32 bar 1e-4; the
    parameters' gradients with every other weight zero."""
    K = 40
    w = _small_workload(d=d, n=n, N=9, K=K, seed=20 + d)
    w.N = np.random.default_rng(d).integers(1, 10, n).astype(np.int32)
    idx = np.array([0, 1, n // 3, n // 2, n - 2, n - 1])
    ws = w.subset(idx)
    wts = np.random.default_rng(d + 1).uniform(0.5, 1.5, n)
    phi, dx, de, dA, dQ = _reference_gradients(oracle_mod, ws, K, wts[idx])
    g = _gpu_lt(w, K, 50, wts)
    assert np.all(g["iters"] == K) and np.all(np.isfinite(g["phi"])) and np.all(np.isfinite(g["dx"]))
    assert rel_err(g["phi"][idx], phi).max() <= 1e-4 and rel_err(g["phi_solve"][idx], phi).max() <= 1e-4
    assert np.max(np.abs(g["dx"][idx] - dx)) <= 1e-4 * max(1.0, np.abs(dx).max())
    some = np.zeros(n)
    some[idx] = wts[idx]
    g = _gpu_lt(w, K, 50, some)
    rest = np.setdiff1d(np.arange(n), idx)
    assert np.all(g["dx"][rest] == 0.0)
    for got, want in ((g["dx"][idx], dx), (g["dh"][:1], de.reshape(1)), (g["dh"][1:], dA.ravel()), (g["dg"], dQ.ravel())):
        assert np.max(np.abs(got - want)) <= 1e-4 * max(1.0, np.abs(want).max())
