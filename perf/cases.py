"""What this library is used for, as cases that can be timed: reconstructions of a
multi-echo series (small to large, every prior, coils, batches, serving) and the
public single steps a caller runs by themselves (the weight update, the CG operator).

``listed`` gives the fixed cases, ``draw`` more of the same ranges, ``prepare`` what a
program holds before the call (plans and device inputs), ``run`` one pass through the
public entry points, ``exact`` the same outputs in float64 by plain torch, ``work`` the
bytes and operations one pass cannot do without.
"""
import ctypes
import math
import random

import torch

import paper_1704_04511_amd as slrx

DEV = "cuda"
LAM, P_NORM, GAMMA, EPS0 = 1e-3, 0.6, 1.4, 0.01

# Slices of the uneven batch: frames of 96..256 squared with 8..20 echoes, as acquired
# with different protocols.
BATCH_P, BATCH_T = (96, 128, 160, 192, 256), (8, 12, 16, 20)


def listed():
    return [
        # one application of the CG normal operator on a small series, from a caller's own
        # solver loop: the smallest call, launches and latency
        dict(name="apply_64", kind="apply", P=64, Q=64, T=8, N1=5, N2=5, M=3),
        # the weight update alone (eigenvalues, H and the masks in device memory), for a
        # caller with its own least-squares solver
        dict(name="weights_128", kind="weights", P=128, Q=128, T=16, N1=9, N2=9, M=5),
        # a small, an ordinary and a large single-channel reconstruction (the large ones of ten
        # outer iterations: with a smaller eps their images follow the rounding of complex64)
        dict(name="recon_64", kind="recon", P=64, Q=64, T=8, N1=5, N2=5, M=3, n_irls=15, n_cg=10),
        dict(name="recon_128", kind="recon", P=128, Q=128, T=16, N1=9, N2=9, M=5, n_irls=15, n_cg=10),
        dict(name="recon_256", kind="recon", P=256, Q=256, T=20, N1=15, N2=15, M=5, n_irls=10, n_cg=15),
        # an odd shape: uneven frame, even filter sides, circular along the echoes (GIRAF)
        dict(name="giraf_160x96", kind="recon", giraf=True, P=160, Q=96, T=11, N1=8, N2=7, M=4, n_irls=10, n_cg=8),
        # twelve receive coils, the size of the multichannel experiment
        dict(name="coils_128", kind="coils", nc=12, P=128, Q=128, T=12, N1=9, N2=9, M=5, n_irls=15, n_cg=10),
        # the pixel-wise prior, the comparison method of the large series
        dict(name="voxel_256", kind="voxel", P=256, Q=256, T=20, N1=1, N2=1, M=5, n_irls=10, n_cg=15),
        # the explicit lifting without FFT approximations, for the approximation study
        dict(name="direct_64", kind="direct", P=64, Q=64, T=8, N1=5, N2=5, M=3, n_irls=15, n_cg=10),
        # a study of many uneven slices in one call, and one of many small equal slices
        dict(name="batch_32", kind="batch", slices=32, uneven=True, P=256, Q=256, T=20, N1=9, N2=9, M=5, n_irls=15,
             n_cg=10),
        dict(name="batch_small", kind="batch", slices=32, uneven=False, P=64, Q=64, T=8, N1=5, N2=5, M=3, n_irls=15,
             n_cg=10),
        # a burst of requests to the server: host data in, host images out
        dict(name="serve_10", kind="serve", slices=10, uneven=True, P=192, Q=192, T=16, N1=9, N2=9, M=5, n_irls=15,
             n_cg=10),
    ]


def draw(rng):
    """One more case: any kind, frame sides over the supported transform lengths, filters from
    3x3x2 up, Gram sizes up to 1125 for one series and 605 in batches."""
    kind = rng.choice(["apply", "weights", "recon", "recon", "recon", "coils", "voxel", "direct", "batch", "serve"])
    small = kind in ("direct", "batch", "serve", "coils")
    sides = [32, 64, 96, 128] if kind == "direct" else [32, 64, 96, 128, 160, 192] + ([] if small else [256])
    c = dict(kind=kind, P=rng.choice(sides), Q=rng.choice(sides), T=rng.randint(6, 12 if kind == "direct" else 20))
    c["M"] = rng.randint(2, 5)
    cap = {"direct": 150, "batch": 605, "serve": 500, "coils": 605}.get(kind, 1125)
    s = math.exp(rng.uniform(math.log(18), math.log(cap)))
    side = max(3.0, math.sqrt(s / c["M"]))
    c["N1"] = max(3, min(15, round(side * rng.uniform(0.8, 1.2))))
    c["N2"] = max(3, min(15, round(s / c["M"] / c["N1"])))
    while c["N1"] * c["N2"] * c["M"] > cap:
        c["N1"] -= 1
    if kind == "voxel":
        c["N1"] = c["N2"] = 1
    if kind not in ("apply", "weights"):
        c["n_irls"], c["n_cg"] = rng.randint(4, 10), rng.randint(5, 15)
    if kind in ("recon", "apply"):
        c["giraf"] = rng.random() < 0.3
    if kind == "coils":
        c["nc"] = rng.randint(2, 12)
    if kind in ("batch", "serve"):
        c["slices"] = rng.randint(3, 24 if kind == "batch" else 10)
        c["uneven"] = rng.random() < 0.5
    return c


# ------------------------------------------------------------------ inputs
class _Rng:
    """Uniform numbers and normal fields of a seed, on the device."""

    def __init__(self, seed):
        self.cpu = torch.Generator().manual_seed(int(seed))
        self.gpu = torch.Generator(device=DEV).manual_seed(int(seed))

    def uniform(self, lo, hi):
        return lo + (hi - lo) * float(torch.rand((), generator=self.cpu, dtype=torch.float64))

    def choice(self, seq):
        return seq[int(torch.randint(len(seq), (), generator=self.cpu))]


def _grid(P, Q):
    r1 = torch.arange(P, device=DEV, dtype=torch.float64)[:, None]
    r2 = torch.arange(Q, device=DEV, dtype=torch.float64)[None, :]
    return r1, r2


def _bumps(g, P, Q, lo, hi):
    """A smooth map in [lo, hi]: six Gaussian bumps."""
    r1, r2 = _grid(P, Q)
    f = torch.zeros(P, Q, device=DEV, dtype=torch.float64)
    for _ in range(6):
        c1, c2, w = g.uniform(0, P), g.uniform(0, Q), g.uniform(0.08, 0.25) * P
        f += g.uniform(0.3, 1.0) * torch.exp(-((r1 - c1) ** 2 + (r2 - c2) ** 2) / (2.0 * w * w))
    f -= f.min()
    return lo + (hi - lo) * f / f.max()


def _series(g, P, Q, T):
    """Two damped exponentials per pixel (T2 of 15..40 and 60..200 ms, 10 ms echoes) with a
    smooth phase, complex128 [T][P][Q]."""
    te = 10.0 * (torch.arange(T, device=DEV, dtype=torch.float64) + 1.0)[:, None, None]
    rho, fr = _bumps(g, P, Q, 0.0, 1.0), _bumps(g, P, Q, 0.0, 1.0)
    sig = fr * torch.exp(-te / _bumps(g, P, Q, 15.0, 40.0)) + (1 - fr) * torch.exp(-te / _bumps(g, P, Q, 60.0, 200.0))
    return rho * sig * torch.exp(1j * _bumps(g, P, Q, -math.pi, math.pi))


def _masks(g, P, Q, T, R):
    """One variable-density mask per echo with exactly round(PQ/R) samples (a random draw
    without replacement, the low frequencies always sampled), uint8 [T][P][Q]."""
    k1, k2 = torch.fft.fftfreq(P, device=DEV)[:, None], torch.fft.fftfreq(Q, device=DEV)[None, :]
    kr = torch.sqrt(k1.double() ** 2 + k2.double() ** 2)
    key = 2.0 * torch.log(torch.clamp(1.0 - kr / kr.max(), min=1e-6)).reshape(1, -1)
    u = torch.rand(T, P * Q, generator=g.gpu, device=DEV, dtype=torch.float64)
    key = key - torch.log(-torch.log(u.clamp(1e-300, 1 - 1e-16)))
    key[:, (kr < 4.0 / P).reshape(-1)] = math.inf
    S = torch.zeros(T, P * Q, device=DEV, dtype=torch.uint8)
    S.scatter_(1, key.topk(round(P * Q / R), dim=1).indices, 1)
    return S.reshape(T, P, Q)


def _noisy(g, x, S):
    """S o (x + noise) at 40 dB of the sampled entries, complex64."""
    sel = S.bool().expand_as(x)
    sig = torch.linalg.vector_norm(x[sel]) / math.sqrt(int(sel.sum())) * 1e-2
    n = torch.randn(*x.shape, 2, generator=g.gpu, device=DEV, dtype=torch.float64)
    return (S * (x + torch.view_as_complex(n) * (sig / math.sqrt(2.0)))).to(torch.complex64)


def _coil_maps(g, P, Q, nc):
    r1, r2 = _grid(P, Q)
    r1, r2, maps = r1 - P / 2, r2 - Q / 2, []
    for j in range(nc):
        a = 2 * math.pi * j / nc + g.uniform(-0.2, 0.2)
        w = g.uniform(0.35, 0.55) * P
        m = torch.exp(-((r1 - 0.7 * P * math.cos(a)) ** 2 + (r2 - 0.7 * Q * math.sin(a)) ** 2) / (2 * w * w))
        ph = g.uniform(-math.pi, math.pi) * r1 / P + g.uniform(-math.pi, math.pi) * r2 / Q + g.uniform(-3.0, 3.0)
        maps.append(m * torch.exp(1j * ph))
    C = torch.stack(maps)
    return (C / torch.sqrt((C.abs() ** 2).sum(0, keepdim=True))).to(torch.complex64)


def _data(case, seed):
    """Sampled k-space, masks and (coils) the maps of one series."""
    P, Q, T, g = case["P"], case["Q"], case["T"], _Rng(seed)
    img = _series(g, P, Q, T)
    S = _masks(g, P, Q, T, g.choice([4, 6, 8]))
    if case["kind"] != "coils":
        return _noisy(g, torch.fft.fft2(img, norm="ortho"), S), S, None
    C = _coil_maps(g, P, Q, case["nc"])
    return _noisy(g, torch.fft.fft2(C[:, None] * img[None], norm="ortho"), S), S, C


def _slices(case, seed):
    """The cases of a batch's slices: equal, or frames and echo counts drawn per slice."""
    one = {k: v for k, v in case.items() if k not in ("slices", "uneven", "name")}
    if not case["uneven"]:
        return [dict(one, kind="recon") for _ in range(case["slices"])]
    g, out = random.Random(case["slices"]), []  # the shapes belong to the case, the data to the seed
    for _ in range(case["slices"]):
        P = min(g.choice(BATCH_P), max(case["P"], case["Q"]))
        out.append(dict(one, kind="recon", P=P, Q=P, T=max(min(g.choice(BATCH_T), case["T"]), case["M"])))
    return out


def _params(case):
    return slrx.make_params(lam=LAM, n_irls=case.get("n_irls", 1), n_cg=case.get("n_cg", 1), p=P_NORM, gamma=GAMMA,
                            eps0_frac=EPS0, giraf=bool(case.get("giraf")), voxel=case["kind"] == "voxel",
                            direct=case["kind"] == "direct")


def _plan(case):
    return slrx.Plan(case["P"], case["Q"], case["T"], case["N1"], case["N2"], case["M"], _params(case))


def _operator(case, seed):
    """Masks E [W][P][Q] of a plausible weight update and a CG direction, for the operator alone."""
    P, Q, T, M, g = case["P"], case["Q"], case["T"], case["M"], _Rng(seed)
    W = M * (M + 1) // 2
    E = torch.view_as_complex(torch.randn(W, P, Q, 2, generator=g.gpu, device=DEV)) * 0.3
    w = 0
    for m in range(M):
        E[w] = 1.0 + torch.rand(P, Q, generator=g.gpu, device=DEV)
        w += M - m
    v = torch.view_as_complex(torch.randn(T, P, Q, 2, generator=g.gpu, device=DEV))
    return _masks(g, P, Q, T, 6), E, v


def prepare(case, seed):
    kind = case["kind"]
    if kind == "apply":
        S, E, v = _operator(case, seed)
        dims = slrx.Dims(case["P"], case["Q"], case["T"], case["N1"], case["N2"], case["M"])
        st = dict(case=case, dims=dims, S=S, E=E, v=v, out=torch.empty_like(v))
    elif kind == "batch":
        items = []
        for j, c in enumerate(_slices(case, seed)):
            b, S, _ = _data(c, 1000 * seed + j)
            items.append(dict(plan=_plan(c), b=b, S=S, out=torch.empty_like(b)))
        st = dict(case=case, items=items)
    elif kind == "serve":
        reqs = []
        for j, c in enumerate(_slices(case, seed)):
            b, S, _ = _data(c, 1000 * seed + j)
            reqs.append((b.cpu().numpy(), S.cpu().numpy()))
        st = dict(case=case, reqs=reqs, params=_params(case), server=slrx.Server(32 << 30, max_slots=8))
    else:
        b, S, C = _data(case, seed)
        st = dict(case=case, plan=_plan(case), b=b, S=S, C=C)
        if kind == "weights":
            s, W = st["plan"].s, st["plan"].W
            st.update(lam=torch.empty(s, dtype=torch.float64, device=DEV),
                      H=torch.empty(s, s, dtype=torch.complex128, device=DEV),
                      E=torch.empty(W, case["P"], case["Q"], dtype=torch.complex64, device=DEV))
        else:
            st["out"] = torch.empty(case["T"], case["P"], case["Q"], dtype=torch.complex64, device=DEV)
    torch.cuda.synchronize()
    return st


WEIGHTS_EPS = 50.0  # as in the later outer iterations (the largest eigenvalue is about 1e5 at 128 x 128 x 16)


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "apply":
        slrx.apply_noalloc(state["dims"], LAM, state["S"], state["E"], state["v"], state["out"],
                           stream=torch.cuda.current_stream().cuda_stream, giraf=bool(case.get("giraf")))
        return state["out"]
    if kind == "batch":
        for it in state["items"]:
            it["plan"].set_kspace(it["b"])
            it["plan"].set_mask(it["S"])
        slrx.run_batch([it["plan"] for it in state["items"]])
        for it in state["items"]:
            it["plan"].images(it["out"])
        for it in state["items"]:
            it["plan"].sync()
        return [it["out"] for it in state["items"]]
    if kind == "serve":
        srv = state["server"]
        tickets = [srv.submit_data(b, S, case["N1"], case["N2"], case["M"], state["params"]) for b, S in state["reqs"]]
        out = []
        for t, (b, _) in zip(tickets, state["reqs"]):
            srv.wait(t)
            out.append(srv.fetch(t, b.shape))
            srv.release(t)
        return out
    plan = state["plan"]
    if kind == "coils":
        plan.set_coils(state["C"], state["b"])
    else:
        plan.set_kspace(state["b"])
    plan.set_mask(state["S"])
    if kind == "weights":
        ptr = [ctypes.c_void_p(state[k].data_ptr()) for k in ("lam", "H", "E")]
        status = slrx.lib().slrx_step_weights(plan.handle, WEIGHTS_EPS, *ptr, slrx.SLRX_MEM_DEVICE)
        if status != 0:
            raise slrx.SlrxError(status, slrx.lib().slrx_last_error(plan.handle).decode())
        return [state["lam"], state["H"], state["E"]]
    plan.run()
    plan.sync()
    plan.images(state["out"])
    plan.sync()
    return state["out"]


# ------------------------------------------------- the same outputs in float64
def _offsets(c):
    a1 = torch.arange(c["N1"], device=DEV) - c["N1"] // 2
    a2 = torch.arange(c["N2"], device=DEV) - c["N2"] // 2
    A1, A2 = torch.meshgrid(a1, a2, indexing="ij")
    return A1.reshape(-1), A2.reshape(-1)


def _windows(c, rho):
    """rho_{n-m} for the valid (GIRAF: all) echo shifts n, one volume per tap m."""
    T, M = c["T"], c["M"]
    return [torch.roll(rho, m, 0) if c.get("giraf") else rho[M - 1 - m:T - m] for m in range(M)]


def _gram(c, x):
    """R = T(x)^H T(x) of the lifting, circular in space."""
    M, NN = c["M"], c["N1"] * c["N2"]
    a1, a2 = _offsets(c)
    d1, d2 = (a1[:, None] - a1[None]) % c["P"], (a2[:, None] - a2[None]) % c["Q"]
    z = _windows(c, torch.fft.ifft2(x, norm="ortho"))
    R = torch.empty(M * NN, M * NN, dtype=torch.complex128, device=DEV)
    for m in range(M):
        for k in range(M):
            R[m * NN:(m + 1) * NN, k * NN:(k + 1) * NN] = torch.fft.fft2((z[m].conj() * z[k]).sum(0))[d1, d2]
    return R


def _power(lam, U, eps):
    return (U * (lam.clamp(min=0.0) + eps) ** (P_NORM / 2 - 1)) @ U.conj().T


def _penalty_masks(c, H):
    """E[m][m'] = sum over filter taps a, a' of conj(H[(m,a),(m',a')]) e^{2 pi i (a'-a).r}."""
    P, Q, M, NN = c["P"], c["Q"], c["M"], c["N1"] * c["N2"]
    a1, a2 = _offsets(c)
    at = (((a1[None] - a1[:, None]) % P) * Q + (a2[None] - a2[:, None]) % Q).reshape(-1)
    E = []
    for m in range(M):
        for k in range(M):
            w = torch.zeros(P * Q, dtype=torch.complex128, device=DEV)
            w.index_add_(0, at, H[m * NN:(m + 1) * NN, k * NN:(k + 1) * NN].conj().reshape(-1))
            E.append(torch.fft.ifft2(w.reshape(P, Q), norm="forward"))
    return [E[m * M:(m + 1) * M] for m in range(M)]


def _penalty(c, E, rho):
    T, M, out = c["T"], c["M"], torch.zeros_like(rho)
    z = _windows(c, rho)
    for m in range(M):
        u = sum(E[m][k] * z[k] for k in range(M))
        if c.get("giraf"):
            out += torch.roll(u, -m, 0)
        else:
            out[M - 1 - m:T - m] += u
    return out


def _fp(rho):
    return torch.fft.fft2(rho, norm="ortho")


def _cg(op, rhs, x, n):
    r = rhs - op(x)
    p, rr = r.clone(), float(torch.linalg.vector_norm(r)) ** 2
    for _ in range(n):
        q = op(p)
        pq = float(torch.vdot(p.reshape(-1), q.reshape(-1)).real)
        if rr == 0.0 or pq <= 0.0:
            break
        x = x + (rr / pq) * p
        r = r - (rr / pq) * q
        new = float(torch.linalg.vector_norm(r)) ** 2
        p, rr = r + (new / rr) * p, new
    return x


def _voxel_masks(c, x, eps):
    """Per pixel: the Gram matrix of its Toeplitz lifting by a batched cyclic Jacobi method
    (complex Hermitian M x M), its largest eigenvalue and the masks conj((G + eps)^(p/2-1))."""
    M = c["M"]
    z = _windows(c, torch.fft.ifft2(x, norm="ortho"))
    A = torch.stack([torch.stack([(z[m].conj() * z[k]).sum(0).reshape(-1) for k in range(M)]) for m in range(M)])
    V = torch.eye(M, dtype=torch.complex128, device=DEV)[:, :, None].repeat(1, 1, A.shape[2])
    for _ in range(12):
        for p in range(M):
            for q in range(p + 1, M):
                apq = A[p, q]
                mag = apq.abs()
                ph = torch.where(mag > 0, apq / mag.clamp(min=1e-300), torch.ones_like(apq))
                th = 0.5 * torch.atan2(2 * mag, A[q, q].real - A[p, p].real)
                cs, sn = torch.cos(th), torch.sin(th)
                for X in (A, V):  # columns: x_p' = c x_p - s conj(ph) x_q, x_q' = s ph x_p + c x_q
                    xp, xq = X[:, p].clone(), X[:, q].clone()
                    X[:, p], X[:, q] = cs * xp - sn * ph.conj() * xq, sn * ph * xp + cs * xq
                xp, xq = A[p].clone(), A[q].clone()
                A[p], A[q] = cs * xp - sn * ph * xq, sn * ph.conj() * xp + cs * xq
    lam = torch.stack([A[m, m].real for m in range(M)])
    top = float(lam.max())
    if eps is None:
        eps = EPS0 * top
    al = (lam.clamp(min=0.0) + eps) ** (P_NORM / 2 - 1)
    shape = (c["P"], c["Q"])
    E = [[(al * V[m].conj() * V[k]).sum(0).reshape(shape) for k in range(M)] for m in range(M)]
    return E, eps


def _lift(c, x):
    """The lifted matrix that is linear in all three dimensions, (n, w1, w2) x (m, a1, a2)."""
    xc = torch.fft.fftshift(x, dim=(1, 2))
    win = xc.unfold(1, c["N1"], 1).unfold(2, c["N2"], 1).flip(3, 4)  # [T][w1][w2][a1][a2]
    T, M = c["T"], c["M"]
    X = torch.stack([win[M - 1 - m:T - m] for m in range(M)], dim=3)
    return X.reshape(-1, M * c["N1"] * c["N2"])


def _lift_adjoint(c, Y):
    T, P, Q, N1, N2, M = (c[k] for k in ("T", "P", "Q", "N1", "N2", "M"))
    Y = Y.reshape(T - M + 1, P - N1 + 1, Q - N2 + 1, M, N1, N2)
    out = torch.zeros(T, P, Q, dtype=Y.dtype, device=DEV)
    for m in range(M):
        for i in range(N1):
            for j in range(N2):
                o1, o2 = N1 - 1 - i, N2 - 1 - j
                out[M - 1 - m:T - m, o1:o1 + P - N1 + 1, o2:o2 + Q - N2 + 1] += Y[:, :, :, m, i, j]
    return torch.fft.ifftshift(out, dim=(1, 2))


def _recon(c, b, S, C):
    S, b, C = S.double(), S * b.to(torch.complex128), None if C is None else C.to(torch.complex128)
    data = lambda v: S * v  # noqa: E731
    if C is not None:
        b = _fp((C.conj()[:, None] * torch.fft.ifft2(b, norm="ortho")).sum(0))

        def data(v):
            rho = torch.fft.ifft2(v, norm="ortho")
            return _fp(sum(Cj.conj() * torch.fft.ifft2(S * _fp(Cj * rho), norm="ortho") for Cj in C))
    x, eps = b, None
    for _ in range(c["n_irls"]):
        if c["kind"] == "voxel":
            E, eps = _voxel_masks(c, x, eps)
        else:
            X = _lift(c, x) if c["kind"] == "direct" else None
            lam, U = torch.linalg.eigh(_gram(c, x) if X is None else X.conj().T @ X)
            if eps is None:
                eps = EPS0 * float(lam.max())
            H = _power(lam, U, eps)
            E = None if c["kind"] == "direct" else _penalty_masks(c, H)
        if c["kind"] == "direct":
            op = lambda v: data(v) + LAM * _lift_adjoint(c, _lift(c, v) @ H)  # noqa: E731,B023
        else:
            op = lambda v: data(v) + LAM * _fp(_penalty(c, E, torch.fft.ifft2(v, norm="ortho")))  # noqa: E731,B023
        x = _cg(op, b, x, c["n_cg"])
        eps /= GAMMA
    return torch.fft.ifft2(x, norm="ortho")


def exact(case, seed):
    kind = case["kind"]
    if kind == "apply":
        S, E, v = _operator(case, seed)
        M, E, v = case["M"], E.to(torch.complex128), v.to(torch.complex128)
        full = [[None] * M for _ in range(M)]
        w = 0
        for m in range(M):
            for k in range(m, M):
                full[m][k], full[k][m] = E[w], E[w].conj()
                w += 1
        return S * v + LAM * _fp(_penalty(case, full, torch.fft.ifft2(v, norm="ortho")))
    if kind in ("batch", "serve"):  # the first slices only: each is a whole reconstruction
        out = []
        for j, c in enumerate(_slices(case, seed)):
            out.append(_recon(c, *_data(c, 1000 * seed + j)) if j < 3 else None)
        return out
    b, S, C = _data(case, seed)
    if kind != "weights":
        return _recon(case, b, S, C)
    lam, U = torch.linalg.eigh(_gram(case, S * b.to(torch.complex128)))
    H = _power(lam, U, WEIGHTS_EPS)
    E = _penalty_masks(case, H)
    return [lam, H, torch.stack([E[m][k] for m in range(case["M"]) for k in range(m, case["M"])])]


# -------------------------------------------------------------------- work
def _fft_flops(n, P, Q):
    return 5.0 * n * math.log2(P * Q)


def _operator_flops(c, V, pq):
    f = 2 * _fft_flops(V, c["P"], c["Q"]) + 8.0 * (2 * c["M"] - 1) * V + 6.0 * V
    if c["kind"] == "coils":
        f += c["nc"] * (2 * _fft_flops(V, c["P"], c["Q"]) + 16.0 * V)
    return f


def _update_flops(c, V, pq):
    """One weight update: the Gram matrix, its eigen-decomposition, the masks."""
    M, N1, N2, k = c["M"], c["N1"], c["N2"], c["T"] - c["M"] + 1
    W, L1, L2, s = M * (M + 1) / 2, 2 * N1 - 1, 2 * N2 - 1, N1 * N2 * M
    if c["kind"] == "voxel":
        return _fft_flops(V, c["P"], c["Q"]) + pq * (8.0 * W * k + 40.0 * M ** 3)
    eig = (16 / 3 + 4 / 3 + 8) * s ** 3
    if c["kind"] == "direct":
        return 4.0 * s * s * k * (c["P"] - N1 + 1) * (c["Q"] - N2 + 1) + eig + 4.0 * s ** 3
    gram = _fft_flops(V, c["P"], c["Q"]) + 8.0 * W * (k * pq + pq * L2 + c["P"] * L1 * L2)
    masks = 8.0 * s * (M * L1 * L2 * N2 / N1 + W * L1 * L2) + 8.0 * W * (L1 * L2 * c["Q"] + L1 * pq)
    return gram + eig + masks


def work(case):
    kind, V, pq = case["kind"], float(case["T"] * case["P"] * case["Q"]), float(case["P"] * case["Q"])
    W, s = case["M"] * (case["M"] + 1) // 2, case["N1"] * case["N2"] * case["M"]
    if kind == "apply":
        return {"bytes": 17 * V + 8 * W * pq, "flops": _operator_flops(case, V, pq)}
    if kind == "weights":
        return {"bytes": 9 * V + 8 * s + 16 * s * s + 8 * W * pq, "flops": _update_flops(case, V, pq) + 8.0 * s ** 3}
    if kind in ("batch", "serve"):
        each = [work(c) for c in _slices(case, 0)]
        return {k: sum(e[k] for e in each) for k in ("bytes", "flops")}
    if kind == "direct":
        rows = (case["T"] - case["M"] + 1) * (case["P"] - case["N1"] + 1) * (case["Q"] - case["N2"] + 1)
        op = 8.0 * s * s * rows
    else:
        op = _operator_flops(case, V, pq) + 24.0 * V
    data = 8 * V * case.get("nc", 1) + V + 8 * V + (8 * pq * case["nc"] if kind == "coils" else 0)
    return {"bytes": data, "flops": case["n_irls"] * (_update_flops(case, V, pq) + (case["n_cg"] + 1) * op)}
