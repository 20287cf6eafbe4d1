"""Workloads of the library as a user's program calls them, for timing.

Families (the ``kind`` of a case):
  dirac       one application of D, or of a Dirichlet slab block, to 1-12 columns
  solve       one linear solve D x = b on the lattice or a slab, 1-12 columns
  factorised  the factorised propagator, the exact one and both pion correlators
  batched     one batch of uneven independent Dirichlet domains
  force       the pseudofermion action of a Dirichlet domain and its gradients
  blocks      baryon blocks of a set of quark lines
  basis       quark-line projection vectors by inverse iteration

Sizes are those of the package's workloads (16x4^3, 32x16^3, 64x32^3, the 96-domain
batch and its shapes) and generic ones between them, odd extents among them.  A
program keeps one context per lattice for all its gauge fields, so contexts are kept
per lattice here too; links, sources and output buffers belong to one state.  Links
are SU(3) matrices exp(i eps H) as in ``inputs.py``, made on the GPU from the seed.
Solves run to 1e-12, so that the answers of two correct solvers agree far better than
1e-9.
"""
import math

import torch

import paper_1612_06424_amd.dd as dd

DEV = "cuda:0"
_CONTEXTS = {}


def _ctx(T, L, bc):
    key = (T, L, bc)
    if key not in _CONTEXTS:
        _CONTEXTS[key] = dd.Context(T, L, bc)
    return _CONTEXTS[key]


# ------------------------------------------------------------------ the cases

def listed():
    return [
        # the smallest call: D on the smallest workload, one column (launch latency)
        dict(name="dirac_16x4_fp64_1", kind="dirac", T=16, L=4, bc=-1, t0=0, nt=0, ncol=1, fp64=True),
        # an odd slab across the time edge, 5 columns in FP32: nothing is a multiple of a tile
        dict(name="dirac_slab_11x15_fp32_5", kind="dirac", T=24, L=15, bc=-1, t0=18, nt=11, ncol=5, fp64=False),
        # one column on the ordinary lattice's slab, the domain of its factorised propagator
        dict(name="dirac_slab_16x16_fp64_1", kind="dirac", T=32, L=16, bc=-1, t0=0, nt=16, ncol=1, fp64=True),
        # the headline lattice, all 12 spin-colour columns of a propagator, both precisions
        dict(name="dirac_64x32_fp32_12", kind="dirac", T=64, L=32, bc=-1, t0=0, nt=0, ncol=12, fp64=False),
        dict(name="dirac_64x32_fp64_12", kind="dirac", T=64, L=32, bc=-1, t0=0, nt=0, ncol=12, fp64=True),
        # the 12 point sources of a propagator on one domain of the headline lattice, mixed precision
        dict(name="solve_slab_16x32_mixed_12", kind="solve", T=64, L=32, bc=-1, t0=0, nt=16, ncol=12, mixed=True,
             cgnr=True, point=True, eps=0.15, kappa=0.135, iters=350),
        # Gaussian volume sources on the ordinary lattice, FP64 throughout
        dict(name="solve_32x16_fp64_12", kind="solve", T=32, L=16, bc=-1, t0=0, nt=0, ncol=12, mixed=False,
             cgnr=True, point=False, eps=0.2, kappa=0.13, iters=120),
        # a whole calculation on the smallest workload: slab solves, frontier hops, exact
        # propagator, correlators (many small launches)
        dict(name="factorised_16x4", kind="factorised", T=16, L=4, bc=-1, ndom=2, overlap=0, mixed=True, eps=0.3,
             kappa=0.125, iters=50),
        # many local problems at once: 24 uneven domains, 12 point sources each
        dict(name="batched_24", kind="batched", ndom=24, ncol=12, mixed=True, shapes=4),
        # one step of a molecular-dynamics force on a Dirichlet domain: two solves, forward and backward
        dict(name="force_32x16", kind="force", T=32, L=16, bc=0, t0=0, nt=0, ncol=1, mixed=True, eps=0.2, kappa=0.13,
             iters=140),
        # nucleon blocks of 120 lines on one 32^3 time slice (the source slice)
        dict(name="blocks_120_32", kind="blocks", n=120, L=32, nt=1),
        # 24 projection vectors of a frontier, one inverse iteration on 8 slices of 16^3
        dict(name="basis_24_8x16", kind="basis", T=32, L=16, bc=-1, t0=12, nt=8, nvec=24, n_iter=1, mixed=True, eps=0.2,
             kappa=0.125, iters=70),
    ]


def _logint(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["dirac", "dirac", "dirac", "solve", "solve", "factorised", "batched", "force", "blocks", "basis"])
    if kind == "dirac":
        while True:
            T, L, ncol = _logint(rng, 4, 64), _logint(rng, 4, 32), rng.randint(1, 12)
            if T * L ** 3 * ncol <= 64 * 32 ** 3 * 12 // 2:
                break
        nt = 0 if rng.random() < 0.5 else rng.randint(1, T - 1)
        return dict(kind=kind, T=T, L=L, bc=rng.choice([-1, 0, 1]), t0=0 if nt == 0 else rng.randrange(T), nt=nt,
                    ncol=ncol, fp64=rng.random() < 0.5)
    if kind == "solve":
        while True:
            T, L, ncol = _logint(rng, 8, 48), _logint(rng, 4, 32), rng.randint(1, 12)
            nt = 0 if rng.random() < 0.5 else rng.randint(2, T - 1)
            if (nt or T) * L ** 3 * ncol <= 32 * 16 ** 3 * 12 * 2 and T * L ** 3 <= 32 * 32 ** 3:
                break
        return dict(kind=kind, T=T, L=L, bc=-1, t0=0 if nt == 0 else rng.randrange(T), nt=nt, ncol=ncol,
                    mixed=rng.random() < 0.6, cgnr=rng.random() < 0.7, point=rng.random() < 0.5, eps=0.2,
                    kappa=round(rng.uniform(0.115, 0.128), 4))
    if kind == "factorised":
        T, L = rng.choice([8, 12, 16, 24]), rng.choice([4, 5, 6, 8])
        return dict(kind=kind, T=T, L=L, bc=-1, ndom=rng.choice([2, 3, 4]), overlap=rng.choice([0, 0, 1]),
                    mixed=rng.random() < 0.7, eps=0.3, kappa=round(rng.uniform(0.115, 0.125), 4))
    if kind == "batched":
        return dict(kind=kind, ndom=_logint(rng, 2, 24), ncol=rng.randint(1, 12), mixed=rng.random() < 0.7,
                    shapes=rng.randint(1, 4))
    if kind == "force":
        T, L = _logint(rng, 6, 32), _logint(rng, 4, 16)
        nt = 0 if rng.random() < 0.5 else rng.randint(2, T - 1)
        return dict(kind=kind, T=T, L=L, bc=0, t0=0 if nt == 0 else rng.randrange(T - nt + 1), nt=nt,
                    ncol=rng.randint(1, 4), mixed=rng.random() < 0.7, eps=0.2, kappa=round(rng.uniform(0.115, 0.128), 4))
    if kind == "blocks":
        n, nt = _logint(rng, 4, 120), rng.randint(1, 4)
        return dict(kind=kind, n=n, L=_logint(rng, 4, 32 if n <= 60 else 20), nt=nt)
    T, L = rng.choice([16, 24, 32]), rng.choice([5, 8, 9, 12, 16])
    nt = rng.randint(4, 8)
    return dict(kind="basis", T=T, L=L, bc=-1, t0=rng.randrange(T - nt), nt=nt, nvec=rng.randint(4, 36), n_iter=1,
                mixed=True, eps=0.2, kappa=round(rng.uniform(0.115, 0.125), 4))


# ------------------------------------------------------------------ inputs

def _mul3(a, b):
    return [[a[i][0] * b[0][j] + a[i][1] * b[1][j] + a[i][2] * b[2][j] for j in range(3)] for i in range(3)]


def _links(T, L, eps, gen):
    """SU(3) links exp(i eps H), H traceless Hermitian with Gaussian entries: (4, 9, V) complex128.
    Ten terms of the Taylor series of exp(i eps H / 8), squared three times."""
    V = T * L ** 3
    h = torch.randn((9, 4, V), dtype=torch.float64, device=DEV, generator=gen) * (eps / 8)
    tr = (h[0] + h[1] + h[2]) / 3
    z = torch.zeros_like(tr)
    d = [torch.complex(z, h[k] - tr) for k in range(3)]  # i times the entries of eps H / 8
    u01, u02, u12 = (torch.complex(-h[4 + 2 * k], h[3 + 2 * k]) for k in range(3))
    a = [[d[0], u01, u02], [-u01.conj().resolve_conj(), d[1], u12],
         [-u02.conj().resolve_conj(), -u12.conj().resolve_conj(), d[2]]]
    e = [[a[i][j] / 10 + (1.0 if i == j else 0.0) for j in range(3)] for i in range(3)]
    for k in range(9, 0, -1):
        m = _mul3(a, e)
        e = [[m[i][j] / k + (1.0 if i == j else 0.0) for j in range(3)] for i in range(3)]
    for _ in range(3):
        e = _mul3(e, e)
    return torch.stack([e[i][j] for i in range(3) for j in range(3)], dim=1).contiguous()


def _gauss(shape, gen, dtype=torch.complex128):
    return torch.randn(shape, dtype=dtype, device=DEV, generator=gen)


def _dom(case):
    return None if case["nt"] == 0 else (case["t0"], case["nt"])


def _nsite(case):
    return (case["nt"] or case["T"]) * case["L"] ** 3


def _params(case):
    return dd.solver_params(tol=1e-12, max_iter=20000, prec=dd.DD_MIXED if case["mixed"] else dd.DD_FP64,
                            solver=dd.DD_CGNR if case.get("cgnr", True) else dd.DD_BICGSTAB)


def _slabs(case):
    T, n = case["T"], case["ndom"]
    cut = [T * k // n for k in range(n + 1)]
    return [(cut[k], cut[k + 1] - cut[k]) for k in range(n)]


#: (T, L) of the domains of the uneven batch
SHAPES = [(8, 8), (8, 12), (16, 8), (16, 16)]


def prepare(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    kind = case["kind"]
    s = dict(case=case, kind=kind)
    if kind == "batched":
        s["ctx"] = _ctx(8, 8, 0)
        s["params"] = _params(case)
        s["items"] = []
        for i in range(case["ndom"]):
            # every shape of the case in turn, so that the work does not depend on the seed
            T, L = SHAPES[i % case["shapes"]]
            b = torch.zeros((case["ncol"], 12, T * L ** 3), dtype=torch.complex128, device=DEV)
            for j in range(case["ncol"]):
                b[j, j, (T // 2) * L ** 3] = 1.0
            kappa = 0.125 + 0.005 * ((i * 7) % case["ndom"]) / case["ndom"]
            s["items"].append(dict(T=T, L=L, time_bc=0, U=_links(T, L, 0.2, gen), kappa=kappa, b=b,
                                   x=torch.empty_like(b)))
        return s
    if kind == "blocks":
        s["ctx"] = _ctx(max(2, case["nt"]), case["L"], -1)
        # quark lines come from solves with orthonormal sources: entries of order one
        s["s"] = _gauss((case["n"], 12, case["nt"] * case["L"] ** 3), gen)
        return s
    T, L = case["T"], case["L"]
    s["ctx"] = _ctx(T, L, case["bc"])
    U = _links(T, L, case.get("eps", 0.15), gen)
    if kind == "dirac":
        dt = torch.complex128 if case["fp64"] else torch.complex64
        s["U"] = U.to(dt)
        s["kappa"] = 0.135
        s["psi"] = _gauss((case["ncol"], 12, _nsite(case)), gen, dt)
        s["out"] = torch.empty_like(s["psi"])
        return s
    s["U"], s["kappa"], s["params"] = U, case["kappa"], _params(case)
    if kind == "solve":
        n = _nsite(case)
        if case["point"]:
            b = torch.zeros((case["ncol"], 12, n), dtype=torch.complex128, device=DEV)
            site = int(torch.randint(n, (1,), device=DEV, generator=gen).item())
            for j in range(case["ncol"]):
                b[j, j, site] = 1.0
        else:
            b = _gauss((case["ncol"], 12, n), gen)
        s["b"], s["x"] = b, torch.empty_like(b)
    elif kind == "factorised":
        s["S"] = [torch.empty((12, 12, T * L ** 3), dtype=torch.complex128, device=DEV) for _ in range(2)]
    elif kind == "force":
        s["phi"] = _gauss((case["ncol"], 12, _nsite(case)), gen)
        s["U"].requires_grad_(True)
        s["phi"].requires_grad_(True)
    elif kind == "basis":
        s["v0"] = _gauss((case["nvec"], 12, _nsite(case)), gen)
    return s


# ------------------------------------------------------------------ one pass

def run(s):
    kind, case, ctx = s["kind"], s["case"], s["ctx"]
    if kind == "dirac":
        return dd.apply_dirac(ctx, s["U"], s["kappa"], s["psi"], _dom(case), s["out"])
    if kind == "solve":
        return dd.block_solve(ctx, s["U"], s["kappa"], s["b"], _dom(case), s["params"], s["x"])[0]
    if kind == "factorised":
        Sf, Se, _ = dd.factorized_propagator(ctx, s["U"], s["kappa"], (0, 0, 0, 0), _slabs(case), s["params"],
                                             exact=True, S_fact=s["S"][0], S_exact=s["S"][1], overlap=case["overlap"])
        return dict(S_fact=Sf, S_exact=Se, C_fact=dd.pion_correlator(ctx, Sf, 0), C_exact=dd.pion_correlator(ctx, Se, 0))
    if kind == "batched":
        dd.block_solve_batched(ctx, s["items"], s["params"])
        return [it["x"] for it in s["items"]]
    if kind == "force":
        s["U"].grad = s["phi"].grad = None
        S = dd.DomainActionFn.apply(s["U"], s["phi"], ctx, s["kappa"], _dom(case), s["params"])
        S.backward()
        return dict(S=S, grad_U=s["U"].grad, grad_phi=s["phi"].grad)
    if kind == "blocks":
        return dd.baryon_blocks(ctx, s["s"])
    return dd.projection_basis(ctx, s["U"], s["kappa"], _dom(case), case["t0"] + case["nt"] // 2 - 1, +1, s["v0"],
                               case["n_iter"], s["params"])[0]


# ------------------------------------------------------------------ work

def _iterations(case):
    """Krylov iterations (two applications of the operator each) of a solve to 1e-12: about those
    that CG on the even-odd operator takes (a little fewer), measured for the listed cases, else
    a line through the easy ones."""
    return case.get("iters") or int(40 + 2500 * max(0.0, case["kappa"] - 0.115))


def _solve_work(nsite, ncol, iters, real):
    # per iteration: two applications of the operator (spinors in and out, links once each) and the
    # update of three vectors; 1320 flops per site and hop sum
    per_site = 2 * (48 * ncol + 72) + 6 * 24 * ncol
    return dict(bytes=iters * nsite * per_site * real / 2, flops=iters * nsite * ncol * 2 * 1400.0)


def work(case):
    kind = case["kind"]
    if kind == "dirac":
        n, r = _nsite(case), 8 if case["fp64"] else 4
        return dict(bytes=n * (48 * case["ncol"] + 72) * r, flops=1392.0 * n * case["ncol"])
    if kind == "blocks":
        n, X = case["n"], case["L"] ** 3 * case["nt"]
        # (i, j) symmetric: n (n + 1) / 2 pairs, 4 n spin-line columns, 3 colours, 8 flops
        return dict(bytes=16.0 * (12 * n * X + 4 * n ** 3 * case["nt"]), flops=8.0 * 3 * 4 * n * (n * (n + 1) / 2) * X)
    real = 4 if case["mixed"] else 8
    if kind == "batched":
        n = sum(T * L ** 3 for T, L in (SHAPES[i % case["shapes"]] for i in range(case["ndom"])))
        return _solve_work(n, case["ncol"], 80, real)
    V = case["T"] * case["L"] ** 3
    it = _iterations(case)
    if kind == "factorised":
        return _solve_work(2 * V, 12, it, real)
    if kind == "force":
        return _solve_work(2 * _nsite(case), case["ncol"], it, real)
    if kind == "basis":
        return _solve_work(_nsite(case), case["nvec"], it, real)
    return _solve_work(_nsite(case), case["ncol"], it, real)


# ------------------------------------------------------------------ 64-bit values

_GAMMA = {  # (gamma_mu psi)_s = factor * psi_{column}, chiral basis
    0: [(2, -1), (3, -1), (0, -1), (1, -1)],
    1: [(3, -1j), (2, -1j), (1, 1j), (0, 1j)],
    2: [(3, -1), (2, 1), (1, 1), (0, -1)],
    3: [(2, -1j), (3, 1j), (0, 1j), (1, -1j)],
}


def _gamma(mu, p):
    return torch.stack([f * p[:, j] for j, f in _GAMMA[mu]], dim=1)


def _colour(u, p, adj):
    """u or u^+ times the colour index of p (col, 4, 3, t, z, y, x); u (3, 3, t, z, y, x)."""
    w = u.conj().transpose(0, 1) if adj else u
    return torch.stack([sum(w[i, j] * p[:, :, j] for j in range(3)) for i in range(3)], dim=2)


def _dirac64(U, kappa, psi, T, L, bc, dom, dag=False):
    """D psi (or D^+ psi) in complex128 with plain torch operations; psi (ncol, 12, nsite)."""
    t0, nt = dom if dom is not None else (0, T)
    ts = [(t0 + k) % T for k in range(nt)]
    u = U.reshape(4, 3, 3, T, L, L, L)[:, :, :, torch.tensor(ts, device=U.device)]
    p = psi.reshape(-1, 4, 3, nt, L, L, L)
    fac = [float(bc) if t == T - 1 else 1.0 for t in ts]  # of the hop between slices k and k + 1
    if dom is not None:
        fac[-1] = 0.0
    ph = torch.tensor(fac, dtype=torch.float64, device=U.device).reshape(1, 1, 1, nt, 1, 1, 1)
    sg = -1.0 if dag else 1.0
    out = p / (2 * kappa)
    for mu, dim in ((0, 3), (1, 6), (2, 5), (3, 4)):  # time, x, y, z
        f = torch.roll(p, -1, dim)
        h = _colour(u[mu], f - sg * _gamma(mu, f), False)
        q = _colour(u[mu], p + sg * _gamma(mu, p), True)
        if mu == 0:
            h, q = ph * h, ph * q
        out = out - 0.5 * (h + torch.roll(q, 1, dim))
    return out.reshape(psi.shape)


def _cg64(U, kappa, b, T, L, bc, dom, dag=False):
    """D^-1 b (or D^-+ b), conjugate gradients on the normal equations, columns independent."""
    x, r = torch.zeros_like(b), b.clone()
    op = lambda v, d: _dirac64(U, kappa, v, T, L, bc, dom, d)  # noqa: E731
    dot = lambda v: (v.real ** 2 + v.imag ** 2).sum(dim=(1, 2), keepdim=True)  # noqa: E731
    for _ in range(3):  # restarted from the true residual
        z = op(r, not dag)
        p, zz = z.clone(), dot(z)
        for k in range(3000):
            w = op(p, dag)
            al = zz / dot(w).clamp_min(1e-300)
            x, r = x + al * p, r - al * w
            z = op(r, not dag)
            z2 = dot(z)
            p, zz = z + (z2 / zz.clamp_min(1e-300)) * p, z2
            if k % 10 == 9 and bool((dot(r) <= 1e-28 * dot(b)).all()):
                break
        r = b - op(x, dag)
    return x


def exact(case, seed):
    kind = case["kind"]
    if kind in ("basis", "batched"):
        return None  # tens of solves: too long
    s = prepare(case, seed)
    if kind == "blocks":
        return _blocks64(s["s"], case)
    T, L, bc = case["T"], case["L"], case["bc"]
    U = s["U"].detach().to(torch.complex128)
    if kind == "dirac":
        out = torch.empty(s["psi"].shape, dtype=torch.complex128, device=DEV)
        for j in range(case["ncol"]):
            out[j] = _dirac64(U, s["kappa"], s["psi"][j:j + 1].to(torch.complex128), T, L, bc, _dom(case))[0]
        return out
    if _nsite(case) * case.get("ncol", 12) > 1 << 18 if kind != "factorised" else T * L ** 3 > 1 << 15:
        return None  # over the time that this takes with plain operations
    if kind == "solve":
        return _cg64(U, s["kappa"], s["b"], T, L, bc, _dom(case))
    if kind == "force":
        phi = s["phi"].detach()
        Y = _cg64(U, s["kappa"], phi, T, L, bc, _dom(case), True)
        X = _cg64(U, s["kappa"], Y, T, L, bc, _dom(case))
        V = U.clone().requires_grad_(True)
        F = -2 * (Y.conj() * _dirac64(V, s["kappa"], X, T, L, bc, _dom(case))).real.sum()
        F.backward()
        return dict(S=(Y.abs() ** 2).sum(), grad_U=V.grad, grad_phi=2 * X)
    eta = torch.zeros((12, 12, T * L ** 3), dtype=torch.complex128, device=DEV)
    for j in range(12):
        eta[j, j, 0] = 1.0
    Se = _cg64(U, s["kappa"], eta, T, L, bc, None)
    corr = lambda S: (S.abs() ** 2).reshape(12, 12, T, L ** 3).sum(dim=(0, 1, 3)).cpu().numpy()  # noqa: E731
    res = dict(S_fact=None, S_exact=Se, C_fact=None, C_exact=corr(Se))
    if case["ndom"] == 2 and case["overlap"] == 0:
        # psi_0 = D_0^-1 eta, psi_1 = -D_1^-1 D_{1,0} psi_0 (D applied to psi_0 extended by zero)
        L3, doms = L ** 3, _slabs(case)
        n0 = doms[0][1] * L3
        Sf = torch.zeros_like(eta)
        Sf[:, :, :n0] = _cg64(U, s["kappa"], eta[:, :, :n0].contiguous(), T, L, bc, doms[0])
        h = _dirac64(U, s["kappa"], Sf, T, L, bc, None)[:, :, n0:].contiguous()
        Sf[:, :, n0:] = -_cg64(U, s["kappa"], h, T, L, bc, doms[1])
        res.update(S_fact=Sf, C_fact=corr(Sf))
    return res


def _blocks64(s, case):
    """B[t][k][alpha][i][j] from the definition, chunks of sites."""
    n, L3, nt = case["n"], case["L"] ** 3, case["nt"]
    B = torch.zeros((nt, n, 4, n, n), dtype=torch.complex128, device=DEV)
    step = max(1, (1 << 25) // (n * n * 3))
    for t in range(nt):
        acc = torch.zeros((n * n, 4 * n), dtype=torch.complex128, device=DEV)
        for x0 in range(t * L3, (t + 1) * L3, step):
            f = s[:, :, x0:min((t + 1) * L3, x0 + step)].reshape(n, 4, 3, -1)
            dq = {}
            for a in range(3):
                for b in range(3):
                    if a != b:  # s_i^a (C gamma5) s_j^b
                        dq[a, b] = (f[:, None, 1, a] * f[None, :, 0, b] - f[:, None, 0, a] * f[None, :, 1, b]
                                    + f[:, None, 3, a] * f[None, :, 2, b] - f[:, None, 2, a] * f[None, :, 3, b])
            for a, b, c in ((1, 2, 0), (2, 0, 1), (0, 1, 2)):
                E = (dq[a, b] - dq[b, a]).reshape(n * n, -1)
                acc += E @ f[:, :, c].reshape(4 * n, -1).transpose(0, 1).contiguous()
        B[t] = acc.reshape(n, n, n, 4).permute(2, 3, 0, 1)
    return B
