"""The workloads the library's speed is measured on: products with the CCSD Jacobian (the sigma vector),
its transpose and its vector-Jacobian product, and the solves built from them, over the sizes, precisions
and directions that response calculations meet.

A case is a dict of plain values:
  op         "forward" | "adjoint" (device buffers), "grad" (forward and backward through autograd),
             "host" (forward on host arrays), "solve" (response equations on host arrays),
             "alpha" (polarizability at converged amplitudes)
  n0, n1, n2 k mesh (n1 = n2 = 1: a chain); o, v, naux orbitals and Cholesky vectors per k
  rhs        right-hand sides (frequencies, for "alpha")
  prec       "f64", or "f32": complex64 matrix-core products ("solve" and "alpha": complex64 corrections
             inside complex128 refinement)
  graph      replay the application as a HIP graph on a stream of its own
  tune       let the library time its launch variants once

Results of complex64 products are kept as complex64 vectors, as a mixed-precision Krylov basis keeps them.
"""
import math

import numpy as np
import torch

import paper_2508_01266_amd as lr
from paper_2508_01266_amd import autograd as lr_autograd

C = torch.complex128


def _case(op, mesh, o, v, naux, rhs, prec, graph=False, tune=False, name=None):
    n = tuple(mesh) + (1,) * (3 - len(mesh))
    c = dict(op=op, n0=n[0], n1=n[1], n2=n[2], o=o, v=v, naux=naux, rhs=rhs, prec=prec, graph=graph, tune=tune)
    return dict(c, name=name) if name else c


def listed():
    return [
        # one molecule in a cell: the smallest product, three axes at 0 and +-w in one batch
        _case("forward", (1,), 4, 12, 48, 9, "f64", name="molecule_f64"),
        # the same in complex64 as a long solve replays it, captured once
        _case("forward", (1,), 4, 12, 48, 9, "f32", graph=True, name="molecule_f32_graph"),
        # a three-k chain, two frequencies: one step of an ordinary complex128 solve
        _case("forward", (3,), 4, 20, 72, 12, "f64", name="chain3_f64"),
        # transposed products of a chain of ragged sizes, as the perturbed multipliers take them
        _case("adjoint", (3,), 5, 23, 61, 7, "f32", name="ragged3_adjoint_f32"),
        # forward and backward of a differentiable product inside a larger program
        _case("grad", (4,), 6, 26, 80, 6, "f64", name="chain4_grad_f64"),
        # a three-dimensional mesh, inner step of a mixed solve
        _case("forward", (2, 2, 2), 4, 16, 56, 12, "f32", name="mesh222_f32"),
        # complex64 product of the batched workload: three axes, +-w, eight frequencies
        _case("forward", (5,), 8, 40, 144, 48, "f32", tune=True, name="batch5_f32"),
        # complex128 residuals of the same system at two frequencies
        _case("forward", (5,), 8, 40, 144, 12, "f64", name="batch5_f64"),
        # one vector through the transposed product: a step of the multiplier equations
        _case("adjoint", (5,), 8, 40, 144, 1, "f64", name="lambda5_f64"),
        # wide virtual space, transposed products in complex64
        _case("adjoint", (3,), 10, 60, 210, 6, "f32", name="wide3_adjoint_f32"),
        # response equations of a molecule from host arrays, complex64 corrections
        _case("solve", (1,), 4, 12, 48, 6, "f32", name="molecule_solve_mixed"),
        # polarizability of the three-k chain at its own CCSD amplitudes, two frequencies
        _case("alpha", (3,), 4, 20, 72, 2, "f32", name="chain3_alpha_mixed"),
    ]


# most that a drawn product may take: the listed complex64 batch, one complex128 vector set of its size
_MOST_FLOPS = 2.0e12
_MOST_VECTOR = 48 * (5 ** 3) * 64 * 1600


def draw(rng):
    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    while True:
        op = rng.choice(["forward"] * 5 + ["adjoint"] * 3 + ["grad", "host", "solve"])
        prec = rng.choice(["f64", "f32"])
        mesh = rng.choice([(1,), (2,), (3,), (3,), (4,), (5,), (6,), (2, 2), (3, 2), (2, 2, 2)])
        nk = math.prod(mesh)
        o, v = rng.randint(2, 10), log(8, 60)
        naux = rng.randint(2 * (o + v), 3 * (o + v))
        rhs = rng.choice([1, 1, log(2, 48), 3 * rng.randint(1, 16)])
        if op == "solve":
            mesh, nk, o, v, rhs = rng.choice([(1,), (2,)]), 1, rng.randint(2, 5), log(8, 20), rng.randint(1, 8)
            naux = rng.randint(2 * (o + v), 3 * (o + v))
        if op == "host" and rhs * nk ** 3 * (o * v) ** 2 > 4_000_000:
            continue
        c = _case(op, mesh, o, v, naux, rhs, prec, graph=op in ("forward", "adjoint") and rng.random() < 0.25)
        n = nk * nk * naux * (o + v) ** 2
        cost = _flops(c) * (2.5 if prec == "f64" else 1.0)
        if rhs * nk ** 3 * (o * v) ** 2 <= _MOST_VECTOR / 4 and n <= 12_000_000 and nk ** 3 * (o * v) ** 2 <= 16_000_000 \
                and cost <= _MOST_FLOPS:
            return c


# ---------------------------------------------------------------- inputs
def _mesh(c):
    return c["n0"], c["n1"], c["n2"]


def _nk(c):
    return c["n0"] * c["n1"] * c["n2"]


def _kb(c):
    """kb[ki][kj][ka] = ki + kj - ka on the mesh (flat indices)."""
    n0, n1, n2 = _mesh(c)
    k = np.arange(_nk(c))
    comp = np.stack([k // (n1 * n2), (k // n2) % n1, k % n2])
    j = comp[:, :, None, None] + comp[:, None, :, None] - comp[:, None, None, :]
    j = [j[d] % n for d, n in enumerate((n0, n1, n2))]
    return torch.from_numpy((j[0] * n1 + j[1]) * n2 + j[2])


def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _normal(gen, shape, sigma):
    x = torch.randn(*shape, 2, generator=gen, device=gen.device, dtype=torch.float64)
    return torch.view_as_complex(x).mul_(sigma)


def _antisym(c, raw):
    """Doubles [nk]^3[o][o][v][v] antisymmetric in (ki,i),(kj,j) and in (ka,a),(kb,b)."""
    kb = _kb(c).to(raw.device)
    nk = raw.shape[0]
    a = raw - raw.permute(1, 0, 2, 4, 3, 5, 6)
    ki, kj = torch.meshgrid(torch.arange(nk, device=raw.device), torch.arange(nk, device=raw.device), indexing="ij")
    out = a.clone()
    for ka in range(nk):
        out[:, :, ka] -= a[ki, kj, kb[:, :, ka]].transpose(-1, -2)
    return out.mul_(0.5)


def _system(c, seed):
    """Hamiltonian, amplitudes and vectors of a case as device tensors, from the seed alone: band
    energies with a cosine shift, Cholesky vectors scaled so that the coupling of an amplitude row does
    not grow with the size, amplitudes of the magnitude that converged ones have."""
    dev = _device()
    gen = torch.Generator(device=dev)
    gen.manual_seed(1266 + 7919 * int(seed))
    nk, o, v, naux = _nk(c), c["o"], c["v"], c["naux"]
    n = o + v

    def uniform(lo, hi, m):
        return torch.sort(torch.rand(m, generator=gen, device=dev, dtype=torch.float64) * (hi - lo) + lo)[0]

    band = torch.cat([uniform(-1.5, -0.3, o), uniform(0.2, 3.0, v)])
    k = torch.arange(nk, device=dev)
    n0, n1, n2 = _mesh(c)
    comp = [k // (n1 * n2), (k // n2) % n1, k % n2]
    per = [d for d in range(3) if _mesh(c)[d] > 1]
    shift = sum(torch.cos(2 * math.pi * comp[d] / _mesh(c)[d]) for d in per) / len(per) if per else torch.zeros(1, device=dev)
    fock = torch.diag_embed(band[None] + 0.1 * shift.to(torch.float64)[:, None]).to(C)
    sigma = 0.05 * min(1.0, math.sqrt(12 * math.sqrt(48.0) / (v * math.sqrt(naux / nk))))
    raw = _normal(gen, (nk, nk, naux, n, n), sigma)
    herm = raw.permute(1, 0, 2, 4, 3).conj()
    low = (k[:, None] < k[None, :])[:, :, None, None, None]
    same = (k[:, None] == k[None, :])[:, :, None, None, None]
    chol = torch.where(low, raw, herm)
    chol = torch.where(same, (raw + herm) / math.sqrt(2.0), chol).resolve_conj()
    dip = _normal(gen, (3, nk, n, n), 0.5)
    dip = ((dip + dip.transpose(-1, -2).conj()) / 2).resolve_conj()
    t1 = _normal(gen, (nk, o, v), 0.02)
    t2 = _antisym(c, _normal(gen, (nk, nk, nk, o, o, v, v), 0.02 * nk))
    s = dict(fock=fock, chol=chol, dip=dip, t1=t1, t2=t2)
    if c["op"] != "alpha":
        R = c["rhs"]
        s["x1"] = _normal(gen, (R, nk, o, v), 0.1)
        s["x2"] = torch.empty((R, nk, nk, nk, o, o, v, v), dtype=C, device=dev)
        for r in range(R):
            s["x2"][r] = _antisym(c, _normal(gen, (nk, nk, nk, o, o, v, v), 0.1 * nk))
        s["omega"] = torch.linspace(-0.1, 0.1, R, dtype=torch.float64, device=dev) if R > 1 else \
            torch.full((1,), 0.0656, dtype=torch.float64, device=dev)
        if c["op"] == "grad":
            s["g1"] = _normal(gen, (R, nk, o, v), 0.1)
            s["g2"] = _normal(gen, (R, nk, nk, nk, o, o, v, v), 0.1)
    else:
        s["omegas"] = [0.0656 * (j + 0.1 * float(torch.rand(1, generator=gen, device=dev))) for j in range(c["rhs"])]
    return s


def _host(t):
    return np.ascontiguousarray(t.cpu().numpy())


def prepare(case, seed):
    c = dict(case)
    s = _system(c, seed)
    ctx = lr.Context(0)
    if c["n1"] * c["n2"] > 1:
        ctx.set_kmesh(*_mesh(c))
    ctx.set_hamiltonian(c["o"], _host(s["fock"]), _host(s["chol"]), _host(s["dip"]))
    if c["op"] == "alpha":
        ctx.solve_ccsd(tol=1e-11, max_iter=300)
        return dict(c=c, ctx=ctx, omegas=s["omegas"])
    ctx.set_amplitudes(_host(s["t1"]), _host(s["t2"]))
    ctx.set_autotune(c["tune"])
    st = dict(c=c, ctx=ctx, prec=lr.FP64 if c["prec"] == "f64" else lr.FP32)
    if c["op"] in ("host", "solve"):
        st.update(x1=_host(s["x1"]), x2=_host(s["x2"]), omega=_host(s["omega"]))
        return st
    st.update(x1=s["x1"], x2=s["x2"], omega=s["omega"])
    if c["op"] == "grad":
        st["x1"].requires_grad_(True)
        st["x2"].requires_grad_(True)
        st.update(g1=s["g1"], g2=s["g2"])
        return st
    st.update(y1=torch.empty_like(s["x1"]), y2=torch.empty_like(s["x2"]))
    if c["graph"]:
        ctx.set_graphs(True)
        st["stream"] = torch.cuda.Stream()
    if c["graph"] or c["tune"]:      # captured or tuned once, before the solve's iterations
        torch.cuda.synchronize()
        run(st)
        torch.cuda.synchronize()
    return st


# ---------------------------------------------------------------- one pass
def _product(st):
    c, ctx = st["c"], st["ctx"]
    stream = torch.cuda.current_stream()
    ctx.apply_sigma_dev(st["x1"], st["x2"], st["y1"], st["y2"], st["omega"], st["prec"], stream.cuda_stream,
                        adjoint=c["op"] == "adjoint")
    if c["prec"] == "f32":
        return st["y1"].to(torch.complex64), st["y2"].to(torch.complex64)
    return st["y1"], st["y2"]


def run(st):
    c, ctx = st["c"], st["ctx"]
    if c["op"] == "alpha":
        a, _ = ctx.solve(st["omegas"], axis_mask=7, tol=1e-11, precision=lr.FP32, reuse_lambda=0)
        return (a, *ctx.get_lambda())
    if c["op"] == "solve":
        y1, y2, _ = ctx.solve_response(st["x1"], st["x2"], st["omega"], tol=1e-12, precision=st["prec"])
        return y1, y2
    if c["op"] == "host":
        y1, y2 = ctx.apply_sigma(st["x1"], st["x2"], st["omega"], st["prec"])
        return (y1.astype(np.complex64), y2.astype(np.complex64)) if c["prec"] == "f32" else (y1, y2)
    if c["op"] == "grad":
        y1, y2 = lr_autograd.sigma(ctx, st["x1"], st["x2"], st["omega"], st["prec"])
        d1, d2 = torch.autograd.grad((y1, y2), (st["x1"], st["x2"]), (st["g1"], st["g2"]))
        out = [y1.detach(), y2.detach(), d1, d2]
        return [t.to(torch.complex64) for t in out] if c["prec"] == "f32" else out
    if c["graph"]:
        s = st["stream"]
        s.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(s):
            out = _product(st)
        torch.cuda.current_stream().wait_stream(s)
        for t in out:
            t.record_stream(torch.cuda.current_stream())
        return out
    return _product(st)


# ---------------------------------------------------------------- what a pass cannot do without
def _flops(c):
    """Real operations of one pass, 8 per complex multiply-add, over the unique antisymmetric index pairs
    where a product has them: the particle-particle ladder, the ring, the hole-hole products and the
    one-body terms."""
    nk, o, v = _nk(c), c["o"], c["v"]
    po, pv = nk * o * (nk * o - 1) / 2, nk * v * (nk * v - 1) / 2   # unique pairs, all momenta
    per = po * pv * pv / nk ** 2 + 2 * po * po * pv / nk ** 2 + nk ** 4 * (o * v) ** 3 \
        + 4 * nk ** 3 * (o * v) ** 2 * (o + v) / 2
    passes = {"forward": 1, "adjoint": 1, "host": 1, "grad": 2, "solve": 20, "alpha": 300}[c["op"]]
    return 8.0 * per * passes * c["rhs"]


def work(case):
    c = dict(case)
    nk, o, v, naux = _nk(c), c["o"], c["v"], c["naux"]
    vec = 16.0 * (nk * o * v + nk ** 3 * (o * v) ** 2)
    out = (0.5 if c["prec"] == "f32" and c["op"] not in ("solve", "alpha") else 1.0) * vec
    ham = 16.0 * nk * nk * naux * (o + v) ** 2 + vec
    if c["op"] == "alpha":
        return {"bytes": ham + 16.0 * 9 * c["rhs"], "flops": _flops(c)}
    n = 2 if c["op"] == "grad" else 1
    return {"bytes": ham + n * c["rhs"] * (vec + out), "flops": _flops(c)}


# ---------------------------------------------------------------- the same in plain torch, 64 bits
def _dense(c, s):
    """Fock matrix and antisymmetrised integrals <PQ||RS> on collective indices, occupied first."""
    nk, o, v, naux = _nk(c), c["o"], c["v"], c["naux"]
    dev = s["fock"].device
    N, kb = nk * (o + v), _kb(c)
    idx = torch.stack([torch.cat([k * o + torch.arange(o), nk * o + k * v + torch.arange(v)]) for k in range(nk)]).to(dev)
    f = torch.zeros(N, N, dtype=C, device=dev)
    L = torch.zeros(nk, naux, N, N, dtype=C, device=dev)
    for k1 in range(nk):
        f[idx[k1][:, None], idx[k1][None, :]] = s["fock"][k1]
        for k2 in range(nk):
            q = int(kb[k2, 0, k1])                    # momentum transfer k2 - k1
            L[q][:, idx[k1][:, None], idx[k2][None, :]] = s["chol"][k1, k2]
    return f, L.reshape(nk * naux, N, N) / math.sqrt(nk)


def _to_dense(c, x1, x2):
    nk, o, v = _nk(c), c["o"], c["v"]
    kb = _kb(c)
    d1 = torch.zeros(nk * o, nk * v, dtype=C, device=x1.device)
    d2 = torch.zeros(nk * o, nk * o, nk * v, nk * v, dtype=C, device=x1.device)
    for i in range(nk):
        d1[i * o:(i + 1) * o, i * v:(i + 1) * v] = x1[i]
        for j in range(nk):
            for a in range(nk):
                b = int(kb[i, j, a])
                d2[i * o:(i + 1) * o, j * o:(j + 1) * o, a * v:(a + 1) * v, b * v:(b + 1) * v] = x2[i, j, a]
    return d1, d2


def _to_blocks(c, d1, d2):
    nk, o, v = _nk(c), c["o"], c["v"]
    kb = _kb(c)
    x1 = torch.stack([d1[k * o:(k + 1) * o, k * v:(k + 1) * v] for k in range(nk)])
    x2 = torch.empty(nk, nk, nk, o, o, v, v, dtype=C, device=d1.device)
    for i in range(nk):
        for j in range(nk):
            for a in range(nk):
                b = int(kb[i, j, a])
                x2[i, j, a] = d2[i * o:(i + 1) * o, j * o:(j + 1) * o, a * v:(a + 1) * v, b * v:(b + 1) * v]
    return x1, x2


def _residual(t1, t2, f, W, no):
    """The spin-orbital CCSD residual (singles, doubles) in the factorisation of Stanton and Gauss, with
    the full Fock matrix; W: the integral classes by their orbital letters."""
    e = torch.einsum
    fo, fv = slice(0, no), slice(no, None)
    fov, foo, fvv, fvo = f[fo, fv], f[fo, fo], f[fv, fv], f[fv, fo]
    pair = e("ia,jb->ijab", t1, t1)
    pair = pair - pair.transpose(2, 3)
    tau, half = t2 + pair, t2 + 0.5 * pair
    Fv = fvv - 0.5 * e("me,ma->ae", fov, t1) + e("mf,mafe->ae", t1, W["ovvv"]) - 0.5 * e("mnaf,mnef->ae", half, W["oovv"])
    Fo = foo + 0.5 * e("ie,me->mi", t1, fov) + e("ne,mnie->mi", t1, W["ooov"]) + 0.5 * e("inef,mnef->mi", half, W["oovv"])
    Fx = fov + e("nf,mnef->me", t1, W["oovv"])
    w = e("je,mnie->mnij", t1, W["ooov"])
    Wo = W["oooo"] + w - w.transpose(2, 3) + 0.25 * e("ijef,mnef->mnij", tau, W["oovv"])
    w = e("mb,amef->abef", t1, -W["ovvv"].transpose(0, 1))
    Wv = W["vvvv"] - w + w.transpose(0, 1) + 0.25 * e("mnab,mnef->abef", tau, W["oovv"])
    Wx = W["ovvo"] + e("jf,mbef->mbej", t1, W["ovvv"]) + e("nb,mnje->mbej", t1, W["ooov"]) \
        - e("jnfb,mnef->mbej", 0.5 * t2 + e("jf,nb->jnfb", t1, t1), W["oovv"])
    r1 = fvo.T + t1 @ Fv.T - e("ma,mi->ia", t1, Fo) + e("imae,me->ia", t2, Fx) + e("nf,nafi->ia", t1, W["ovvo"]) \
        - 0.5 * e("imef,maef->ia", t2, W["ovvv"]) + 0.5 * e("mnae,nmie->ia", t2, W["ooov"])
    x = e("ijae,be->ijab", t2, Fv - 0.5 * t1.T @ Fx)
    r2 = W["oovv"].conj() + x - x.transpose(2, 3)
    x = e("imab,mj->ijab", t2, Fo + 0.5 * e("je,me->mj", t1, Fx))
    r2 = r2 - x + x.transpose(0, 1)
    r2 = r2 + 0.5 * e("mnab,mnij->ijab", tau, Wo) + 0.5 * e("ijef,abef->ijab", tau, Wv)
    x = e("imae,mbej->ijab", t2, Wx) - e("ie,mbej,ma->ijab", t1, W["ovvo"], t1)
    x = x - x.transpose(2, 3)
    r2 = r2 + x - x.transpose(0, 1)
    x = e("ie,jeba->ijab", t1, W["ovvv"].conj())           # <ab||ej> = conj <ej||ab>
    r2 = r2 + x - x.transpose(0, 1)
    x = e("ma,ijmb->ijab", t1, W["ooov"].conj())           # <mb||ij> = conj <ij||mb>
    return r1, r2 - x + x.transpose(2, 3)


def _both(x):
    x = x - x.transpose(0, 1)
    return x - x.transpose(2, 3)


def exact(case, seed):
    c = dict(case)
    nk, o, v = _nk(c), c["o"], c["v"]
    NO, NV, R = nk * o, nk * v, c["rhs"]
    dims = NO * NV + (NO * (NO - 1) // 2) * (NV * (NV - 1) // 2)
    dense = 16.0 * R * (NO ** 2 * NV ** 4 + 4 * (NO * NV) ** 3)
    if c["op"] == "alpha" or NV > 130 or dense > 2e14 or (c["op"] == "solve" and (nk > 1 or dims > 800)):
        return None
    s = _system(c, seed)
    f, L = _dense(c, s)
    chem = torch.einsum("xpr,xsq->prqs", L, L.conj())
    part = {"o": slice(0, NO), "v": slice(NO, None)}

    def eri(p, q, r, t):
        a = chem[part[p], part[r], part[q], part[t]].permute(0, 2, 1, 3)
        return (a - chem[part[p], part[t], part[q], part[r]].permute(0, 2, 3, 1)).contiguous()

    W = {k: eri(*k) for k in ("oovv", "ovvv", "ooov", "ovvo", "oooo", "vvvv")}
    del chem, L
    T = _to_dense(c, s["t1"], s["t2"] / nk)

    def omega(t1, t2):
        return _residual(t1, t2, f, W, NO)

    def product(x1, x2, w):
        d = _to_dense(c, x1, x2 / nk)
        y = torch.func.jvp(omega, T, d)[1]
        y1, y2 = _to_blocks(c, y[0], y[1])
        return y1 - w * x1, nk * y2 - w * x2

    out = []
    if c["op"] == "solve":
        i, j = torch.triu_indices(NO, NO, 1, device=f.device)
        a, b = torch.triu_indices(NV, NV, 1, device=f.device)

        def column(u):
            d2 = torch.zeros(NO, NO, NV, NV, dtype=C, device=f.device)
            d2[i[:, None], j[:, None], a[None], b[None]] = u[NO * NV:].reshape(len(i), len(a))
            return u[:NO * NV].reshape(NO, NV), _both(d2)

        cols = []
        for m in range(dims):
            u = torch.zeros(dims, dtype=C, device=f.device)
            u[m] = 1
            y1, y2 = torch.func.jvp(omega, T, column(u))[1]
            cols.append(torch.cat([y1.reshape(-1), y2[i[:, None], j[:, None], a[None], b[None]].reshape(-1)]))
        A = torch.stack(cols, 1)
        for r in range(R):
            b1, b2 = _to_dense(c, s["x1"][r], s["x2"][r] / nk)
            rhs = torch.cat([b1.reshape(-1), b2[i[:, None], j[:, None], a[None], b[None]].reshape(-1)])
            u = torch.linalg.solve(A - s["omega"][r] * torch.eye(dims, dtype=C, device=f.device), rhs)
            y1, y2 = _to_blocks(c, *column(u))
            out.append((y1, nk * y2))
    else:
        for r in range(R):
            x1, x2, w = s["x1"][r], s["x2"][r], s["omega"][r]
            if c["op"] == "adjoint":    # transposed in the pairing sum u1 w1 + 1/4 sum u2 w2
                z1, z2 = _to_dense(c, x1, x2 * nk)
                back = torch.func.vjp(omega, *T)[1]
                y1, y2 = (g.conj() for g in back((z1.conj(), 0.25 * z2.conj())))
                y1, y2 = _to_blocks(c, y1, _both(y2))
                out.append((y1 - w * x1, y2 / nk - w * x2))
            elif c["op"] == "grad":     # conjugate transpose, within the antisymmetric doubles
                z1, z2 = _to_dense(c, s["g1"][r], s["g2"][r] * nk)
                back = torch.func.vjp(omega, *T)[1]
                g1, g2 = back((z1, 0.25 * _both(z2)))
                g1, g2 = _to_blocks(c, g1, 0.25 * _both(g2) / nk)
                p2 = _to_blocks(c, z1, 0.25 * _both(z2) / nk)[1]
                out.append((*product(x1, x2, w), g1 - w * s["g1"][r], g2 - w * p2))
            else:
                out.append(product(x1, x2, w))
    out = [torch.stack(t) for t in zip(*out)]
    return [_host(t) for t in out] if c["op"] in ("host", "solve") else out
