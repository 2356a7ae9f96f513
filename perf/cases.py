"""The performance cases of the library: what its users have it compute.

Operator applications (Wilson, even-odd Schur, domain wall) on packed fields
and whole solves on canonical torch tensors, from lattices of a few hundred
sites, where launches and latency count, to 32^3 x 64; every storage
precision; one and several right-hand sides; the operator and its adjoint;
forward and backward of the differentiable solve.  Sizes, couplings and
tolerances are those of the benchmark and the tests, or generic.  No case runs the
autotuner: the entry points used here never call it, so a program gets the
launch shapes that the library picks by itself.

Inputs are drawn on the GPU from the seed: links exp(i eps H) with eps = 0.3
(as the benchmark's) and Gaussian spinors.
"""
import torch

from paper_1712_01505_amd import wilson as W
from paper_1712_01505_amd.autograd import wilson_solve

EPS = 0.3
BC = (1, 1, 1, -1)
SITE_BYTES = {"f64": 192, "f32": 96, "bf16": 52, "f16": 52}   # packed spinor
LINK_BYTES = {"f64": 96, "f32": 48, "bf16": 24, "f16": 24}    # packed link
KAPPA = 0.1255
M0, MQ = -1.8, 0.05
TOL = 1e-11      # one digit under the benchmark's 1e-10, so that two solutions agree to 1e-9


def _case(name, kind, dims, prec, **more):
    c = {"name": name, "kind": kind, "lx": dims[0], "ly": dims[1], "lz": dims[2], "lt": dims[3], "prec": prec,
         "nrhs": 1, "dagger": False}
    c.update(more)
    return c


def listed():
    return [
        # the smallest call: one application on a few hundred sites, as in a unit test, a small
        # block of a preconditioner or a toy lattice; all launch and latency
        _case("apply_f64_4x4x4x8", "apply", (4, 4, 4, 8), "f64"),
        # the operator in double precision on the benchmark's lattice: the true residual of
        # every solve and what eigensolvers and measurements apply
        _case("apply_f64_32x32x32x64", "apply", (32, 32, 32, 64), "f64"),
        # the adjoint with 16-bit storage: one half of a normal-equations step in an inner solver
        _case("apply_bf16_dag_32x32x32x64", "apply", (32, 32, 32, 64), "bf16", dagger=True),
        # extents that no tile divides, an odd number of right-hand sides
        _case("apply_f16_3rhs_22x18x14x27", "apply", (22, 18, 14, 27), "f16", nrhs=3),
        # the twelve spin-colour columns of a propagator at once
        _case("apply_f32_12rhs_24x24x24x48", "apply", (24, 24, 24, 48), "f32", nrhs=12),
        # the even-odd Schur operator, what preconditioned solvers apply
        _case("schur_f32_32x32x32x64", "schur", (32, 32, 32, 64), "f32"),
        # the domain-wall operator with Table I's eight slices; the largest field
        _case("dw_f32_32x32x32x64_ns8", "dw", (32, 32, 32, 64), "f32", ns=8),
        # CG on the domain-wall normal equations on the paper's smaller lattice
        _case("dw_solve_f32_16x16x16x32_ns8", "dw_solve", (16, 16, 16, 32), "f32", ns=8),
        # a small solve from canonical tensors: a few thousand sites, launches and reductions count
        _case("solve_f64_8x8x8x16", "solve", (8, 8, 8, 16), "f64", eo=False),
        # the benchmark's step: FP16 inner BiCGStab inside FP64 refinement
        _case("solve_f16_32x32x32x64", "solve", (32, 32, 32, 64), "f16", eo=False),
        # the fastest solver offered: even-odd, FP16 inner with reliable updates
        _case("solve_eo_f16_32x32x32x64", "solve", (32, 32, 32, 64), "f16", eo=True),
        # forward and backward of the differentiable solve: two solves and the link force
        _case("grad_f32_16x16x16x32", "grad", (16, 16, 16, 32), "f32"),
    ]


def _dims(c):
    return c["lx"], c["ly"], c["lz"], c["lt"]


def _vol(c):
    return c["lx"] * c["ly"] * c["lz"] * c["lt"]


def _log_int(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    """Extents of 4 to 32 (64 in t), log-uniform; odd ones except where the even-odd
    split needs even extents; solves up to 32^3 x 64 as listed, mixed ones on at least a few
    thousand sites."""
    most = max(w["bytes"] for w in map(work, listed()))
    while True:
        kind = rng.choice(["apply", "apply", "apply", "schur", "dw", "solve", "solve", "dw_solve", "grad"])
        top = {"dw_solve": 16, "grad": 16}.get(kind, 32)
        dims = [_log_int(rng, 4, top) for _ in range(3)] + [_log_int(rng, 4, 2 * top)]
        prec = rng.choice(["f64", "f32", "bf16", "f16"])
        more = {}
        if kind == "apply":
            more = {"nrhs": rng.choice([1, 1, 1, 2, 3, 4, 5, 8, 12]), "dagger": rng.random() < 0.5}
        elif kind == "schur":
            more = {"nrhs": rng.choice([1, 1, 2, 3, 12]), "dagger": rng.random() < 0.5}
        elif kind == "dw":
            more = {"ns": rng.choice([4, 6, 8, 12]), "dagger": rng.random() < 0.5}
        elif kind == "dw_solve":
            prec, more = rng.choice(["f64", "f32"]), {"ns": rng.choice([4, 6, 8])}
        elif kind == "solve":
            more = {"eo": rng.random() < 0.5, "nrhs": rng.choice([1, 1, 1, 3])}
        else:
            prec = rng.choice(["f64", "f32"])
        if kind == "schur" or more.get("eo"):
            dims = [d + d % 2 for d in dims]
        c = _case("", kind, dims, prec, **more)
        del c["name"]
        if kind in ("solve", "dw_solve", "grad") and prec != "f64" and _vol(c) < 2048:
            continue
        if work(c)["bytes"] <= most:
            return c


# ---------------------------------------------------------------- inputs
def _rand(gen, *shape):
    return torch.randn(*shape, 2, dtype=torch.float64, device="cuda", generator=gen)


def _spinor(gen, c, *lead):
    x, y, z, t = _dims(c)
    return torch.view_as_complex(_rand(gen, *lead, t, z, y, x, 4, 3))


def _gauge(gen, c):
    """exp(i eps H) with H = sum_a h_a lambda_a / 2, h_a ~ N(0, 1); rows made orthonormal and the
    third the conjugate cross product of the first two, so that each link is in SU(3) to rounding."""
    x, y, z, t = _dims(c)
    out = torch.empty(4, t, z, y, x, 3, 3, dtype=torch.complex128, device="cuda")
    n = t * z * y * x
    for mu in range(4):
        h = torch.randn(8, n, dtype=torch.float64, device="cuda", generator=gen) * (0.5 * EPS)
        d8 = h[7] / 3.0 ** 0.5
        o01, o02, o12 = (torch.complex(h[i], -h[i + 1]) for i in (0, 3, 5))
        A = torch.stack([torch.complex(h[2] + d8, 0 * d8), o01, o02, o01.conj(), torch.complex(d8 - h[2], 0 * d8),
                         o12, o02.conj(), o12.conj(), torch.complex(-2 * d8, 0 * d8)], 0).reshape(3, 3, n) * 1j
        U = torch.zeros_like(A)
        for i in range(3):
            U[i, i] = 1.0
        for k in range(12, 0, -1):  # Horner: U = 1 + (A / k) U
            B = A / k
            U = torch.stack([torch.stack([B[i, 0] * U[0, j] + B[i, 1] * U[1, j] + B[i, 2] * U[2, j]
                                          for j in range(3)], 0) for i in range(3)], 0)
            for i in range(3):
                U[i, i] += 1.0
        r0 = U[0] / U[0].abs().square().sum(0).sqrt()
        r1 = U[1] - (r0.conj() * U[1]).sum(0) * r0
        r1 = r1 / r1.abs().square().sum(0).sqrt()
        r2 = torch.stack([r0[1] * r1[2] - r0[2] * r1[1], r0[2] * r1[0] - r0[0] * r1[2],
                          r0[0] * r1[1] - r0[1] * r1[0]], 0).conj()
        out[mu] = torch.stack([r0, r1, r2], 0).permute(2, 0, 1).reshape(t, z, y, x, 3, 3)
    return out


def _inputs(c, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    U = _gauge(gen, c)
    kind = c["kind"]
    if kind in ("dw", "dw_solve"):
        return U, _spinor(gen, c, c["ns"])
    if kind == "grad":
        return U, _spinor(gen, c), _spinor(gen, c)
    return U, _spinor(gen, c, *([c["nrhs"]] if c["nrhs"] > 1 or kind in ("apply", "schur") else []))


def prepare(case, seed):
    c, kind, p = case, case["kind"], W.PREC[case["prec"]]
    if kind == "grad":
        U, b, g = _inputs(c, seed)
        return {"case": c, "U": U.requires_grad_(), "b": b.requires_grad_(), "g": g}
    U, psi = _inputs(c, seed)
    if kind == "apply":
        op = W.Operator.create(U, KAPPA, p, BC)
        return {"case": c, "op": op, "in": op.pack(psi), "out": op.new_field(c["nrhs"])}
    if kind == "schur":
        op = W.Operator.create(U, KAPPA, p, BC)
        even, odd = op.eo_split(op.pack(psi), c["nrhs"])
        return {"case": c, "op": op, "in": even, "tmp": odd, "out": op.new_half(c["nrhs"])}
    if kind == "dw":
        op = W.DWOperator.create(U, M0, MQ, c["ns"], p, BC)
        return {"case": c, "op": op, "in": op.pack(psi), "out": op.new_field()}
    if kind == "dw_solve":
        hi = W.DWOperator.create(U, M0, MQ, c["ns"], W.WL_F64, BC)
        lo = None if c["prec"] == "f64" else W.DWOperator.create(U, M0, MQ, c["ns"], p, BC)
        return {"case": c, "ops": (hi, lo), "b": psi}
    hi = W.Operator.create(U, KAPPA, W.WL_F64, BC)
    lo = None if c["prec"] == "f64" else W.Operator.create(U, KAPPA, p, BC)
    return {"case": c, "ops": (hi, lo), "b": psi}


def _numbers(packed, c, cols, sites):
    """A packed field as the numbers it holds: FP64 or FP32 reals, or 16-bit reals and the
    FP32 scale of each site."""
    prec = c["prec"]
    if prec == "f64":
        return packed.view(torch.float64)
    if prec == "f32":
        return packed.view(torch.float32)
    n = cols * sites * 48
    return packed[:n].view(torch.bfloat16 if prec == "bf16" else torch.float16), packed[n:].view(torch.float32)


def run(state):
    c = state["case"]
    kind, mixed = c["kind"], c["prec"] if c["prec"] == "f64" else "mixed-" + c["prec"]
    if kind == "apply":
        state["op"].apply_packed(state["out"], state["in"], c["nrhs"], c["dagger"])
        return _numbers(state["out"], c, c["nrhs"], _vol(c))
    if kind == "schur":
        state["op"].schur_packed(state["out"], state["in"], state["tmp"], c["nrhs"], c["dagger"])
        return _numbers(state["out"], c, c["nrhs"], _vol(c) // 2)
    if kind == "dw":
        state["op"].apply_packed(state["out"], state["in"], 1, c["dagger"])
        return _numbers(state["out"], c, c["ns"], _vol(c))
    if kind == "dw_solve":
        return W.dw_solve(None, state["b"], M0, MQ, precision=mixed, tol=TOL, ops=state["ops"],
                          reliable=c["prec"] == "f32")
    if kind == "solve":
        return W.solve(None, state["b"], KAPPA, method="bicgstab", precision=mixed, tol=TOL, ops=state["ops"],
                       eo=c["eo"], reliable=c["eo"] and c["prec"] != "f64")
    x = wilson_solve(state["U"], state["b"], KAPPA, precision=mixed, tol=TOL, bc=BC)
    grad_U, grad_b = torch.autograd.grad(x, (state["U"], state["b"]), state["g"])
    return x.detach(), grad_U, grad_b


# ---------------------------------------------------------------- the work of one pass
def work(case):
    """Bytes: for an application, each spinor and link read and written once (the Schur operator's
    two half-lattice hops each read all links); for a solve, those bytes for every application of
    the operator in the inner precision plus the vectors of one update each, at a nominal number of
    iterations.  Flops: Table I's 1368 per site and application (domain wall: 1440 per 5-d site)."""
    c, kind, v = case, case["kind"], _vol(case)
    s, l = SITE_BYTES[c["prec"]], 4 * LINK_BYTES[c["prec"]]
    n = c["nrhs"]
    if kind == "apply":
        return {"bytes": v * (2 * s * n + l), "flops": 1368.0 * v * n}
    if kind == "schur":  # in -> odd, odd and in -> out
        return {"bytes": v * (2.5 * s * n + 2 * l), "flops": 1368.0 * v * n}
    if kind == "dw":
        return {"bytes": v * (2 * s * c["ns"] + l), "flops": 1440.0 * v * c["ns"]}
    if kind == "dw_solve":  # CG on the normal equations: two products, x r p updates
        return {"bytes": 500.0 * v * (13 * s * c["ns"] + 2 * l), "flops": 500 * 2 * 1440.0 * v * c["ns"]}
    iters, half = (55, 0.5) if c.get("eo") else (110, 1.0)
    solves = 2 if kind == "grad" else 1
    links = 2 * l / half  # both products; a Schur product reads the links twice
    return {"bytes": solves * iters * v * ((15 * s * n) * half + links), "flops": solves * iters * 2 * 1368.0 * v * n}


# ---------------------------------------------------------------- the same in plain torch, 64 bits
# gamma_mu psi = phase * psi[perm] over the four spins (chiral basis, gamma_5 = diag(1, 1, -1, -1))
_PERM = ((3, 2, 1, 0), (3, 2, 1, 0), (2, 3, 0, 1), (2, 3, 0, 1))
_PHASE = ((1j, 1j, -1j, -1j), (-1, 1, 1, -1), (1j, -1j, -1j, 1j), (1, 1, 1, 1))


def _gamma(mu, psi):
    ph = torch.tensor(_PHASE[mu], dtype=psi.dtype, device=psi.device)[:, None]
    return ph * psi[..., list(_PERM[mu]), :]


def _shift(f, mu, step, axis):
    """f(x + step mu) with the boundary sign of the hop; `axis`: where mu's axis is in f."""
    f = torch.roll(f, -step, axis)
    if BC[mu] < 0:
        f.narrow(axis, f.shape[axis] - 1 if step > 0 else 0, 1).neg_()
    return f


def _mv(u, h, adj):
    if adj:
        return sum(u[..., None, b, :].conj() * h[..., :, b, None] for b in range(3))
    return sum(u[..., None, :, b] * h[..., :, b, None] for b in range(3))


def _hop(U, psi, dagger):
    s = -1 if dagger else 1
    out = torch.zeros_like(psi)
    for mu in range(4):
        axis = -3 - mu
        f = _shift(psi, mu, 1, axis)
        out += _mv(U[mu], f - s * _gamma(mu, f), False)
        b = _mv(U[mu], psi + s * _gamma(mu, psi), True)
        out += _shift(b, mu, -1, axis)
    return out


def _apply(U, psi, dagger=False):
    return psi - KAPPA * _hop(U, psi, dagger)


def _dw(U, psi, dagger=False):
    """psi (Ns, ...)"""
    out = (M0 + 5.0) * psi - 0.5 * _hop(U, psi, dagger)
    up, dn = torch.roll(psi, -1, 0), torch.roll(psi, 1, 0)
    up[-1] *= -MQ
    dn[0] *= -MQ
    lo, hi = (slice(0, 2), slice(2, 4)) if dagger else (slice(2, 4), slice(0, 2))
    out[..., lo, :] -= up[..., lo, :]
    out[..., hi, :] -= dn[..., hi, :]
    return out


def _parity(c):
    x, y, z, t = (torch.arange(n, device="cuda") for n in _dims(c))
    return (t[:, None, None, None] + z[:, None, None] + y[:, None] + x) & 1


def _cg(mul, mul_dag, b, iters):
    """Normal equations, to 1e-13 of b's norm (checked on the true residual)."""
    x, r, bn = torch.zeros_like(b), b.clone(), float(b.norm())
    for _ in range(4):
        z = mul_dag(r)
        p, zz = z.clone(), float(z.norm()) ** 2
        for _ in range(iters):
            w = mul(p)
            a = zz / float(w.norm()) ** 2
            x += a * p
            r -= a * w
            if float(r.norm()) < 5e-14 * bn:
                break
            z = mul_dag(r)
            zz, old = float(z.norm()) ** 2, zz
            p = z + (zz / old) * p
        r = b - mul(x)
        if float(r.norm()) < 2e-13 * bn:
            break
    return x


def _solve(U, b, dagger=False):
    """BiCGStab, restarted from the true residual until it is under 1e-13."""
    x, bn = torch.zeros_like(b), float(b.norm())
    for _ in range(12):
        r = b - _apply(U, x, dagger)
        if float(r.norm()) < 2e-13 * bn:
            break
        rh, p, rn = r.clone(), r.clone(), float(r.norm())
        rho = torch.vdot(rh.reshape(-1), r.reshape(-1)).item()
        for _ in range(400):
            v = _apply(U, p, dagger)
            al = rho / torch.vdot(rh.reshape(-1), v.reshape(-1)).item()
            r -= al * v
            t = _apply(U, r, dagger)
            om = torch.vdot(t.reshape(-1), r.reshape(-1)).item() / float(t.norm()) ** 2
            x += al * p + om * r
            r -= om * t
            if float(r.norm()) < 1e-3 * rn and float(r.norm()) < 1e-13 * bn:
                break
            rho, old = torch.vdot(rh.reshape(-1), r.reshape(-1)).item(), rho
            p = r + (rho / old) * (al / om) * (p - om * v)
    return x


def _packed(psi, c):
    """The numbers of the packed layout: [column][chunk][site][complex of the chunk] (and scales)."""
    per = {"f64": 1, "f32": 2}.get(c["prec"], 4)
    f = torch.view_as_real(psi.resolve_conj().contiguous()).reshape(psi.shape[0], -1, 12 // per, per, 2)  # col, site
    if c["prec"] in ("f64", "f32"):
        return f.transpose(1, 2).reshape(-1)
    sc = f.abs().amax((2, 3, 4))
    return (f / sc[:, :, None, None, None]).transpose(1, 2).reshape(-1), sc.reshape(-1)


def _gradient(U, x, mu_):
    """i P U with P the traceless Hermitian part of i U G, dL = Re sum Tr[dU G]."""
    out = torch.empty_like(U)
    for mu in range(4):
        axis = -3 - mu
        xf, mf = _shift(x, mu, 1, axis), _shift(mu_, mu, 1, axis)
        v, w = xf - _gamma(mu, xf), x + _gamma(mu, x)
        G = sum(v[..., s, :, None] * mu_[..., s, None, :].conj() + mf[..., s, :, None] * w[..., s, None, :].conj()
                for s in range(4)) * KAPPA
        A = 1j * sum(U[mu][..., :, k, None] * G[..., k, None, :] for k in range(3))
        P = 0.5 * (A + A.mH)
        P -= torch.diag_embed((P.diagonal(dim1=-2, dim2=-1).sum(-1) / 3.0)[..., None].expand(*P.shape[:-1]))
        out[mu] = 1j * sum(P[..., :, k, None] * U[mu][..., k, None, :] for k in range(3))
    return out


def exact(case, seed):
    c, kind = case, case["kind"]
    if kind == "grad":
        U, b, g = _inputs(c, seed)
        x, m = _solve(U, b), _solve(U, g, True)
        return x, _gradient(U, x, m), m
    U, psi = _inputs(c, seed)
    if kind == "apply":
        return _packed(torch.stack([_apply(U, p, c["dagger"]) for p in psi]), c)
    if kind == "schur":
        even = _parity(c) == 0
        keep = even[..., None, None]
        out = torch.stack([torch.where(keep, p - KAPPA ** 2 * _hop(U, _hop(U, torch.where(keep, p, 0.0), c["dagger"]),
                                                                   c["dagger"]), 0.0) for p in psi])
        return _packed(out.reshape(len(psi), -1, 12)[:, even.reshape(-1)], c)
    if kind == "dw":
        return _packed(_dw(U, psi, c["dagger"]), c)
    if kind == "dw_solve":
        return _cg(lambda p: _dw(U, p), lambda p: _dw(U, p, True), psi, 1500)
    if c["nrhs"] > 1:
        return torch.stack([_solve(U, b) for b in psi])
    return _solve(U, psi)
