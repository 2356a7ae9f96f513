"""Schur operator over the tile orders, workgroup sizes and right-hand-side
groupings of the half-lattice hop, against its definition through the
oracle's hopping term: slab order (z extent divisible by 8), contiguous
order, 64- and 256-site workgroups, partly filled and padded tiles, rows of
one and two half-lattice sites, every boundary sign.

Tolerances are those of the two chained hops in the storage type: a few
roundings of FP64 / FP32 per term, and the stored format's rounding (2^-9
BF16, 2^-12 FP16, relative to a site's largest component) times the few such
roundings that reach an output.
"""
import numpy as np
import pytest

from paper_1712_01505_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = {"f64": 1e-12, "f32": 1e-5, "bf16": 2e-2, "f16": 3e-3}


@pytest.fixture(scope="module")
def W():
    from paper_1712_01505_amd import wilson
    assert torch.cuda.is_available()
    wilson.lib()
    return wilson


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


def _odd(dims):
    Lx, Ly, Lz, Lt = dims
    t, z, y, x = np.meshgrid(np.arange(Lt), np.arange(Lz), np.arange(Ly), np.arange(Lx), indexing="ij")
    return ((x + y + z + t) % 2)[..., None, None] == 1


@pytest.mark.parametrize("dims,prec,nrhs,bc", [
    ((8, 4, 8, 16), "f64", 1, (1, 1, 1, -1)),       # slabs, 64-site workgroups
    ((8, 4, 8, 16), "f64", 3, (-1, -1, -1, -1)),
    ((16, 16, 16, 32), "f64", 1, (1, -1, 1, -1)),   # slabs, 256-site workgroups
    ((16, 16, 16, 32), "f32", 2, (1, 1, 1, -1)),    # contiguous, 256
    ((16, 16, 16, 64), "f32", 1, (-1, 1, 1, -1)),   # slabs above 2^17 half sites
    ((16, 16, 16, 64), "bf16", 1, (1, 1, 1, -1)),
    ((16, 16, 16, 64), "f16", 1, (1, 1, -1, -1)),
    ((2, 2, 2, 2), "f32", 5, (-1, 1, -1, 1)),       # part of one wavefront, padded tiles
    ((6, 10, 4, 14), "f16", 3, (1, 1, 1, -1)),      # no power of two
    ((10, 6, 14, 22), "f64", 2, (1, -1, 1, 1)),
    ((4, 2, 16, 6), "f64", 1, (-1, 1, 1, -1)),      # z divisible, the slab is not a multiple of 64
])
def test_schur_orders(W, oracle_mod, dims, prec, nrhs, bc):
    kappa = 0.1255
    U = inputs.near_unity_gauge(dims, 0.3, seed=3)
    psi = inputs.gaussian_spinor(dims, seed=4, nrhs=nrhs)
    odd = _odd(dims)
    x_e = np.where(odd, 0.0, psi)
    op = W.Operator.create(dev(U), kappa, W.PREC[prec], bc)
    ev, zero_o = op.eo_split(op.pack(dev(x_e)), nrhs)
    for dagger in (False, True):
        out_e, tmp_o = op.new_half(nrhs), op.new_half(nrhs)
        op.schur_packed(out_e, ev, tmp_o, nrhs, dagger)
        got = op.unpack(op.eo_merge(out_e, zero_o, nrhs), nrhs).cpu().numpy()
        for k in range(nrhs):
            tmp = np.where(odd, oracle_mod.hop(U, x_e[k], bc=bc, dagger=dagger), 0.0)
            ref = np.where(odd, 0.0, x_e[k] - kappa ** 2 * oracle_mod.hop(U, tmp, bc=bc, dagger=dagger))
            assert np.linalg.norm(got[k] - ref) / np.linalg.norm(ref) < TOL[prec], (dagger, k)


def test_solve_residual_in_one_pass(W, oracle_mod):
    """Reported residuals of even-odd solves, several right-hand sides, against the oracle's."""
    dims, kappa = (8, 4, 8, 16), 0.1255
    U = inputs.near_unity_gauge(dims, 0.3, seed=5)
    b = inputs.gaussian_spinor(dims, seed=6, nrhs=3)
    for precision in ("f64", "mixed-f32"):
        x, st = W.solve(dev(U), dev(b), kappa, method="bicgstab", precision=precision, tol=1e-10, eo=True,
                        return_stats=True)
        for k in range(3):
            r = np.linalg.norm(oracle_mod.apply(U, x[k].cpu().numpy(), kappa) - b[k]) / np.linalg.norm(b[k])
            assert st[k]["converged"] and r <= 1e-10
            assert abs(r - st[k]["true_rel_res"]) < 1e-12
