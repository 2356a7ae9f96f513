"""Fused inner products over many launch shapes: the wavefront and workgroup
sums of the stencil kernels and the finalize that adds their partials, at the
edges of its slices (rows of 1, 511, 512, 513 and more than 8192 partials),
for every grouping of right-hand sides, against FP64 sums of the stored
fields.

Tolerance: both sides sum n FP64 products of values of order one, in
different orders.  Such sums differ by at most about log2(n) rounding steps
of the sum of magnitudes for the tree of partial sums and by sqrt(n) of them
for torch's; 2^-52 * 1e3 of the norms' product covers n up to 1e6 lattice
components per chunk.
"""
import numpy as np
import pytest

from paper_1712_01505_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# V / 64 = 1 (a part of a wavefront), 511, 512, 513, 8256
DIMS = [(2, 2, 2, 4), (8, 8, 7, 73), (16, 16, 16, 8), (8, 8, 9, 57), (16, 16, 16, 129)]
TOL = 1e3 * 2.0 ** -52


@pytest.fixture(scope="module")
def W():
    from paper_1712_01505_amd import wilson
    assert torch.cuda.is_available()
    wilson.lib()
    return wilson


def _spinor(dims, n, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    x, y, z, t = dims
    return torch.view_as_complex(torch.randn(n, t, z, y, x, 4, 3, 2, dtype=torch.float64, device="cuda", generator=g))


def _check(W, dims, prec, nrhs, shape):
    U = torch.from_numpy(inputs.unit_gauge(dims)).to("cuda")
    op = W.Operator.create(U, 0.11, W.PREC[prec])
    if not W.try_set_launch(op.handle, nrhs, *shape):
        pytest.skip("launch shape not offered here")
    psi, phi = _spinor(dims, nrhs, 1), _spinor(dims, nrhs, 2)
    a, v = op.pack(psi), op.pack(phi)
    out = op.new_field(nrhs)
    A, V = op.unpack(a, nrhs).reshape(nrhs, -1), op.unpack(v, nrhs).reshape(nrhs, -1)

    def dot(x, y):
        return (x.conj() * y).sum(-1)

    for kind in (W.WL_DOT_BICG, W.WL_DOT_V, W.WL_DOT_NORM):
        d = W.apply_dot(op, out, a, v, nrhs=nrhs, kind=kind)
        O = op.unpack(out, nrhs).reshape(nrhs, -1)
        io, vi, vo = dot(A, O), dot(V, A), dot(V, O)
        oo, ii, vv = dot(O, O).real, dot(A, A).real, dot(V, V).real
        if kind == W.WL_DOT_BICG:
            ref = torch.stack([io.real, io.imag, oo, vi.real, vi.imag, vo.real, vo.imag, ii])
            mag = torch.stack([ii * oo, ii * oo, oo * oo, vv * ii, vv * ii, vv * oo, vv * oo, ii * ii]).sqrt()
        elif kind == W.WL_DOT_V:
            ref, mag = torch.stack([vo.real, vo.imag]), torch.stack([vv * oo, vv * oo]).sqrt()
        else:
            ref, mag = oo[None], oo[None]
        assert float(((d - ref).abs() / mag).max()) <= TOL, (kind, d, ref)


@pytest.mark.parametrize("dims", DIMS)
@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_partial_counts(W, dims, prec):
    _check(W, dims, prec, 1, (64, 1, 0, 1))


# (block, rhs per thread, tile order, variant, rhs across lanes)
@pytest.mark.parametrize("nrhs,shape", [
    (8, (512, 1, 0, 1, 8)), (8, (256, 1, 0, 2, 4)), (8, (128, 1, 1, 2, 2)), (8, (64, 1, 0, 0, 1)),
    (4, (256, 4, 0, 0, 1)), (6, (128, 2, 1, 0, 1)), (3, (128, 1, 0, 1, 1)),
    (8, (256, 1, 0, 4, 8)), (2, (64, 1, 0, 5, 2)), (1, (512, 1, 0, 1, 1)),
    (4, (256, 1, 0, 7, 4, (8, 8, 1), 4)), (2, (256, 1, 0, 7, 2, (8, 8, 2), 8)), (1, (128, 1, 0, 7, 1, (8, 4, 4), 4)),
])
def test_right_hand_side_groupings(W, nrhs, shape):
    _check(W, (8, 8, 8, 8), "f32", nrhs, shape)
