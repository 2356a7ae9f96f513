"""Launch shapes chosen without a tuner: valid for every geometry (on the
CPU), and the same results as the straight-line kernel on the GPU."""
import ctypes
import random

import numpy as np
import pytest

from paper_1712_01505_amd import inputs, wilson


def _op(dims, prec, ns=0):
    g = wilson.make_geom(dims)
    if ns:
        h = ctypes.c_void_p()
        assert wilson.lib().wl_dw_op_create(ctypes.byref(g), -1.8, 0.05, ns, prec, 16, ctypes.byref(h)) == wilson.WL_OK
        return h.value
    return wilson.wl_op_create(g, 0.12, prec, 16)  # a dummy address: nothing is launched


def test_default_shape_is_valid_everywhere():
    rng = random.Random(1)
    some = [2, 3, 4, 5, 6, 8, 10, 12, 14, 16, 18, 20, 22, 24, 28, 31, 32, 40, 48, 64]
    seen = set()
    for k in range(1500):
        dims = [rng.choice(some) for _ in range(4)] if k % 10 else [32, 32, 32, rng.choice([48, 64])]
        prec, ns = rng.randrange(4), rng.choice([0, 0, 0, 1, 4, 6, 8])
        nrhs = rng.choice([1, 1, 1, 2, 3, 4, 5, 8, 12, 16])
        if max(ns, 1) * nrhs > 64:
            continue
        h = _op(dims, prec, ns)
        c = wilson.wl_launch()
        assert wilson.lib().wl_get_launch(h, nrhs, ctypes.byref(c)) == wilson.WL_OK
        assert wilson.lib().wl_set_launch(h, nrhs, ctypes.byref(c)) == wilson.WL_OK, (dims, prec, ns, nrhs, c.variant)
        if ns and c.variant == wilson.VAR_BRICK:  # the library's own choice: taken back, no other is taken
            o = wilson.wl_launch()
            ctypes.memmove(ctypes.byref(o), ctypes.byref(c), ctypes.sizeof(c))
            c.block, c.variant, c.t_steps, c.xcd_remap, c.rhs_lanes, c.brick[:] = 64, 0, 0, 0, 1, [0, 0, 0]
            assert wilson.lib().wl_set_launch(h, nrhs, ctypes.byref(c)) == wilson.WL_OK
            assert wilson.lib().wl_set_launch(h, nrhs, ctypes.byref(o)) == wilson.WL_OK
            o.xcd_remap = 1 - o.xcd_remap
            assert wilson.lib().wl_set_launch(h, nrhs, ctypes.byref(o)) == wilson.WL_EINVAL
            c.variant = wilson.VAR_BRICK
        seen.add((prec, c.variant, ns > 0, nrhs > 1))
        wilson.lib().wl_op_destroy(h)
    for prec in (wilson.WL_F64, wilson.WL_F32, wilson.WL_F16S):
        assert (prec, wilson.VAR_BRICK, False, False) in seen  # the sample reaches the bricks


@pytest.mark.gpu
@pytest.mark.parametrize("dims,nrhs", [((32, 32, 32, 20), 1), ((24, 12, 16, 12), 12), ((16, 16, 16, 20), 1),
                                       ((20, 20, 12, 8), 3), ((18, 14, 10, 9), 5), ((32, 16, 16, 16), 2),
                                       ((8, 8, 8, 16), 1), ((16, 16, 12, 40), 4), ((32, 32, 32, 25), 1)])
@pytest.mark.parametrize("prec", ["f64", "f32", "bf16", "f16"])
def test_default_matches_straight_line(dims, nrhs, prec):
    """FP64 / FP32: the same bits in every shape.  16 bits: the walks form a site in another
    grouping, so results agree to the storage rounding (2^-8 BF16, 2^-11 FP16 of a site's
    largest component, a few of them)."""
    torch = pytest.importorskip("torch")
    U = torch.from_numpy(inputs.near_unity_gauge((2, 2, 2, 2), 0.3, seed=3)).to("cuda")
    Lx, Ly, Lz, Lt = dims
    rep = [-(-n // 2) for n in (Lt, Lz, Ly, Lx)]
    U = U.repeat(1, *rep, 1, 1)[:, :Lt, :Lz, :Ly, :Lx].contiguous()
    g = torch.Generator(device="cuda").manual_seed(1)
    psi = torch.view_as_complex(torch.randn(nrhs, Lt, Lz, Ly, Lx, 4, 3, 2, dtype=torch.float64, device="cuda",
                                            generator=g))
    op = wilson.Operator.create(U, 0.1255, wilson.PREC[prec])
    src = op.pack(psi)
    outs = []
    for shape in (None, (64, 1, 0, 0, 1)):
        if shape:
            assert wilson.try_set_launch(op.handle, nrhs, *shape)
        for dagger in (False, True):
            out = op.new_field(nrhs)
            op.apply_packed(out, src, nrhs, dagger)
            outs.append(out)
    for got, ref in ((outs[0], outs[2]), (outs[1], outs[3])):
        if prec in ("f64", "f32"):
            assert torch.equal(got, ref)
        else:
            a, b = op.unpack(got, nrhs), op.unpack(ref, nrhs)
            assert float((a - b).norm() / b.norm()) < (2.0 ** -7 if prec == "bf16" else 2.0 ** -10)


@pytest.mark.gpu
@pytest.mark.parametrize("dims,ns,prec", [((32, 32, 32, 4), 4, "f32"), ((32, 32, 32, 2), 4, "f64"),
                                          ((32, 32, 32, 3), 8, "bf16"), ((32, 32, 32, 4), 7, "f16"),
                                          ((64, 16, 32, 6), 4, "f32")])
def test_domain_wall_bricks(dims, ns, prec):
    """The brick walk's fifth-dimension terms: the bits of the straight-line kernel in FP64 and
    FP32, the storage rounding (as above) in 16 bits; D and D^dag, and the fused |D x|^2 of CG."""
    torch = pytest.importorskip("torch")
    Lx, Ly, Lz, Lt = dims
    U = torch.from_numpy(inputs.near_unity_gauge((2, 2, 2, 2), 0.3, seed=3)).to("cuda")
    U = U.repeat(1, -(-Lt // 2), Lz // 2, Ly // 2, Lx // 2, 1, 1)[:, :Lt].contiguous()
    g = torch.Generator(device="cuda").manual_seed(2)
    psi = torch.view_as_complex(torch.randn(ns, Lt, Lz, Ly, Lx, 4, 3, 2, dtype=torch.float64, device="cuda", generator=g))
    op = wilson.DWOperator.create(U, -1.8, 0.05, ns, wilson.PREC[prec])
    assert wilson.wl_get_launch(op.handle, 1)[3] == wilson.VAR_BRICK
    src = op.pack(psi)
    outs = []
    for shape in (None, (64, 1, 0, 0, 1)):
        if shape:
            assert wilson.try_set_launch(op.handle, 1, *shape)
        for dagger in (False, True):
            out = op.new_field()
            op.apply_packed(out, src, 1, dagger)
            outs.append(out)
    for got, ref in ((outs[0], outs[2]), (outs[1], outs[3])):
        if prec in ("f64", "f32"):
            assert torch.equal(got, ref)
        else:
            a, b = op.unpack(got), op.unpack(ref)
            assert float((a - b).norm() / b.norm()) < (2.0 ** -7 if prec == "bf16" else 2.0 ** -10)
    if prec == "f64":  # CG with the fused norms; its solution against the operator itself
        x, st = wilson.dw_solve(U, psi, -1.8, 0.05, precision="f64", tol=1e-9, return_stats=True)
        r = psi - wilson.dw_apply(U, x, -1.8, 0.05, op=op)
        assert st["converged"] and float(r.norm() / psi.norm()) <= 1e-9


@pytest.mark.gpu
@pytest.mark.parametrize("dims,nrhs,prec", [((32, 32, 32, 20), 1, "bf16"), ((20, 20, 12, 8), 3, "f16"),
                                            ((32, 32, 32, 24), 1, "f64")])
def test_untuned_reduction_shape_does_not_depend_on_earlier_calls(dims, nrhs, prec):
    """A fused reduction on an operator that has already been applied: the same bits as on a new
    operator (each launch keeps its own untuned shape)."""
    torch = pytest.importorskip("torch")
    Lx, Ly, Lz, Lt = dims
    U = torch.from_numpy(inputs.near_unity_gauge((2, 2, 2, 2), 0.3, seed=3)).to("cuda")
    U = U.repeat(1, Lt // 2, Lz // 2, Ly // 2, Lx // 2, 1, 1)
    g = torch.Generator(device="cuda").manual_seed(4)
    psi = torch.view_as_complex(torch.randn(nrhs, Lt, Lz, Ly, Lx, 4, 3, 2, dtype=torch.float64, device="cuda",
                                            generator=g))
    got = []
    for first in (False, True):
        op = wilson.Operator.create(U, 0.1255, wilson.PREC[prec])
        src, out = op.pack(psi), op.new_field(nrhs)
        v = op.pack(psi.roll(1, 1))
        if first:
            op.apply_packed(out, src, nrhs)
        for kind in (wilson.WL_DOT_BICG, wilson.WL_DOT_V):
            dots = wilson.apply_dot(op, out, src, v, nrhs=nrhs, kind=kind)
            got.append((first, kind, out.clone(), dots))
    for a, b in zip(got[:2], got[2:]):
        assert torch.equal(a[2], b[2]) and torch.equal(a[3], b[3])
