"""One-column solves on small lattices, where each update does the scalar step
in front of it (up to 64 workgroups of 256 sites), against the same system as
the first of two columns, which goes through the finalize launches."""
import pytest

from paper_1712_01505_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
KAPPA = 0.12


@pytest.fixture(scope="module")
def W():
    from paper_1712_01505_amd import wilson
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    wilson.lib()
    return wilson


def _system(dims, seed):
    U = torch.from_numpy(inputs.near_unity_gauge(dims, 0.3, seed=seed)).cuda()
    return U, torch.from_numpy(inputs.gaussian_spinor(dims, seed=seed + 1, nrhs=2)).cuda()


# sites: two workgroups with a remainder, one full one, 64 full workgroups (the last size that
# does its own scalar steps), 65
FULL = [((5, 3, 7, 3), True), ((8, 8, 2, 2), True), ((16, 16, 16, 4), True), ((16, 16, 13, 5), False)]
HALF = [((2, 2, 2, 2), True), ((16, 16, 16, 8), True), ((16, 16, 12, 12), False)]


@pytest.mark.parametrize("method", ["bicgstab", "cgnr"])
@pytest.mark.parametrize("dims,small,eo", [(d, s, False) for d, s in FULL] + [(d, s, True) for d, s in HALF])
def test_iterates_match_the_finalize_path(W, dims, small, eo, method):
    """The iterate after a few steps: FP64 scalars and sums in either path, so it differs by
    their rounding only (7 steps, each amplifying 2^-53 by the condition number, below 10^3 for
    D^dag D at this mass); in FP32 by the rounding of the vectors, 2^-24 in place of 2^-53."""
    U, b = _system(dims, 31)
    for prec, eps in (("f64", 2.0 ** -53), ("f32", 2.0 ** -24)):
        fins = []
        for steps in (1, 2, 7):
            kw = dict(precision=prec, method=method, tol=1e-14, maxiter=steps, eo=eo, return_stats=True)
            x1, s1 = W.solve(U, b[0], KAPPA, **kw)
            x2, s2 = W.solve(U, b, KAPPA, **kw)
            assert s1["iters"] == s2[0]["iters"] == steps
            fins.append((s1["finalizes"], s2[0]["finalizes"]))
            assert float((x1 - x2[0]).norm()) <= 7e3 * eps * float(x2[0].norm())
        # launches inside the loop: those of 7 steps less those of 1
        grown = [b - a for a, b in zip(fins[0], fins[2])]
        per_step = 3 if method == "bicgstab" else 2
        assert grown == [0 if small else 6 * per_step, 6 * per_step]


@pytest.mark.parametrize("method", ["bicgstab", "cgnr"])
@pytest.mark.parametrize("precision", ["f64", "mixed-f32", "mixed-bf16", "mixed-f16"])
@pytest.mark.parametrize("dims,eo", [((8, 8, 4, 4), False), ((16, 16, 16, 4), False), ((16, 16, 16, 8), True)])
def test_solves_match_the_finalize_path(W, dims, eo, precision, method):
    """Both reach 1e-10; ||D^{-1}|| <= 1 / (1 - 8 kappa) = 25 and ||b|| <= 2 ||x||, so the two
    solutions differ by at most 2 x 1e-10 x 25 x 2 = 1e-8 of x."""
    U, b = _system(dims, 57)
    kw = dict(precision=precision, method=method, tol=1e-10, eo=eo, return_stats=True)
    x1, s1 = W.solve(U, b[0], KAPPA, **kw)
    x2, s2 = W.solve(U, b, KAPPA, **kw)
    assert s1["converged"] and s2[0]["converged"] and s2[1]["converged"]
    if precision == "f64":
        assert abs(s1["iters"] - s2[0]["iters"]) <= 1
    assert float((x1 - x2[0]).norm()) <= 1e-8 * float(x2[0].norm())


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("dims", [(8, 8, 4, 4), (16, 16, 16, 8)])
def test_cgnr_columns_that_stop_apart(W, dims, precision):
    """A column that starts near its solution stops early and keeps the last alpha p: its x is
    that of the column alone.  Bound as above for the tolerance that either reaches."""
    U, b = _system(dims, 83)
    tol = 1e-9 if precision == "f64" else 1e-5
    near = W.solve(U, b[0], KAPPA, method="cgnr", tol=100 * tol)
    x0 = torch.stack([near, torch.zeros_like(near)])
    kw = dict(precision=precision, method="cgnr", tol=tol, return_stats=True)
    x, s = W.solve(U, b, KAPPA, x0=x0, **kw)
    assert s[0]["iters"] < s[1]["iters"] and s[0]["converged"] and s[1]["converged"]
    for r in range(2):
        xr, sr = W.solve(U, b[r], KAPPA, x0=x0[r], **kw)
        assert sr["converged"] and abs(sr["iters"] - s[r]["iters"]) <= 1
        assert float((x[r] - xr).norm()) <= 100 * tol * float(xr.norm())


def test_runs_on_the_current_stream(W):
    """The default stream and a side stream: the handle passed is torch's, and a solve gives the
    same bits on either."""
    U, b = _system((8, 8, 4, 4), 5)
    ref = W.solve(U, b[0], KAPPA, precision="f64", tol=1e-10)
    side = torch.cuda.Stream()
    for stream in (torch.cuda.default_stream(), side):
        stream.wait_stream(torch.cuda.default_stream())
        with torch.cuda.stream(stream):
            assert W._stream() == torch.cuda.current_stream().cuda_stream == stream.cuda_stream
            x = W.solve(U, b[0], KAPPA, precision="f64", tol=1e-10)
        stream.synchronize()
        assert torch.equal(x, ref)
    assert side.cuda_stream != torch.cuda.default_stream().cuda_stream
