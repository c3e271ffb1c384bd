"""Edges of the kernels' size ranges and of the rules that choose between them: scalings of the matrix
exponential around its first squarings, tridiagonalisation of matrices with nothing to reflect, the
switches of the D = 8 launch shape, the bound without its reverse sweep."""
import numpy as np
import pytest

import lrh_workloads as W
from oracle import lrh_oracle as O
from test_gpu_parity import (EXPM_PROBLEMS, lrhmod, max_pair_err, need_gpu, oracle_marginals, say,  # noqa: F401
                             sites_per_instance)

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("wg32", [False, True])
@pytest.mark.parametrize("name", ["randchain_Y5_complex", "k5_complete_real", "heis_Y7_real", "gue_Y8_complex"])
def test_gibbs_around_the_first_squarings(name, wg32):
    """beta from no squaring at all through one, two and a few, every dimension 16 to 256.  Entry
    tolerance as for larger beta: 1e-10 below beta = 10 and 2e-9 above; float messages 5e-5."""
    lrh = lrhmod()
    make, dims = EXPM_PROBLEMS[name]
    if wg32 and 32 not in dims:
        pytest.skip("no 32-dimensional clusters")
    d = make()
    P = lrh.Problem(d, 0)
    R = O.Relaxation(d)
    if wg32:
        P.force_shape(32, 4)
    nu_o = R.draw(71, 0.5)
    nu = P.from_dense(R.to_pairs(nu_o))
    nu32 = P.from_dense(R.to_pairs(nu_o), f32=True)
    nu_r = R.from_pairs(P.to_dense(nu32))
    n = sites_per_instance(d)
    for beta in (1e-9, 0.02, 0.1, 0.25, 0.55, 1.3, 40.0):
        say(f"[expm scale] {name} beta={beta} wg32={wg32}")
        q, g, m = P.dual_eval(nu, beta, grad=True, marg=True)
        q32, g32, _ = P.dual_eval(nu32, beta, grad=True)
        torch.cuda.synchronize()
        tol = 1e-10 if beta < 10 else 2e-9
        q_o, g_o = R.grad_beta(nu_o, beta)
        _, rho = R.gibbs(nu_o, beta)
        # F = mu - log Z / beta: at small beta a rounding of log Z ~ log D counts 1 / beta
        assert np.all(np.abs(q.cpu().numpy() - q_o) <= (1e-9 + 1e-13 / beta) * n)
        assert max_pair_err(P.to_dense(g), R.to_pairs(g_o)) < tol
        assert max_pair_err(P.marg_dense(m), oracle_marginals(R, rho)) < tol
        _, g_o = R.grad_beta(nu_r, beta)
        assert max_pair_err(P.to_dense(g32), R.to_pairs(g_o)) < 5e-5
    assert P.check() == (0, 0)


@pytest.mark.parametrize("k", [6, 7])
@pytest.mark.parametrize("kind", ["zero", "identity", "diagonal", "one_row", "random"])
@pytest.mark.parametrize("cplx", [False, True])
def test_certify_matrices_with_nothing_to_reflect(k, kind, cplx):
    """One cluster of 64 or 128 dimensions: lambda_min within the margin, 8 D eps ||theta||_F, of the
    eigenvalues by LAPACK (whose own error is far below it)."""
    lrh = lrhmod()
    say(f"[tridiag] 2^{k} {kind} cplx={cplx}")
    D = 2 ** k
    rng = np.random.default_rng(5 + k)
    z = rng.normal(size=(D, D)) + (1j * rng.normal(size=(D, D)) if cplx else 0.0)
    h = np.diag(np.diag(z + z.conj().T)).astype(z.dtype)
    if kind == "zero":
        h = 0 * h
    elif kind == "identity":
        h = -1.25 * np.eye(D, dtype=z.dtype)
    elif kind == "one_row":   # a column whose only element below the diagonal is the last
        h[D - 1, 0] = z[D - 1, 0]
        h[0, D - 1] = np.conj(z[D - 1, 0])
    elif kind == "random":
        h = z + z.conj().T
    b = W._Builder("dense", k)
    b.add_term(tuple(range(k)), h)
    d = b.build(real=not cplx)
    P = lrh.Problem(d, 0)
    q, mg, _ = P.certify(P.zeros())
    torch.cuda.synchronize()
    want = np.linalg.eigvalsh(h)[0]
    margin = 8 * D * np.finfo(np.float64).eps * np.linalg.norm(h)
    assert abs(q.item() - want) <= margin + np.finfo(np.float64).tiny   # the bracket of a zero matrix
    assert mg.item() >= margin * (1 - 1e-9)


@pytest.mark.parametrize("n", [1, 5, 2048, 2049, 32769])
@pytest.mark.parametrize("beta", [0.0, 2.0])
def test_eight_dimensional_shape_switches(n, beta):
    """A real chain with n three-site clusters in the default shape against one lane per cluster: both FP64
    Jacobi, so to rounding (the dual value per site, the oracle's entry tolerance)."""
    lrh = lrhmod()
    say(f"[D=8 default] n={n} beta={beta}")
    d = W.with_tops(W.heisenberg_chain(n + 2, field_x=0.4), [tuple(range(i, i + 3)) for i in range(n)])
    P = lrh.Problem(d, 0)
    g0 = torch.Generator(device="cpu").manual_seed(3)
    nu = P.zeros()
    nu.copy_(0.3 * torch.randn(nu.shape, generator=g0, dtype=torch.float64))
    q, g, m = P.dual_eval(nu, beta, grad=True, marg=True)
    P.force_shape(8, 1)
    q1, g1, m1 = P.dual_eval(nu, beta, grad=True, marg=True)
    torch.cuda.synchronize()
    assert (q - q1).abs().max().item() <= 1e-12 * d.n_sites
    assert g.numel() == 0 or (g - g1).abs().max().item() < 1e-10
    assert (m - m1).abs().max().item() < 1e-10


@pytest.mark.parametrize("T", [0, 1, 7])
def test_bound_without_gradient_is_the_bound(T):
    lrh = lrhmod()
    say(f"[unrolled value] T={T}")
    d = W.xxz_triangular(4, 0.5, seed=5)
    P = lrh.Problem(d, 0)
    b, _, _ = P.unrolled_bound_grad(4.0, T)
    v = lrh.unrolled_bound(torch.tensor(d.params, dtype=torch.float64, device="cuda"), P, 4.0, T)
    torch.cuda.synchronize()
    assert (v - b).abs().max().item() <= 1e-12 * d.n_sites


@pytest.mark.parametrize("L", [5, 64, 96])
@pytest.mark.parametrize("beta", [0.0, 3.0])
def test_adjoint_of_the_value_is_the_gradient(L, beta):
    """Dimensions 8, 4 and 2 in one launch (L = 5, 64) and one by one (96): the adjoint of Q alone is
    the gradient of the evaluation, two FP64 eigensolvers apart (the oracle's entry tolerance)."""
    lrh = lrhmod()
    say(f"[vjp group] L={L} beta={beta}")
    P = lrh.Problem(W.xxz_triangular(L, 0.5, seed=5), 0)
    nu = P.zeros()
    nu.copy_(0.3 * torch.randn(nu.shape, generator=torch.Generator().manual_seed(8), dtype=torch.float64))
    _, g, _ = P.dual_eval(nu, beta, grad=True)
    nb, _ = P.dual_vjp(nu, beta, qbar=P.qbuf(1.0))
    torch.cuda.synchronize()
    # (cotangents of the Frobenius inner product, as the gradient is)
    assert (nb - g).abs().max().item() < 1e-10


@pytest.mark.parametrize("beta", [0.0, 3.0])
def test_complex_sixteen_dimensional_adjoint_switch(beta):
    """1024 complex 16 x 16 windows (a wave each) and 1025 (16 lanes each) of one chain: the same messages away from
    the end, so the same cotangents there, two FP64 eigensolvers apart (the entry tolerance)."""
    lrh = lrhmod()
    say(f"[vjp D=16 switch] beta={beta}")
    rng = np.random.default_rng(12)
    draws = {}
    out = []
    for n in (1025, 1024):
        P = lrh.Problem(W.random_chain(n + 3, seed=6, top_len=4, two_level=True), 0)
        assert sum(s["n"] for s in P.shapes() if s["De"] == 16) == n
        for k in P.message_keys():
            if k not in draws:
                z = rng.normal(size=(2, 8, 8)) + 1j * rng.normal(size=(2, 8, 8))
                draws[k] = 0.2 * (z + np.conj(np.swapaxes(z, 1, 2)))
        nu, gb = (P.from_dense({k: v[i] for k, v in draws.items()}) for i in (0, 1))
        nb, _ = P.dual_vjp(nu, beta, qbar=P.qbuf(0.7), gbar=gb if beta > 0 else None)
        torch.cuda.synchronize()
        assert P.check() == (0, 0)
        out.append(P.to_dense(nb))
    keys = [k for k in out[1] if k[0][-1] < 1000]
    assert len(keys) > 1900
    assert max(np.abs(out[0][k] - out[1][k]).max() for k in keys) < 1e-10


@pytest.mark.parametrize("n,other", [(32768, 1), (32769, 8)])
@pytest.mark.parametrize("beta", [0.0, 2.0])
def test_eight_dimensional_double_shapes_on_both_sides_of_the_last_switch(n, other, beta):
    """8 lanes per cluster up to 32768 real clusters, one above: against the shape of the other side, both FP64
    Jacobi (the dual value per site, the oracle's entry tolerance)."""
    lrh = lrhmod()
    say(f"[D=8 double switch] n={n} beta={beta}")
    d = W.with_tops(W.heisenberg_chain(n + 2, field_x=0.4), [tuple(range(i, i + 3)) for i in range(n)])
    P = lrh.Problem(d, 0)
    nu = P.zeros()
    nu.copy_(0.3 * torch.randn(nu.shape, generator=torch.Generator().manual_seed(3), dtype=torch.float64))
    q, g, m = P.dual_eval(nu, beta, grad=True, marg=True)
    P.force_shape(8, other, f32=False)
    q1, g1, m1 = P.dual_eval(nu, beta, grad=True, marg=True)
    torch.cuda.synchronize()
    assert not torch.equal(m, m1)   # (another order of rotations, so another shape did run)
    assert (q - q1).abs().max().item() <= 1e-12 * d.n_sites
    assert (g - g1).abs().max().item() < 1e-10
    assert (m - m1).abs().max().item() < 1e-10


@pytest.mark.parametrize("cplx,n,default,other", [(False, 2048, 16, 1), (False, 2049, 8, 1), (False, 13000, 8, 1),
                                                  (False, 13001, 1, 8), (True, 2048, 16, 1), (True, 2049, 8, 1),
                                                  (True, 24576, 8, 1), (True, 24577, 1, 8)])
def test_eight_dimensional_float_iterations_at_the_switches(cplx, n, default, other):
    """Float iterations on n three-site clusters with their bonds and sites (one launch with the 8 x 8 clusters while
    their blocks are few, apart above) in the default shape, against another: float Jacobi solvers of the same
    Gibbs states, three steps, at the float entry tolerance."""
    lrh = lrhmod()
    say(f"[D=8 float switch] cplx={cplx} n={n}")
    d = (W.random_chain(n + 2, seed=7, top_len=3, subintervals=True) if cplx else
         W.with_tops(W.heisenberg_chain(n + 2, field_x=0.4), [tuple(range(i, i + 3)) for i in range(n)],
                     subintervals=True))
    P = lrh.Problem(d, 0)
    x = 0.3 * torch.randn(P.nu_len, generator=torch.Generator().manual_seed(3), dtype=torch.float64)
    out = {}
    for shape in (None, default, other):
        if shape:
            P.force_shape(8, shape, f32=True)
        nu = P.zeros(True)
        nu.copy_(x)
        ze = nu.clone()
        P.step_nesterov(nu, ze, P.new_nesterov_state(2.0), 3)
        torch.cuda.synchronize()
        assert P.check() == (0, 0)
        out[shape] = (nu, ze)
    for k in (0, 1):
        assert torch.equal(out[None][k], out[default][k])
        assert not torch.equal(out[None][k], out[other][k])
        assert (out[None][k] - out[other][k]).abs().max().item() < 5e-5


@pytest.mark.parametrize("f32", [True, False])
def test_plaquettes_on_both_sides_of_the_merged_launch(f32):
    """199 809 plaquettes (in float one launch with their bonds and sites) and 200 704 (apart): from zero messages every
    periodic lattice iterates translation-invariantly, so both have one bound per site (to rounding of the sums)."""
    lrh = lrhmod()
    out = []
    for L in (447, 448, 5):
        say(f"[plaquette merge] L={L} f32={f32}")
        P = lrh.Problem(W.tfim_plaquette_batch([L], [1.7]), 0)
        nu, ze = P.zeros(f32), P.zeros(f32)
        P.step_nesterov(nu, ze, P.new_nesterov_state(3.0), 4)
        q, _, _ = P.certify(nu)
        torch.cuda.synchronize()
        assert P.check() == (0, 0)
        out.append(q.item() / L ** 2)
    assert abs(out[0] - out[1]) <= 1e-9 and abs(out[0] - out[2]) <= (1e-5 if f32 else 1e-9)


@pytest.mark.parametrize("n", [6, 900, 9400])
def test_float_iterations_of_triples_and_quadruples_in_one_pass(n):
    """8 x 8 clusters in lanes share the bonds' launch, 16 x 16 ones go apart (up to some 9000 complex triples; the other
    way round above): against one lane per 8 x 8 cluster, at the float entry tolerance."""
    lrh = lrhmod()
    say(f"[triples and quadruples] n={n}")
    P = lrh.Problem(W.random_chain(n, seed=11, top_len=4, subintervals=True), 0)
    x = 0.3 * torch.randn(P.nu_len, generator=torch.Generator().manual_seed(3), dtype=torch.float64)
    out = []
    for shape in (None, 1):
        if shape:
            P.force_shape(8, shape, f32=True)
        for fused in (False, True):
            nu = P.zeros(True)
            nu.copy_(x)
            ze = nu.clone()
            P.step_nesterov(nu, ze, P.new_nesterov_state(2.0), 3, fused=fused)
            torch.cuda.synchronize()
            out.append((nu, ze))
    assert P.check() == (0, 0)
    for k in (0, 1):
        assert torch.equal(out[0][k], out[1][k]) and torch.equal(out[2][k], out[3][k])
        assert (out[0][k] - out[2][k]).abs().max().item() < 5e-5
