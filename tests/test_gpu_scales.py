"""Magnitudes far from one: certified values of matrices whose squares underflow or overflow, or that hold
single entries of such a size, and of matrices that are not finite; states and iterations of Hamiltonians
times a power of two."""
import numpy as np
import pytest

import lrh_workloads as W
from test_gpu_parity import PROBLEMS, lrhmod, need_gpu, say  # noqa: F401

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def dense(k, seed, cplx):
    rng = np.random.default_rng(seed)
    z = rng.normal(size=(2 ** k, 2 ** k)) + (1j * rng.normal(size=(2 ** k, 2 ** k)) if cplx else 0.0)
    return z + z.conj().T


def one_cluster(h, cplx):
    k = int(np.log2(len(h)))
    b = W._Builder("dense", k)
    b.add_term(tuple(range(k)), h)
    return lrhmod().Problem(b.build(real=not cplx), 0)


def certified(P, method):
    P.set_certify_method(method)
    q, mg, _ = P.certify(P.zeros())
    torch.cuda.synchronize()
    assert P.check() == (0, 0)
    return q.item(), mg.item()


TRIDIAG = [(k, cplx) for k in (4, 5, 6, 7, 8) for cplx in (False, True)]


@pytest.mark.parametrize("k,cplx", TRIDIAG)
def test_certified_value_scales_exactly_by_powers_of_two(k, cplx):
    """The tridiagonalisation of 2^e h is that of h times 2^e, bit for bit, value and margin, also where every
    square underflows (1e-163) or overflows (1e156)."""
    h = dense(k, 3 + k, cplx)
    q0, m0 = certified(one_cluster(h, cplx), 1)
    for e in (-540, -400, 520):
        say(f"[tridiag scale] 2^{k} cplx={cplx} e={e}")
        q, m = certified(one_cluster(np.ldexp(1.0, e) * h, cplx), 1)
        assert q == np.ldexp(q0, e) and m == np.ldexp(m0, e)


@pytest.mark.parametrize("k,cplx", TRIDIAG)
@pytest.mark.parametrize("kind", ["first", "column"])
def test_certified_value_with_entries_whose_squares_underflow(k, cplx, kind):
    """One first-subdiagonal entry of 2e-162, or a column whose only entries off the diagonal are near 1e-158,
    in a matrix of entries near one: lambda_min within the margin, 8 D eps ||h||_F, of LAPACK's."""
    say(f"[tridiag tiny] 2^{k} {kind} cplx={cplx}")
    D = 2 ** k
    h = dense(k, 20 + k, cplx)
    if kind == "first":
        h[1, 0] = 2.3e-162 * (0.8 + 0.6j if cplx else 1.0)
        h[0, 1] = np.conj(h[1, 0])
    else:
        h[1:, 0] = h[0, 1:] = 0.0
        h[1, 0] = h[0, 1] = 1.0e-158
        h[D - 1, 0] = -0.7e-158 * (0.6 + 0.8j if cplx else 1.0)
        h[0, D - 1] = np.conj(h[D - 1, 0])
    q, mg = certified(one_cluster(h, cplx), 1)
    margin = 8 * D * np.finfo(np.float64).eps * np.linalg.norm(h)
    assert abs(q - np.linalg.eigvalsh(h)[0]) <= margin
    assert mg >= margin * (1 - 1e-9)


@pytest.mark.parametrize("e", [0, -540, 520])
def test_certified_value_without_workspace_scales_exactly(e):
    """The one-wave tridiagonalisation, which the allocation-free call takes where the slabs of 128
    256-dimensional clusters fill its workspace, on one 16- and one 32-dimensional cluster."""
    lrh = lrhmod()
    say(f"[tridiag one wave] e={e}")
    b = W._Builder("hog", 144)
    for i in range(128):
        b.add_top(tuple(range(i, i + 8)))
    hs = [dense(4, 41, False), dense(5, 42, False)]
    hs[0][1, 0] = hs[0][0, 1] = 2.3e-162 if e == 0 else hs[0][0, 1]
    for h, first in zip(hs, (135, 139)):
        b.add_term(tuple(range(first, first + int(np.log2(len(h))))), np.ldexp(1.0, e) * h)
    P = lrh.Problem(b.build(), 0)
    q, mg = P.qbuf(), P.qbuf()
    lm = torch.empty(P.n_clusters, dtype=torch.float64, device="cuda")
    lrh.lrh_certify_noalloc(P.h, P.zeros(), 0, q, mg, lm)
    torch.cuda.synchronize()
    assert P.check() == (0, 0)
    lm = dict(zip(P.clusters, lm.cpu().numpy()))
    for h, first in zip(hs, (135, 139)):
        got = np.ldexp(lm[tuple(range(first, first + int(np.log2(len(h)))))], -e)
        margin = 8 * len(h) * np.finfo(np.float64).eps * np.linalg.norm(h)
        assert abs(got - np.linalg.eigvalsh(h)[0]) <= margin


@pytest.mark.parametrize("k,cplx", TRIDIAG)
@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_certified_value_of_a_matrix_that_is_not_finite(k, cplx, bad):
    """A NaN or infinite message component: the cluster's value is NaN and counted, whatever rows the
    component does not reach."""
    lrh = lrhmod()
    say(f"[tridiag not finite] 2^{k} cplx={cplx} {bad}")
    h = np.diag(np.arange(2.0 ** k)).astype(complex if cplx else float)   # rows that do not mix
    P = one_cluster(h, cplx)
    P.set_certify_method(1)
    nu = P.zeros()
    nu[0] = bad
    _, _, lm = P.certify(nu, lmin=True)
    torch.cuda.synchronize()
    top = P.clusters.index(tuple(range(k)))
    assert np.isnan(lm[top].item())
    with pytest.raises(lrh.LrhError) as err:
        P.check()
    assert err.value.code == 6


def scaled(name, e, f32, seed=3):
    """Problem and messages of PROBLEMS[name] times 2^e."""
    P = lrhmod().Problem(W.batch_scaled([PROBLEMS[name]()], [2.0 ** e]), 0)
    x = 0.3 * torch.randn(P.nu_len, generator=torch.Generator().manual_seed(seed), dtype=torch.float64)
    nu = P.zeros(f32)
    nu.copy_(x.float().double() * 2.0 ** e)
    return P, nu


@pytest.mark.parametrize("name", ["c1_tfim16_complex", "randchain_Y3", "randchain_Y4", "randchain_T4_two_level",
                                  "xxz_tri3", "spin1_Y3_complex", "gue_Y5"])
@pytest.mark.parametrize("e", [-440, 400])
def test_double_states_and_iterations_at_any_magnitude(name, e):
    """H and messages times 2^e (1e-133: squares near the smallest normal number), beta over 2^e: the states,
    iterates and cotangents are those of H to the entry tolerance of the parity tests, and no solve misses its
    tolerance.  At beta = 0 every eigenvalue of the small one lies in the ground window, 1e-9 wide: mu = 1 / D."""
    lrh = lrhmod()
    out = []
    for k in (0, e):
        say(f"[scale] {name} 2^{k}")
        P, nu = scaled(name, k, False)
        sc = 2.0 ** k
        q, g, m = P.dual_eval(nu, 0.7 / sc, grad=True, marg=True)
        b, mg, lm = P.certify(nu, lmin=True)
        x, z = nu.clone(), nu.clone()
        P.step_nesterov(x, z, P.new_nesterov_state(4.0 / sc), 5)
        r = [q / sc, g, m, lm / sc, mg / sc, x / sc, z / sc]
        if not name.startswith("spin1"):
            r.append(P.dual_vjp(nu, 3.0 / sc, qbar=P.qbuf(0.7))[0])
        if k < 0:
            assert P.dual_eval(nu, 0.0, grad=True)[1].abs().max().item() < 1e-10
        torch.cuda.synchronize()
        assert P.check() == (0, 0)
        out.append(r)
    n = P.desc.n_sites
    for i, (a, b) in enumerate(zip(*out)):
        assert (a - b).abs().max().item() <= (1e-9 * n if i == 0 else 1e-10)


@pytest.mark.parametrize("W_", [8, 16])
@pytest.mark.parametrize("e", [-43, -58, 40])
def test_float_lanes_solver_at_any_magnitude(W_, e):
    """Complex 8 x 8 clusters in lanes, float: as above, at the float tolerance."""
    out = []
    for k in (0, e):
        say(f"[scale float] W={W_} 2^{k}")
        P, nu = scaled("randchain_T4_two_level", k, True)
        P.force_shape(8, W_, f32=True)
        q, g, m = P.dual_eval(nu, 2.0 / 2.0 ** k, grad=True, marg=True)
        torch.cuda.synchronize()
        assert P.check() == (0, 0)
        out.append((q / 2.0 ** k, g, m))
    for a, b in zip(*out):
        assert (a - b).abs().max().item() <= 5e-5
