"""The forms of FP32 complex products whose operators are formed per step
(oscillator, midpoint) or kept as L - I by the caller.

Far from the identity they keep the two components apart (four real products):
with a real-valued operator the imaginary part of the result is that of the
state times the operator, to FP32 rounding of its own size, also where it is
10^-5 of the real part.  In three products its error would be rounding at the
size of the real part, 10^-2 of it.

Near the identity they run on L - I with the input added back: a short product
rounds once, at 2^-24 of its result or less, and P of them in sequence add up to
sqrt(P) 2^-24 (1.5 of it is the tolerance); products on L itself round at every
partial sum, two to five times that."""
import numpy as np
import pytest

import synth
from gpu_util import REL_TOL, cast, from_gpu, note, rel, to_gpu
from oracle import mumode as om
from oracle import operators as op
from oracle import schemes as sc

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2103_01691_amd as mm
    c = mm.Context(0)
    yield c
    c.close()


def _state(dims, k):
    g = synth.rng(2001, k)
    return cast(synth.random_tensor(dims, False, g) + 1e-5j * synth.random_tensor(dims, False, g), "fp32", True)


@pytest.mark.parametrize("n", [24, 40, 100])
def test_midpoint_step_far(ctx, n):
    dims = (n, 12, 7)
    U = _state(dims, n)
    g = synth.rng(2002, n)
    B = [3.0 * np.linalg.qr(synth.random_matrix(m, m, False, g))[0] + 0j for m in dims]
    tau = 1.0
    ref = sc.magnus_midpoint(U, B, [np.zeros(m) for m in dims], lambda mu, t: 0.0, tau, 2)
    T = to_gpu(U, "fp32", True)
    ctx.mumode_magnus_step(T, B, None, None, tau, 2, "fp32")
    got = from_gpu(T)
    assert rel(got.real, ref.real) < 2 * REL_TOL["fp32"]
    assert rel(got.imag, ref.imag) < 2 * REL_TOL["fp32"]


@pytest.mark.parametrize("m", [24, 40, 100])
def test_oscillator_step_far(ctx, m):
    # a step of length zero on a quarter of the Hermite functions: the
    # projection on them, real and far from the identity
    import paper_2103_01691_amd as mm
    Phi, Psi = op.hermite_forward(m), op.hermite_backward(m)
    X, _ = mm.hermite_nodes(m)
    K = m // 4
    F, B = mm.hermite_matrices(m)
    F, B = np.ascontiguousarray(F[:K]), np.ascontiguousarray(B[:, :K])
    g = synth.rng(2003, m)
    full = np.zeros((m, m, m), complex)
    full[:6, :6, :6] = g.standard_normal((6, 6, 6)) + 1e-5j * g.standard_normal((6, 6, 6))
    U = cast(om.tucker(full, [Psi] * 3), "fp32", True)
    ref = om.tucker(U, [Psi[:, :K] @ Phi[:K]] * 3)
    T = to_gpu(U, "fp32", True)
    ctx.ho_strang_step(T, [ctx.mm_op_prepare(F, "fp32")] * 3, [ctx.mm_op_prepare(B, "fp32")] * 3, [X] * 3, 0.2, 0.0,
                       0.1, 1)
    got = from_gpu(T)
    assert rel(got.real, ref.real) < REL_TOL["fp32"]
    assert rel(got.imag, ref.imag) < REL_TOL["fp32"]


@pytest.mark.parametrize("n", [24, 81, 200])
def test_callers_identity_split_far_from_the_identity(ctx, n):
    dims = (5, n, 9)
    U = _state(dims, n)
    Q = np.linalg.qr(synth.random_matrix(n, n, False, synth.rng(2004, n)))[0]
    T = to_gpu(U, "fp32", True)
    ctx.mumode_expstep(T, [None, ctx.mm_op_prepare(-Q.T @ Q + 0.3 * Q + 0j, "fp32", identity_split=True), None], 1)
    ref = om.mode_product(U, -Q.T @ Q + 0.3 * Q, 2)
    got = from_gpu(T)
    assert rel(got.real, ref.real) < REL_TOL["fp32"]
    assert rel(got.imag, ref.imag) < REL_TOL["fp32"]


def _smooth(dims):
    U = np.ones(dims, complex)
    for k, n in enumerate(dims):
        x = np.linspace(-3.0, 3.0, n)
        U *= np.exp(-(x - 0.3 * k) ** 2 / 2 + 0.7j * x).reshape([-1 if j == k else 1 for j in range(len(dims))])
    return cast(U, "fp32", True)


@pytest.mark.parametrize("timed", [False, True])
@pytest.mark.parametrize("n", [24, 40, 100])
def test_midpoint_step_near(ctx, n, timed):
    dims, tau, steps = (n, n, n), 0.01, 4
    g = synth.rng(2005, n)
    U = _smooth(dims)
    B = []
    for m in dims:
        H = synth.random_matrix(m, m, True, g)
        B.append(-1j * (H + H.conj().T))
    d = [g.uniform(-1.0, 1.0, m) for m in dims]
    gf = (lambda mu, t: -1j * np.cos(t + mu)) if timed else (lambda mu, t: 0.0)
    coef = np.array([[gf(mu, (j + 0.5) * tau) for mu in range(3)] for j in range(steps)])
    ref = sc.magnus_midpoint(U, B, d, gf, tau, steps)
    T = to_gpu(U, "fp32", True)
    ctx.mumode_magnus_step(T, B, d if timed else None, coef if timed else None, tau, steps, "fp32")
    err = rel(from_gpu(T), ref)
    note(f"midpoint near n={n} timed={timed}: {err:.3e}")
    assert err < 1.5 * np.sqrt(3 * steps) * 2.0 ** -24


@pytest.mark.parametrize("eps", [0.0, 0.1])
@pytest.mark.parametrize("m", [24, 40, 100])
def test_oscillator_step_near(ctx, m, eps):
    import paper_2103_01691_amd as mm
    steps, tau = 4, 2e-4
    Phi, Psi, X = op.hermite_forward(m), op.hermite_backward(m), op.hermite_nodes(m)
    Xl, _ = mm.hermite_nodes(m)
    F, B = mm.hermite_matrices(m)
    U = cast(om.tucker(synth.hermite_coefficients(m, 8, 3, cfg_id=3), [Psi] * 3), "fp32", True)
    ref = sc.ho_strang(U, [Phi] * 3, [Psi] * 3, [X] * 3, 0.3, tau, eps, steps)
    T = to_gpu(U, "fp32", True)
    ctx.ho_strang_step(T, [ctx.mm_op_prepare(F, "fp32")] * 3, [ctx.mm_op_prepare(B, "fp32")] * 3, [Xl] * 3, 0.3, tau,
                       eps, steps)
    err = rel(from_gpu(T), ref)
    note(f"oscillator near m={m} eps={eps}: {err:.3e}")
    assert err < 1.5 * np.sqrt(3 * steps) * 2.0 ** -24
