"""The resident-tile FP64 / FP32 product kernels at the edges of their tiles:
row counts around whole fragments and around the fragment-count rule, fibre
counts that leave a partial tile, odd strides, every operator form, phases
with real operators, repeated products in one launch, and non-finite entries.
Tolerances are the precisions' own (gpu_util.REL_TOL) times the products."""
import numpy as np
import pytest

import synth
from gpu_util import REL_TOL, cast, empty_gpu, from_gpu, note, rel, to_gpu
from oracle import mumode as om
from oracle import schemes as sc

pytestmark = pytest.mark.gpu

# (n, m): fragment edges, the largest complex / real sides, rectangles
COMPLEX = [(1, 1), (3, 16), (16, 17), (31, 64), (64, 65), (80, 80), (81, 81), (129, 128), (141, 145), (192, 193), (256, 256)]
REAL = COMPLEX + [(257, 300), (512, 512)]


@pytest.fixture(scope="module")
def ctx():
    import paper_2103_01691_amd as mm
    c = mm.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("form", ["cc", "cc-near-identity", "rc", "rr"])
def test_products_at_tile_edges(ctx, prec, form):
    cplx_op, cplx = form.startswith("cc"), form != "rr"
    g = synth.rng(1601, 0)
    for n, m in (COMPLEX if cplx_op else REAL):
        if form == "cc-near-identity":      # kept as L - I, the input added back
            m = n
        for dims, mu in (((n, 7, 5), 1), ((3, n, 11), 2), ((n, 33), 1), ((37, n), 2)):
            U = cast(synth.random_tensor(dims, cplx, g), prec, cplx)
            L = synth.random_matrix(m, n, cplx_op, g)
            if form == "cc-near-identity":
                L = np.eye(n) + 0.1 * L
            od = tuple(m if k == mu - 1 else x for k, x in enumerate(dims))
            op = ctx.mm_op_prepare(L, prec)
            out = empty_gpu(od, prec, cplx)
            ctx.mumode_apply(out, to_gpu(U, prec, cplx), op, mu)
            err = rel(from_gpu(out), om.mode_product(U, L, mu))
            op.destroy()
            assert err < REL_TOL[prec], (prec, form, dims, mu, m, err)
    note(f"resident tile edges {prec} {form}: last rel err {err:.3e}")


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("dims", [(33, 20, 9), (70, 5, 18)])
def test_phases_with_real_operators(ctx, prec, dims):
    g = synth.rng(1602, dims[0])
    U = cast(synth.random_tensor(dims, True, g), prec, True)
    E = [np.eye(n) + 0.2 * synth.random_matrix(n, n, False, g) for n in dims]
    T = to_gpu(U, prec, True)
    ctx.gpe_strang_step(T, [ctx.mm_op_prepare(e, prec) for e in E], 0.02, 1.5, 2)
    assert rel(from_gpu(T), sc.gpe_strang(U, E, 0.02, 1.5, 2)) < 6 * REL_TOL[prec]


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("cplx", [True, False])
@pytest.mark.parametrize("scale", [1.0, 4.0])
def test_repeated_products_in_one_launch(ctx, prec, cplx, scale):
    # all steps of a mode in one launch, in blocks that keep the reordered
    # products in range: with operators of norm 4 and 1/4 a reordering of all
    # 40 steps would pass 4^40 in FP32's 2^127 range only by the blocks
    dims, steps = (40, 23, 6), 40
    g = synth.rng(1603, int(cplx))
    U = cast(synth.random_tensor(dims, cplx, g), prec, cplx)
    E = [np.linalg.qr(synth.random_matrix(n, n, cplx, g))[0] * s for n, s in zip(dims, (scale, 1.0 / scale, 1.0))]
    T = to_gpu(U, prec, cplx)
    ctx.mumode_expstep(T, [ctx.mm_op_prepare(e, prec) for e in E], steps)
    assert rel(from_gpu(T), om.expstep(U, E, steps)) < steps * REL_TOL[prec]


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_non_finite_entries_stay_in_their_fibre(ctx, prec):
    dims = (21, 18, 3)
    g = synth.rng(1604, 0)
    for mu, bad in ((1, np.inf), (2, np.nan)):
        U = cast(synth.random_tensor(dims, True, g), prec, True)
        U[4, 5, 1] = bad
        n = dims[mu - 1]
        out = empty_gpu(dims, prec, True)
        ctx.mumode_apply(out, to_gpu(U, prec, True), ctx.mm_op_prepare(synth.random_matrix(n, n, True, g), prec), mu)
        got = np.isfinite(from_gpu(out))
        want = np.ones(dims, dtype=bool)
        want[(slice(None), 5, 1) if mu == 1 else (4, slice(None), 1)] = False
        assert np.array_equal(got, want)
