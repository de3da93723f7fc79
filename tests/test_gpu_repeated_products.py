"""Several steps of a mode in one launch (mumode_expstep in FP64 and FP32).

The growth bound: the modes' operators grow and shrink the state by the same
factor per step, so the step order stays at one size while all steps of the
first mode at once would pass the type's range (16^40 = 2^160 in FP32,
2^(30 40) = 2^1200 in FP64); only the blocks keep the result finite.

Mode lengths: every fragment count per wave of the resident tile's loop over
products (one at 65 and 80 rows, two at 81 and 193, three at 129, four at 300
real rows), and the tuner's choices of it by a tune file.  Tolerance: the
precision's own (gpu_util.REL_TOL) per step."""
import numpy as np
import pytest

import synth
from gpu_util import REL_TOL, cast, from_gpu, rel, to_gpu
from oracle import mumode as om

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2103_01691_amd as mm
    c = mm.Context(0)
    yield c
    c.close()


def _orthogonal(n, cplx, g):
    return np.linalg.qr(synth.random_matrix(n, n, cplx, g))[0]


@pytest.mark.parametrize("prec,log2scale", [("fp32", 4), ("fp64", 30)])
@pytest.mark.parametrize("cplx", [True, False])
@pytest.mark.parametrize("dims", [(40, 23, 6), (81, 66, 3)])
def test_growth_is_bounded_by_blocks(ctx, prec, log2scale, cplx, dims):
    steps = 40
    assert log2scale * steps > (1024 if prec == "fp64" else 128)
    g = synth.rng(2101, dims[0] + int(cplx))
    U = cast(synth.random_tensor(dims, cplx, g), prec, cplx)
    s = 2.0 ** log2scale
    E = [_orthogonal(n, cplx, g) * f for n, f in zip(dims, (s, 1.0 / s, 1.0))]
    T = to_gpu(U, prec, cplx)
    ctx.mumode_expstep(T, [ctx.mm_op_prepare(e, prec) for e in E], steps)
    got = from_gpu(T)
    assert np.all(np.isfinite(got))
    assert rel(got, om.expstep(U, E, steps)) < steps * REL_TOL[prec]


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("cplx,n", [(c, n) for c in (True, False) for n in (65, 80, 81, 129, 193, 256)] + [(False, 300)])
@pytest.mark.parametrize("near", [False, True])
def test_every_fragment_count(ctx, prec, cplx, n, near):
    g = synth.rng(2102, n + int(cplx))
    for dims in ((n, 37), (19, n), (3, n, 7)):
        U = cast(synth.random_tensor(dims, cplx, g), prec, cplx)
        E = [_orthogonal(m, cplx, g) if m == n or not near else np.eye(m) for m in dims]
        if near:
            E = [np.eye(m) + 0.05 * e if m == n else e for m, e in zip(dims, E)]
        T = to_gpu(U, prec, cplx)
        ctx.mumode_expstep(T, [ctx.mm_op_prepare(e, prec) for e in E], 5)
        assert rel(from_gpu(T), om.expstep(U, E, 5)) < 5 * REL_TOL[prec], dims


@pytest.mark.parametrize("prec,code", [("fp64", 0), ("fp32", 1)])
@pytest.mark.parametrize("cplx", [True, False])
@pytest.mark.parametrize("cls", [0, 1, 2, 3])
def test_tuned_fragment_counts(ctx, tmp_path, prec, code, cplx, cls):
    g = synth.rng(2103, 10 * code + cls)
    for n in (40, 81, 200) + (() if cplx else (300,)):
        dims, c = (5, n, 9), 2 if cplx else 1
        f = tmp_path / "t.txt"
        f.write_text("mumode-tune 2\n" + "".join(f"{code} {int(cplx)} {ld} {c * n} {c * n} 45 {cls} 0.0\n"
                                                 for ld in (0, 1, 2, 3)))
        ctx.mm_tune_clear()
        ctx.mm_tune_load(f)
        U = cast(synth.random_tensor(dims, cplx, g), prec, cplx)
        E = synth.random_matrix(n, n, cplx, g)
        T = to_gpu(U, prec, cplx)
        ctx.mumode_expstep(T, [None, ctx.mm_op_prepare(E, prec), None], 1)
        ctx.mm_tune_clear()
        assert rel(from_gpu(T), om.mode_product(U, E, 2)) < REL_TOL[prec], n
