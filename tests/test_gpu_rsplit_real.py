"""Real operators on the resident-tile split kernels (real fibres, and the two
planes of complex ones) at the edges of their tiles: row counts around 32-row
fragments, partial fibre tiles, odd strides, the largest mode that fits, the
identity add and the running bound along a chain of products.
Tolerances are the precisions' own (gpu_util.REL_TOL) times the products."""
import numpy as np
import pytest

import synth
from gpu_util import REL_TOL, cast, empty_gpu, from_gpu, rel, to_gpu
from oracle import mumode as om

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2103_01691_amd as mm
    c = mm.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("prec", ["fp16x2", "bf16x3"])
@pytest.mark.parametrize("complex_state", [False, True])
def test_real_products_at_tile_edges(ctx, prec, complex_state):
    g = synth.rng(1901, 0)
    for n, m in ((1, 1), (3, 32), (8, 7), (31, 33), (64, 64), (81, 80), (128, 129), (200, 199), (257, 255), (511, 512)):
        for dims, mu in (((n, 7, 5), 1), ((3, n, 11), 2), ((4, n, 33), 2), ((n, 65), 1), ((37, n), 2), ((n, 13000), 1)):
            if dims[-1] == 13000 and n not in (31, 64):
                continue
            U = cast(synth.random_tensor(dims, complex_state, g), prec, complex_state)
            L = synth.random_matrix(m, n, False, g)
            od = tuple(m if k == mu - 1 else x for k, x in enumerate(dims))
            op = ctx.mm_op_prepare(L, prec)
            out = empty_gpu(od, prec, complex_state)
            ctx.mumode_apply(out, to_gpu(U, prec, complex_state), op, mu)
            err = rel(from_gpu(out), om.mode_product(U, L, mu))
            op.destroy()
            assert err < REL_TOL[prec], (prec, dims, mu, m, err)


@pytest.mark.parametrize("prec", ["fp16x2", "bf16x3"])
@pytest.mark.parametrize("identity", [False, True])
@pytest.mark.parametrize("complex_state", [False, True])
def test_real_chain(ctx, prec, identity, complex_state):
    dims = (33, 40, 18)
    g = synth.rng(1902, 0)
    U = cast(synth.random_tensor(dims, complex_state, g), prec, complex_state)
    E = [np.eye(n) + 0.2 * synth.random_matrix(n, n, False, g) for n in dims]
    ops = [ctx.mm_op_prepare(e, prec, identity_split=identity) for e in E]
    T = to_gpu(U, prec, complex_state)
    ctx.mumode_expstep(T, ops, 2)
    want = U
    for _ in range(2):
        want = om.tucker(want, E)
    assert rel(from_gpu(T), want) < 6 * REL_TOL[prec]
