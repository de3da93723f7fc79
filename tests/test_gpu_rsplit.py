"""The resident-tile split kernels (tile class 6, the built-in choice of short
and of unaligned modes) at the edges of their tiles: row counts around whole
32-row fragments, partial fibre tiles of 32 and 64, odd strides, the largest
mode, the identity add, the fused phases and the running bound along a chain.
Tolerances are the precisions' own (gpu_util.REL_TOL) times the products."""
import numpy as np
import pytest

import synth
from gpu_util import REL_TOL, cast, empty_gpu, from_gpu, note, rel, to_gpu
from oracle import mumode as om
from oracle import schemes as sc

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2103_01691_amd as mm
    c = mm.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("prec", ["fp16x2", "bf16x3"])
def test_products_at_tile_edges(ctx, prec):
    g = synth.rng(1801, 0)
    worst = 0.0
    for n, m in ((1, 1), (3, 16), (16, 17), (31, 32), (33, 48), (81, 81), (128, 129), (141, 140), (199, 200), (255, 256)):
        for dims, mu in (((n, 7, 5), 1), ((3, n, 11), 2), ((5, n, 2600), 2), ((n, 65), 1), ((37, n), 2)):
            if n > 60 and dims[-1] == 2600 and n not in (81, 141):
                continue
            U = cast(synth.random_tensor(dims, True, g), prec, True)
            L = synth.random_matrix(m, n, True, g)
            od = tuple(m if k == mu - 1 else x for k, x in enumerate(dims))
            op = ctx.mm_op_prepare(L, prec)
            out = empty_gpu(od, prec, True)
            ctx.mumode_apply(out, to_gpu(U, prec, True), op, mu)
            err = rel(from_gpu(out), om.mode_product(U, L, mu))
            op.destroy()
            worst = max(worst, err)
            assert err < REL_TOL[prec], (prec, dims, mu, m, err)
    note(f"resident split edges {prec}: worst rel err {worst:.3e}")


@pytest.mark.parametrize("prec", ["fp16x2", "bf16x3"])
@pytest.mark.parametrize("identity", [False, True])
@pytest.mark.parametrize("dims", [(17, 21, 13), (64, 33, 20), (1, 40, 3)])
def test_phases_identity_and_chain(ctx, prec, identity, dims):
    g = synth.rng(1802, dims[0])
    U = cast(synth.random_tensor(dims, True, g), prec, True)
    E = [np.eye(n) + 0.2 * synth.random_matrix(n, n, True, g) for n in dims]
    ops = [ctx.mm_op_prepare(e, prec, identity_split=identity) for e in E]
    T = to_gpu(U, prec, True)
    ctx.gpe_strang_step(T, ops, 0.02, 1.5, 3)
    assert rel(from_gpu(T), sc.gpe_strang(U, E, 0.02, 1.5, 3)) < 9 * REL_TOL[prec]
