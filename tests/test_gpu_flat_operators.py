"""Operators of few rows and long columns (transforms that keep a few modes of
a long axis) on many fibres, where the resident tile's LDS is bounded by the
columns: every combination of waves along the fibres and fibre fragments that
the LDS limit changes, against the oracle.  Tolerance: the precision's own
(gpu_util.REL_TOL)."""
import numpy as np
import pytest

import synth
from gpu_util import REL_TOL, cast, empty_gpu, from_gpu, rel, to_gpu
from oracle import mumode as om

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,cplx_op,cplx,m,n,side", [
    ("fp64", True, True, 1, 145, 182), ("fp64", False, True, 16, 200, 200), ("fp64", True, True, 16, 256, 256),
    ("fp64", False, False, 16, 256, 257), ("fp64", False, True, 32, 400, 182), ("fp64", False, False, 17, 512, 182),
    ("fp32", False, True, 16, 512, 182), ("fp32", False, False, 8, 256, 257)])
def test_few_rows_long_columns(prec, cplx_op, cplx, m, n, side):
    import paper_2103_01691_amd as mm
    g = synth.rng(1901, m + n)
    L = synth.random_matrix(m, n, cplx_op, g)
    U = cast(synth.random_tensor((n, side, side), cplx, g), prec, cplx)
    with mm.Context(0) as ctx:
        op = ctx.mm_op_prepare(L, prec)
        for mu in (1, 2):
            X = U if mu == 1 else np.ascontiguousarray(U.transpose(1, 0, 2))
            dims = tuple(m if k == mu - 1 else x for k, x in enumerate(X.shape))
            out = empty_gpu(dims, prec, cplx)
            ctx.mumode_transform(out, to_gpu(X, prec, cplx), [op if k == mu - 1 else None for k in range(3)])
            assert rel(from_gpu(out), om.mode_product(X, L, mu)) < REL_TOL[prec], (mu, dims)
