"""The batched device exponentials of the exponential midpoint step: modes of
different sizes and norms (batches split by size and by the number of
squarings), every mode or some timed, more steps than one block holds, modes
above the batched kernels' size, against the oracle.  Tolerance: the
precision's own (gpu_util.REL_TOL) per step."""
import numpy as np
import pytest

import synth
from gpu_util import REL_TOL, cast, from_gpu, rel, to_gpu
from oracle import schemes as sc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "fp32", "fp16x2"])
@pytest.mark.parametrize("dims,timed,nsteps", [((16, 17, 5), (1, 1, 1), 3), ((33, 16, 16), (0, 1, 0), 70),
                                               ((1, 40, 3), (0, 0, 1), 2), ((256, 4), (1, 0), 2), ((260, 3), (1, 1), 2)])
def test_batched_exponentials(prec, dims, timed, nsteps):
    import paper_2103_01691_amd as mm
    g = synth.rng(1701, dims[0])
    U = cast(synth.random_tensor(dims, True, g), prec, True)
    tau = 0.05
    B, d = [], []
    for k, n in enumerate(dims):
        H = synth.random_matrix(n, n, True, g, scale=1.0)
        B.append(-1j * (H + H.conj().T) * (0.5 + 2.0 * k))     # skew-Hermitian, norms a few squarings apart
        d.append(g.uniform(-3.0, 3.0, n) if timed[k] else None)
    gf = lambda mu, t: -1j * np.cos(3.0 * t + mu)
    coef = np.array([[gf(mu, (j + 0.5) * tau) for mu in range(len(dims))] for j in range(nsteps)])
    ref = sc.magnus_midpoint(U, B, [x if x is not None else np.zeros(n) for x, n in zip(d, dims)], gf, tau, nsteps)
    with mm.Context(0) as ctx:
        T = to_gpu(U, prec, True)
        ctx.mumode_magnus_step(T, B, d, coef, tau, nsteps, prec)
        assert rel(from_gpu(T), ref) < nsteps * REL_TOL[prec]
