"""More fibres than one launch dimension takes threads for: 2^30 and some, of a
unit mode (8.6 GB of complex FP32 state), one product and a run of two."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nsteps", [1, 2])
def test_unit_mode_of_2_to_30_fibres(nsteps):
    import paper_2103_01691_amd as mm
    import torch
    a, b = 32768, 32769
    T = torch.empty((b, 1, a), dtype=torch.complex64, device="cuda")     # dims (a, 1, b)
    row = torch.arange(a, device="cuda", dtype=torch.float32) / a
    for i in range(b):
        T[i, 0] = torch.complex(row, row * 0 + (i % 1024) / 1024.0)
    z = 0.8 - 0.6j
    with mm.Context(0) as ctx:
        op = ctx.mm_op_prepare(np.array([[z]]), "fp32")
        ctx.mumode_expstep(T, [None, op, None], nsteps)
        torch.cuda.synchronize()
    w = torch.tensor(z ** nsteps, dtype=torch.complex128, device="cuda")
    worst = 0.0
    for i in range(0, b, 2048):
        rows = torch.arange(i, min(i + 2048, b), device="cuda")
        want = torch.complex(row.double()[None, :].expand(len(rows), a),
                             ((rows % 1024) / 1024.0).double()[:, None].expand(len(rows), a)) * w
        worst = max(worst, float((T[i:i + 2048, 0] - want).abs().max()))
    assert worst < 1e-6 * nsteps
