"""GPU parity of the bias gradient (column sums of dY) at the edges of its row and column blocks, with the workspace of a
data gradient to cut the rows in and with what both factors frozen and no dX leave: from 512 tokens on that of the sliced
weight gradients, below it none."""
import numpy as np
import pytest
import torch

from parity import dev, empty, f32, host, workspace
from paper_2309_03824_amd import binding as lrd

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dt", ["bf16", "f32"])
@pytest.mark.parametrize("T,n", [(1, 8), (31, 24), (33, 257), (256, 264), (1000, 520), (4099, 1000), (2048, 37)])
@pytest.mark.parametrize("with_dx", [True, False])
def test_bias_gradient_is_the_column_sum(dt, T, n, with_dx):
    rng = np.random.default_rng(T * 1000 + n)
    n_in, r = 16, 8
    dY = dev(rng.standard_normal((T, n)), dt)
    V, U = dev(rng.standard_normal((r, n_in)), dt), dev(rng.standard_normal((n, r)), dt)
    dX = empty((T, n_in), dt) if with_dx else None
    db = f32((n,))
    ws = workspace(lrd.linear_workspace_bytes(T, n_in, n, r, lrd.BF16 if dt == "bf16" else lrd.F32, 3))
    lrd.linear_bwd(dY, None, None, V, U, dX, None, None, db, 3, ws)
    torch.cuda.synchronize()
    ref = dY.double().cpu().numpy()
    # T fp32 terms in any order: the error of a column is at most T * 2^-24 times the sum of magnitudes
    bound = T * 2.0 ** -24 * np.abs(ref).sum(0) + 1e-30
    assert np.all(np.abs(host(db).astype(np.float64) - ref.sum(0)) <= bound)
