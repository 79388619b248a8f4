"""GPU parity of the fp32 products at the edges of their tiles (16, 32 and 64 wide), of the 16-deep K-steps and
of the K cut over waves and workgroups: forward, data gradient and weight gradient of a dense layer."""
import numpy as np
import pytest
import torch

from parity import dev, f32, host, workspace
from paper_2309_03824_amd import binding as lrd

pytestmark = pytest.mark.gpu


def bounded(got, a, b, what):
    """|got - a.b| <= K * 2^-24 * |a|.|b|: fp32 products summed in any order."""
    got = host(got)
    bound = a.shape[1] * 2.0 ** -24 * (np.abs(a) @ np.abs(b)) + 1e-30
    assert np.all(np.abs(got - a @ b) <= bound), what


@pytest.mark.parametrize("T,n_in,n_out", [(1, 5, 3), (2, 2, 2), (15, 17, 16), (16, 16, 16), (33, 31, 47), (64, 129, 65), (7, 1040, 2),
                                          (1030, 33, 18), (2051, 64, 40), (600, 250, 900), (777, 1001, 1003)])
def test_f32_products(T, n_in, n_out):
    rng = np.random.default_rng(T + 7 * n_in + 31 * n_out)
    X, W, dY = (dev(rng.standard_normal(s), "f32") for s in ((T, n_in), (n_out, n_in), (T, n_out)))
    b = dev(rng.standard_normal(n_out), "f32")
    Y, dX, dW = f32((T, n_out)), f32((T, n_in)), f32((n_out, n_in))
    ws = workspace(lrd.dense_linear_workspace_bytes(T, n_in, n_out, lrd.F32))
    lrd.dense_linear_fwd(X, W, b, Y, ws)
    lrd.dense_linear_bwd(dY, X, W, dX, dW, ws)
    torch.cuda.synchronize()
    x, w, g, bias = host(X), host(W), host(dY), host(b)
    bounded(Y, np.concatenate([x, np.ones((T, 1))], 1), np.concatenate([w.T, bias[None]], 0), "Y")
    bounded(dX, g, w, "dX")
    bounded(dW, g.T, x, "dW")
