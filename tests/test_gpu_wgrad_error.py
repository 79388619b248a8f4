"""The fp32 sums of weight gradients: their error against 64 bits is that of the slices that the reduction is cut into, on
the aligned, the unaligned and the fp32 engine, for one layer and for a batch."""
import math

import pytest
import torch

from paper_2309_03824_amd import binding as lrd

pytestmark = pytest.mark.gpu
BF = torch.bfloat16


def bound(K, slices, depth=16):
    """Relative error (2-norm) of a sum of K random products in `slices` chains, one fp32 addition per `depth` products
    (16: the depth of a bf16 matrix instruction; 1: every fp32 product is rounded).  An addition's error is at most
    2^-24 / sqrt(3) of the running sum in the root mean square; the running sum of i products has variance i, so n
    additions give n / 2 of its square per chain, the sum over the chains slices / 2.  Chains are whole steps of 64."""
    n = math.ceil(math.ceil(K / slices) / 64) * 64 / depth
    return 2.0 ** -24 / math.sqrt(3) * math.sqrt((n + slices) / 2)


def normal(gen, *shape, dt=BF):
    return torch.randn(*shape, device="cuda", generator=gen).to(dt)


def dense_error(M, N, K, dt):
    gen = torch.Generator(device="cuda").manual_seed(M + N + K)
    dY, X, W = normal(gen, K, M, dt=dt), normal(gen, K, N, dt=dt), normal(gen, M, N, dt=dt)
    dW = torch.full((M, N), float("nan"), device="cuda")
    code = lrd.BF16 if dt == BF else lrd.F32
    ws = torch.empty(max(lrd.dense_linear_workspace_bytes(K, N, M, code), 256), dtype=torch.uint8, device="cuda")
    lrd.dense_linear_bwd(dY, X, W, None, dW, ws)
    torch.cuda.synchronize()
    ref = dY.double().t().contiguous() @ X.double()
    return ((dW - ref).norm() / ref.norm()).item()


# (rows and columns of the gradient, tokens, slices): at least 480 workgroups of 128 x 128 tiles (432 of 64 x 64) or 256
# tokens a slice
@pytest.mark.parametrize("M,N,K,slices", [(4096, 256, 4096, 8), (3072, 192, 8192, 10), (192, 768, 8192, 12), (264, 1024, 4100, 16),
                                          (2048, 104, 4099, 7), (1001, 1003, 4000, 8), (1001, 192, 8192, 9)])
def test_weight_gradient_error(M, N, K, slices):
    assert dense_error(M, N, K, BF) <= bound(K, slices)


# few and many tiles of 32 x 32 and 64 x 64 (waves of a workgroup that share a reduction: 8 and 2)
@pytest.mark.parametrize("M,N,K,slices", [(2048, 1024, 1024, 4), (1000, 1000, 20000, 8), (640, 640, 16384, 20),
                                          (771, 705, 8191, 12), (130, 70, 5000, 19)])
def test_f32_weight_gradient_error(M, N, K, slices):
    assert dense_error(M, N, K, torch.float32) <= bound(K, slices, depth=1)


@pytest.mark.parametrize("L,M,N,K,slices", [(12, 1024, 256, 8192, 4), (4, 2048, 128, 4096, 7), (3, 520, 136, 8000, 15)])
def test_batched_weight_gradient_error(L, M, N, K, slices):
    gen = torch.Generator(device="cuda").manual_seed(M + N + K)
    dY, H = normal(gen, L, K, M), normal(gen, L, K, N)
    dU = torch.full((L, M, N), float("nan"), device="cuda")
    ws = torch.empty(max(lrd.linear_wgrad_batched_workspace_bytes(L, K, M, M, N, lrd.BF16, lrd.FREEZE_L0), 256), dtype=torch.uint8, device="cuda")
    lrd.linear_wgrad_batched(dY, H, None, None, None, dU, lrd.FREEZE_L0, ws)
    torch.cuda.synchronize()
    ref = torch.stack([dY[l].double().t().contiguous() @ H[l].double() for l in range(L)])
    assert ((dU - ref).norm() / ref.norm()).item() <= bound(K, slices)


# Every tile that weight gradients are given (rows, columns, waves down and across, stages), off its edges
@pytest.mark.parametrize("M,N,K,slices,tile", [(3080, 1000, 8001, 3, "256,256,2,4,2"), (264, 4104, 6001, 5, "128,256,2,4,3"),
                                               (200, 3080, 8201, 10, "128,128,2,4,2"), (104, 1000, 16001, 14, "64,128,2,4,4"),
                                               (776, 200, 2001, 7, "64,64,2,2,4"), (24, 40, 70, 1, "64,64,2,2,4")])
def test_weight_gradient_tiles(M, N, K, slices, tile):
    with lrd.ProfileLog(2) as log:
        error = dense_error(M, N, K, BF)
    assert (log.rows()[0]["kernel"], log.rows()[0]["splits"]) == (f"gemm2_kernel<{tile},A_KM,B_KM,f32>", slices)
    assert error <= bound(K, slices)


@pytest.mark.parametrize("N,hw,C,S,slices,tile", [(37, 14, 128, 128, 12, "128,64,4,2,4"), (33, 7, 312, 312, 6, "128,128,2,4,2"),
                                                  (21, 28, 72, 64, 40, "64,128,2,4,4"), (5, 9, 24, 40, 1, "64,64,2,2,4")])
def test_convolution_weight_gradient_tiles(N, hw, C, S, slices, tile):
    gen = torch.Generator(device="cuda").manual_seed(N + C)
    geo = lrd.conv_geom(N, hw, hw, C, S, 1, 1, 3, 1, 1)
    X, dY, W = normal(gen, N, hw, hw, C), normal(gen, N, hw, hw, S), normal(gen, S, 3, 3, C)
    dW = torch.full((S, 3, 3, C), float("nan"), device="cuda")
    ws = torch.empty(lrd.dense_conv_workspace_bytes(geo, lrd.BF16) + 16, dtype=torch.uint8, device="cuda")
    with lrd.ProfileLog(2) as log:
        lrd.dense_conv_bwd(dY, X, W, None, dW, geo, ws)
        torch.cuda.synchronize()
    assert (log.rows()[0]["kernel"], log.rows()[0]["splits"]) == (f"gemm2_kernel<{tile},A_KM,B_KM,f32,conv>", slices)
    pad, rows = torch.nn.functional.pad(X.double(), (0, 0, 1, 1, 1, 1)), dY.double().reshape(-1, S).t().contiguous()
    ref = torch.stack([torch.stack([rows @ pad[:, u:u + hw, v:v + hw].reshape(-1, C) for v in range(3)], 1) for u in range(3)], 1)
    assert ((dW - ref).norm() / ref.norm()).item() <= bound(N * hw * hw, slices)
