"""The output tiles of the MFMA product kernel, each at sizes off its edges: rows, columns and K that end inside a tile, a
load and a K-step; against fp32 products of the same bf16 operands.  Each shape names its tile, and the event log has to
agree."""
import pytest
import torch

from paper_2309_03824_amd import binding as lrd

BF = torch.bfloat16

# (tokens, in, out, rank), and the tile (rows, columns, waves down and across, stages) that the products
# tokens x rank over in and tokens x out over rank are given
SHAPES = [((200, 1000, 520, 72), "64,64,2,2,4", "64,64,2,2,2"),
          ((200, 1000, 520, 264), "64,64,2,2,4", "64,64,2,2,4"),
          ((8201, 600, 640, 184), "128,64,4,2,4", "128,128,2,4,2"),
          ((4100, 1032, 1024, 264), "64,128,2,4,4", "128,128,2,4,2"),
          ((16001, 584, 600, 256), "128,128,2,4,4", "128,128,2,4,2"),
          ((7999, 1032, 776, 760), "128,256,2,4,3", "128,256,2,4,3"),
          ((16264, 1032, 1032, 1024), "256,256,2,4,2", "128,256,2,4,3"),
          ((64, 8, 16, 8), "64,64,2,2,1", "64,64,2,2,1")]      # less than one of anything


def kernel(tile, b_km=False, epilogue=""):
    return f"gemm2_kernel<{tile},A_KC,{'B_KM' if b_km else 'B_KC'},bf16{epilogue}>"


@pytest.mark.gpu
@pytest.mark.parametrize("shape,first,second", SHAPES)
def test_tiles(shape, first, second):
    T, n_in, n_out, r = shape
    gen = torch.Generator(device="cuda").manual_seed(T + r)

    def normal(*shape, std=1.0):
        return torch.randn(*shape, device="cuda", generator=gen).mul_(std).to(BF)

    def rel(a, b):
        return ((a.float() - b).norm() / b.norm()).item()

    X, dY = normal(T, n_in), normal(T, n_out)
    U, V = normal(n_out, r, std=r ** -0.5), normal(r, n_in, std=n_in ** -0.5)
    Y, H, dX = (torch.full((T, n), float("nan"), device="cuda", dtype=BF) for n in (n_out, r, n_in))
    dU, dV = (torch.full(s, float("nan"), device="cuda") for s in ((n_out, r), (r, n_in)))
    ws = torch.empty(lrd.linear_workspace_bytes(T, n_in, n_out, r, lrd.BF16, 0), dtype=torch.uint8, device="cuda")
    with lrd.ProfileLog(8) as log:
        lrd.linear_fwd(X, V, U, None, Y, H, ws)
        torch.cuda.synchronize()
    assert [row["kernel"] for row in log.rows()] == [kernel(first), kernel(second)]
    lrd.linear_bwd(dY, X, H, V, U, dX, dV, dU, None, 0, ws)
    torch.cuda.synchronize()
    # one rounding to bf16 is at most 2^-9 of a value; dX and dV go through a dH rounded on either side, whose
    # roundings may differ by one step where the fp32 sums do
    dH = (dY.float() @ U.float()).to(BF).float()
    assert rel(H, X.float() @ V.float().t()) < 2e-3
    assert rel(Y, H.float() @ U.float().t()) < 2e-3
    assert rel(dX, dH @ V.float()) < 4e-3
    assert rel(dU, dY.float().t() @ H.float()) < 2e-5
    assert rel(dV, dH.t() @ X.float()) < 2e-3


# Short reductions with the activation in the epilogue, off every edge of their tiles: (tokens, narrow side, wide side, rank)
# and the tile of tokens x wide over rank with GELU, with the gradient of GELU
ACTIVATIONS = [((4100, 1024, 3080, 192), "128,128,2,4,2", "128,128,2,4,1"),
               ((8201, 1032, 4104, 256), "128,128,2,4,2", "128,128,2,4,1"),
               ((12300, 1032, 3080, 264), "128,128,2,4,1", "128,128,2,4,1"),
               ((16200, 2056, 3080, 456), "256,256,2,4,2", "256,256,2,4,2"),
               ((6100, 512, 520, 72), "128,128,2,4,2", "128,128,2,4,2"),
               ((300, 512, 520, 72), "64,64,2,2,2", "64,64,2,2,2")]


@pytest.mark.gpu
@pytest.mark.parametrize("shape,forward,gradient", ACTIVATIONS)
def test_tiles_with_activation(shape, forward, gradient):
    """The fused epilogues against the plain product followed by the elementwise kernels (the same values, bit for bit),
    and the plain product against fp32."""
    T, narrow, wide, r = shape
    gen = torch.Generator(device="cuda").manual_seed(T + r)

    def normal(*shape, std=1.0, dt=BF):
        return torch.randn(*shape, device="cuda", generator=gen).mul_(std).to(dt)

    def nan(*shape):
        return torch.full(shape, float("nan"), device="cuda", dtype=BF)

    def rel(a, b):
        return ((a.float() - b).norm() / b.norm()).item()

    def logged(call, *args):
        with lrd.ProfileLog(4) as log:
            call(*args)
            torch.cuda.synchronize()
        return log.rows()[-1]["kernel"]

    # forward, narrow -> wide, with a bias
    X, bias = normal(T, narrow), normal(wide, std=0.1, dt=torch.float32)
    U, V = normal(wide, r, std=r ** -0.5), normal(r, narrow, std=narrow ** -0.5)
    ws = torch.empty(lrd.linear_workspace_bytes(T, narrow, wide, r, lrd.BF16, 0), dtype=torch.uint8, device="cuda")
    Y, A, H, plain, A2 = nan(T, wide), nan(T, wide), nan(T, r), nan(T, wide), nan(T, wide)
    assert logged(lrd.linear_fwd_act, X, V, U, bias, Y, A, H, lrd.ACT_GELU, ws) == kernel(forward, epilogue=",gelu")
    lrd.linear_fwd(X, V, U, bias, plain, None, ws)
    lrd.gelu_fwd(plain, A2)
    torch.cuda.synchronize()
    # one rounding to bf16 is at most 2^-9 of a value
    assert rel(plain, H.float() @ U.float().t() + bias) < 2e-3
    assert torch.equal(Y, plain) and torch.equal(A, A2)
    # data gradient of a layer wide -> narrow whose input is an activation
    dY, Z = normal(T, narrow), normal(T, wide)
    U, V = normal(narrow, r, std=r ** -0.5), normal(r, wide, std=wide ** -0.5)
    dX, plain, dH, dX2 = nan(T, wide), nan(T, wide), nan(T, r), nan(T, wide)
    assert logged(lrd.linear_bwd_data, dY, V, U, dX, dH, Z, lrd.ACT_GELU, ws) == kernel(gradient, True, ",gelu_grad")
    lrd.linear_bwd_data(dY, V, U, plain, dH, None, lrd.ACT_NONE, ws)
    lrd.gelu_bwd(plain, Z, dX2)
    torch.cuda.synchronize()
    assert rel(plain, dH.float() @ V.float()) < 2e-3
    assert torch.equal(dX, dX2)


# Gathers with many workgroups, off the edges of their tiles: (images, height, width, C, S, k, stride), and the tiles of the
# forward pass and of the data gradient
GATHERS = [((37, 56, 55, 24, 40, 5, 1), "64,64,2,2,2", "128,32,4,1,4"),
           ((37, 79, 79, 40, 56, 3, 2), "64,64,2,2,2", "64,64,2,2,2"),
           ((11, 57, 57, 72, 104, 3, 2), "128,64,4,2,4", "64,64,2,2,2"),
           ((9, 57, 57, 136, 160, 3, 2), "128,64,4,2,4", "64,64,2,2,2"),
           ((20, 50, 50, 40, 72, 5, 3), "64,64,2,2,4", "64,64,2,2,2"),
           ((5, 19, 19, 40, 72, 5, 3), "64,64,2,2,4", "64,64,2,2,4")]


@pytest.mark.gpu
@pytest.mark.parametrize("shape,forward,gradient", GATHERS)
def test_gather_tiles(shape, forward, gradient):
    N, hh, ww, C, S, k, s = shape
    gen = torch.Generator(device="cuda").manual_seed(N + C)

    def normal(*shape, std=1.0):
        return torch.randn(*shape, device="cuda", generator=gen).mul_(std).to(BF)

    geo = lrd.conv_geom(N, hh, ww, C, S, 1, 1, k, s, k // 2)
    ho, wo = geo.out_hw()
    X, W, dY = normal(N, hh, ww, C), normal(S, k, k, C, std=(k * k * C) ** -0.5), normal(N, ho, wo, S)
    Y, dX = (torch.full(t, float("nan"), device="cuda", dtype=BF) for t in ((N, ho, wo, S), (N, hh, ww, C)))
    ws = torch.empty(lrd.dense_conv_workspace_bytes(geo, lrd.BF16) + 16, dtype=torch.uint8, device="cuda")
    with lrd.ProfileLog(4) as log:
        lrd.dense_conv_fwd(X, W, Y, geo, ws)
        lrd.dense_conv_bwd(dY, X, W, dX, None, geo, ws)
        torch.cuda.synchronize()
    # (a data gradient of stride 1 is a forward gather with flipped weights)
    assert [row["kernel"] for row in log.rows()] == [f"gemm2_kernel<{forward},A_KC,B_KC,bf16,conv>",
                                                    f"gemm2_kernel<{gradient},A_KC,{'B_KC' if s == 1 else 'B_KM'},bf16,conv>"]
    # the same sums in fp32, tap by tap
    pad = torch.nn.functional.pad(X.float(), (0, 0, k // 2, k // 2, k // 2, k // 2))
    dpad, want = torch.zeros_like(pad), torch.zeros(N, ho, wo, S, device="cuda")
    for u in range(k):
        for v in range(k):
            at = (slice(None), slice(u, u + (ho - 1) * s + 1, s), slice(v, v + (wo - 1) * s + 1, s))
            want += pad[at] @ W[:, u, v].float().t()
            dpad[at] += dY.float() @ W[:, u, v].float()
    dwant = dpad[:, k // 2:k // 2 + hh, k // 2:k // 2 + ww]
    # one rounding to bf16 is at most 2^-9 of a value
    assert ((Y.float() - want).norm() / want.norm()).item() < 2e-3
    assert ((dX.float() - dwant).norm() / dwant.norm()).item() < 2e-3
