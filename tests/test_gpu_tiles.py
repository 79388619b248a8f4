"""The output tiles of the MFMA product kernel, each at sizes off its edges: rows, columns and K that end inside a tile, a
load and a K-step; against fp32 products of the same bf16 operands."""
import pytest
import torch

from paper_2309_03824_amd import binding as lrd

BF = torch.bfloat16

# (tokens, in, out, rank): the tile that the first product, tokens x rank over in, is given
SHAPES = [(200, 1000, 520, 72),        # 64 x 64
          (200, 1000, 520, 264),       # 64 x 64, second product of more than 256
          (8201, 600, 640, 184),       # 128 x 64
          (4100, 1032, 1024, 264),     # 64 x 128
          (16001, 584, 600, 256),      # 128 x 128
          (7999, 1032, 776, 760),      # 128 x 256
          (16264, 1032, 1032, 1024),   # 256 x 256
          (64, 8, 16, 8)]              # less than one of anything


@pytest.mark.gpu
@pytest.mark.parametrize("T,n_in,n_out,r", SHAPES)
def test_tiles(T, n_in, n_out, r):
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
    lrd.linear_fwd(X, V, U, None, Y, H, ws)
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
