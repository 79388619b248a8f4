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
