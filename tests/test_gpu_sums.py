"""The sums over K-slices that a backward pass puts off to one launch, against the same sums in launches of their own: the dense
gradients of the same operands, the bias gradient of a pass without others, and the smallest workspace that a call accepts, which
has no room to keep the partial sums apart.  The same bits either way."""
import pytest
import torch
from test_gpu_wgrad_error import bound

from paper_2309_03824_amd import binding as lrd

BF = torch.bfloat16
pytestmark = pytest.mark.gpu


def smallest(call, most):
    """The fewest bytes of workspace, in steps of 256, with which call(workspace) is accepted."""
    low, high = 0, most // 256
    while low < high:
        mid = (low + high) // 2
        try:
            call(torch.empty(mid * 256 + 256, dtype=torch.uint8, device="cuda")[:mid * 256])
            high = mid
        except lrd.LrdError:
            low = mid + 1
    torch.cuda.synchronize()
    return low * 256


def compare(call, outputs, most, sums):
    """call(workspace) in `most` bytes and in the fewest gives `outputs` the same bits, with sums[0] and sums[1] of them put off."""
    least = smallest(call, most)
    assert least < most
    results, put_off = [], []
    for n in (most, least):
        for t in outputs:
            t.fill_(float("nan"))
        with lrd.ProfileLog(16) as log:
            call(torch.empty(n + 256, dtype=torch.uint8, device="cuda")[:n])
            torch.cuda.synchronize()
        results.append([t.clone() for t in outputs])
        put_off.append(sum(row["batch"] for row in log.rows() if row["role"] == lrd.ROLE_SUMS))
    assert all(torch.equal(a, b) and not a.isnan().any() for a, b in zip(*results))
    assert tuple(put_off) == sums


def normals(seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    return lambda *shape, std=1.0: torch.randn(*shape, device="cuda", generator=gen).mul_(std).to(BF)


def dense_gradient(dY, X):
    """dY^T X in the same slices, their sum a launch of its own; against 64 bits within the error of its chains."""
    T, M, N = *dY.shape, X.shape[1]
    dW = torch.full((M, N), float("nan"), device="cuda")
    ws = torch.empty(max(lrd.dense_linear_workspace_bytes(T, N, M, lrd.BF16), 256), dtype=torch.uint8, device="cuda")
    with lrd.ProfileLog(4) as log:
        lrd.dense_linear_bwd(dY, X, torch.empty(M, N, device="cuda", dtype=BF), None, dW, ws)
        torch.cuda.synchronize()
    row, = log.rows()
    assert row["splits"] > 1
    ref = dY.double().t().contiguous() @ X.double()
    assert ((dW - ref).norm() / ref.norm()).item() <= bound(T, row["splits"])
    return dW


# tokens, in, out, rank, and the sums put off in the largest and in the smallest workspace: of one lane a group (large gradients), of 16
# (small ones over many slices), cropped (a raw rank), and fewer rows than the partial rows of the bias gradient need (wide, rank 16)
@pytest.mark.parametrize("T,n_in,n_out,r,sums", [(4100, 1024, 2048, 264, (3, 2)), (20000, 64, 128, 32, (3, 2)), (3000, 520, 1032, 101, (3, 2)),
                                                 (2100, 256, 4096, 16, (2, 1))])
def test_linear_sums(T, n_in, n_out, r, sums):
    normal = normals(T)
    X, dY, U, V = normal(T, n_in), normal(T, n_out), normal(n_out, r, std=r ** -0.5), normal(r, n_in, std=n_in ** -0.5)
    H, dX = torch.empty(T, r, device="cuda", dtype=BF), torch.empty(T, n_in, device="cuda", dtype=BF)
    dU, dV, db = torch.empty(n_out, r, device="cuda"), torch.empty(r, n_in, device="cuda"), torch.empty(n_out, device="cuda")
    most = lrd.linear_workspace_bytes(T, n_in, n_out, r, lrd.BF16, 0)
    ws = torch.empty(most, dtype=torch.uint8, device="cuda")
    lrd.linear_fwd(X, V, U, None, torch.empty(T, n_out, device="cuda", dtype=BF), H, ws)
    compare(lambda ws: lrd.linear_bwd(dY, X, H, V, U, dX, dV, dU, db, 0, ws), [dX, dU, dV, db], most, sums)
    # a raw rank is computed with zeros up to a multiple of 8
    more = -r % 8
    U, V, H = torch.nn.functional.pad(U, (0, more)), torch.nn.functional.pad(V, (0, 0, 0, more)), torch.nn.functional.pad(H, (0, more))
    dH = torch.empty_like(H)
    lrd.linear_bwd_data(dY, V, U, dX, dH, None, lrd.ACT_NONE, ws)
    assert torch.equal(dV, dense_gradient(dH, X)[:r]) and torch.equal(dU, dense_gradient(dY, H)[:, :r])
    alone = torch.full_like(db, float("nan"))
    with lrd.ProfileLog(4) as log:
        lrd.linear_bwd(dY, None, None, V, U, dX, None, None, alone, 3, ws)
        torch.cuda.synchronize()
    assert lrd.ROLE_SUMS not in [row["role"] for row in log.rows()]
    assert torch.equal(db, alone)
    assert ((db.double() - dY.double().sum(0)).norm() / dY.double().sum(0).norm()).item() < 1e-6


# (the gradients of both 1x1 layers and of the core; the direct kernels of a 32-channel core sum by themselves)
@pytest.mark.parametrize("N,hw,C,S,r1,r2,k,sums", [(40, 28, 64, 64, 32, 32, 3, (2, 0)), (30, 14, 96, 136, 45, 72, 3, (3, 0)),
                                                   (64, 7, 256, 256, 128, 128, 3, (3, 0))])
def test_convolution_sums(N, hw, C, S, r1, r2, k, sums):
    normal = normals(N)
    geo = lrd.conv_geom(N, hw, hw, C, S, r1, r2, k, 1, k // 2)
    X, dY, A, B = normal(N, hw, hw, C), normal(N, hw, hw, S), normal(N, hw, hw, r1), normal(N, hw, hw, r2)
    P1, G, P2 = normal(r1, C, std=C ** -0.5), normal(r2, k, k, r1, std=(k * k * r1) ** -0.5), normal(S, r2, std=r2 ** -0.5)
    dX = torch.empty(N, hw, hw, C, device="cuda", dtype=BF)
    dP1, dG, dP2 = (torch.empty(*s, device="cuda") for s in ((r1, C), (r2, k, k, r1), (S, r2)))
    compare(lambda ws: lrd.tucker_conv_bwd(dY, X, A, B, P1, G, P2, dX, dP1, dG, dP2, 0, geo, ws), [dX, dP1, dG, dP2],
            lrd.tucker_conv_workspace_bytes(geo, lrd.BF16, 0), sums)
