"""Short reductions with a wide result (the kernel that keeps the rows of its left operand in registers): rows, k and column
ranges that end inside a workgroup, every depth, a group's members, bias and the fused activations; against fp32 products of
the same bf16 operands and the elementwise kernels."""
import pytest
import torch

from paper_2309_03824_amd import binding as lrd

BF = torch.bfloat16


class Maker:
    def __init__(self, seed):
        self.gen = torch.Generator(device="cuda").manual_seed(seed)

    def normal(self, *shape, std=1.0, dt=BF):
        return torch.randn(*shape, device="cuda", generator=self.gen).mul_(std).to(dt)


def nan(*shape):
    return torch.full(shape, float("nan"), device="cuda", dtype=BF)


def rel(a, b):
    return ((a.float() - b).norm() / b.norm()).item()


def workspace(T, n_in, n_out, r):
    return torch.empty(lrd.linear_workspace_bytes(T, n_in, n_out, r, lrd.BF16, 0), dtype=torch.uint8, device="cuda")


def logged(call, *args):
    with lrd.ProfileLog(4) as log:
        call(*args)
        torch.cuda.synchronize()
    return log.rows()[-1]["kernel"]


# (tokens, narrow side, wide side, rank) and the depth and waves of the kernel: ranks that end inside 32, 64 and 16-byte
# chunks; tokens that leave a workgroup, a wave and a block of 16 unfilled; column ranges with a last one of fewer chunks
SHAPES = [((7873, 64, 1536, 8), "64,4"), ((5000, 128, 2560, 64), "64,4"), ((6177, 128, 1984, 104), "128,4"),
          ((4100, 192, 3072, 136), "192,4"), ((8191, 256, 1536, 192), "192,4"), ((3001, 256, 4160, 256), "256,4"),
          ((10001, 512, 3264, 264), "320,8"), ((8193, 384, 4096, 376), "384,8"), ((21000, 512, 1600, 424), "448,8"),
          ((8200, 512, 4096, 512), "512,8"),
          # many more columns than rows: dealt to the dies by columns
          ((1000, 256, 12544, 120), "128,4"), ((97, 256, 125056, 160), "192,4"), ((701, 512, 46080, 296), "320,8")]


@pytest.mark.gpu
@pytest.mark.parametrize("shape,depth", SHAPES)
def test_wide_products(shape, depth):
    T, narrow, wide, r = shape
    m = Maker(T + r)
    # forward, narrow -> wide, plain and with GELU, each with a bias
    X, bias = m.normal(T, narrow), m.normal(wide, std=0.1, dt=torch.float32)
    U, V = m.normal(wide, r, std=r ** -0.5), m.normal(r, narrow, std=narrow ** -0.5)
    ws = workspace(T, narrow, wide, r)
    Y, A, H, plain, A2 = nan(T, wide), nan(T, wide), nan(T, r), nan(T, wide), nan(T, wide)
    assert logged(lrd.linear_fwd_act, X, V, U, bias, Y, A, H, lrd.ACT_GELU, ws) == f"wide_kernel<{depth},B_KC,gelu>"
    assert logged(lrd.linear_fwd, X, V, U, bias, plain, None, ws) == f"wide_kernel<{depth},B_KC>"
    lrd.gelu_fwd(plain, A2)
    torch.cuda.synchronize()
    # one rounding to bf16 is at most 2^-9 of a value
    assert rel(plain, H.float() @ U.float().t() + bias) < 2e-3
    assert torch.equal(Y, plain) and torch.equal(A, A2)
    # data gradient, wide -> narrow layer, plain and times the gradient of GELU
    dY, Z = m.normal(T, narrow), m.normal(T, wide)
    U, V = m.normal(narrow, r, std=r ** -0.5), m.normal(r, wide, std=wide ** -0.5)
    dX, plain, dH, dX2 = nan(T, wide), nan(T, wide), nan(T, r), nan(T, wide)
    assert logged(lrd.linear_bwd_data, dY, V, U, dX, dH, Z, lrd.ACT_GELU, ws) == f"wide_kernel<{depth},B_KM,gelu_grad>"
    assert logged(lrd.linear_bwd_data, dY, V, U, plain, dH, None, lrd.ACT_NONE, ws) == f"wide_kernel<{depth},B_KM>"
    lrd.gelu_bwd(plain, Z, dX2)
    torch.cuda.synchronize()
    assert rel(plain, dH.float() @ V.float()) < 2e-3
    assert torch.equal(dX, dX2)


# Wide results that are faster in tiles: most of the last row block would be empty, or a very short reduction
@pytest.mark.gpu
@pytest.mark.parametrize("T,wide,r,act", [(48, 262144, 64, False), (130, 100032, 192, False), (300, 128256, 320, False), (1100, 24064, 64, False),
                                          (1024, 24064, 128, False), (1100, 24064, 128, True)])
def test_not_wide(T, wide, r, act):
    m = Maker(T + r)
    X, U, V = m.normal(T, r), m.normal(wide, r, std=r ** -0.5), m.normal(r, r, std=r ** -0.5)
    ws, H, Y, A = workspace(T, r, wide, r), nan(T, r), nan(T, wide), nan(T, wide) if act else None
    args = (X, V, U, None, Y, A, H, lrd.ACT_GELU, ws) if act else (X, V, U, None, Y, H, ws)
    assert logged(lrd.linear_fwd_act if act else lrd.linear_fwd, *args).startswith("gemm2_kernel")
    assert rel(Y, H.float() @ U.float().t()) < 2e-3


@pytest.mark.gpu
def test_members_of_a_group():
    """Each member reads its columns of the stacked intermediate (a row pitch of three ranks) and its own factor and bias."""
    T, n_in, n_out, r, G = 2500, 256, 1664, 184, 3
    m = Maker(5)
    X, V, U = m.normal(T, n_in), m.normal(G * r, n_in, std=n_in ** -0.5), m.normal(G, n_out, r, std=r ** -0.5)
    bias = m.normal(G, n_out, std=0.1, dt=torch.float32)
    Y, H = nan(G, T, n_out), nan(T, G * r)
    ws = torch.empty(lrd.linear_group_workspace_bytes(T, n_in, n_out, r, G, lrd.BF16, 0), dtype=torch.uint8, device="cuda")
    assert logged(lrd.linear_group_fwd, X, V, U, bias, Y, H, ws) == "wide_kernel<192,4,B_KC>"
    for i in range(G):
        assert rel(Y[i], H[:, i * r:(i + 1) * r].float() @ U[i].float().t() + bias[i]) < 2e-3
