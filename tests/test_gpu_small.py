"""Layers with few tokens: the kernels that take whole reductions on their way at once and share launches in the backward pass, at
rows, columns and k that end inside a block, a step and a group of steps; against fp32 products of the same bf16 operands."""
import pytest
import torch
from test_gpu_wgrad_error import bound

from paper_2309_03824_amd import binding as lrd

BF, F32 = torch.bfloat16, torch.float32

# (tokens, in, out, rank) and the columns of a block where these kernels run the products H, Y, dH, dX by themselves, and the launches
# of dH with dU and of dX with dV; "-": output tiles
SHAPES = [((1, 64, 96, 32), "- - 32 - 32 32"), ((7, 1024, 160, 64), "32 - 32 - 32 32"), ((33, 96, 1056, 96), "32 32 32 32 32 32"),
          ((48, 1024, 4096, 256), "32 32 - 32 - 32"), ((100, 2080, 544, 160), "- 32 32 64 32 64"), ((509, 768, 3072, 192), "32 - - 64 32 64"),
          ((509, 544, 512, 256), "32 32 32 64 32 64"), ((1000, 512, 480, 128), "32 64 - - 32 64"), ((1024, 1536, 256, 96), "32 32 - - 32 128"),
          ((300, 208, 336, 48), "32 - 32 - 32 32"), ((130, 1040, 1136, 144), "32 32 32 32 32 32"), ((700, 4096, 1024, 256), "- - - - 32 128"),
          ((600, 2048, 2048, 512), "- - - - 64 128"), ((40, 96, 4160, 32), "32 - - - - 32")]


def rel(a, b):
    return ((a.float() - b).norm() / b.norm()).item()


def inputs(T, n_in, n_out, r):
    gen = torch.Generator(device="cuda").manual_seed(T + n_in + r)

    def normal(*shape, std=1.0, dt=BF):
        return torch.randn(*shape, device="cuda", generator=gen).mul_(std).to(dt)

    return (normal(T, n_in), normal(T, n_out), normal(n_out, r, std=r ** -0.5), normal(r, n_in, std=n_in ** -0.5), normal(n_out, std=0.1, dt=F32),
            normal(T, n_in))


def nan(*shape, dt=BF):
    return torch.full(shape, float("nan"), device="cuda", dtype=dt)


@pytest.mark.gpu
@pytest.mark.parametrize("shape,blocks", SHAPES)
@pytest.mark.parametrize("with_h,with_dx,act", [(True, True, False), (False, True, True), (True, False, False)])
def test_small_layers(shape, blocks, with_h, with_dx, act):
    T, n_in, n_out, r = shape
    X, dY, U, V, bias, Z = inputs(*shape)
    Y, H, dX = nan(T, n_out), nan(T, r), nan(T, n_in)
    dU, dV, db = nan(n_out, r, dt=F32), nan(r, n_in, dt=F32), nan(n_out, dt=F32)
    ws = torch.empty(lrd.linear_workspace_bytes(T, n_in, n_out, r, lrd.BF16, 0), dtype=torch.uint8, device="cuda")
    with lrd.ProfileLog(16) as log:
        lrd.linear_fwd(X, V, U, bias, Y, H, ws)
        lrd.linear_bwd_act(dY, X, H if with_h else None, V, U, dX if with_dx else None, dV, dU, db, 0, Z if act else None,
                           lrd.ACT_GELU if act else lrd.ACT_NONE, ws)
        torch.cuda.synchronize()
    names = [row["kernel"] for row in log.rows() if row["role"] != lrd.ROLE_SUMS]
    h, y, dh, dx, dh_du, dx_dv = (None if b == "-" else b for b in blocks.split())
    recomputed = [] if with_h else [("fwd", h)]
    want = [("fwd", h), ("fwd", y)]
    want += recomputed + [("bwd", dh_du)] * 2 if dh_du else [("bwd", dh)]
    want += [("bwd", dx_dv)] * 2 if with_dx else []
    want += [] if dh_du else recomputed + [("bwd", None)]
    want += [] if with_dx else [("bwd", None)]
    assert len(names) == len(want) and all(n == f"small_{kind}_kernel<{b}>" if b else n.startswith("gemm2") or T < 8 for n, (kind, b) in zip(names, want)), names
    # one rounding to bf16 is at most 2^-9 of a value; dX and dV go through a dH rounded on either side, whose roundings may
    # differ by one step where the fp32 sums do; the gradient of GELU rounds dX once more (and is off by 2.6e-4 itself)
    dH = (dY.float() @ U.float()).to(BF).float()
    assert rel(H, X.float() @ V.float().t()) < 2e-3
    assert rel(Y, H.float() @ U.float().t() + bias) < 2e-3
    if with_dx:
        z = Z.float().requires_grad_()
        slope = torch.autograd.grad(torch.nn.functional.gelu(z).sum(), z)[0] if act else 1.0
        assert rel(dX, (dH @ V.float()) * slope) < (7e-3 if act else 4e-3)
    assert rel(dU, dY.float().t() @ H.float()) < 2e-5
    assert rel(dV, dH.t() @ X.float()) < 2e-3
    assert rel(db, dY.double().sum(0)) < 1e-6


@pytest.mark.gpu
def test_small_frozen_factors_and_no_bias():
    """Jobs that are absent from a launch: each mask gives the same bits for what it computes, and leaves the rest alone."""
    T, n_in, n_out, r = 200, 512, 768, 128
    X, dY, U, V, bias, _ = inputs(T, n_in, n_out, r)
    ws = torch.empty(lrd.linear_workspace_bytes(T, n_in, n_out, r, lrd.BF16, 0), dtype=torch.uint8, device="cuda")
    Y, H = nan(T, n_out), nan(T, r)
    lrd.linear_fwd(X, V, U, bias, Y, H, ws)
    full = None
    for mask in range(4):
        for with_dx, with_bias in ((True, True), (True, False), (False, False)):
            dX, dU, dV, db = nan(T, n_in), nan(n_out, r, dt=F32), nan(r, n_in, dt=F32), nan(n_out, dt=F32)
            lrd.linear_bwd(dY, X, H, V, U, dX if with_dx else None, None if mask & 1 else dV, None if mask & 2 else dU, db if with_bias else None, mask, ws)
            torch.cuda.synchronize()
            full = full or (dX, dU, dV, db)
            for got, ref, there in zip((dX, dU, dV, db), full, (with_dx, not mask & 2, not mask & 1, with_bias)):
                assert torch.equal(got, ref) if there else got.isnan().all()


# Layers on which the launches of a call depend on what it wants: a factor's gradient, dX, an optimizer step, the data gradient alone
WANTED = [(1024, 3072, 3072, 384), (600, 2048, 2048, 512), (512, 4096, 4096, 512), (768, 1536, 3072, 512), (509, 768, 3072, 192), (48, 1024, 4096, 256),
          (40, 96, 4160, 32), (900, 512, 768, 176), (2, 80, 112, 48), (500, 768, 1024, 104), (500, 768, 1024, 101)]


@pytest.mark.gpu
@pytest.mark.parametrize("shape", WANTED)
def test_results_do_not_depend_on_what_else_is_wanted(shape):
    """The same bits from every freeze mask, with and without dX, from lrd_linear_bwd_sgd (learning rate and decay zero: the momentum
    buffer receives the gradient) and from lrd_linear_bwd_data (ranks that are padded aside)."""
    T, n_in, n_out, r = shape
    X, dY, U, V, bias, _ = inputs(*shape)
    ws = torch.empty(max(f(T, n_in, n_out, r, lrd.BF16, 0) for f in (lrd.linear_workspace_bytes, lrd.linear_sgd_workspace_bytes)), dtype=torch.uint8,
                     device="cuda")
    H, Y = nan(T, r), nan(T, n_out)
    lrd.linear_fwd(X, V, U, bias, Y, H, ws)
    ref, dX, dH = {}, nan(T, n_in), nan(T, r)

    def same(**got):
        torch.cuda.synchronize()
        for name, t in got.items():
            assert t is None or torch.equal(t, ref.setdefault(name, t.clone())) and not t.isnan().any(), name

    for mask in range(4):
        tv, tu = not mask & 1, not mask & 2
        for with_dx in (True, False):
            dX, dU, dV, db = nan(T, n_in) if with_dx else None, nan(n_out, r, dt=F32) if tu else None, nan(r, n_in, dt=F32) if tv else None, nan(n_out, dt=F32)
            lrd.linear_bwd(dY, X, H, V, U, dX, dV, dU, db, mask, ws)
            same(dX=dX, dU=dU, dV=dV, db=db if with_dx else None)      # (its runs of rows follow the workspace that a call needs)
        dX, masters = nan(T, n_in), [U.float() if tu else None, V.float() if tv else None]
        momenta = [torch.zeros_like(m) if m is not None else None for m in masters]
        lrd.linear_bwd_sgd(dY, X, H, V.clone(), U.clone(), dX, masters[1], masters[0], momenta[1], momenta[0], None, mask, None, lrd.ACT_NONE,
                           lrd.Sgd(0.0, 0.9, 0.0), ws)
        same(dX=dX, dU=momenta[0], dV=momenta[1])
    if r % 8 == 0:
        dX = nan(T, n_in)
        lrd.linear_bwd_data(dY, V, U, dX, dH, None, lrd.ACT_NONE, ws)
        same(dX=dX)


@pytest.mark.gpu
@pytest.mark.parametrize("n_in,n_out,r", [(768, 1024, 192), (1472, 512, 64), (320, 1456, 240)])
def test_few_tokens_are_rows_of_many(n_in, n_out, r):
    """Unsliced products, whose rows are the same chains in these kernels and in the output tiles that more tokens go to."""
    X, dY, U, V, bias, Z = inputs(1100, n_in, n_out, r)
    results = []
    for T in (1100, 1024, 300, 33):
        ws = torch.empty(lrd.linear_workspace_bytes(T, n_in, n_out, r, lrd.BF16, 0), dtype=torch.uint8, device="cuda")
        Y, A, H, dH, dX = nan(T, n_out), nan(T, n_out), nan(T, r), nan(T, r), nan(T, n_in)
        with lrd.ProfileLog(8) as log:
            lrd.linear_fwd_act(X[:T], V, U, bias, Y, A, H, lrd.ACT_GELU, ws)
            lrd.linear_bwd_data(dY[:T], V, U, dX, dH, Z[:T], lrd.ACT_GELU, ws)
            torch.cuda.synchronize()
        assert any(row["kernel"].startswith("small") for row in log.rows()) == (T <= 1024)
        results.append((Y, A, H, dH, dX))
        assert all(torch.equal(full[:T], part) for full, part in zip(results[0], results[-1]))


@pytest.mark.gpu
@pytest.mark.parametrize("T", [1, 300, 1024])
def test_small_weight_gradients_are_as_exact_as_their_chains(T):
    """A chain of additions for each slice of the rows, of at least 256 rows for a result this small."""
    n_in, n_out, r = 256, 320, 64
    X, dY, U, V, bias, _ = inputs(T, n_in, n_out, r)
    ws = torch.empty(lrd.linear_workspace_bytes(T, n_in, n_out, r, lrd.BF16, 0), dtype=torch.uint8, device="cuda")
    Y, H, dX = nan(T, n_out), nan(T, r), nan(T, n_in)
    dU, dV = nan(n_out, r, dt=F32), nan(r, n_in, dt=F32)
    lrd.linear_fwd(X, V, U, bias, Y, H, ws)
    lrd.linear_bwd(dY, X, H, V, U, dX, dV, dU, None, 0, ws)
    torch.cuda.synchronize()
    assert ((dU.double() - (ref := dY.double().t() @ H.double())).norm() / ref.norm()).item() <= bound(T, max(1, T // 256))
