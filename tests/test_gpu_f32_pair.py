"""fp32 layers whose data gradient and weight gradient share a launch: each has the bits that it has alone, in every form of the launch
(blocks of 16 x 16 or 32 x 32 for either), at extents off the blocks and reductions off the steps of 16."""
import pytest
import torch

from paper_2309_03824_amd import binding as lrd

pytestmark = pytest.mark.gpu


# tokens, in, out, rank, and the blocks of dH and dU, and of dX and dV; None: gradients that would run on after everything else, alone
@pytest.mark.parametrize("T,n_in,n_out,r,up,down", [(33, 47, 65, 17, "1,1", "1,1"), (1001, 259, 130, 103, "2,1", "2,1"), (100, 700, 520, 301, "1,2", "1,2"),
                                                    (500, 401, 530, 303, "2,2", "2,2"), (500, 1000, 384, 150, "1,1", None), (1700, 770, 770, 209, None, None), (2, 35, 34, 2, "1,1", "1,1"), (256, 768, 768, 208, "1,2", "2,2")])
@pytest.mark.parametrize("act", [False, True])
def test_products_of_a_pair_have_the_bits_of_each_alone(T, n_in, n_out, r, up, down, act):
    gen = torch.Generator(device="cuda").manual_seed(T + r)
    X, dY, U, V, Z, H = (torch.randn(*s, device="cuda", generator=gen) for s in ((T, n_in), (T, n_out), (n_out, r), (r, n_in), (T, n_in), (T, r)))
    ws = torch.empty(lrd.linear_workspace_bytes(T, n_in, n_out, r, lrd.F32, 0), dtype=torch.uint8, device="cuda")
    ref = {}
    for mask in (3, 2, 1, 0):
        dX, dU, dV = (torch.full(s, float("nan"), device="cuda") for s in ((T, n_in), (n_out, r), (r, n_in)))
        with lrd.ProfileLog(16) as log:
            lrd.linear_bwd_act(dY, X, H, V, U, dX, None if mask & 1 else dV, None if mask & 2 else dU, None, mask, Z if act else None,
                               lrd.ACT_GELU if act else lrd.ACT_NONE, ws)
            torch.cuda.synchronize()
        kernels = [row["kernel"] for row in log.rows()]
        alone = ["f32_gemm_kernel"]
        pair1, pair2 = up and not mask & 2, down and not mask & 1
        want = ([f"f32_pair_kernel<{up}>"] * 2 if pair1 else alone) + ([f"f32_pair_kernel<{down}>"] * 2 if pair2 else alone)
        want += alone * ((not mask & 2 and not pair1) + (not mask & 1 and not pair2))
        assert kernels == want, mask
        for name, t, there in (("dX", dX, True), ("dU", dU, not mask & 2), ("dV", dV, not mask & 1)):
            assert torch.equal(t, ref.setdefault(name, t)) and not t.isnan().any() if there else t.isnan().all(), (name, mask)
    # dU alone: rows and columns of a dense layer's gradient; dV alone, of the dH that dX has gone through
    dH = torch.empty(T, r, device="cuda")
    lrd.linear_bwd_data(dY, V, U, dX, dH, None, lrd.ACT_NONE, ws)
    for name, rows, cols in (("dU", dY, H), ("dV", dH, X)):
        got = torch.full((rows.shape[1], cols.shape[1]), float("nan"), device="cuda")
        dense = torch.empty(max(lrd.dense_linear_workspace_bytes(T, cols.shape[1], rows.shape[1], lrd.F32), 256), dtype=torch.uint8, device="cuda")
        with lrd.ProfileLog(4) as log:
            lrd.dense_linear_bwd(rows, cols, torch.empty_like(got), None, got, dense)
            torch.cuda.synchronize()
        assert [row["kernel"] for row in log.rows()] == ["f32_gemm_kernel"]
        assert torch.equal(got, ref[name]), name
        # K products of 24 bits, summed in any order
        bound = T * 2.0 ** -24 * (rows.abs().double().t() @ cols.abs().double()) + 1e-30
        assert ((got.double() - rows.double().t() @ cols.double()).abs() <= bound).all()
