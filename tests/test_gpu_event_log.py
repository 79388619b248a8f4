"""The event log of a backward pass: sums that are put off have a record of their own, two products of one launch have their time
once, so that the logged times add up to no more than the pass takes."""
import pytest
import torch

import bench
from paper_2309_03824_amd import binding as lrd

pytestmark = pytest.mark.gpu
BF = torch.bfloat16


def logged_backward(T, n_in, n_out, r):
    def normal(*shape, std=1.0):
        return torch.randn(*shape, device="cuda").mul_(std).to(BF)

    X, dY, U, V = normal(T, n_in), normal(T, n_out), normal(n_out, r, std=r ** -0.5), normal(r, n_in, std=n_in ** -0.5)
    H, dX = torch.empty(T, r, device="cuda", dtype=BF), torch.empty(T, n_in, device="cuda", dtype=BF)
    dU, dV, db = torch.empty(n_out, r, device="cuda"), torch.empty(r, n_in, device="cuda"), torch.empty(n_out, device="cuda")
    ws = torch.empty(lrd.linear_workspace_bytes(T, n_in, n_out, r, lrd.BF16, 0), dtype=torch.uint8, device="cuda")
    lrd.linear_fwd(X, V, U, None, torch.empty(T, n_out, device="cuda", dtype=BF), H, ws)
    lrd.linear_bwd(dY, X, H, V, U, dX, dV, dU, db, 0, ws)
    torch.cuda.synchronize()
    start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    with lrd.ProfileLog(16) as log:
        start.record()
        lrd.linear_bwd(dY, X, H, V, U, dX, dV, dU, db, 0, ws)
        end.record()
        torch.cuda.synchronize()
    return log.rows(), start.elapsed_time(end) * 1e3


def test_sums_that_are_put_off_have_a_record():
    T, n_in, n_out, r = 4100, 1024, 2048, 264
    rows, total = logged_backward(T, n_in, n_out, r)
    assert [row["role"] for row in rows] == [lrd.ROLE_DGRAD_UP, lrd.ROLE_DGRAD_DOWN, lrd.ROLE_WGRAD_U, lrd.ROLE_WGRAD_V, lrd.ROLE_SUMS]
    assert not any(row["shared"] for row in rows)
    sums = rows[-1]
    assert sums["kernel"] == "sums_kernel" and sums["us"] > 0
    # the gradients of both factors and of the bias
    assert sums["batch"] == 3 and sums["M"] == n_out * r + r * n_in + n_out
    assert sums["splits"] >= max(row["splits"] for row in rows[2:4]) > 1
    assert sum(row["us"] for row in rows) <= total
    roof, by_kernel = bench.kernel_roofline(rows)
    assert roof["kernel"] != "sums_kernel" and by_kernel["sums_kernel"]["total_us"] == sums["us"]
    assert sum(k["total_us"] for k in by_kernel.values()) == pytest.approx(sum(row["us"] for row in rows))


def test_products_of_one_launch_have_its_time_once():
    rows, total = logged_backward(600, 2048, 2048, 512)
    assert [(row["role"], row["shared"]) for row in rows] == [(lrd.ROLE_DGRAD_UP, False), (lrd.ROLE_WGRAD_U, True), (lrd.ROLE_DGRAD_DOWN, False),
                                                              (lrd.ROLE_WGRAD_V, True)]
    assert [row["splits"] for row in rows] == [2, 2, 1, 2]      # (chains of additions, in the same kernel)
    once = sum(row["us"] for row in rows if not row["shared"])
    assert once <= total
    roof, by_kernel = bench.kernel_roofline(rows)
    assert sum(k["total_us"] for k in by_kernel.values()) == pytest.approx(once) and sum(k["launches"] for k in by_kernel.values()) == 2
