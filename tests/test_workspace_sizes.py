"""A workspace for the largest batch serves every smaller one: the size queries never fall as tokens or images grow, and
the calls run in it, to the same results as in a workspace of their own."""
import pytest
import torch

from paper_2309_03824_amd import binding as lrd

SHAPES = [(768, 3072, 192), (3072, 768, 192), (1024, 4096, 256), (4096, 4096, 512), (8192, 8192, 2048), (4096, 4096, 16), (1000, 1024, 257),
          (512, 512, 64), (2048, 2048, 33), (64, 64, 8), (4096, 512, 100)]


def rising(query, counts):
    sizes = [query(n) for n in counts]
    return all(a <= b for a, b in zip(sizes, sizes[1:]))


@pytest.mark.parametrize("dt", [lrd.BF16, lrd.F32])
@pytest.mark.parametrize("n_in,n_out,r", SHAPES)
def test_linear_queries_never_fall(n_in, n_out, r, dt):
    tokens = list(range(1, 1400)) + list(range(1400, 18000, 37))
    assert rising(lambda T: lrd.linear_workspace_bytes(T, n_in, n_out, r, dt, 0), tokens)
    assert rising(lambda T: lrd.linear_sgd_workspace_bytes(T, n_in, n_out, r, dt, 1), tokens)
    assert rising(lambda T: lrd.linear_group_workspace_bytes(T, n_in, n_out, r, 3, dt, 0), tokens)
    assert rising(lambda T: lrd.dense_linear_workspace_bytes(T, n_in, n_out, dt), tokens)
    for layers in (1, 2, 5, 12):
        assert rising(lambda T: lrd.linear_wgrad_batched_workspace_bytes(layers, T, n_in, n_out, r, dt, 0), tokens)


@pytest.mark.parametrize("dt", [lrd.BF16, lrd.F32])
@pytest.mark.parametrize("hw,C,S,r1,r2,stride", [(56, 64, 64, 32, 32, 1), (14, 256, 256, 128, 128, 1), (10, 64, 32, 29, 32, 1), (7, 512, 512, 309, 309, 1),
                                                 (28, 128, 256, 64, 128, 2), (9, 40, 24, 17, 9, 1)])
def test_convolution_queries_never_fall(hw, C, S, r1, r2, stride, dt):
    images = range(1, 300)
    assert rising(lambda N: lrd.tucker_conv_workspace_bytes(lrd.conv_geom(N, hw, hw, C, S, r1, r2, 3, stride, 1), dt, 0), images)
    assert rising(lambda N: lrd.dense_conv_workspace_bytes(lrd.conv_geom(N, hw, hw, C, S, r1, r2, 3, stride, 1), dt), images)


@pytest.mark.parametrize("n_in,n_out,r", SHAPES)
def test_linear_queries_ask_for_a_second_set_of_slices_only_where_two_gradients_use_it(n_in, n_out, r):
    def query(T, dt, mask):
        return lrd.linear_workspace_bytes(T, n_in, n_out, r, dt, mask)

    for T in (100, 511, 513, 4100, 16384):
        # fp32 sums at once; a frozen factor has no slices
        assert len({query(T, lrd.F32, mask) for mask in range(4)}) == 1
        assert len({query(T, lrd.BF16, mask) for mask in (1, 2, 3)}) == 1
        extra = query(T, lrd.BF16, 0) - query(T, lrd.BF16, 3)
        rank = r if r % 8 == 0 else (r + 7) // 8 * 8
        assert extra % (rank * n_in * 4) < 256 and (extra == 0 or T >= 512), (T, extra)
        assert extra > 0 or T < 512 or n_out * r > 4 << 20, T      # (the largest gradients are never cut)
        for mask in range(4):
            sgd = lrd.linear_sgd_workspace_bytes(T, n_in, n_out, r, lrd.BF16, mask)
            assert sgd - query(T, lrd.BF16, mask) == sgd_extra(n_in, n_out, r)


def sgd_extra(n_in, n_out, r):
    return sum((n * 4 + 255) // 256 * 256 for n in (n_out * r, r * n_in))


def test_convolution_queries_ask_for_slices_of_their_own_only_where_they_are_summed_together():
    geo = lrd.conv_geom(128, 14, 14, 256, 256, 128, 128, 3, 1, 1)

    def query(mask, dt=lrd.BF16):
        return lrd.tucker_conv_workspace_bytes(geo, dt, mask)

    assert len({query(mask, lrd.F32) for mask in range(8)}) == 1
    alone = query(7)
    assert query(5) == query(6) == query(3) == alone        # one layer trained
    first, last = query(4) - alone, query(1) - alone        # with the core
    assert first > 0 and last > 0 and query(0) - alone == first + last
    assert query(2) - alone == first                        # the 1x1 layers: one of them has the shared region


@pytest.mark.parametrize("n_in,n_out,r", SHAPES)
def test_a_query_within_the_static_scratch_fits_it(n_in, n_out, r):
    for T in range(1, 9000, 61):
        need = lrd.linear_workspace_bytes(T, n_in, n_out, r, lrd.BF16, 0)
        assert lrd.linear_bwd_static_fits(T, n_in, n_out, r, lrd.BF16, 0) or need > lrd.STATIC_SCRATCH_BYTES


@pytest.mark.gpu
@pytest.mark.parametrize("n_in,n_out,r,most,tokens", [(1024, 4096, 256, 4096, (4032, 1500, 64)), (4096, 4096, 512, 2048, (1984, 300)),
                                                      (768, 3072, 192, 8192, (8000, 200)), (1000, 1024, 257, 700, (640, 65))])
def test_smaller_batches_run_in_the_largest_one_s_workspace(n_in, n_out, r, most, tokens):
    gen = torch.Generator(device="cuda").manual_seed(most)
    bf = torch.bfloat16

    def normal(*shape, std=1.0):
        return torch.randn(*shape, device="cuda", generator=gen).mul_(std).to(bf)

    U, V = normal(n_out, r, std=r ** -0.5), normal(r, n_in, std=n_in ** -0.5)

    def step(T, X, dY, ws):
        Y, dX = torch.empty(T, n_out, device="cuda", dtype=bf), torch.empty(T, n_in, device="cuda", dtype=bf)
        dV, dU = torch.empty(r, n_in, device="cuda"), torch.empty(n_out, r, device="cuda")
        lrd.linear_fwd(X, V, U, None, Y, None, ws)
        lrd.linear_bwd(dY, X, None, V, U, dX, dV, dU, None, 0, ws)
        torch.cuda.synchronize()
        return Y, dX, dV, dU

    shared = torch.empty(lrd.linear_workspace_bytes(most, n_in, n_out, r, lrd.BF16, 0), dtype=torch.uint8, device="cuda")
    for T in tokens:
        X, dY = normal(T, n_in), normal(T, n_out)
        own = torch.empty(lrd.linear_workspace_bytes(T, n_in, n_out, r, lrd.BF16, 0), dtype=torch.uint8, device="cuda")
        for a, b in zip(step(T, X, dY, shared), step(T, X, dY, own)):
            assert torch.equal(a, b)
