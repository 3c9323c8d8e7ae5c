"""Every tile shape of the block product (fd_block_gemm_f64) at the edges of its tiles and
K stages, against the FP64 oracle: small integer operands, exact in any order of
summation, so the products are equal bit for bit."""
import numpy as np
import pytest
import torch

import oracle as ora

pytestmark = pytest.mark.gpu

api = pytest.importorskip("paper_2506_02486_amd.api")


def _check(m, n, k, accumulate, pad=(3, 5, 2)):
    rng = np.random.default_rng(m + 7 * n + 31 * k)
    A = rng.integers(-9, 10, (m, k)).astype(np.float64)
    B = rng.integers(-9, 10, (k, n)).astype(np.float64)
    C0 = rng.integers(-99, 100, (m, n)).astype(np.float64)
    dev = []
    for x, extra in zip((A, B, C0), pad):  # leading dimensions wider than the rows
        t = torch.full((x.shape[0], x.shape[1] + extra), float("nan"), dtype=torch.float64,
                       device="cuda")
        t[:, :x.shape[1]] = torch.from_numpy(x)
        dev.append(t)
    a, b, c = dev
    api.block_gemm(a[:, :k], b[:, :n], c[:, :n], accumulate=accumulate)
    want = ora.block_gemm(A, B, C0.copy(), accumulate=accumulate)
    assert np.array_equal(c[:, :n].cpu().numpy(), want)
    assert bool(torch.isnan(c[:, n:]).all())  # nothing outside C is written


# 32 x 32 and 32 x 64 tiles (stages of 32), 64 x 64 and 128 x 128 (stages of 16)
@pytest.mark.parametrize("m,n", [(33, 65), (31, 31), (65, 4095), (511, 4090), (2045, 2047)])
@pytest.mark.parametrize("k", [1, 2, 15, 16, 17, 31, 32, 33, 47, 64, 97])
def test_pair_kernel_tiles(m, n, k):
    _check(m, n, k, accumulate=k % 2 == 1)


@pytest.mark.parametrize("k", [1, 16, 17, 33, 50])
def test_large_tiles(k):  # 256 x 128
    _check(4095, 4094, k, accumulate=k % 2 == 1)


@pytest.mark.parametrize("ld", [(1 << 23) + 1, (1 << 23) - 1])
def test_large_leading_dimension(ld):  # 64-bit offsets, and the last 32-bit ones
    _check(3, 70, 37, True, pad=(ld - 37, 5, 2))


# several products in one launch (tiles of 64 x 64 at 4096, 32 x 64 at 1124, 32 x 32; stages of a product that are
# whole, ragged and, at 32, single) and in several (the larger tiles, at 4400 and 6146), in
# the ring order from any rank
@pytest.mark.parametrize("N,P,rank", [(64, 2, 1), (99, 3, 0), (160, 5, 3), (185, 5, 4), (96, 4, 2),
                                      (1026, 6, 5), (1124, 4, 3), (4096, 8, 7), (4400, 5, 1), (6146, 2, 1)])
def test_cannon_launch_gives_the_bits_of_its_products(N, P, rank):
    ns = N // P
    g = torch.Generator(device="cuda").manual_seed(N + P)
    A = torch.randn((ns, N + 3), generator=g, dtype=torch.float64, device="cuda")[:, :N]
    B = torch.randn((N, N + 1), generator=g, dtype=torch.float64, device="cuda")[:, :N]
    C = torch.randn((ns, N + 2), generator=g, dtype=torch.float64, device="cuda")
    want = C.clone()
    for q in api.cannon_order(rank, P):
        api.block_gemm(A[:, q * ns:(q + 1) * ns], B[q * ns:(q + 1) * ns, :], want[:, :N], True)
    api.cannon_rank(A, B, C[:, :N], rank, P)
    assert torch.equal(C, want)
