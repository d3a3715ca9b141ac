"""mpq_hutchinson_quad_signs where its layout changes: rows around the 32-row block, k around the 128-k block and
no multiple of it (sign words cut out of two Philox blocks), 1 to 8 waves sharing k, several trips per
workgroup with a ragged last one, both probe widths and several passes; the exactness of the three-way split;
and sums over the rows in double."""
import numpy as np
import pytest

from test_gpu_parity import data, dev, host, mpq

pytestmark = pytest.mark.gpu


def want(x, v):
    return ((x.astype(np.float64) @ v.astype(np.float64).T) ** 2).sum(0)


@pytest.mark.parametrize("mkp", [(1, 16, 1), (31, 48, 3), (32, 128, 32), (33, 144, 33), (65, 256, 64), (40, 272, 65),
                                 (300, 1040, 5), (70, 2064, 130), (200, 4096, 3), (9000, 256, 4), (20000, 80, 7)])
def test_layouts(mkp):
    M, K, P = mkp
    x = data((M, K), 110)
    v = host(mpq.rademacher(7, 3, P, K))
    got = host(mpq.hutchinson_quad_signs(dev(x), 7, 3, P))
    # exact products; sums of K terms and of M squares in fp32: far below 1e-5 of a sum of squares
    np.testing.assert_allclose(got, want(x, v), rtol=1e-5)


# K <= 256: a wave per 32 k while there are at most as many row blocks as CUs, whole blocks per wave from 8193 rows on
@pytest.mark.parametrize("P", [5, 40])
@pytest.mark.parametrize("M", [1, 33, 8192, 8193])
@pytest.mark.parametrize("K", [16, 32, 48, 80, 112, 128, 144, 208, 256, 272])
def test_a_wave_per_tile_of_k(M, K, P):
    x = data((M, K), 114)
    v = host(mpq.rademacher(9, 1, P, K))
    got = host(mpq.hutchinson_quad_signs(dev(x), 9, 1, P))
    # exact products, so a row's s = sum of +-x is off by e <= 2^-24 (terms added) sum |x| (three parts per x, and one
    # row can cancel: s << sum |x|), its square by 2 |s| e + e^2; squares and 32 of them in fp32: 33 roundings
    e = 2.0 ** -24 * 3 * K * np.abs(x.astype(np.float64)).sum(1)
    s = np.abs(x.astype(np.float64) @ v.astype(np.float64).T)
    exact = want(x, v)
    assert (np.abs(got - exact) <= (2 * s * e[:, None] + e[:, None] ** 2).sum(0) + 33 * 2.0 ** -24 * exact).all()


# grid times row blocks per workgroup is 2048 at most, so these take two trips or more whatever the layout, the
# last one partly past M: k in whole 128-k blocks and not, one probe block and two; a K long enough for 8 waves each
@pytest.mark.parametrize("mkp", [(70001, 512, 33), (70001, 80, 5), (66000, 208, 64), (35003, 4096, 3)])
def test_several_trips(mkp):
    import torch
    M, K, P = mkp
    x = torch.randn((M, K), generator=torch.Generator(device="cuda").manual_seed(113), device="cuda")
    v = mpq.rademacher(7, 3, P, K).double().t().contiguous()
    exact = torch.zeros(P, dtype=torch.float64, device="cuda")
    for r in range(0, M, 8192):
        exact += (x[r:r + 8192].double() @ v).square().sum(0)
    got = mpq.hutchinson_quad_signs(x, 7, 3, P)
    # products exact, sums over k of one row in fp32: relative 2^-24 sqrt(K) of a row's, far less of their sum
    np.testing.assert_allclose(host(got), host(exact), rtol=1e-7)


@pytest.mark.parametrize("M", [16384, 9001, 40007])
def test_row_blocks_are_added_in_double(M):
    """2^24 in the first 32 rows, 1 in each 32 after them: whole numbers that an fp32 running sum would drop."""
    x = np.zeros((M, 16), np.float32)
    x[::32, 3] = 1.0
    x[0, 3] = 4096.0
    blocks = (M + 31) // 32
    np.testing.assert_array_equal(host(mpq.hutchinson_quad_signs(dev(x), 5, 0, 40)), np.full(40, 2.0 ** 24 + blocks - 1))


def test_the_split_is_exact_over_the_exponent_range():
    """One column per row: a row's product is +-x itself, so the quadratic form is the sum of exact squares."""
    M, K = 64, 16
    r = np.random.Generator(np.random.PCG64(111))
    for scale in (-18, -6, 0, 6, 18):       # squares stay in the range of fp32
        x = np.zeros((M, K), np.float32)
        x[np.arange(M), r.integers(0, K, M)] = (r.standard_normal(M) * 10.0 ** scale).astype(np.float32)
        got = host(mpq.hutchinson_quad_signs(dev(x), 5, 0, 4))
        np.testing.assert_allclose(got, np.full(4, (x.astype(np.float64) ** 2).sum()), rtol=2e-6)  # fp32 squares and their sum


def test_replay_in_a_graph():
    import torch
    x = dev(data((500, 272), 112))
    ws, out = mpq.Workspace(), torch.empty(9, dtype=torch.float64, device="cuda")
    mpq.init()
    eager = host(mpq.hutchinson_quad_signs(x, 1, 2, 9, ws=ws)).copy()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        mpq.hutchinson_quad_signs(x, 1, 2, 9, out=out, ws=ws)
    for _ in range(3):
        out.zero_()
        g.replay()
        torch.cuda.synchronize()
        np.testing.assert_array_equal(host(out), eager)


@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
def test_values_that_are_not_finite_make_the_form_nan(bad):
    x = data((70, 144), 114)
    x[33, 20] = bad
    assert np.all(np.isnan(host(mpq.hutchinson_quad_signs(dev(x), 5, 0, 35))))
