"""The quantized layer at any K and any alignment: operand tiles go through registers in 16-byte chunks, the
last chunk of a row is loaded to end with the row and shifted into place, rows shorter than 16 bytes are read
byte by byte.  Accumulators are integers, so every comparison with the oracle is exact."""
import numpy as np
import pytest

import oracle
from test_gpu_parity import dev, host, mpq, rand_codes

pytestmark = pytest.mark.gpu


def misaligned(a, by):
    import torch
    raw = a.reshape(-1).view(np.uint8)
    buf = torch.zeros(raw.size + 16, dtype=torch.uint8, device="cuda")
    buf[by:by + raw.size] = torch.from_numpy(raw.copy())
    t = buf[by:by + raw.size]
    return (t if a.dtype == np.uint8 else t.view(torch.int8)).reshape(a.shape)


# K around the 16-byte chunk, the 128-byte k tile and the two register sets; M, N around the 64-wide tile
@pytest.mark.parametrize("K", [1, 2, 15, 16, 17, 30, 31, 33, 46, 127, 128, 129, 143, 255, 256, 258, 385, 527])
@pytest.mark.parametrize("wbits,by", [(8, 0), (8, 1), (8, 13), (4, 0), (4, 3)])
def test_every_chunk_remainder(K, wbits, by):
    if wbits == 4 and K % 2:
        K += 1
    M, N = (65, 67) if K % 3 else (64, 130)
    a, w = rand_codes((M, K), 127, 70), rand_codes((N, K), 127 if wbits == 8 else 7, 71)
    ws = w if wbits == 8 else oracle.pack4(w)
    _, acc_o = oracle.qgemm(a, ws, [1.0], [1.0], wbits)
    _, acc = mpq.qgemm(misaligned(a, by), misaligned(ws, by), None, None, wbits, want_y=False, want_acc=True)
    np.testing.assert_array_equal(host(acc), acc_o)


@pytest.mark.parametrize("K,wbits", [(515, 8), (526, 4)])
def test_the_128_tile(K, wbits):
    """Enough 128 x 128 tiles to select them; rows are independent, so a sample of them is checked."""
    M, N = 2950, 2901
    a, w = rand_codes((M, K), 127, 72), rand_codes((N, K), 127 if wbits == 8 else 7, 73)
    ws = w if wbits == 8 else oracle.pack4(w)
    rows = np.array([0, 1, 63, 64, 127, 128, 2815, 2816, M - 2, M - 1])
    _, acc_o = oracle.qgemm(a[rows], ws, [1.0], [1.0], wbits)
    _, acc = mpq.qgemm(dev(a), dev(ws), None, None, wbits, want_y=False, want_acc=True)
    np.testing.assert_array_equal(host(acc)[rows], acc_o)
    np.testing.assert_array_equal(host(acc).astype(np.int64).sum(0), a.astype(np.int64).sum(0) @ w.astype(np.int64).T)


# rows that start at a multiple of 4 and at every other byte, ending in every byte of a dword, in the last lane's
# chunk and in the first of a k tile; both tiles, every epilogue against the plain float64 product
@pytest.mark.parametrize("mn", [(700, 131), (1500, 1500)])
@pytest.mark.parametrize("K", [256, 257, 258, 259, 260, 371, 383, 385, 512, 515])
@pytest.mark.parametrize("wbits,by", [(8, 0), (8, 2), (8, 3), (4, 0), (4, 1)])
def test_rows_at_any_byte(mn, K, wbits, by):
    import torch
    (M, N), K = mn, K + (K & 1 if wbits == 4 else 0)
    a, w = rand_codes((M, K), 127, 76), rand_codes((N, K), 127 if wbits == 8 else 7, 77)
    qa, qw = misaligned(a, by), misaligned(w if wbits == 8 else oracle.pack4(w), by)
    acc = dev(a).double() @ dev(w).double().t().contiguous()
    sa, sw = torch.full((1,), 0.01, device="cuda"), torch.rand(N, device="cuda") + 0.5
    y = (acc.float() * sa) * sw
    got, acc_k = mpq.qgemm(qa, qw, sa, sw, wbits, mpq.PER_ROW, want_acc=True)
    assert torch.equal(acc_k.double(), acc) and torch.equal(got, y)
    relu, top = mpq.qgemm_act(qa, qw, sa, sw, mpq.ACT_RELU, wbits, mpq.PER_ROW)
    assert torch.equal(relu, y.clamp(min=0)) and float(top) == float(y.max().clamp(min=0))
    codes = mpq.qgemm_act_codes(qa, qw, sa, sw, mpq.ACT_RELU, top, 8, wbits, mpq.PER_ROW)
    assert torch.equal(codes, mpq.fake_quant(relu, top, 8, want_y=False, want_codes=True)[1])
    ref = y + torch.rand_like(y)
    sse, _ = mpq.qgemm_score(qa, qw, sa, sw, ref, wbits, mpq.PER_ROW)
    want = float((y.double() - ref.double()).square().sum())
    assert abs(float(sse) - want) <= 4e-6 * want  # a lane's squares by eights, at most four times, its wave in 6 steps, the difference: (8 + 4 + 6 + 2) * 2^-24 = 1.2e-6


# one 16 x 16 tile per CU at most, 4 waves (K < 2048) and 8; two per CU; K around the step of 128, fewer
# steps than waves, more steps than one round of loads; ragged M and N; any alignment
@pytest.mark.parametrize("mnk", [(1, 1, 128), (7, 250, 96), (16, 16, 129), (49, 512, 640), (64, 256, 256), (33, 31, 2047),
                                 (17, 65, 2048), (250, 250, 2050), (5, 100, 8320), (256, 512, 2304), (500, 250, 130)])
@pytest.mark.parametrize("wbits,by", [(8, 0), (8, 5), (4, 0), (4, 1)])
def test_layers_of_few_tiles(mnk, wbits, by):
    import torch
    M, N, K = mnk
    K += K & 1 if wbits == 4 else 0
    a, w = rand_codes((M, K), 127, 74), rand_codes((N, K), 127 if wbits == 8 else 7, 75)
    ws = w if wbits == 8 else oracle.pack4(w)
    sa = np.array([0.013], np.float32)
    sw = (np.random.Generator(np.random.PCG64(76)).random(N).astype(np.float32) + 0.5) * np.float32(1e-2)
    y_o, acc_o = oracle.qgemm(a, ws, sa, sw, wbits, oracle.PER_ROW)
    da, dw = misaligned(a, by), misaligned(ws, by)
    y, acc = mpq.qgemm(da, dw, dev(sa), dev(sw), wbits, mpq.PER_ROW, want_acc=True)
    np.testing.assert_array_equal(host(acc), acc_o)
    np.testing.assert_array_equal(host(y), y_o)          # two fp32 products in a fixed order
    # activation, running maximum and codes in the epilogue
    r, m = mpq.qgemm_act(da, dw, dev(sa), dev(sw), mpq.ACT_RELU, wbits, mpq.PER_ROW)
    np.testing.assert_array_equal(host(r), np.maximum(y_o, 0))
    assert host(m)[0] == np.maximum(y_o, 0).max()
    codes = mpq.qgemm_act_codes(da, dw, dev(sa), dev(sw), mpq.ACT_RELU, m, 5, wbits, mpq.PER_ROW)
    _, c_o, _ = oracle.fake_quant(np.maximum(y_o, 0), host(m), 5)
    np.testing.assert_array_equal(host(codes), c_o)
    # an output that is only 4-byte aligned takes the scalar stores
    buf = torch.zeros(M * N + 4, dtype=torch.float32, device="cuda")[1:1 + M * N].view(M, N)
    mpq.qgemm(da, dw, dev(sa), dev(sw), wbits, mpq.PER_ROW, y=buf)
    np.testing.assert_array_equal(host(buf), y_o)


# k tiles around the number of LDS stages, last tile whole and ragged: 64 x 64 tiles in two stages (up to a k of 512, or with
# more than two tiles per CU) and in three
@pytest.mark.parametrize("mnk", [(1000, 520, 256), (1000, 520, 224), (1000, 520, 512), (1000, 520, 416), (1000, 520, 128), (1000, 520, 384),
                                 (1000, 520, 640), (1001, 530, 1024), (1001, 530, 1008), (2100, 1030, 256), (2100, 1030, 512),
                                 (2100, 1030, 448)])
@pytest.mark.parametrize("wbits", [8, 4])
def test_short_k_in_two_stages(mnk, wbits):
    M, N, K = mnk
    K = (K + 31) // 32 * 32 if wbits == 4 else K
    a, w = rand_codes((M, K), 127, 77), rand_codes((N, K), 127 if wbits == 8 else 7, 78)
    ws = w if wbits == 8 else oracle.pack4(w)
    _, acc = mpq.qgemm(dev(a), dev(ws), None, None, wbits, want_y=False, want_acc=True)
    # products of codes are whole numbers below 2^31: exact in double
    np.testing.assert_array_equal(host(acc), (a.astype(np.float64) @ w.astype(np.float64).T).astype(np.int64))
    sa, sw = np.array([0.01], np.float32), np.array([0.02], np.float32)
    r, m = mpq.qgemm_act(dev(a), dev(ws), dev(sa), dev(sw), mpq.ACT_RELU, wbits)   # one scale for all channels
    y = np.maximum((host(acc).astype(np.float32) * sa) * sw, 0)
    np.testing.assert_array_equal(host(r), y)
    assert host(m)[0] == y.max()


# one 16 x 16 tile per CU at most: a long k (int8 above 9216, packed int4 above 13312 in eight ranges or more) is cut over
# workgroups where there is a workspace, over the waves of a workgroup where there is none; on either side of the limits
@pytest.mark.parametrize("mnk", [(5, 40, 9216), (5, 40, 9232), (49, 130, 12304), (16, 4096, 9248), (33, 72, 13312), (33, 72, 13344), (1, 60, 40000), (1, 60, 28672)])
@pytest.mark.parametrize("wbits", [8, 4])
def test_long_k_of_few_tiles(mnk, wbits):
    M, N, K = mnk
    K += -K % 32 if wbits == 4 else 0
    a, w = rand_codes((M, K), 127, 79), rand_codes((N, K), 127 if wbits == 8 else 7, 80)
    ws = w if wbits == 8 else oracle.pack4(w)
    sa = np.array([0.013], np.float32)
    sw = (np.random.Generator(np.random.PCG64(81)).random(N).astype(np.float32) + 0.5) * np.float32(1e-3)
    want = (a.astype(np.float64) @ w.astype(np.float64).T).astype(np.int64)
    y_o = (want.astype(np.float32) * sa) * sw
    for use in (True, False):
        y, acc = mpq.qgemm(dev(a), dev(ws), dev(sa), dev(sw), wbits, mpq.PER_ROW, want_acc=True, use_workspace=use)
        np.testing.assert_array_equal(host(acc), want)
        np.testing.assert_array_equal(host(y), y_o)


# with a running maximum up to one tile per CU in one launch, above that in 64 x 64 tiles
@pytest.mark.parametrize("mnk", [(256, 256, 300), (256, 257, 300), (128, 768, 768), (130, 500, 272), (130, 500, 270)])
@pytest.mark.parametrize("wbits", [8, 4])
def test_running_maximum_of_few_tiles(mnk, wbits):
    M, N, K = mnk
    a, w = rand_codes((M, K), 127, 82), rand_codes((N, K), 127 if wbits == 8 else 7, 83)
    ws = w if wbits == 8 else oracle.pack4(w)
    sa, sw = np.array([0.013], np.float32), np.array([0.002], np.float32)
    want = np.maximum(((a.astype(np.float64) @ w.astype(np.float64).T).astype(np.float32) * sa) * sw, 0)
    y, m = mpq.qgemm_act(dev(a), dev(ws), dev(sa), dev(sw), mpq.ACT_RELU, wbits)
    np.testing.assert_array_equal(host(y), want)
    assert host(m)[0] == want.max()


@pytest.mark.parametrize("M,N", [(1024, 1024), (2048, 1024)])
def test_score_of_equal_differences(M, N):
    """All squares equal, so that the roundings of a running sum pull one way: a chain of n of them is off by up to (n + 1) / 2
    * 2^-24 of its sum.  A lane of either tile adds them up by eights, four times at most: 4.5 + 2.5 = 7; doubling along the
    wave is exact.  1.9405739: one chain of 32 is off by 8.5, of 16 by nothing."""
    import torch
    a, w = torch.zeros((M, 257), dtype=torch.int8, device="cuda"), torch.zeros((N, 257), dtype=torch.int8, device="cuda")
    one = torch.ones(1, device="cuda")
    for d in (1.9405739, 1.382529, 1.8926064, 1.1, 1.7):
        ref = torch.full((M, N), -d, device="cuda")
        want = M * N * float(np.float32(d)) ** 2
        sse, _ = mpq.qgemm_score(a, w, one, one, ref)
        assert abs(float(sse) - want) <= 7 * 2.0 ** -24 * want, (d, (float(sse) / want - 1) * 2 ** 24)
