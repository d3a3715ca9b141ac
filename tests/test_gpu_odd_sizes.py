"""The streaming calls at odd sizes and alignments: 16-byte accesses at any element, the last cols % 4 (or
n % 4) elements by themselves, columns in groups of four with a ragged last group, several row chunks."""
import numpy as np
import pytest

import oracle
from test_gpu_parity import data, dev, host, mpq

pytestmark = pytest.mark.gpu

# rows, cols: remainders 0..3 of the vector, short rows, more than one wave / workgroup of columns, several
# trips of four loads, more row chunks than waves; 16390 columns are two segments of a row
SHAPES = [(1, 1), (3, 2), (5, 3), (2, 5), (67, 7), (130, 66), (33, 255), (33, 257), (40, 1023), (70, 1030), (1500, 5),
          (2100, 70), (9, 2049), (3, 16390),
          # around the sizes up to which one workgroup reduces a whole tensor (16384 and 32768 elements)
          (128, 128), (5, 3277), (128, 256), (2731, 12)]


def at(a, off):
    """a on the device, `off` elements behind a 16-byte boundary."""
    import torch
    t = torch.from_numpy(np.ascontiguousarray(a))
    buf = torch.zeros(t.numel() + 4, dtype=t.dtype, device="cuda")
    buf[off:off + t.numel()] = t.reshape(-1).cuda()
    return buf[off:off + t.numel()].view(t.shape)


@pytest.mark.parametrize("gran", [mpq.PER_TENSOR, mpq.PER_ROW, mpq.PER_COL])
@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("off", [0, 1, 3])
def test_streaming_calls(shape, off, gran):
    import torch
    x = data(shape, 90 + off)
    dx = at(x, off)
    m_o = oracle.absmax(x, gran)
    m = mpq.calibrate_absmax(dx, gran)
    np.testing.assert_array_equal(host(m), m_o)
    run = dev(np.full_like(m_o, m_o.max() / 2))       # running maximum
    mpq.calibrate_absmax(dx, gran, out=run, accumulate=True)
    np.testing.assert_array_equal(host(run), np.maximum(m_o, m_o.max() / 2))
    for lo, hi in ((2, 8), (5, 5)):
        sse = host(mpq.quant_error(dx, m, lo, hi, gran))
        want = oracle.quant_error(x, m_o, lo, hi, gran)
        # fp32 partial sums: 1e-4 relative; an element on the grid (its channel's maximum) has an error of
        # one rounding of its product, hence the floor at (2^-24 max)^2 per element of a channel
        np.testing.assert_allclose(sse, want, rtol=1e-4, atol=(2.0 ** -24 * float(m_o.max())) ** 2 * x.size)
    for bits in (8, 3):
        packed = bits == 3 and shape[1] % 2 == 0
        y = at(np.zeros(shape, np.float32), off)
        codes = torch.zeros(x.size + 8, dtype=torch.int8, device="cuda")[off:off + x.size].view(shape)
        p4 = torch.zeros(x.size // 2 + 8, dtype=torch.uint8, device="cuda")[off:off + x.size // 2].view(shape[0], -1) if packed else None
        mpq.fake_quant(dx, m, bits, gran, y=y, codes=codes, packed4=p4)
        y_o, c_o, p_o = oracle.fake_quant(x, m_o, bits, gran, want_packed4=packed)
        np.testing.assert_array_equal(host(codes), c_o)
        np.testing.assert_array_equal(host(y), y_o)
        if packed:
            np.testing.assert_array_equal(host(p4), p_o)
    if gran == mpq.PER_TENSOR:
        ref = data(shape, 95)
        got = host(mpq.sse_pair(dx, at(ref, (off + 2) % 4)))[0]
        assert got == pytest.approx(oracle.sse_pair(x, ref), rel=1e-4)


@pytest.mark.parametrize("gran", [mpq.PER_TENSOR, mpq.PER_ROW])
@pytest.mark.parametrize("shape", [(1, 1), (5, 3), (67, 7), (33, 255), (20, 256), (9, 257), (70, 1030), (6, 4099), (2, 9001), (300, 64)])
@pytest.mark.parametrize("off", [0, 3])
def test_scale_adjustment(shape, off, gran):
    """4, 16 (up to 256 columns) lanes or a wave per row, pieces past the row's end, rows cut into segments."""
    x, g = data(shape, 96), data(shape, 97)
    m = oracle.absmax(x, gran)
    for bits in (3, 8):
        qmax = np.float32(2 ** (bits - 1) - 1)
        inv, scale = (qmax / m * np.float32(1.3)).astype(np.float32), (m / qmax).astype(np.float32)
        y, codes = mpq.fake_quant_scales(at(x, off), dev(inv), dev(scale), bits, gran, want_codes=True)
        y_o, c_o = oracle.fake_quant_scales(x, inv, scale, bits, gran)
        np.testing.assert_array_equal(host(codes), c_o)
        np.testing.assert_array_equal(host(y), y_o)
        for up in (None, g):
            got = mpq.scale_grad(at(x, off), dev(inv), dev(scale), bits, None if up is None else at(up, (off + 1) % 4), gran)
            want = oracle.scale_grad(x, inv, scale, bits, up, gran)
            # fp32 partial sums of terms of either sign: 1e-4 of the sum of their absolute values
            for a, key, lim in zip(got, ("dinv", "dscale", "loss"), ("abs_dinv", "abs_dscale", "loss")):
                assert np.all(np.abs(host(a) - want[key]) <= 1e-4 * want[lim] + 1e-12)


@pytest.mark.parametrize("gran", [mpq.PER_TENSOR, mpq.PER_ROW, mpq.PER_COL])
@pytest.mark.parametrize("shape", [(1, 1), (5, 3), (7, 4), (9, 5), (67, 7), (33, 255), (20, 256), (70, 1030), (3, 4099)])
@pytest.mark.parametrize("off", [0, 1])
def test_noise(shape, off, gran):
    """Groups of four elements in one row, in two rows and (rows of three elements) in more; the last n % 4; planes
    that start at any element.  Bit for bit."""
    import torch
    x = data(shape, 98)
    m = oracle.absmax(x, gran)
    want = {b: oracle.noise_inject(x, m, b, 0.3, 9, 2, gran) for b in (2, 5, 8)}
    got = at(np.zeros(shape, np.float32), off)
    mpq.noise_inject(at(x, off), dev(m), 5, 0.3, 9, 2, gran, out=got)
    np.testing.assert_array_equal(host(got), want[5])
    n, stride = x.size, x.size + 3
    buf = torch.zeros(7 * stride + 4, dtype=torch.float32, device="cuda")
    out = buf[off:off + 7 * stride].view(7, stride)[:, :n].unflatten(1, shape)
    mpq.noise_inject_sweep(at(x, off), dev(m), 2, 8, 0.3, 9, 2, gran, out=out)
    for b in want:
        np.testing.assert_array_equal(host(out[b - 2]), want[b])
    inplace = at(x, off)
    mpq.noise_inject(inplace, dev(m), 8, 0.3, 9, 2, gran, out=inplace)
    np.testing.assert_array_equal(host(inplace), want[8])


# per column: up to 8, 32 and 512 rows a workgroup of 1, 4 and 16 waves writes the result itself (1 up to 64 rows from
# 2048 groups of 64 columns on, 4 up to 512 rows from 512 groups on); above, two launches
@pytest.mark.parametrize("shape", [(1, 65), (8, 130), (9, 63), (32, 129), (33, 64), (512, 70), (513, 70), (64, 131073), (65, 131009),
                                   (100, 32769), (600, 9)])
@pytest.mark.parametrize("widths", [(2, 8), (4, 4), (3, 5)])
def test_sweep_per_column_of_few_rows(shape, widths):
    x = data(shape, 99)
    m = oracle.absmax(x, oracle.PER_COL) * np.float32(1.25)     # off the grid: no element's error is a rounding alone
    for off in (0, 1):
        got = host(mpq.quant_error(at(x, off), dev(m), *widths, mpq.PER_COL))
        np.testing.assert_allclose(got, oracle.quant_error(x, m, *widths, oracle.PER_COL), rtol=1e-5)


def test_per_column_fp32_sums_stay_short():
    """Errors of 1/4 in the first rows, of 1/4 2^-13 below: an fp32 sum that holds one of the former drops the
    squares of the latter.  A lane adds at most max(8, rows * groups of 256 columns / 8192) rows in fp32."""
    rows, cols = 2 ** 17, 4
    x = np.full((rows, cols), 0.25 * 2.0 ** -13, np.float32)
    x[:4096] = 0.25
    got = host(mpq.quant_error(dev(x), dev(np.ones(cols, np.float32)), 2, 2, mpq.PER_COL))
    want = oracle.quant_error(x, np.ones(cols, np.float32), 2, 2, oracle.PER_COL)
    assert np.all(np.abs(got / want - 1) <= (rows / 8192) * 2.0 ** -26)


# rows that no sweep plan holds: 16 lanes or a wave per row; whole trips of four vectors and every way to fall short
@pytest.mark.parametrize("shape", [(3, 5), (5, 64), (9, 65), (40, 127), (40, 255), (33, 257), (17, 1021), (17, 1026), (3, 2500), (600, 75),
                                   (600, 76), (8192, 131), (8191, 1025), (8200, 771), (8200, 2047), (8200, 2050)])
@pytest.mark.parametrize("widths", [(2, 8), (4, 4), (3, 5)])
def test_sweep_per_row_at_any_size(shape, widths):
    """As close to the sums in 64 bits as fp32 sums of 64 lanes, each over every 64th column, that meet in a
    tree: the random part of the roundings of such sums, with 15 % for the spread of the estimate."""
    x = data(shape, 100)
    m = oracle.absmax(x, oracle.PER_ROW) * np.float32(1.25)
    off = 1 if shape[1] % 4 == 0 else 0
    got = host(mpq.quant_error(at(x, off), dev(m), *widths, mpq.PER_ROW))
    want = oracle.quant_error(x, m, *widths, oracle.PER_ROW)
    np.testing.assert_allclose(got, want, rtol=1e-5)
    if shape[0] < 2000:
        return
    b = widths[1]
    qmax = np.float32(2 ** (b - 1) - 1)
    inv, sc = (qmax / m)[:, None], (m / qmax)[:, None]
    q = np.rint(x.astype(np.float64) * inv)
    e = (q * sc.astype(np.float64) - x).astype(np.float32)          # one fused multiply-add
    lanes = np.zeros((shape[0], 64), np.float32)
    exact = (e.astype(np.float64) ** 2).sum(1)
    for c in range(0, shape[1], 64):
        p = e[:, c:c + 64]
        lanes[:, :p.shape[1]] = (p.astype(np.float64) ** 2 + lanes[:, :p.shape[1]]).astype(np.float32)
    while lanes.shape[1] > 1:
        lanes = lanes[:, 0::2] + lanes[:, 1::2]
    rms = np.sqrt(np.mean((lanes[:, 0] / exact - 1) ** 2))
    assert np.sqrt(np.mean((got[:, -1] / exact - 1) ** 2)) <= 1.15 * rms


def lane_sums(e):
    """Sums of squares as 64-lane waves of fp32 sums of four vectors a lane form them, the waves in double."""
    n = e.size // 4096 * 4096
    v = e[:n].reshape(-1, 4, 64, 4)                                  # tile of a wave, vector, lane, element
    acc = np.zeros((v.shape[0], 64), np.float32)
    for k in range(4):
        for c in range(4):
            acc = (v[:, k, :, c].astype(np.float64) ** 2 + acc).astype(np.float32)
    while acc.shape[1] > 1:
        acc = acc[:, 0::2] + acc[:, 1::2]
    return acc.astype(np.float64).sum() + (e[n:].astype(np.float64) ** 2).sum()


@pytest.mark.parametrize("n", [4096, 16384, 32768, 65536, 69632])
@pytest.mark.parametrize("off", [0, 1])
def test_small_tensors_are_summed_as_closely_as_larger_ones(n, off):
    """One workgroup up to 65536 elements (one width; 16384 unaligned) and 32768 (squared distance): rms error over 24
    inputs no larger than that of lane_sums, with 25 % for the spread of either estimate."""
    err = np.zeros((24, 4))
    for i in range(24):
        x, ref = data((1, n), 300 + i), data((1, n), 400 + i)
        d = (x - ref).reshape(-1)
        m = oracle.absmax(x) * np.float32(1.25)
        inv, sc = np.float32(7) / m, m / np.float32(7)
        e = (np.rint(x.astype(np.float64) * inv) * sc.astype(np.float64) - x).astype(np.float32).reshape(-1)
        for k, (v, got) in enumerate(((d, host(mpq.sse_pair(at(x, off), at(ref, off)))[0]),
                                      (e, host(mpq.quant_error(at(x, off), dev(m), 4, 4))[0, 0]))):
            exact = (v.astype(np.float64) ** 2).sum()
            err[i, 2 * k:2 * k + 2] = got / exact - 1, lane_sums(v) / exact - 1
    rms = np.sqrt((err ** 2).mean(0))
    assert rms[0] <= 1.25 * rms[1] and rms[2] <= 1.25 * rms[3], rms


# 16 lanes or a wave per row, one load in flight or four, streamed or cached; per tensor in tiles or one vector a trip
@pytest.mark.parametrize("gran,shape", [(mpq.PER_ROW, s) for s in [(5, 64), (5, 65), (3, 768), (3, 769), (2100, 64), (2100, 66), (8200, 256),
                                                                  (8210, 257), (3, 1800001), (5300, 1000), (42000, 130)]] +
                         [(mpq.PER_TENSOR, s) for s in [(1, 524288), (1, 524293), (7, 100001)]])
def test_scale_gradients_where_the_layout_changes(gran, shape):
    x, g = data(shape, 101), data(shape, 102)
    m = oracle.absmax(x, gran)
    inv, scale = (np.float32(7) / m * np.float32(1.3)).astype(np.float32), (m / np.float32(7)).astype(np.float32)
    for off in (0, 1):
        for up in (None, g):
            got = mpq.scale_grad(at(x, off), dev(inv), dev(scale), 4, None if up is None else at(up, (off + 1) % 4), gran)
            want = oracle.scale_grad(x, inv, scale, 4, up, gran)
            for a, key, lim in zip(got, ("dinv", "dscale", "loss"), ("abs_dinv", "abs_dscale", "loss")):
                # rms of a million random roundings of fp32 sums, far below 1e-6 of the sum of absolute values
                assert np.all(np.abs(host(a) - want[key]) <= 1e-6 * want[lim] + 1e-12)


@pytest.mark.parametrize("shape", [(4000, 256), (4000, 255), (8200, 250)])
def test_scale_gradients_are_summed_as_closely_as_by_64_lanes(shape):
    x, g = data(shape, 103), data(shape, 104)
    m = oracle.absmax(x, oracle.PER_ROW)
    inv, scale = (np.float32(7) / m).astype(np.float32), (m / np.float32(7)).astype(np.float32)
    dscale = host(mpq.scale_grad(dev(x), dev(inv), dev(scale), 4, dev(g), mpq.PER_ROW)[1])
    gq = g.astype(np.float64) * np.clip(np.rint(x.astype(np.float64) * inv[:, None]), -7, 7)
    lanes = np.zeros((shape[0], 64), np.float32)
    for c in range(0, shape[1], 64):
        p = gq[:, c:c + 64]
        lanes[:, :p.shape[1]] = (p + lanes[:, :p.shape[1]]).astype(np.float32)
    while lanes.shape[1] > 1:
        lanes = lanes[:, 0::2] + lanes[:, 1::2]
    rms = [np.sqrt(np.mean(((v - gq.sum(1)) / np.abs(gq).sum(1)) ** 2)) for v in (dscale, lanes[:, 0])]
    assert rms[0] <= 1.06 * rms[1], rms     # thousands of rows: either estimate is good to 2 %


# lanes per row (4 up to 32 columns, 16 up to 256), rows per wave of a narrow tensor's columns (16, 64 and 128 columns),
# one row chunk of column maxima (64 and 128 rows), long rows in segments of 1024 columns and of 16384
@pytest.mark.parametrize("gran", [mpq.PER_ROW, mpq.PER_COL])
@pytest.mark.parametrize("shape", [(70, 31), (70, 32), (70, 33), (300, 16), (300, 17), (64, 64), (65, 65), (128, 128), (129, 129), (130, 256), (70, 258),
                                   (129, 3), (3, 70001), (2, 70002), (1, 5), (1100, 2050), (2060, 1030), (4000, 20), (1, 36866)])
@pytest.mark.parametrize("off", [0, 1])
def test_streaming_calls_where_the_layout_changes(shape, off, gran):
    test_streaming_calls(shape, off, gran)


@pytest.mark.parametrize("shape", [(300, 16), (70, 31), (70, 32), (70, 33), (5000, 7)])
def test_explicit_scales_of_short_rows(shape):
    test_scale_adjustment(shape, 0, mpq.PER_ROW)
    test_scale_adjustment(shape, 1, mpq.PER_ROW)


# one vector a trip up to 2^19 elements, tiles above, streamed where the tensor is aligned
@pytest.mark.parametrize("n", [2 ** 19, 2 ** 19 + 1, 2 ** 19 + 4098])
def test_per_tensor_sums_where_the_layout_changes(n):
    x, ref = data((1, n), 105), data((1, n), 106)
    m = oracle.absmax(x) * np.float32(1.25)
    for off in (0, 1, 3):
        for widths in ((2, 8), (3, 3)):
            np.testing.assert_allclose(host(mpq.quant_error(at(x, off), dev(m), *widths)), oracle.quant_error(x, m, *widths), rtol=1e-6)
        assert host(mpq.sse_pair(at(x, off), at(ref, (off + 1) % 4)))[0] == pytest.approx(oracle.sse_pair(x, ref), rel=1e-6)
