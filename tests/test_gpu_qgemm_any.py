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
