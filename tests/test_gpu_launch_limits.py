"""Tensors whose one-workgroup-per-piece grid would pass what a launch can count (2^32 work items in x, 65535
workgroups in y): zero but for planted values, whose results the oracle gives."""
import numpy as np
import pytest

import oracle
from test_gpu_parity import host, mpq

pytestmark = pytest.mark.gpu


def planted(rows, cols, seed, n=64):
    """Zeros with n planted values, the first and the last element among them: tensor, flat indexes, values."""
    import torch
    r = np.random.Generator(np.random.PCG64(seed))
    flat = np.unique(np.concatenate([[0, rows * cols - 1], r.integers(0, rows * cols, n)]))
    vals = r.standard_normal(flat.size).astype(np.float32)
    x = torch.zeros(rows * cols, dtype=torch.float32, device="cuda")
    x[torch.from_numpy(flat).cuda()] = torch.from_numpy(vals).cuda()
    return x.view(rows, cols), flat, vals


def test_layer_of_more_than_65535_row_tiles():
    """M between 64 * 65535 and 128 * 65535 at sizes that no 16-byte load fits."""
    import torch
    M, N, K = 64 * 65535 + 37, 3, 17
    g = torch.Generator(device="cuda").manual_seed(3)
    a = torch.randint(-127, 128, (M, K), dtype=torch.int8, device="cuda", generator=g)
    w = torch.randint(-127, 128, (N, K), dtype=torch.int8, device="cuda", generator=g)
    _, acc = mpq.qgemm(a, w, None, None, 8, want_y=False, want_acc=True)
    want = torch.stack([(a.int() * w[n].int()).sum(1) for n in range(N)], 1)
    assert torch.equal(acc, want.int())
    one = torch.ones(1, device="cuda")
    y, m = mpq.qgemm_act(a, w, one, one, mpq.ACT_RELU)
    assert torch.equal(y, want.clamp(min=0).float()) and m.item() == want.max().item()


def test_rows_beyond_the_grid_per_row():
    """A wave (four rows a workgroup) and 16 lanes (sixteen rows) per row."""
    import torch
    for rows, cols in ((2 ** 26 + 9, 3), (2 ** 28 + 33, 1)):
        x, flat, vals = planted(rows, cols, rows % 97)
        m = x.abs().amax(dim=1) if cols > 1 else x.abs().view(-1)
        live = torch.from_numpy(np.unique(flat // cols)).cuda()
        xr, mr = host(x[live]), host(m[live])
        _, codes, _ = mpq.fake_quant(x, m, 5, mpq.PER_ROW, want_y=False, want_codes=True)
        _, want, _ = oracle.fake_quant(xr, mr, 5, oracle.PER_ROW)
        np.testing.assert_array_equal(host(codes[live]), want)
        assert int(torch.count_nonzero(codes)) == int(np.count_nonzero(want))
        inv, scale = torch.where(m > 0, 15 / m, torch.zeros_like(m)), m / 15
        del codes
        _, codes = mpq.fake_quant_scales(x, inv, scale, 5, mpq.PER_ROW, want_y=False, want_codes=True)
        _, want = oracle.fake_quant_scales(xr, host(inv[live]), host(scale[live]), 5, oracle.PER_ROW)
        np.testing.assert_array_equal(host(codes[live]), want)
        assert int(torch.count_nonzero(codes)) == int(np.count_nonzero(want))


def test_columns_beyond_the_grid_per_column():
    """256 columns per workgroup of 1024 threads (maximum) and of 512 (sweep); 64 sums per workgroup of 256 (finish)."""
    import torch
    cols = 2 ** 30 + 5
    x, flat, vals = planted(1, cols, 5)
    m = mpq.calibrate_absmax(x, mpq.PER_COL)
    np.testing.assert_array_equal(host(m[torch.from_numpy(flat).cuda()]), np.abs(vals))
    assert int(torch.count_nonzero(m)) == int(np.count_nonzero(vals))
    _, codes, _ = mpq.fake_quant(x, m, 8, mpq.PER_COL, want_y=False, want_codes=True)
    np.testing.assert_array_equal(host(codes[0, torch.from_numpy(flat).cuda()]), (127 * np.sign(vals)).astype(np.int8))
    assert int(torch.count_nonzero(codes)) == flat.size
    del x, m, codes
    cols = 160_000_001                     # times seven widths: more sums than 2^32 / 4
    x, flat, vals = planted(1, cols, 6)
    m = (2 * x.abs()).view(-1)             # off the grid, so that the errors are not zero
    sse = mpq.quant_error(x, m, 2, 8, mpq.PER_COL)
    idx = torch.from_numpy(flat).cuda()
    want = oracle.quant_error(vals.reshape(1, -1), host(m[idx]), 2, 8, oracle.PER_COL)
    np.testing.assert_allclose(host(sse[idx]), want, rtol=1e-4)
    assert int(torch.count_nonzero(sse[:, 0])) == int(np.count_nonzero(want[:, 0]))
