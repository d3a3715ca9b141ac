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
