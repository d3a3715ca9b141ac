"""The tiled kernels of the quantized linear layer at the edges of their tiles and k loops: one k tile, an odd and an even
number of them, a tail of 16 and of 112, fewer k tiles than stages, several output tiles per workgroup (which sizes give
them is asserted in test_launch_shapes.py), M and N past a tile's edge, outputs that cannot be stored 16 bytes at a
time; int8 and packed int4 weights, every epilogue.

The accumulators are exact: 127 * 127 * K < 2^53, so a float64 product is the reference.  Y = (acc * s_A) * s_W is two
fp32 products, rounded once each, in every implementation: compared for equality.  The score is a double sum of fp32 sums
per wave.  A lane adds up at most 16 squares in a chain and at most eight such chains per output tile (64 x 128 values a wave in
the 256 tile) over at most four output tiles; its wave is summed in 6 steps, the difference is rounded before it is
squared: (16 + 8 * 4 + 6 + 2) * 2^-24 = 3.4e-6 relative at most."""
import pytest
import torch

from paper_2302_01382_amd import mpq

pytestmark = pytest.mark.gpu

# M x N: 256 tiles, one and two per workgroup; 192, 128 and 64 tiles, one per workgroup
TILES = [(16381, 1024), (32700, 1021), (12288, 768), (4093, 1022), (1000, 512), (333, 102)]
# M x N x K with several output tiles per workgroup in 128 and in 64 tiles: fewer k tiles than stages, as many, more; two and
# three stages; the last workgroup's tiles fewer than the others', the last tile ragged
TALL = [(140001, 128, 32), (140001, 101, 416), (70001, 128, 2176), (200001, 100, 160), (140001, 61, 32), (140001, 61, 160), (70001, 61, 1152)]


def _unpack(p):
    v = torch.stack((p & 15, p >> 4), dim=-1).reshape(p.shape[0], -1).to(torch.int32)
    return torch.where(v > 7, v - 16, v)


def _layer(M, N, K, w_bits):
    g = torch.Generator(device="cuda")
    g.manual_seed(M + N + K + w_bits)
    a = torch.randint(-127, 128, (M, K), dtype=torch.int8, device="cuda", generator=g)
    if w_bits == 8:
        w = wv = torch.randint(-127, 128, (N, K), dtype=torch.int8, device="cuda", generator=g)
    else:
        w = torch.randint(0, 256, (N, K // 2), dtype=torch.uint8, device="cuda", generator=g)
        wv = _unpack(w)
    sa = torch.rand(1, device="cuda", generator=g) + 0.5
    sw = torch.rand(N, device="cuda", generator=g) + 0.5
    acc = a.double() @ wv.double().t().contiguous()
    return a, w, sa, sw, acc


@pytest.mark.parametrize("w_bits", [8, 4])
@pytest.mark.parametrize("mnk", [(*mn, K) for mn in TILES for K in (32, 128, 160, 224, 256, 384, 416, 640, 1024)] + TALL)
def test_tiles_accumulators_and_outputs(mnk, w_bits):
    a, w, sa, sw, acc = _layer(*mnk, w_bits)
    y, got = mpq.qgemm(a, w, sa, sw, w_bits, mpq.PER_ROW, want_acc=True)
    assert torch.equal(got.double(), acc)
    assert torch.equal(y, (acc.float() * sa) * sw)


@pytest.mark.parametrize("w_bits", [8, 4])
@pytest.mark.parametrize("mnk", [(*mn, K) for mn in TILES for K in (128, 416, 1152)] + TALL)
def test_tiles_epilogues(mnk, w_bits):
    a, w, sa, sw, acc = _layer(*mnk, w_bits)
    y = (acc.float() * sa) * sw
    one, _ = mpq.qgemm(a, w, sa, sw[:1].contiguous(), w_bits, mpq.PER_TENSOR)
    assert torch.equal(one, (acc.float() * sa) * sw[0])
    relu, top = mpq.qgemm_act(a, w, sa, sw, mpq.ACT_RELU, w_bits, mpq.PER_ROW)
    assert torch.equal(relu, y.clamp(min=0)) and float(top) == float(y.max().clamp(min=0))
    codes = mpq.qgemm_act_codes(a, w, sa, sw, mpq.ACT_RELU, top, 8, w_bits, mpq.PER_ROW)
    assert torch.equal(codes, mpq.fake_quant(relu, top, 8, want_y=False, want_codes=True)[1])
    small = torch.full_like(sa, 1e-5)
    t = ((acc.float() * small) * sw).double()
    gelu, _ = mpq.qgemm_act(a, w, small, sw, mpq.ACT_GELU, w_bits, mpq.PER_ROW)
    exact = 0.5 * t * torch.special.erfc(-t / 2 ** 0.5)
    assert float((gelu.double() - exact).abs().max()) <= 1e-6 * float(t.abs().max())  # 4e-7 |y| by the fit, and its roundings
    ref = y + torch.rand_like(y)
    sse, kept = mpq.qgemm_score(a, w, sa, sw, ref, w_bits, mpq.PER_ROW, want_y=True)
    want = float((y.double() - ref.double()).square().sum())
    assert torch.equal(kept, y) and abs(float(sse) - want) <= 3.4e-6 * want
