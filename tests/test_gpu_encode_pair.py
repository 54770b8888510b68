"""The last two encoder layers in one kernel: its logits are those of two
kernels bit for bit (a 2-layer encoder against the same layers behind an
identity layer of whole numbers, which keeps every value but takes the inputs
through another kernel), at row counts around the blocks and at widths that are
no multiple of a tile; and against fp64."""
import numpy as np
import pytest
import torch

from paper_2608_15438_amd import index_build as IB
from paper_2608_15438_amd import neuroute as NR

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("u8", [True, False])
@pytest.mark.parametrize("d,h,b", [(128, 256, 24), (96, 200, 15), (48, 64, 30), (36, 1, 1),
                                   (20, 65, 16), (1536, 33, 9)])
@pytest.mark.parametrize("m", [33, 16_383, 16_385, 49_151, 49_153])
def test_pair_logits(u8, d, h, b, m):
    if u8 and d % 16:
        d = d + 16 - d % 16
    rng = np.random.default_rng(d * m)
    W = [rng.standard_normal((h, d)).astype(np.float32) / np.float32(np.sqrt(d)),
         rng.standard_normal((b, h)).astype(np.float32) / np.float32(np.sqrt(h))]
    bias = [rng.standard_normal(h).astype(np.float32), rng.standard_normal(b).astype(np.float32)]
    g = torch.Generator(device="cuda").manual_seed(m)
    if u8:
        x = torch.randint(0, 256, (m, d), generator=g, device="cuda", dtype=torch.uint8)
    else:
        x = torch.rand((m, d), generator=g, device="cuda")
    dt = NR.NR_U8 if u8 else NR.NR_F32
    ix = NR.Index.encoder_only(IB.Encoder(W, bias, 1.0), dt)
    got = ix.nr_encode(x)
    xd = x.double()
    hid = xd @ torch.from_numpy(W[0]).cuda().double().T + torch.from_numpy(bias[0]).cuda().double()
    w1 = torch.from_numpy(W[1]).cuda().double()
    want = hid.clamp_min(0) @ w1.T + torch.from_numpy(bias[1]).cuda().double()
    mag = (xd.abs() @ torch.from_numpy(np.abs(W[0])).cuda().double().T + 3) @ w1.abs().T + 3
    # two chains of d and h products: at most d + h + 4 roundings of the magnitudes
    assert ((got - want).abs() <= (d + h + 4) * 2.0 ** -24 * mag).all()
    if d <= 128:
        eye = IB.Encoder([np.eye(d, dtype=np.float32)] + W, [np.zeros(d, np.float32)] + bias, 1.0)
        ix3 = NR.Index.encoder_only(eye, dt)
        assert torch.equal(got, ix3.nr_encode(x))
        ix3.close()
    # rows do not depend on the batch they come in
    assert torch.equal(got[m // 2:m // 2 + 1], ix.nr_encode(x[m // 2:m // 2 + 1].clone()))
    ix.close()


@pytest.mark.parametrize("widths,m", [((16, 3), (1 << 29) + 77), ((16, 4, 2), (1 << 30) + 77)])
def test_more_rows_than_one_launch(widths, m):
    # 32 rows of a one-layer encoder, or 64 of a two-layer one, take a block of
    # 256 threads; a launch takes fewer than 2^32
    rng = np.random.default_rng(len(widths))
    W = [rng.standard_normal((o, i)).astype(np.float32) for i, o in zip(widths, widths[1:])]
    bias = [rng.standard_normal(o).astype(np.float32) for o in widths[1:]]
    ix = NR.Index.encoder_only(IB.Encoder(W, bias, 1.0), NR.NR_U8)
    x = torch.empty((m, 16), dtype=torch.uint8, device="cuda")
    x.random_(0, 256, generator=torch.Generator(device="cuda").manual_seed(1))
    got = ix.nr_encode(x)
    step = 1 << 24
    for i in list(range(0, m, 7 * step)) + [m - 1000]:
        assert torch.equal(got[i:i + step], ix.nr_encode(x[i:i + step])), i
    ix.close()


@pytest.mark.parametrize("u8,widths", [(True, (512, 448, 9)), (True, (528, 512, 16)),
                                       (True, (496, 513, 16)), (False, (512, 520, 30)),
                                       (False, (36, 511, 7)), (False, (1532, 448, 5))])
def test_tiles_agree(u8, widths):
    # 12,000 rows go in 64 x 64 tiles and 100 in 32 x 64 ones, in either order of
    # their K-tiles: every logit is the same chain
    rng = np.random.default_rng(widths[0])
    W = [(rng.standard_normal((o, i)) / np.sqrt(i)).astype(np.float32)
         for i, o in zip(widths, widths[1:])]
    ix = NR.Index.encoder_only(IB.Encoder(W, [np.zeros(o, np.float32) for o in widths[1:]], 1.0),
                               NR.NR_U8 if u8 else NR.NR_F32)
    g = torch.Generator(device="cuda").manual_seed(1)
    x = torch.rand((12_000, widths[0]), generator=g, device="cuda")
    if u8:
        x = (x * 256).to(torch.uint8)
    got = ix.nr_encode(x)
    for i in (0, 7777, 11_900):
        assert torch.equal(got[i:i + 100], ix.nr_encode(x[i:i + 100].clone()))
    h = (x.double() @ torch.from_numpy(W[0]).cuda().double().T).clamp_min(0)
    w1 = torch.from_numpy(W[1]).cuda().double()
    mag = (x.double().abs() @ torch.from_numpy(np.abs(W[0])).cuda().double().T) @ w1.abs().T
    # two chains: at most one rounding of the magnitudes per product
    assert ((got - h @ w1.T).abs() <= (widths[0] + widths[1] + 4) * 2.0 ** -24 * mag).all()
    ix.close()
