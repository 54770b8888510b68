"""The training kernels at their edges: the pair quantile against
torch.quantile (the same bits) over batch sizes, limits that cut a row, ties
and ranks; the distances at sizes that are no multiple of a tile; the gradient
for every latent width around the vector groups; thresholds read on the
device."""
import math

import numpy as np
import pytest
import torch

from paper_2608_15438_amd import neuroute as NR
from paper_2608_15438_amd import train as TR

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,limit", [(2, 1 << 24), (3, 4), (63, 1 << 24), (257, 1 << 24),
                                     (257, 12_345), (1500, 1 << 24), (4200, 1 << 24)])
@pytest.mark.parametrize("kind", ["batch", "ties", "wide"])
def test_pair_quantile(B, limit, kind):
    g = torch.Generator(device="cuda").manual_seed(B)
    if kind == "wide":       # any magnitudes, so that every digit decides
        v = torch.randint(0, 0x7F000000, (B, B), generator=g, device="cuda", dtype=torch.int32)
        d2 = v.view(torch.float32).contiguous()
    else:
        x = torch.randn((B, 24), generator=g, device="cuda")
        if kind == "ties":
            x = x.round()
        d2 = NR.nr_pair_sqdist(x)
    off = d2[~torch.eye(B, dtype=torch.bool, device="cuda")][:limit]
    for q in (0.0, 0.005, 0.37, 0.5, 0.99999, 1.0):
        want = torch.quantile(off, q)
        assert float(NR.nr_pair_quantile(d2, q, limit)) == float(want), (q, float(want))


@pytest.mark.parametrize("B,D", [(1, 1), (5, 3), (64, 16), (65, 17), (130, 100), (1003, 31)])
def test_pair_sqdist_edges(B, D):
    g = torch.Generator(device="cuda").manual_seed(D)
    x = torch.randn((B, D), generator=g, device="cuda") + 3.0
    d2 = NR.nr_pair_sqdist(x)
    xd = x.double()
    want = ((xd[:, None] - xd[None]) ** 2).sum(-1)
    scale = float(((xd - xd.mean(0)) ** 2).sum(1).max())
    # rounding of the norms and of 2 x.y: at most D + 4 roundings of the scale each
    assert float((d2 - want).abs().max()) <= 4 * (D + 4) * 2.0 ** -24 * max(scale, 1e-3)
    assert torch.equal(d2, d2.T)


@pytest.mark.parametrize("offset", [0.0, 1e3, 1e4, 1e5, -3e5])
@pytest.mark.parametrize("B,D", [(256, 128), (300, 20), (65, 200)])
def test_pair_sqdist_offset(B, D, offset):
    # columns far from zero: the centring takes the offset out, so the error
    # stays that of the spread (the exact distances of the fp32 rows)
    g = torch.Generator(device="cuda").manual_seed(B)
    sign = torch.where(torch.arange(D, device="cuda") % 3 > 0, 1.0, -1.37)
    x = torch.randn((B, D), generator=g, device="cuda") + offset * sign
    d2 = NR.nr_pair_sqdist(x)
    xd = x.double()
    want = ((xd[:, None] - xd[None]) ** 2).sum(-1)
    scale = float(((xd - xd.mean(0)) ** 2).sum(1).max())
    # as above: at most D + 4 roundings of the scale for each norm and product
    assert float((d2 - want).abs().max()) <= 4 * (D + 4) * 2.0 ** -24 * scale
    assert torch.equal(d2, d2.T)


@pytest.mark.parametrize("B,L", [(17, 1), (300, 3), (1030, 4), (515, 17), (256, 31), (700, 32)])
def test_lsim_grad_widths(B, L):
    g = torch.Generator(device="cuda").manual_seed(L)
    x = torch.randn((B, 40), generator=g, device="cuda")
    lat = torch.randn((B, L), generator=g, device="cuda")
    lat[1] = lat[0]                                  # coinciding latents have no direction
    d2 = NR.nr_pair_sqdist(x)
    gr = 0.6 * math.sqrt(L / 40)
    tau = float(np.float32(math.sqrt(float(torch.quantile(d2[d2 > 0], 0.05)))))
    nc, grad = NR.nr_lsim_grad(d2, lat, gr, tau)
    # the same mask from fp32 square roots of the same fp32 sums
    t = lat[:, None] - lat[None]
    sl2 = torch.zeros((B, B), device="cuda", dtype=torch.float64)
    for c in range(L):
        sl2 = (sl2 + t[..., c].double() ** 2).float().double()
    sl = sl2.float().double().sqrt().float()         # correctly rounded square roots
    se = d2.double().sqrt().float()
    m = (se <= tau) | (sl <= np.float32(np.float32(gr) * np.float32(tau)))
    m.fill_diagonal_(False)
    assert float(nc[1]) == float(m.sum())
    dd = torch.where(m, sl.double() - float(np.float32(gr)) * se.double(), 0.0)
    coef = torch.where(sl > 0, 4 * dd / sl.double().clamp_min(1e-300), 0.0)
    want = (coef[..., None] * t.double()).sum(1)
    mag = (coef.abs()[..., None] * t.double().abs()).sum(1)
    # each term has a few fp32 roundings, the sum at most B / 64 + 22 more
    assert ((grad - want).abs() <= (B / 64 + 40) * 2.0 ** -24 * mag + 1e-12).all()
    assert abs(float(nc[0]) - float((dd * dd).sum())) <= 1e-5 * float((dd * dd).sum())


def test_loss_reads_tau_on_the_device():
    g = torch.Generator(device="cuda").manual_seed(3)
    x = torch.randn((600, 64), generator=g, device="cuda")
    lat = torch.randn((600, 20), generator=g, device="cuda", requires_grad=True)
    loss, tau, frac = TR.lsim_loss_gpu(x, lat, 0.6)
    loss.backward()
    g1 = lat.grad.clone()
    lat.grad = None
    loss2, tau2, frac2 = TR.lsim_loss_gpu(x, lat, 0.6, tau)
    loss2.backward()
    assert tau == tau2 and frac == frac2
    assert torch.equal(g1, lat.grad)
    d2 = NR.nr_pair_sqdist(x)
    off = ~torch.eye(600, dtype=torch.bool, device="cuda")
    assert tau == math.sqrt(float(torch.quantile(d2[off], 0.005)))
    with pytest.raises(RuntimeError):
        TR.lsim_loss_gpu(x[:1], lat[:1], 0.6)
    with pytest.raises(RuntimeError):
        TR.lsim_loss_gpu(x, lat, 0.6, quantile=1.5)


def test_loss_rejects_a_non_finite_tau():
    # distances that overflow at the quantile: an error, as when tau_emb is given
    g = torch.Generator(device="cuda").manual_seed(4)
    lat = torch.randn((128, 8), generator=g, device="cuda", requires_grad=True)
    x = torch.full((128, 16), 1e25, device="cuda")
    x[::2] *= -1                                     # half of the pairs at infinity
    for q in (0.9, 1.0):
        with pytest.raises(NR.NRError) as e:
            TR.lsim_loss_gpu(x, lat, 0.6, quantile=q)
        assert e.value.status == NR.NR_EINVAL
    assert math.isfinite(TR.lsim_loss_gpu(x, lat, 0.6, quantile=0.1)[1])
    # one row out of range: the pairs below the quantile are not concerned
    x = torch.randn((128, 16), generator=g, device="cuda")
    x[5] = 1e25
    assert math.isfinite(TR.lsim_loss_gpu(x, lat, 0.6, quantile=0.0)[1])


@pytest.mark.parametrize("at,limit", [((0, 1), 1 << 24), ((40, 3), 1 << 24), ((69, 68), 1 << 24),
                                      ((5, 5), 1 << 24), ((69, 0), 100)])
def test_pair_quantile_nan(at, limit):
    # a NaN among the elements makes the quantile NaN, as torch.quantile's; on
    # the diagonal or past the limit it is not among them
    g = torch.Generator(device="cuda").manual_seed(2)
    d2 = torch.rand((70, 70), generator=g, device="cuda")
    d2[at] = float("nan")
    off = d2[~torch.eye(70, dtype=torch.bool, device="cuda")][:limit]
    for q in (0.0, 0.005, 1.0):
        got, want = float(NR.nr_pair_quantile(d2, q, limit)), float(torch.quantile(off, q))
        assert got == want or (math.isnan(got) and math.isnan(want)), (q, got, want)


def test_work_space_of_another_stream():
    # the call's work space is freed when it returns: what the current stream
    # allocates next must not land in it while the other stream still waits
    g = torch.Generator(device="cuda").manual_seed(6)
    x = torch.randn((1500, 64), generator=g, device="cuda")
    want = NR.nr_pair_sqdist(x)
    q = NR.nr_pair_quantile(want, 0.005)
    side = torch.cuda.Stream()
    d2, out = torch.empty_like(want), torch.empty_like(q)
    for _ in range(3):
        d2.zero_()
        out.zero_()
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            torch.cuda._sleep(20_000_000)
        NR.nr_pair_sqdist(x, out=d2, stream=side)
        NR.nr_pair_quantile(d2, 0.005, out=out, stream=side)
        junk = [torch.full((n,), 1e9, device="cuda") for n in (1 << 13, 1 << 14, 1 << 16, 1 << 17, 1 << 18)]
        torch.cuda.synchronize()
        del junk
        assert torch.equal(d2, want)
        assert torch.equal(out, q)


def test_wrong_tensors_are_refused():
    # the kernels read and write by the shapes of one argument
    d2, lat = torch.rand((8, 8), device="cuda"), torch.rand((8, 3), device="cuda")
    stats = torch.ones(3, dtype=torch.float64, device="cuda")
    NR.nr_lsim_grad_at(d2, lat, 0.5, stats)
    for a in ((d2, lat, stats.float()), (d2, lat, stats[:2]), (d2[:7], lat, stats),
              (d2, lat.double(), stats), (d2, lat[:7].contiguous(), stats), (d2, lat, stats.cpu())):
        with pytest.raises(ValueError):
            NR.nr_lsim_grad_at(a[0], a[1], 0.5, a[2])
    for a in ((d2.double(), None), (d2[:5], None), (d2, stats.float()), (d2, stats[:0])):
        with pytest.raises(ValueError):
            NR.nr_pair_quantile(a[0], 0.5, out=a[1])
