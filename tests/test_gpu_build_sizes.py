"""Index construction at the bucket sizes where its kernels change (a wave, a
block of 256 or of 1024 threads per bucket; members in registers or in memory;
sorts in LDS or by radix), with duplicate rows, against the reference builder
on the CPU from the same latents: directory, cluster offsets and row order bit
for bit; centroids, whose fp64 means both builders add in id order, within one
fp32 rounding of each other.  And tau at the sample sizes around the
whole-chip select."""
import numpy as np
import pytest
import torch

from paper_2608_15438_amd import index_build as IB
from paper_2608_15438_amd import neuroute as NR
from synth import configs as CF
from synth import generators as G

pytestmark = pytest.mark.gpu

SIZES = [1, 2, 3, 63, 64, 65, 255, 256, 257, 1023, 1025, 2049]
LARGE = [4096, 4097, 9000]


@pytest.mark.parametrize("b,sizes,cap", [(4, SIZES, 20), (9, SIZES + LARGE, 200), (16, SIZES, 3),
                                         (17, SIZES, 30), (12, SIZES + LARGE, 1 << 20)])
def test_build_bucket_sizes(b, sizes, cap):
    check_build(b, sizes, cap)


def check_build(b, sizes, cap, most=0):
    """`most`: the bound on the clusters passed on (0: the plan's)."""
    rng = np.random.default_rng(b)
    n = sum(sizes)
    code = rng.choice(1 << b, len(sizes), replace=False)
    of = rng.permutation(np.repeat(code, sizes))
    lg = (np.abs(rng.standard_normal((n, b))) + 1e-3).astype(np.float32)
    lg *= np.where((of[:, None] >> np.arange(b)) & 1, 1, -1).astype(np.float32)
    first = np.array([np.flatnonzero(of == c)[0] for c in code])
    dup = rng.random(n) < 0.1                      # some rows coincide with their bucket's first
    where = {int(c): int(f) for c, f in zip(code, first)}
    lg[dup] = lg[[where[int(c)] for c in of[dup]]]
    w = CF.scaled(CF.TINY, n, 1, widths=(32, 64, b), tau_mode="zero", cluster_rule="capacity",
                  capacity=cap)
    rows = np.zeros((n, 32), np.float32)
    ref = IB.to_numpy(IB.build_index(w, IB.array_row_source(rows), device="cpu",
                                     logits_fn=lambda ids: lg[np.asarray(ids)]))
    d = torch.from_numpy(lg).cuda()
    tau = torch.zeros(b, device="cuda")
    codes = torch.empty(n, dtype=torch.int32, device="cuda")
    cnt = torch.zeros(1 << b, dtype=torch.int32, device="cuda")
    NR.nr_build_codes(d, tau, codes, cnt)
    assert np.array_equal(codes.cpu().numpy(), of)
    kb, mlist, info = NR.nr_build_plan(cnt, n, b, NR.NR_CLUSTER_CAPACITY, cap)
    nm, kmax, mc = int(info.n_multi), max(2, int(info.kmax)), max(most, int(info.max_clusters))
    u = np.zeros((1, kmax))
    if nm:
        u = G.uniform01(w.seed("sample"), mlist[:nm].cpu().numpy().astype(np.int64), kmax,
                        G.TAG_SAMPLE + 16)
    U = torch.from_numpy(u).cuda()
    row_ids = torch.empty(n, dtype=torch.int64, device="cuda")
    bc = torch.empty((1 << b) + 1, dtype=torch.int32, device="cuda")
    cl = torch.empty(mc + 1, dtype=torch.int64, device="cuda")
    cent = torch.empty((mc, b), device="cuda")
    desc = NR.nr_build_desc(n=n, b=b, logits=d.data_ptr(), codes=codes.data_ptr(),
                            sizes=cnt.data_ptr(), kb=kb.data_ptr(), mlist=mlist.data_ptr(),
                            max_clusters=mc, n_multi=nm, kmax=kmax, uniforms=U.data_ptr(),
                            seed=w.seed("sample"), lloyd=IB.N_LLOYD,
                            sample_per_cluster=IB.SAMPLE_PER_CLUSTER)
    nc = NR.nr_build_index(desc, row_ids, bc, cl, cent)
    assert np.array_equal(bc.cpu().numpy(), np.asarray(ref.bc_off, np.int64))
    assert np.array_equal(cl[:nc + 1].cpu().numpy(), np.asarray(ref.cl_off, np.int64))
    assert np.array_equal(row_ids.cpu().numpy(), np.asarray(ref.row_ids))
    assert np.allclose(cent[:nc].cpu().numpy(), ref.centroids, rtol=2.0 ** -23, atol=0)


@pytest.mark.parametrize("b,most", [(26, 0), (27, 0), (5, (1 << 26) + 9)])
def test_build_more_waves_than_one_launch(b, most):
    # a wave per bucket (2^b) and per cluster slot (the caller's bound on the
    # clusters); a launch takes fewer than 2^26 waves
    check_build(b, SIZES, 20, most)


@pytest.mark.parametrize("ns,b", [(1, 5), (2, 30), (8191, 16), (8192, 16), (8193, 7), (50_001, 30),
                                  (300_000, 11)])
def test_tau_select(ns, b):
    g = torch.Generator(device="cuda").manual_seed(ns)
    lg = torch.randn((ns, b), generator=g, device="cuda")
    lg[::3] = lg[0].clone()                              # ties
    tau = NR.nr_build_tau(lg)
    want = lg.cpu().sort(dim=0).values[(ns - 1) // 2]
    assert torch.equal(tau.cpu(), want)
