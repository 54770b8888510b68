"""The batch-shared schedule against the per-query one (same lists, bit for
bit) over scans of small, middling and large work, the three cases of the
scan's tile size, and over neighbours per query up to the largest k."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def make_index(n, d, b, dtype, head, seed=0, per=1):
    """Random rows in random buckets, up to `per` clusters in each; the latents
    are d -> b random projections."""
    from paper_2608_15438_amd import neuroute as NR
    g = torch.Generator(device="cuda").manual_seed(seed)
    rng = np.random.default_rng(seed)
    if dtype == NR.NR_U8:
        rows = torch.randint(0, 256, (n, d), generator=g, device="cuda", dtype=torch.uint8)
    else:
        rows = torch.randn((n, d), generator=g, device="cuda")
    sizes = np.bincount(rng.integers(0, 1 << b, n), minlength=1 << b)
    k = np.minimum(sizes, rng.integers(1, per + 1, 1 << b))  # clusters of each bucket
    nz = np.concatenate([[s // c + (i < s % c) for i in range(c)] for s, c in zip(sizes, k)])
    nz = nz.astype(np.int64)
    bc = np.concatenate([[0], np.cumsum(k)])
    cl = np.concatenate([[0], np.cumsum(nz)])
    raw = rows.view(torch.uint8)
    pay = torch.cat([raw[:, :head].reshape(-1), raw.reshape(-1)]) if head else raw.reshape(-1)
    W = (rng.standard_normal((b, d)) / np.sqrt(d)).astype(np.float32)
    scale = 1 / 255 if dtype == NR.NR_U8 else 1.0
    tau = np.zeros(b, np.float32)
    ix = NR.Index(n=n, d=d, dtype=dtype, b=b, weights=[W], biases=[np.zeros(b, np.float32)],
                  input_scale=scale, tau=tau, rows=pay.contiguous(),
                  row_ids=torch.randperm(n, generator=g, device="cuda"),
                  bc_off=torch.from_numpy(bc.astype(np.int32)).cuda(),
                  cl_off=torch.from_numpy(cl.astype(np.int64)).cuda(),
                  centroids=torch.randn((len(nz), b), generator=g, device="cuda"),
                  head_bytes=head, head_copy=int(head > 0))
    return ix, rows


def both(ix, q, k, P, b, **kw):
    from paper_2608_15438_amd import neuroute as NR
    r = [ix.nr_search(q, k, P, NR.Params(l_sel=b, r_max=b, k_c=64, refine_mode=m, **kw))
         for m in (NR.NR_REFINE_PER_QUERY, NR.NR_REFINE_SHARED)]
    assert torch.equal(r[0][0], r[1][0])
    assert torch.equal(r[0][1], r[1][1])
    return r[1]


@pytest.mark.parametrize("dtype,d,head", [("u8", 16, 0), ("u8", 128, 16), ("f32", 24, 64),
                                          ("f32", 260, 0)])
@pytest.mark.parametrize("n,b,nq,P,seed_rows", [
    (500, 3, 70, 8, 64),          # less work than one smallest tile per wave
    (60_001, 8, 2049, 256, 64),   # tiles between the smallest and the largest
    (60_001, 8, 300, 100, 0),     # the default seed
])
def test_shared_equals_per_query(dtype, d, head, n, b, nq, P, seed_rows):
    from paper_2608_15438_amd import neuroute as NR
    dt = NR.NR_U8 if dtype == "u8" else NR.NR_F32
    ix, rows = make_index(n, d, b, dt, head)
    g = torch.Generator(device="cuda").manual_seed(1)
    at = torch.randint(0, n, (nq,), generator=g, device="cuda")
    q = rows[at].clone()
    for k in (1, 10, 64):
        ids, dists = both(ix, q, k, P, b, shared_seed_rows=seed_rows)
        if k == 10:   # against plain distances to the rows listed
            pos = torch.empty(n, dtype=torch.int64, device="cuda")
            pos[ix.dev[1]] = torch.arange(n, device="cuda")
            ok = ids >= 0
            x = rows[pos[ids.clamp_min(0)]].double()
            want = ((x - q[:, None].double()) ** 2).sum(-1)
            # fp32 sums of d squares: relative error at most d roundings
            assert ((want - dists.double()).abs() <= d * 2.0 ** -23 * want + 1e-30)[ok].all()
    ix.close()


@pytest.mark.parametrize("dtype,d,nq,P", [
    ("f32", 24, 700, 3), ("f32", 24, 3000, 60), ("f32", 24, 3000, 90), ("f32", 256, 1500, 4),
    ("f32", 260, 700, 4), ("f32", 260, 700, 60), ("u8", 64, 700, 12), ("u8", 64, 3000, 30),
    ("u8", 64, 3000, 40), ("u8", 1024, 700, 4), ("u8", 1040, 700, 4)])
def test_default_seeds(dtype, d, nq, P):
    # lists of 0.7k to 21k rows, batches on both sides of 1.5 GB, rows on both of 1 KB
    from paper_2608_15438_amd import neuroute as NR
    ix, rows = make_index(60_001, d, 8, NR.NR_F32 if dtype == "f32" else NR.NR_U8, 64, seed=d)
    g = torch.Generator(device="cuda").manual_seed(P)
    q = rows[torch.randint(0, 60_001, (nq,), generator=g, device="cuda")].clone()
    for k in (10, 64):
        both(ix, q, k, P, 8)
    ix.close()


def test_shared_equals_per_query_large_scan():
    # more work (rows x groups of 8 queries) than 4 tiles of 4096 per wave
    from paper_2608_15438_amd import neuroute as NR
    ix, rows = make_index(150_000, 16, 8, NR.NR_U8, 0)
    g = torch.Generator(device="cuda").manual_seed(1)
    q = rows[torch.randint(0, 150_000, (8192,), generator=g, device="cuda")].clone()
    both(ix, q, 10, 256, 8, shared_seed_rows=256)
    ix.close()


@pytest.mark.parametrize("d", [272, 528, 1536])
@pytest.mark.parametrize("k", [1, 10, 64])
def test_uint8_keys_past_2_24(d, k):
    # squared distances of whole numbers that fp32 no longer tells apart: both
    # schedules order rows by the exact ones
    from paper_2608_15438_amd import neuroute as NR
    n, nq = 6000, 600
    ix, rows = make_index(n, d, 5, NR.NR_U8, 0, seed=d)
    g = torch.Generator(device="cuda").manual_seed(k)
    rows.copy_(torch.randint(0, 2, (n, d), generator=g, device="cuda"))
    q = torch.randint(253, 256, (nq, d), generator=g, device="cuda").to(torch.uint8)
    ids, dists = both(ix, q, k, 32, 5, shared_seed_rows=64)
    pos = torch.empty(n, dtype=torch.int64, device="cuda")
    pos[ix.dev[1]] = torch.arange(n, device="cuda")
    dist = (q[:, None].long() - rows[pos[ids]].long()).square().sum(-1)
    assert dist.min() > 1 << 24
    key = dist * (1 << 20) + ids
    assert (key[:, 1:] > key[:, :-1]).all()
    ix.close()


@pytest.mark.parametrize("nq", [1, 5, 48, 300, 700])
@pytest.mark.parametrize("k", [1, 9, 32, 33, 64])
@pytest.mark.parametrize("dtype,d,n", [("u8", 16, 7001), ("u8", 144, 3000), ("f32", 4, 5000),
                                       ("f32", 320, 900)])
def test_ties_order_by_id(nq, k, dtype, d, n):
    # rows of few values, so that most distances tie: every list is the exact
    # (distance, id) order, whichever way its entries came in
    from paper_2608_15438_amd import neuroute as NR
    ix, rows = make_index(n, d, 4, NR.NR_U8 if dtype == "u8" else NR.NR_F32, 0, seed=nq)
    g = torch.Generator(device="cuda").manual_seed(k)
    small = torch.randint(0, 2, (n, d), generator=g, device="cuda")
    small[: n // 3] = small[0].clone()
    rows.copy_(small.to(rows.dtype))               # in place: the payload is these rows
    q = rows[torch.randint(0, n, (nq,), generator=g, device="cuda")].clone()
    ids, dists = ix.nr_search(q, k, 16, NR.Params(l_sel=4, r_max=4, k_c=64, shared_seed_rows=64))
    rid = ix.dev[1]
    dist = torch.cdist(q.double(), rows.double()).square().round()   # whole numbers
    key, at = (dist * (1 << 20) + rid).sort(dim=1)
    assert torch.equal(ids, rid[at[:, :k]])
    assert torch.equal(dists.double(), dist.gather(1, at[:, :k]))
    ix.close()


@pytest.mark.parametrize("b,per,P,s_max", [(6, 9, 64, 0.0), (7, 3, 40, 0.0), (6, 30, 64, 4.0),
                                           (5, 1, 32, 0.0), (9, 80, 300, 0.0)])
@pytest.mark.parametrize("nq", [33, 600])
def test_one_gate_equals_batches(b, per, P, s_max, nq):
    # queries whose heap cannot fill are gated once, those that report their
    # counters go batch by batch: the same lists, around the K_c where the two part
    from paper_2608_15438_amd import neuroute as NR
    ix, rows = make_index(20_000, 16, b, NR.NR_F32, 0, seed=b, per=per)
    q = rows[:nq].clone()
    kw = dict(l_sel=b, r_max=b, m_x=[0.0, 4.0], m_y=[1.0, 3.0], shared_seed_rows=64)
    if s_max:
        kw.update(s_max=s_max, n_bins=8)
    stats = ix.nr_search(q, 10, P, NR.Params(k_c=16000, **kw), qstats=True)[2]
    scored = sorted(set(stats[:, 3].tolist()))
    for kc in {1, 64, 512, 600, 2100} | {max(1, scored[len(scored) // 2] + o) for o in (-1, 0, 1)}:
        for stop in (True, False):
            p = NR.Params(k_c=kc, early_stop_on=stop, **kw)
            a = ix.nr_search(q, 10, P, p)
            r = ix.nr_search(q, 10, P, p, qstats=True)
            assert torch.equal(a[0], r[0]) and torch.equal(a[1], r[1]), (kc, stop)
    ix.close()
