"""GPU path (libneuroute.so through its C ABI) against the CPU oracle on the
same seeded inputs.  Given the oracle's logits, probe sequences, candidate
cluster lists and top-k ids are bit-exact; uint8 distances are exact, fp32
distances within 1e-5 relative; encoder logits within 1e-4 of the magnitude
of their terms."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2608_15438_amd import neuroute as NR
from tests.instances import instance, oracle_encoder, split_index
from tests.topk_check import allowed_ids, check_topk

pytestmark = pytest.mark.gpu

CASES = {
    "tiny": (1, 0, 0, ()),
    "sift": (2, 60_000, 300, (("widths", (128, 256, 12)),)),
    "deep": (3, 40_000, 200, (("widths", (96, 256, 12)), ("capacity", 30))),
    # the ablation without bucket-local clustering (every bucket one cluster)
    "sift_noclust": (2, 60_000, 300, (("widths", (128, 256, 12)), ("cluster_rule", "none"))),
    # 1536-d fp32 rows (6 KB) through a five-layer encoder
    "gld": (5, 20_000, 100, (("widths", (1536, 512, 256, 128, 64, 10)),)),
}


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    return torch.device("cuda")


_cache = {}


def setup_case(name, dev):
    if name not in _cache:
        cfg, n, nq, ov = CASES[name]
        w, ix, X, Q = instance(cfg, n, nq, **dict(ov))
        gix = NR.Index.from_built(ix, dev)
        gix_split = NR.Index.from_built(split_index(ix, dev), dev)
        gix_copy = NR.Index.from_built(split_index(ix, dev, copy=True), dev)
        enc = oracle_encoder(ix)
        lg, mag = O.encode(enc, Q, with_mag=True)
        _cache[name] = dict(w=w, ix=ix, X=X, Q=Q, gix=gix, gix_split=gix_split,
                            gix_copy=gix_copy, enc=enc, lg=lg, mag=mag,
                            Qd=torch.from_numpy(Q).to(dev), lgd=torch.from_numpy(lg).to(dev))
    return _cache[name]


def oracle_params(p: NR.Params) -> O.RouteParams:
    return O.RouteParams(n_bins=p.n_bins, s_max=p.s_max, k_c=p.k_c, b_batch=p.b_batch,
                         b_min=p.b_min, t_low=p.t_low, u_heap=p.u_heap, u_front=p.u_front,
                         alpha_front=p.alpha_front, gate_on=p.gate_on,
                         early_stop_on=p.early_stop_on, lowq_or=p.lowq_or,
                         m_x=np.array(p.m_x, np.float32), m_y=np.array(p.m_y, np.float32))


def default_params(case, **kw):
    w = case["w"]
    base = dict(l_sel=min(w.b, 16), r_max=w.r_max, k_c=w.k_c, m_x=[0.0, 4.0], m_y=[1.0, 3.0])
    base.update(kw)
    return NR.Params(**base)


PARAM_SETS = {
    "default": {},
    "no_gate_no_stop": dict(gate_on=False, early_stop_on=False),
    "small_heap_fast_stop": dict(k_c=5, b_batch=3, b_min=1, t_low=1),
    "or_reading": dict(k_c=8, b_batch=7, b_min=1, t_low=2, lowq_or=True),
    "and_reading": dict(k_c=8, b_batch=7, b_min=1, t_low=2, lowq_or=False),
    # the front threshold decides under the OR reading: a wide and a narrow front
    "front_wide": dict(k_c=8, b_batch=5, b_min=1, t_low=1, alpha_front=0.95),
    "front_narrow": dict(k_c=8, b_batch=5, b_min=1, t_low=1, alpha_front=0.05),
    "binned": dict(s_max=1.5, n_bins=6),
    "one_per_batch": dict(b_batch=1, k_c=16),
    # margins through several knots: the segment search and both clamps
    "many_knots": dict(m_x=[0.0, 0.5, 1.5, 3.0, 6.0], m_y=[0.2, 0.8, 1.5, 2.2, 3.0]),
    "knots_flat": dict(m_x=[0.0, 0.3, 0.9, 2.0], m_y=[0.4, 1.2, 1.2, 2.5], k_c=12, b_batch=5),
    # margins below zero: a query near a centroid ends with no gated cluster
    "margin_below_zero": dict(m_x=[0.0, 4.0], m_y=[-3.0, 3.0], early_stop_on=False),
    "margin_below_zero_batches": dict(m_x=[0.0, 2.0], m_y=[-2.0, 5.0], k_c=40, b_batch=5),
    # a heap this large leaves LDS for only the first ~600 probe ranges of a
    # query: the rest of a 1024-probe sequence is read from HBM
    "big_heap": dict(k_c=5000, gate_on=False, early_stop_on=False),
    # K_c past the first pass's 512 heap keys: long queries go to a pass with
    # a K_c-key heap, whose unsorted pool is sorted when it could reach K_c,
    # after which the heap fills and the stop can fire
    "mid_heap_stop": dict(k_c=600, b_batch=16, b_min=2, t_low=1, gate_on=False),
    # K_c past 2048: three passes (512, 2048 and K_c keys)
    "three_tiers": dict(k_c=3000, b_batch=32, gate_on=False, early_stop_on=False),
}


# ------------------------------------------------------------------ step 1
@pytest.mark.parametrize("name", list(CASES))
def test_encoder_logits(dev, name):
    c = setup_case(name, dev)
    got = c["gix"].nr_encode(c["Qd"]).cpu().numpy()
    err = np.abs(got.astype(np.float64) - c["lg"])
    assert np.all(err <= 1e-4 * c["mag"] + 1e-30), float((err / c["mag"]).max())


@pytest.mark.parametrize("widths,dtype,nq,offset", [
    ((36, 50, 13), "f32", 301, 0),     # a hidden width not a multiple of 4: one element per load
    ((32, 64, 9), "f32", 77, 1),       # a query block not 16-byte aligned
    ((32, 66, 30, 9), "u8", 130, 0),   # uint8 rows, odd hidden widths, three layers
    ((128, 256, 24), "u8", 1500, 0),   # the 1B encoder's shape: 32 x 64 tiles, then the code layer
    ((96, 512, 20), "f32", 8200, 0),   # 64 x 64 tiles (the grid fills the chip)
])
def test_encoder_layer_shapes(dev, widths, dtype, nq, offset):
    """Seeded encoders with BatchNorm on the hidden layers, against the
    oracle within 1e-4 of each logit's magnitude: the tile shapes the layer
    sizes select, the four-element loads and the one-element path."""
    from paper_2608_15438_amd import index_build as IB
    rng = np.random.default_rng(sum(widths) + nq)
    L = len(widths) - 1
    Ws = [(rng.standard_normal((widths[l + 1], widths[l])) / np.sqrt(widths[l])).astype(np.float32)
          for l in range(L)]
    bs = [(0.1 * rng.standard_normal(widths[l + 1])).astype(np.float32) for l in range(L)]
    sc = [(1.0 + 0.2 * rng.standard_normal(widths[l + 1])).astype(np.float32) for l in range(L - 1)]
    sh = [(0.1 * rng.standard_normal(widths[l + 1])).astype(np.float32) for l in range(L - 1)]
    scale = 1.0 / 255.0 if dtype == "u8" else 1.0
    enc = IB.Encoder(Ws, bs, scale, sc, sh)
    if dtype == "u8":
        Q = rng.integers(0, 256, size=(nq, widths[0]), dtype=np.uint8)
    else:
        Q = rng.standard_normal((nq, widths[0])).astype(np.float32)
    exp, mag = O.encode(O.Encoder(Ws, bs, sc, sh, scale), Q, with_mag=True)
    gix = NR.Index.encoder_only(enc, NR.NR_U8 if dtype == "u8" else NR.NR_F32)
    flat = torch.from_numpy(np.ascontiguousarray(Q)).reshape(-1)
    buf = torch.zeros(flat.numel() + offset, dtype=flat.dtype, device=dev)
    buf[offset:] = flat.to(dev)
    Qd = buf[offset:].view(nq, widths[0])
    got = gix.nr_encode(Qd).cpu().numpy()
    gix.close()
    err = np.abs(got.astype(np.float64) - exp)
    assert np.all(err <= 1e-4 * mag + 1e-30), float((err / mag).max())


# ------------------------------------------------------------------ step 2
@pytest.mark.parametrize("name", list(CASES))
@pytest.mark.parametrize("P", [1, 7, 64, 300, 1024, 2048, 4096])
@pytest.mark.parametrize("pset", ["default", "binned"])
def test_probe_sequence_bit_exact(dev, name, P, pset):
    c = setup_case(name, dev)
    p = default_params(c, **PARAM_SETS[pset])
    gc, gs, gb, gn = [t.cpu().numpy() for t in c["gix"].nr_probe(c["lgd"], P, p)]
    oc, os_, ob, on = O.probes(c["lg"], c["ix"].tau, p.l_sel, p.r_max, P, p.s_max, p.n_bins)
    assert np.array_equal(gn, on)
    for q in range(len(on)):
        n = on[q]
        assert np.array_equal(gc[q, :n].view(np.uint32), oc[q, :n]), q
        assert np.array_equal(gs[q, :n], os_[q, :n]), q
        assert np.array_equal(gb[q, :n], ob[q, :n]), q


@pytest.mark.parametrize("P", [2048, 4096])
@pytest.mark.parametrize("r_max,s_max,n_bins", [(7, float("inf"), 1), (16, 6.0, 40)])
def test_probe_long_sequences_bit_exact(dev, P, r_max, s_max, n_bins):
    """Sequences of up to 4096 probes over 16 selected dimensions of a 20-bit
    code (26,333 flip sets of radius <= 7), from seeded logits; the lists of
    the merge recursion fill 96 KiB of LDS at P = 4096."""
    b, d, nq = 20, 16, 64
    rng = np.random.default_rng(4096 + P)
    lg = rng.normal(0.0, 1.0, size=(nq, b)).astype(np.float32)
    tau = rng.normal(0.0, 0.2, size=b).astype(np.float32)
    bc_off = np.ones((1 << b) + 1, np.int32)
    bc_off[0] = 0
    gix = NR.Index(n=1, d=d, dtype=NR.NR_U8, b=b, weights=[np.zeros((b, d), np.float32)],
                   biases=[np.zeros(b, np.float32)], input_scale=1.0, tau=tau,
                   rows=torch.zeros((1, d), dtype=torch.uint8, device=dev),
                   row_ids=torch.zeros(1, dtype=torch.int64, device=dev),
                   bc_off=torch.from_numpy(bc_off).to(dev),
                   cl_off=torch.tensor([0, 1], dtype=torch.int64, device=dev),
                   centroids=torch.zeros((1, b), dtype=torch.float32, device=dev))
    p = NR.Params(l_sel=16, r_max=r_max, s_max=s_max, n_bins=n_bins)
    gc, gs, gb, gn = [t.cpu().numpy() for t in gix.nr_probe(torch.from_numpy(lg).to(dev), P, p)]
    oc, os_, ob, on = O.probes(lg, tau, 16, r_max, P, s_max, n_bins)
    assert np.array_equal(gn, on)
    if r_max == 7:
        assert np.all(on == P)
    for q in range(nq):
        n = on[q]
        assert np.array_equal(gc[q, :n].view(np.uint32), oc[q, :n]), q
        assert np.array_equal(gs[q, :n], os_[q, :n]), q
        assert np.array_equal(gb[q, :n], ob[q, :n]), q
    gix.close()


def test_probe_full_budget_covers_all_codes(dev):
    c = setup_case("tiny", dev)
    p = default_params(c, l_sel=8, r_max=8)
    gc, gs, gb, gn = [t.cpu().numpy() for t in c["gix"].nr_probe(c["lgd"], 256, p)]
    assert np.all(gn == 256)
    for q in range(len(gn)):
        assert sorted(gc[q].tolist()) == list(range(256))



def _alg1_cases():
    import os
    rows = []
    path = os.path.join(os.path.dirname(__file__), "golden", "alg1_worked_examples.txt")
    for line in open(path):
        if line.strip() and not line.startswith("#"):
            f = [c.strip() for c in line.split("|")]
            rows.append(dict(name=f[0], b=int(f[1]), tau=np.array(f[2].split(), np.float32),
                             logits=np.array(f[3].split(), np.float32), l_sel=int(f[4]),
                             r_max=int(f[5]), s_max=float(f[6]), n_bins=int(f[7]), P=int(f[8]),
                             codes=[int(x) for x in f[9].split()],
                             costs=[float(x) for x in f[10].split()],
                             bins=[int(x) for x in f[11].split()]))
    return rows


@pytest.mark.parametrize("ex", _alg1_cases(), ids=lambda e: e["name"])
def test_probe_worked_examples(dev, ex):
    """The hand-worked Alg. 1 sequences (ties, a logit exactly at tau, finite
    S_max with bins) on the GPU, through a one-row index with that tau."""
    b, d = ex["b"], 16
    bc_off = np.ones((1 << b) + 1, np.int32)
    bc_off[0] = 0
    gix = NR.Index(n=1, d=d, dtype=NR.NR_U8, b=b, weights=[np.zeros((b, d), np.float32)],
                   biases=[np.zeros(b, np.float32)], input_scale=1.0, tau=ex["tau"],
                   rows=torch.zeros((1, d), dtype=torch.uint8, device=dev),
                   row_ids=torch.zeros(1, dtype=torch.int64, device=dev),
                   bc_off=torch.from_numpy(bc_off).to(dev),
                   cl_off=torch.tensor([0, 1], dtype=torch.int64, device=dev),
                   centroids=torch.zeros((1, b), dtype=torch.float32, device=dev))
    p = NR.Params(l_sel=ex["l_sel"], r_max=ex["r_max"], s_max=ex["s_max"], n_bins=ex["n_bins"])
    lg = torch.from_numpy(ex["logits"][None].copy()).to(dev)
    gc, gs, gb, gn = [t.cpu().numpy() for t in gix.nr_probe(lg, ex["P"], p)]
    n = int(gn[0])
    assert n == len(ex["codes"])
    assert gc[0, :n].view(np.uint32).tolist() == ex["codes"]
    assert gs[0, :n].tolist() == ex["costs"]
    assert gb[0, :n].tolist() == ex["bins"]
    gix.close()

# ------------------------------------------------------------------ steps 3-4
@pytest.mark.parametrize("name", list(CASES))
@pytest.mark.parametrize("pset", list(PARAM_SETS))
@pytest.mark.parametrize("P", [4, 64, 512, 4096])
def test_candidate_clusters_bit_exact(dev, name, pset, P):
    c = setup_case(name, dev)
    p = default_params(c, **PARAM_SETS[pset])
    clus, n = c["gix"].nr_route(c["lgd"], P, p)
    clus, n = clus.cpu().numpy().view(np.uint32), n.cpu().numpy()
    oc, os_, ob, on = O.probes(c["lg"], c["ix"].tau, p.l_sel, p.r_max, P, p.s_max, p.n_bins)
    lists = O.route(c["lg"], oc, ob, on, c["ix"].bc_off, c["ix"].centroids, oracle_params(p))
    for q, L in enumerate(lists):
        assert n[q] == len(L), q
        assert np.array_equal(clus[q, :n[q]], L), q



def _worked_cases():
    import os
    rows = []
    path = os.path.join(os.path.dirname(__file__), "golden", "alg2_worked_example.txt")
    for line in open(path):
        if line.strip() and not line.startswith("#"):
            f = [c.strip() for c in line.split("|")]
            rows.append(dict(name=f[0], k_c=int(f[1]), t_low=int(f[2]), es=int(f[3]),
                             lowq_or=int(f[4]), exp=[int(x) for x in f[5].split()],
                             alpha=float(f[7])))
    return rows


@pytest.mark.parametrize("case", _worked_cases(), ids=lambda c: c["name"])
def test_route_worked_example(dev, case):
    """The hand-worked Alg. 2 cases on the GPU.  Three code bits with
    deviations 1, 2, 4 make the probe sequence codes 0..6 in order, one bin
    each; every centroid differs from the query's logits in dimension 0 only,
    by mu, so d_cent = mu^2 exactly, as in the one-dimensional example."""
    mu = np.array([1, 2, 3, 100, 0.5, 4, 5, 6, 100, 7, 8, 100], np.float32)
    lg = np.array([[-1.0, -2.0, -4.0]], np.float32)
    cent = np.stack([lg[0, 0] - mu, np.full(12, lg[0, 1]), np.full(12, lg[0, 2])], 1)
    cent = np.ascontiguousarray(cent, np.float32)
    n, d = 12, 16
    bc_off = np.array([0, 3, 4, 6, 8, 9, 11, 12, 12], np.int32)
    gix = NR.Index(n=n, d=d, dtype=NR.NR_U8, b=3, weights=[np.zeros((3, d), np.float32)],
                   biases=[np.zeros(3, np.float32)], input_scale=1.0, tau=np.zeros(3, np.float32),
                   rows=torch.zeros((n, d), dtype=torch.uint8, device=dev),
                   row_ids=torch.arange(n, dtype=torch.int64, device=dev),
                   bc_off=torch.from_numpy(bc_off).to(dev),
                   cl_off=torch.arange(n + 1, dtype=torch.int64, device=dev),
                   centroids=torch.from_numpy(cent).to(dev))
    # M(x) = 10 everywhere: two knots with a flat segment
    p = NR.Params(l_sel=3, r_max=3, k_c=case["k_c"], b_batch=2, b_min=1, t_low=case["t_low"],
                  u_heap=1, u_front=1, alpha_front=case["alpha"], gate_on=True,
                  early_stop_on=bool(case["es"]), lowq_or=bool(case["lowq_or"]),
                  m_x=[0.0, 1.0], m_y=[10.0, 10.0])
    gc, _, gb, gn = [t.cpu().numpy() for t in gix.nr_probe(torch.from_numpy(lg).to(dev), 7, p)]
    assert gn[0] == 7 and gc[0].view(np.uint32).tolist() == list(range(7))
    assert gb[0].tolist() == list(range(7))
    clus, cnt = gix.nr_route(torch.from_numpy(lg).to(dev), 7, p)
    got = clus.cpu().numpy()[0, :int(cnt[0])].tolist()
    assert got == case["exp"]
    oc, _, ob, on = O.probes(lg, np.zeros(3, np.float32), 3, 3, 7, p.s_max, p.n_bins)
    assert O.route(lg, oc, ob, on, bc_off.astype(np.uint32), cent, oracle_params(p))[0].tolist() \
        == case["exp"]
    gix.close()

# ------------------------------------------------------------------ step 5
def _assert_topk(c, gi, gd, oi, od, lists=None, ix=None):
    """uint8: ids and distances equal.  fp32: the checks of check_topk (valid
    top-k, near-ties only); lists (the oracle's C(q)) bound the allowed ids."""
    ix = ix if ix is not None else c.get("ix")
    allowed = None
    if lists is not None and ix is not None:
        allowed = lambda q: allowed_ids(ix.cl_off, ix.row_ids, lists[q])
    X = c["X"]
    check_topk(gi, gd, oi, od, is_u8=c["w"].dtype == "u8", X_by_id=lambda ids: X[ids],
               Q=c["Q"], allowed=allowed)


def _oracle_lists(c, p, P):
    """The oracle's C(q) for every query of the case (Alg. 1, then Alg. 2)."""
    oc, _, ob, on = O.probes(c["lg"], c["ix"].tau, p.l_sel, p.r_max, P, p.s_max, p.n_bins)
    return O.route(c["lg"], oc, ob, on, c["ix"].bc_off, c["ix"].centroids, oracle_params(p))


@pytest.mark.parametrize("layout", ["gix", "gix_split", "gix_copy"])
@pytest.mark.parametrize("name", list(CASES))
@pytest.mark.parametrize("k", [1, 10, 64])
def test_refine_given_clusters(dev, name, k, layout):
    c = setup_case(name, dev)
    p = default_params(c)
    P = 128
    oc, os_, ob, on = O.probes(c["lg"], c["ix"].tau, p.l_sel, p.r_max, P)
    lists = O.route(c["lg"], oc, ob, on, c["ix"].bc_off, c["ix"].centroids, oracle_params(p))
    cap = max(1, max(len(L) for L in lists))
    cl = np.zeros((len(lists), cap), np.uint32)
    n = np.zeros(len(lists), np.int32)
    for q, L in enumerate(lists):
        cl[q, :len(L)] = L
        n[q] = len(L)
    gi, gd = c[layout].nr_refine(c["Qd"], k, torch.from_numpy(cl.view(np.int32)).to(dev),
                                 torch.from_numpy(n).to(dev))
    oi, od, _ = O.refine(c["ix"].rows, c["ix"].row_ids, c["ix"].cl_off, c["Q"], lists, k)
    _assert_topk(c, gi.cpu().numpy(), gd.cpu().numpy(), oi, od, lists=lists)


# every refine kernel shape by row length: rows past 8 x 128 bytes keep the
# query in LDS and accumulate 8 segments at a time (in the scan, one 1 KB slab
# of the batch's queries at a time); lengths that are not a
# multiple of 128 bytes (they are multiples of 16) leave a ragged last segment
@pytest.mark.parametrize("cfg,d", [(3, 300), (3, 384), (3, 700), (3, 1536),
                                   (2, 1104), (2, 2048), (2, 4096)])
@pytest.mark.parametrize("layout", ["gix", "gix_split"])
def test_refine_row_lengths(dev, cfg, d, layout):
    ov = dict(d=d, widths=(d, 64, 8), n_centers=30, cluster_rule="capacity", capacity=30)
    w, ix, X, Q = instance(cfg, 3000, 40, **ov)
    gix = NR.Index.from_built(ix if layout == "gix" else split_index(ix, dev), dev)
    rng = np.random.default_rng(7 + d)
    nc = len(ix.cl_off) - 1
    cap = min(nc, 48)
    lists = [np.sort(rng.choice(nc, size=int(rng.integers(0, cap + 1)), replace=False))
             for _ in range(len(Q))]
    cl = np.zeros((len(Q), cap), np.uint32)
    n = np.zeros(len(Q), np.int32)
    for q, L in enumerate(lists):
        cl[q, :len(L)] = L
        n[q] = len(L)
    for k in (1, 10, 64):
        gi, gd = gix.nr_refine(torch.from_numpy(Q).to(dev), k,
                               torch.from_numpy(cl.view(np.int32)).to(dev),
                               torch.from_numpy(n).to(dev))
        oi, od, _ = O.refine(ix.rows, ix.row_ids, ix.cl_off, Q,
                             [L.astype(np.uint32) for L in lists], k)
        _assert_topk(dict(w=w, X=X, Q=Q), gi.cpu().numpy(), gd.cpu().numpy(), oi, od,
                     lists=lists, ix=ix)
    # the whole search: the batch-shared schedule (seed pass of 64 rows, the
    # rest through the scan) returns exactly the per-query schedule's lists
    Qd = torch.from_numpy(Q).to(dev)
    base = dict(l_sel=8, r_max=4, k_c=64, m_x=[0.0, 4.0], m_y=[1.0, 3.0])
    for P in (16, 128):
        pi, pd = gix.nr_search(Qd, 10, P, NR.Params(refine_mode=NR.NR_REFINE_PER_QUERY, **base))
        si, sd = gix.nr_search(Qd, 10, P, NR.Params(refine_mode=NR.NR_REFINE_SHARED,
                                                    shared_seed_rows=64, **base))
        assert gix.nr_last_work()["shared_pairs"] > 0
        assert torch.equal(pi, si) and torch.equal(pd, sd)


# ------------------------------------------------------------------ whole path
# refinement schedule x payload layout; the shared schedule with a tiny seed
# sends nearly every candidate cluster through the scan, even on small cases
MODES = {"per_query": ("gix", dict(refine_mode=NR.NR_REFINE_PER_QUERY)),
         "shared": ("gix", dict(refine_mode=NR.NR_REFINE_SHARED)),
         "shared_seed64": ("gix", dict(refine_mode=NR.NR_REFINE_SHARED, shared_seed_rows=64)),
         "split_per_query": ("gix_split", dict(refine_mode=NR.NR_REFINE_PER_QUERY)),
         "split_shared_seed64": ("gix_split", dict(refine_mode=NR.NR_REFINE_SHARED,
                                                   shared_seed_rows=64)),
         "copy_per_query": ("gix_copy", dict(refine_mode=NR.NR_REFINE_PER_QUERY)),
         "copy_shared_seed64": ("gix_copy", dict(refine_mode=NR.NR_REFINE_SHARED,
                                                 shared_seed_rows=64))}


@pytest.mark.parametrize("mode", list(MODES))
@pytest.mark.parametrize("name", list(CASES))
@pytest.mark.parametrize("pset", ["default", "no_gate_no_stop", "small_heap_fast_stop", "binned"])
@pytest.mark.parametrize("P", [1, 16, 256])
def test_search_given_logits_bit_exact(dev, name, pset, P, mode):
    c = setup_case(name, dev)
    p = default_params(c, **MODES[mode][1], **PARAM_SETS[pset])
    gi, gd = c[MODES[mode][0]].nr_search(c["Qd"], 10, P, p, logits=c["lgd"])
    ix = c["ix"]
    oi, od, _, _ = O.search(c["enc"], ix.tau, ix.rows, ix.row_ids, ix.bc_off, ix.cl_off,
                            ix.centroids, c["Q"], 10, p.l_sel, p.r_max, P, oracle_params(p),
                            n_threads=4)
    _assert_topk(c, gi.cpu().numpy(), gd.cpu().numpy(), oi, od, lists=_oracle_lists(c, p, P))


@pytest.mark.parametrize("mode", ["per_query", "shared", "shared_seed64"])
@pytest.mark.parametrize("name", ["sift", "deep", "gld"])
@pytest.mark.parametrize("P", [2048, 4096])
def test_search_long_probe_sequences(dev, name, P, mode):
    """The whole path at the largest probe budgets."""
    c = setup_case(name, dev)
    p = default_params(c, **MODES[mode][1])
    gi, gd = c[MODES[mode][0]].nr_search(c["Qd"], 10, P, p, logits=c["lgd"])
    ix = c["ix"]
    oi, od, _, _ = O.search(c["enc"], ix.tau, ix.rows, ix.row_ids, ix.bc_off, ix.cl_off,
                            ix.centroids, c["Q"], 10, p.l_sel, p.r_max, P, oracle_params(p),
                            n_threads=4)
    _assert_topk(c, gi.cpu().numpy(), gd.cpu().numpy(), oi, od, lists=_oracle_lists(c, p, P))


@pytest.mark.parametrize("mode", list(MODES))
def test_full_budget_search_is_exact_knn(dev, mode):
    c = setup_case("tiny", dev)
    p = default_params(c, l_sel=8, r_max=8, gate_on=False, early_stop_on=False, k_c=10 ** 9,
                       **MODES[mode][1])
    gi, gd = c[MODES[mode][0]].nr_search(c["Qd"], 10, 256, p)
    bi, bd = O.bruteforce(c["X"], c["Q"], 10)
    _assert_topk(c, gi.cpu().numpy(), gd.cpu().numpy(), bi, bd)


@pytest.mark.parametrize("name", list(CASES))
def test_search_with_gpu_encoder(dev, name):
    """nr_search = nr_encode then the rest; it agrees with the oracle's own
    logits except where a logit sits within rounding of a decision."""
    c = setup_case(name, dev)
    p = default_params(c)
    gi, gd = c["gix"].nr_search(c["Qd"], 10, 64, p)
    lg = c["gix"].nr_encode(c["Qd"])
    gi2, gd2 = c["gix"].nr_search(c["Qd"], 10, 64, p, logits=lg)
    assert torch.equal(gi, gi2) and torch.equal(gd, gd2)
    oi, _, _, _ = O.search(c["enc"], c["ix"].tau, c["ix"].rows, c["ix"].row_ids, c["ix"].bc_off,
                           c["ix"].cl_off, c["ix"].centroids, c["Q"], 10, p.l_sel, p.r_max, 64,
                           oracle_params(p), n_threads=4)
    assert O.recall_at_k(gi.cpu().numpy(), oi, 10) >= 0.98


# ------------------------------------------------------------------ edge cases
def test_empty_and_single_query(dev):
    c = setup_case("sift", dev)
    p = default_params(c)
    gi, gd = c["gix"].nr_search(c["Qd"][:0], 10, 16, p)
    assert gi.shape == (0, 10)
    gi, gd = c["gix"].nr_search(c["Qd"][:1], 10, 16, p, logits=c["lgd"][:1])
    oi, od, _, _ = O.search(c["enc"], c["ix"].tau, c["ix"].rows, c["ix"].row_ids, c["ix"].bc_off,
                            c["ix"].cl_off, c["ix"].centroids, c["Q"][:1], 10, p.l_sel, p.r_max,
                            16, oracle_params(p))
    _assert_topk(c, gi.cpu().numpy(), gd.cpu().numpy(), oi, od,
                 lists=[_oracle_lists(c, p, 16)[0]])


def test_short_lists_are_padded(dev):
    """One probe into a small bucket: fewer than k candidates."""
    c = setup_case("sift", dev)
    p = default_params(c)
    gi, gd, qs = c["gix"].nr_search(c["Qd"], 64, 1, p, logits=c["lgd"], qstats=True)
    gi, gd, qs = gi.cpu().numpy(), gd.cpu().numpy(), qs.cpu().numpy()
    rows = qs[:, NR.QS["rows"]]
    assert np.any(rows < 64)
    for q in range(len(gi)):
        m = min(64, rows[q])
        assert np.all(gi[q, :m] >= 0) and np.all(gi[q, m:] == -1)
        assert np.all(np.isinf(gd[q, m:]))


@pytest.mark.parametrize("mode", list(MODES))
def test_many_queries_span_chunks(dev, mode):
    """More queries than one internal launch sequence handles."""
    c = setup_case("tiny", dev)
    p = default_params(c, **MODES[mode][1])
    reps = 20000 // len(c["Q"]) + 1
    Q = np.tile(c["Q"], (reps, 1))
    lg = np.tile(c["lg"], (reps, 1))
    gi, gd = c[MODES[mode][0]].nr_search(torch.from_numpy(Q).to(dev), 10, 8, p,
                                logits=torch.from_numpy(lg).to(dev))
    gi = gi.cpu().numpy()
    n0 = len(c["Q"])
    for r in range(1, reps):
        assert np.array_equal(gi[r * n0:(r + 1) * n0], gi[:n0])


@pytest.mark.parametrize("mode", list(MODES))
def test_deterministic(dev, mode):
    c = setup_case("deep", dev)
    p = default_params(c, **MODES[mode][1])
    a = c[MODES[mode][0]].nr_search(c["Qd"], 10, 256, p)
    b = c[MODES[mode][0]].nr_search(c["Qd"], 10, 256, p)
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])


def test_argument_errors(dev):
    c = setup_case("tiny", dev)
    p = default_params(c)
    with pytest.raises(NR.NRError) as e:
        c["gix"].nr_search(c["Qd"], 0, 4, p)
    assert e.value.status == NR.NR_EINVAL
    with pytest.raises(NR.NRError) as e:
        c["gix"].nr_search(c["Qd"], 65, 4, p)
    assert e.value.status == NR.NR_EUNSUPPORTED
    with pytest.raises(NR.NRError) as e:
        c["gix"].nr_search(c["Qd"], 10, 0, p)
    assert e.value.status == NR.NR_EINVAL
    with pytest.raises(NR.NRError) as e:
        c["gix"].nr_search(c["Qd"], 10, 4, default_params(c, m_x=[1.0, 0.5], m_y=[0.0, 1.0]))
    assert e.value.status == NR.NR_EINVAL


@pytest.mark.parametrize("what", ["bc_off", "cl_off", "row_ids"])
def test_corrupt_index_rejected(dev, what):
    c = setup_case("tiny", dev)
    ix = c["ix"]
    bc = ix.bc_off.astype(np.int64).copy()
    cl = ix.cl_off.astype(np.int64).copy()
    ids = ix.row_ids.copy()
    if what == "bc_off":
        bc[5], bc[6] = bc[6] + 1, bc[5]
    elif what == "cl_off":
        cl[3] = cl[4] + 1
    else:
        ids[7] = ids[8]
    e = ix.encoder
    with pytest.raises(NR.NRError) as err:
        NR.Index(n=len(ids), d=ix.rows.shape[1], dtype=NR.NR_F32, b=len(ix.tau),
                 weights=e.weights, biases=e.biases, input_scale=e.input_scale, tau=ix.tau,
                 rows=torch.from_numpy(ix.rows).to(dev),
                 row_ids=torch.from_numpy(ids).to(dev),
                 bc_off=torch.from_numpy(bc.astype(np.int32)).to(dev),
                 cl_off=torch.from_numpy(cl).to(dev),
                 centroids=torch.from_numpy(ix.centroids).to(dev))
    assert err.value.status == NR.NR_ECORRUPT


@pytest.mark.parametrize("layout", ["gix", "gix_split", "gix_copy"])
@pytest.mark.parametrize("name", list(CASES))
def test_shared_schedule_work_counters(dev, name, layout):
    """The scan really runs on these cases (pairs, rows read whole,
    survivors), and its counters add up: every (query, cluster) pair is
    scored either by the query's seed pass or by the scan."""
    c = setup_case(name, dev)
    p = default_params(c, **MODES["shared_seed64"][1])
    gi, gd = c[layout].nr_search(c["Qd"], 10, 256, p, logits=c["lgd"])
    w = c[layout].nr_last_work()
    assert w["shared_pairs"] > 0 and w["survivors"] > 0 and w["full_rows"] > 0
    assert w["rows"] == w["own_rows"] + w["shared_pair_rows"]
    assert w["rows_read"] == w["own_rows"] + w["shared_rows"] + w["fallback_rows"]
    assert w["shared_rows"] <= w["shared_pair_rows"] and w["flagged"] == 0
    assert w["full_rows"] <= w["shared_pair_rows"]
    rb = c["w"].row_bytes
    if rb <= 1024:
        assert w["body_bytes"] == w["full_rows"] * rb
    else:  # the first 1 KB slab of every row read past its head; then, per
        # (row, query) pair it left open, the further slabs that pair needed
        assert w["body_bytes"] == w["full_rows"] * 1024
        assert w["open_bytes"] <= w["shared_pair_rows"] * (rb - 1024)
    if c["w"].dtype == "u8" or rb <= 1024:
        assert w["open_bytes"] == 0
        assert w["refine_bytes"] == (w["own_rows"] + w["fallback_rows"]) * rb
    else:
        assert 0 < w["refine_bytes"] <= (w["own_rows"] + w["fallback_rows"]) * rb
    assert w["head_bytes"] == 16 * (1 if c["w"].dtype == "u8" else 4)
    pi, pd = c[layout].nr_search(c["Qd"], 10, 256, default_params(c, **MODES["per_query"][1]),
                                 logits=c["lgd"])
    assert torch.equal(gi, pi) and torch.equal(gd, pd)
    w1 = c[layout].nr_last_work()
    assert w1["rows"] == w["rows"] == w1["rows_read"] == w1["own_rows"]


def test_split_layout_rejects_bad_head(dev):
    c = setup_case("sift", dev)
    ix = c["ix"]
    e = ix.encoder
    for hb, copy in ((8, 0), (48, 0), (128, 0), (256, 1), (16, 2)):
        with pytest.raises(NR.NRError) as err:
            NR.Index(n=ix.workload.n, d=ix.workload.d, dtype=NR.NR_U8, b=len(ix.tau),
                     weights=e.weights, biases=e.biases, input_scale=e.input_scale, tau=ix.tau,
                     rows=c["gix_split"].dev[0], row_ids=c["gix_split"].dev[1],
                     bc_off=c["gix_split"].dev[2], cl_off=c["gix_split"].dev[3],
                     centroids=c["gix_split"].dev[4], head_bytes=hb, head_copy=copy)
        assert err.value.status == NR.NR_EINVAL


@pytest.mark.parametrize("nq", [100, 600])
def test_shared_schedule_survivor_pool_and_fallback(dev, nq):
    """All rows tie and original ids fall along the rows, so after the leading
    clusters every row is a survivor (~15.6k per query).  Past a query's own
    2048 slots they go to the shared pool (4M entries): 100 queries fit; 600
    do not, and the queries that lost a survivor are recomputed per query."""
    n, d, n_cl = 20000, 16, 50
    rows = np.zeros((n, d), np.uint8)
    row_ids = np.arange(n - 1, -1, -1, dtype=np.int64)
    bc_off = np.array([0, 0, n_cl], np.int32)
    cl_off = np.linspace(0, n, n_cl + 1).astype(np.int64)
    cent = np.zeros((n_cl, 1), np.float32)
    W = np.zeros((1, d), np.float32)
    gix = NR.Index(n=n, d=d, dtype=NR.NR_U8, b=1, weights=[W], biases=[np.array([1.0], np.float32)],
                   input_scale=1.0, tau=np.zeros(1, np.float32),
                   rows=torch.from_numpy(rows).to(dev), row_ids=torch.from_numpy(row_ids).to(dev),
                   bc_off=torch.from_numpy(bc_off).to(dev), cl_off=torch.from_numpy(cl_off).to(dev),
                   centroids=torch.from_numpy(cent).to(dev))
    Q = torch.zeros((nq, d), dtype=torch.uint8, device=dev)
    base = dict(l_sel=1, r_max=1, k_c=n_cl, gate_on=False, early_stop_on=False)
    a = gix.nr_search(Q, 10, 2, NR.Params(refine_mode=NR.NR_REFINE_PER_QUERY, **base))
    b = gix.nr_search(Q, 10, 2, NR.Params(refine_mode=NR.NR_REFINE_SHARED, **base))
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
    assert b[0][0].tolist() == list(range(10))          # smallest ids, distance 0
    w = gix.nr_last_work()
    assert w["rows"] == nq * n
    assert w["survivors"] > nq * 4096
    if nq == 100:
        assert w["flagged"] == 0 and w["fallback_rows"] == 0
    else:
        # every query appends while the pool fills, so any number of them may lose one
        assert 0 < w["flagged"] <= nq and w["fallback_rows"] == w["flagged"] * n
    assert w["rows_read"] == w["own_rows"] + w["shared_rows"] + w["fallback_rows"]
    assert w["rows"] == w["own_rows"] + w["shared_pair_rows"]
    gix.close()
