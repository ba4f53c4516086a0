"""Parity of tables, encoding and the whole flat search with the oracle on the trained,
SIFT-like workload (needs an MI355X)."""
import numpy as np
import pytest
import torch

import oracle as O
import workloads as W
from gpu_util import RTOL, assert_topk_matches

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def setup():
    import paper_1609_01882_amd as psc
    out = {}
    for m in (8, 16):
        xt = W.sift_like(4000, seed=60 + m, stream=1)
        xb = W.sift_like(60_001, seed=60 + m, stream=2)
        xq = W.sift_like(50, seed=60 + m, stream=3)
        idx = psc.Index(128, m)
        idx.train_pq(xt, iters=5, seed=1)
        idx.optimize_index_assignment(n_iter=30_000, seed=2)
        out[m] = dict(idx=idx, cb=idx.get_codebook(), xb=xb, xq=xq)
    out["psc"] = psc
    return out


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("m", [8, 16])
def test_tables_and_query_codes(setup, m):
    s = setup[m]
    lut, qc = s["idx"].build_lut(_dev(s["xq"]))
    torch.cuda.synchronize()
    lut, qc = lut.cpu().numpy(), qc.cpu().numpy()
    ref = O.build_lut(s["xq"], s["cb"])
    # The tables come from the expansion |q'|^2 - 2 q'.c' + |c'|^2 in float32 on the matrix
    # cores, entries that cancel to less than 1/16 of those terms being redone by direct
    # differences: every entry is within the path's 1e-5 of its own value.
    allow = RTOL * ref
    assert np.all(np.abs(lut - ref) <= allow), np.max(np.abs(lut - ref) / allow)
    # ADC sums built from these tables stay within the 1e-5 relative bound of the path
    codes = W.random_codes(4000, m, seed=3)
    got = sum(lut[:, j, codes[:, j]].astype(np.float64) for j in range(m))
    want = sum(ref[:, j, codes[:, j]] for j in range(m))
    assert np.max(np.abs(got - want) / want) < RTOL / 10
    # the query code is the arg-min of the float32 table row (lowest index on ties) ...
    assert np.array_equal(qc, lut.argmin(axis=2).astype(np.uint8))
    # ... and a valid code in the oracle's eyes: its entry is within tolerance of the row minimum
    pick = np.take_along_axis(ref, qc[:, :, None].astype(np.int64), axis=2)[:, :, 0]
    assert np.all(pick <= ref.min(axis=2) * (1 + 2 * RTOL))
    assert (qc == O.query_codes(ref)).mean() > 0.999


@pytest.mark.parametrize("m,dsub", [(16, 2), (8, 4), (16, 6), (8, 8), (8, 12), (16, 16), (8, 24), (8, 32), (8, 48), (8, 64)])
def test_tables_without_codes_are_the_same_tables(m, dsub):
    """The table kernel stores the entries by lane where no codes are asked for and whole rows where they are."""
    import paper_1609_01882_amd as psc
    rng = np.random.default_rng(dsub)
    idx = psc.Index(m * dsub, m)
    idx.set_codebook(rng.normal(size=(m, 256, dsub)).astype(np.float32))
    q = _dev(rng.normal(size=(131, m * dsub)).astype(np.float32))
    for nq in (1, 31, 32, 33, 131):
        lut, codes = idx.build_lut(q[:nq].contiguous())
        alone, none = idx.build_lut(q[:nq].contiguous(), want_codes=False)
        assert none is None and torch.equal(lut, alone)
        assert torch.equal(codes.long(), lut.argmin(dim=2))


@pytest.mark.parametrize("m", [8, 16])
def test_encode(setup, m):
    s = setup[m]
    codes = s["idx"].encode(_dev(s["xb"])).cpu().numpy()
    ref = O.encode(s["xb"][:20_000], s["cb"])
    got = codes[:20_000]
    bad = np.argwhere(got != ref)
    assert len(bad) < 20  # only near-ties may differ
    dsub = 128 // m
    for i, j in bad:
        v = s["xb"][i, j * dsub:(j + 1) * dsub].astype(np.float64)
        da = ((v - s["cb"][j, got[i, j]]) ** 2).sum()
        db = ((v - s["cb"][j, ref[i, j]]) ** 2).sum()
        assert abs(da - db) <= RTOL * db
    s["codes"] = codes


@pytest.mark.parametrize("m,dsub", [(16, 1), (8, 6), (8, 8), (8, 12), (8, 16), (16, 24), (8, 32), (16, 48), (8, 64)])
def test_encode_of_many_rows_equals_encode_of_few(m, dsub):
    """The encoder's workgroups take several turns, for sub-vectors of 48 it reads the centroids another way from 1.6M
    codes on: the same sums, so the codes are those of the same rows 1000 at a time, which are the oracle's."""
    import paper_1609_01882_amd as psc
    dim, n = m * dsub, 3_200_000 // m + 259
    rng = np.random.default_rng(dim)
    cb = rng.normal(size=(m, 256, dsub)).astype(np.float32)
    idx = psc.Index(dim, m)
    idx.set_codebook(cb)
    g = torch.Generator(device="cuda")
    g.manual_seed(dim)
    x = torch.randn((n, dim), generator=g, device="cuda")
    few = torch.cat([idx.encode(x[s:s + 1000]) for s in range(0, 20_000, 1000)] + [idx.encode(x[-1000:])])
    for count in (799_999 // m, 800_000 // m, 1_600_000 // m - 1, 1_600_000 // m, n):
        many = idx.encode(x[:count])
        assert torch.equal(many[:20_000], few[:20_000]), count
    assert torch.equal(many[-1000:], few[-1000:])
    ref = O.encode(x[:2000].cpu().numpy(), cb)
    bad = np.argwhere(few[:2000].cpu().numpy() != ref)
    assert len(bad) <= 4
    for i, j in bad:  # only near-ties
        v = x[i, j * dsub:(j + 1) * dsub].cpu().numpy().astype(np.float64)
        da, db = ((v - cb[j, int(few[i, j])]) ** 2).sum(), ((v - cb[j, ref[i, j]]) ** 2).sum()
        assert abs(da - db) <= RTOL * db


@pytest.mark.parametrize("data", ["twins", "one", "far", "tiny", "huge", "wide", "grid", "far and tiny"])
@pytest.mark.parametrize("m,dsub", [(16, 1), (8, 2), (16, 4), (8, 6), (16, 8), (8, 12), (8, 16), (16, 24), (8, 32)])
def test_encode_where_centroids_are_close(m, dsub, data):
    """The search runs on bfloat16 parts, close calls are decided by the float32 distances: the codes are the
    first arg-min of those where nearly every row is a close call (every centroid twice, all centroids one, points
    of a grid halfway between centroids), where one centroid is far out, at the ends of float32's range (in "far and tiny" with
    two centroids far out, so that the squared lengths among the others are below what bfloat16 parts can hold) and
    with infinities and NaNs among the rows; from one row to four turns of a workgroup, of which a
    wave that met many close calls takes two at once."""
    import paper_1609_01882_amd as psc
    dim, turn = m * dsub, 256 * ((512 if dsub <= 16 else 256) // m)  # (rows that the workgroups take in one turn)
    n = 3 * turn + 1_077
    rng = np.random.default_rng(dim + len(data))
    cb = rng.normal(size=(m, 256, dsub)).astype(np.float32)
    x = rng.normal(size=(n, dim)).astype(np.float32)
    if data == "twins":
        cb[:, 128:] = cb[:, 127::-1]
    elif data == "one":
        cb[:] = cb[:, :1]
    elif data == "far":
        cb[:, 77] *= 1000.0
    elif data == "tiny":
        cb, x = cb * np.float32(1e-21), x * np.float32(1e-21)
    elif data == "huge":
        cb, x = cb * np.float32(3e18), x * np.float32(3e18)
    elif data == "far and tiny":
        scale = 10.0 ** np.linspace(-22.0, -17.0, m)[:, None, None]
        cb = (cb * scale).astype(np.float32)
        cb[:, 0], cb[:, min(255, 256 // dsub)] = 1.0, -1.0  # (one after the other in one sum: the mean stays with the others)
        x = (x.reshape(n, m, dsub) * scale[:, 0]).astype(np.float32).reshape(n, dim)
    elif data == "wide":
        x[::3] *= np.float32(1e15)
        x[1::97, 0] = np.inf
        x[2::89, dim - 1] = np.nan
        x[5::83] = 0.0
    else:
        cb, x = np.round(cb * 2), np.round(x * 4) / 2
    idx = psc.Index(dim, m)
    idx.set_codebook(np.ascontiguousarray(cb))
    xd = torch.from_numpy(np.ascontiguousarray(x)).cuda()
    # differences and multiply-adds in ascending order as the encoder states them: a float64 product and sum of
    # float32 values, rounded once to float32, is the fused multiply-add (but for double roundings: near-ties of
    # the last bit, of which a code may be either)
    want = np.zeros((n, m), np.uint8)
    tied = np.zeros((n, m), bool)
    with np.errstate(all="ignore"):
        for j in range(m):
            v = xd[:, j * dsub:(j + 1) * dsub]
            c = torch.from_numpy(np.ascontiguousarray(cb[j])).cuda()
            acc = torch.zeros((n, 256), dtype=torch.float32, device="cuda")
            for t in range(dsub):
                df = (v[:, t:t + 1] - c[None, :, t]).double()
                acc = (df * df + acc.double()).float()
            acc = torch.where(torch.isnan(acc), torch.inf, acc)
            least = acc.min(1, keepdim=True).values
            want[:, j] = (acc == least).int().argmax(1).cpu().numpy()
            got = idx.encode(xd)[:, j:j + 1].long()
            tied[:, j] = (acc.gather(1, got) <= least * (1 + 2e-7))[:, 0].cpu().numpy()
    got = idx.encode(xd).cpu().numpy()
    differs = got != want
    assert np.all(tied[differs]) and differs.sum() <= 1e-4 * differs.size, (int(differs.sum()), int((~tied & differs).sum()))
    for count in (1, 31, 33, 257, turn + 40, 2 * turn + 100, n - 1):
        assert np.array_equal(idx.encode(xd[:count].contiguous()).cpu().numpy(), got[:count]), count


@pytest.mark.parametrize("route", ["auto", "popcount", "mfma"])
@pytest.mark.parametrize("m", [8, 16])
def test_whole_search_matches_oracle(setup, force_route, route, m):
    force_route(route)
    s = setup[m]
    idx = s["idx"]
    if "codes" not in s:
        s["codes"] = idx.encode(_dev(s["xb"])).cpu().numpy()
    codes = s["codes"]
    q_dev, c_dev = _dev(s["xq"]), _dev(codes)
    lut, qc = idx.build_lut(q_dev)
    lut64, qc = lut.cpu().numpy().astype(np.float64), qc.cpu().numpy()
    nb = 8 * m
    for ht, k in ((nb // 4, 10), (nb * 3 // 8, 10), (nb * 3 // 8, 100), (nb // 2, 100), (nb, 100)):
        print(f"search m={m} ht={ht} k={k}", flush=True)
        ids, d = idx.search(q_dev, c_dev, ht, k)
        torch.cuda.synchronize()
        ref = O.scan(lut64, qc, codes, ht, k)
        assert_topk_matches(ids.cpu().numpy(), d.cpu().numpy(), ref, lut64, qc, codes, ht, what=f"m={m} ht={ht}")
        # and against the oracle's own double-precision tables: same ranking up to tolerance ties
        ref2 = O.search_flat(s["xq"], s["cb"], codes, ht, k)
        same_codes = np.all(O.query_codes(O.build_lut(s["xq"], s["cb"])) == qc, axis=1)
        assert same_codes.mean() > 0.9
        gd = d.cpu().numpy()[same_codes]
        fin = np.isfinite(ref2["dists"][same_codes])
        assert np.allclose(gd[fin], ref2["dists"][same_codes][fin], rtol=RTOL)


@pytest.mark.parametrize("m", [8, 16])
def test_small_searches_on_a_workspace_of_earlier_ones(setup, m):
    """The words by which a query's slices find out which ends last are set while the tables are built: searches of
    changing sizes on one workspace, which holds the words, keys and tables of the calls before."""
    psc, s = setup["psc"], setup[m]
    idx, codes = s["idx"], W.random_codes(100_001, m, seed=m)
    q = _dev(W.sift_like(129, seed=60 + m, stream=4))
    lut, qc = idx.build_lut(q)
    lut, qc, codes_d = lut.cpu().numpy().astype(np.float64), qc.cpu().numpy(), _dev(codes)
    calls = ((1, 10), (128, 10), (129, 10), (3, 100), (128, 513), (1, 1024), (100, 10), (128, 1024), (1, 10), (2, 1))
    need = max(idx.search_workspace_bytes(nq, len(codes), k) for nq, k in calls)
    ws = torch.full((need,), 0xa5, dtype=torch.uint8, device="cuda")
    sliced = 0
    for nq, k in calls:
        ids, d = idx.search(q[:nq], codes_d, 3 * m, k, workspace=ws)
        torch.cuda.synchronize()
        words = psc.last_scan_route().split()
        sliced += words[0] == "scan_pool_kernel" and words[4] != "slices=1"
        ref = O.scan(lut[:nq], qc[:nq], codes, 3 * m, k)
        assert_topk_matches(ids.cpu().numpy(), d.cpu().numpy(), ref, lut[:nq], qc[:nq], codes, 3 * m, what=f"{nq} queries, k={k}")
    assert sliced >= 5, sliced  # (the others take the tiles or one workgroup per query)


def test_tiny_workload_as_configured():
    """The smallest named workload, whole: 10k training vectors, product quantizer with optimised
    index assignment (the paper's annealing constants), 100 000 database vectors, 100 queries,
    ht = 24, k = 10 -- every query checked against the oracle, on the library's tables and on the
    oracle's own double-precision path from the raw vectors; recall@10 of both sides coincides."""
    import paper_1609_01882_amd as psc
    cfg = W.get_config("tiny")
    assert (cfg.n_train, cfg.n_db, cfg.n_query, cfg.hts, cfg.k) == (10_000, 100_000, 100, (24,), 10)
    xt, xb, xq = cfg.vectors("train"), cfg.vectors("db"), cfg.vectors("query")
    idx = psc.Index(cfg.dim, cfg.m)
    idx.train_pq(xt, iters=20, seed=cfg.seed)
    idx.optimize_index_assignment(seed=cfg.seed)
    cb = idx.get_codebook()
    ht, k = cfg.hts[0], cfg.k
    codes = idx.encode(_dev(xb))
    ids, d = idx.search(_dev(xq), codes, ht, k)
    lut, qc = idx.build_lut(_dev(xq))
    torch.cuda.synchronize()
    ids, d, codes_h = ids.cpu().numpy(), d.cpu().numpy(), codes.cpu().numpy()
    lut64, qc = lut.cpu().numpy().astype(np.float64), qc.cpu().numpy()
    # same tables and bit strings on both sides: survivor counts exact, ids and distances to the bar
    ref = O.scan(lut64, qc, codes_h, ht, k)
    assert_topk_matches(ids, d, ref, lut64, qc, codes_h, ht, what="tiny")
    ns = psc.hamming_filter(_dev(qc), codes, ht)
    assert np.array_equal(ns.cpu().numpy(), ref["nsurv"])
    # the oracle's own path from the raw vectors (its encoding, its tables, its query codes)
    ref_codes = O.encode(xb, cb)
    bad = np.argwhere(ref_codes != codes_h)
    assert len(bad) < 50
    dsub = cfg.dim // cfg.m
    for i, j in bad:  # only near-ties may be encoded differently
        v = xb[i, j * dsub:(j + 1) * dsub].astype(np.float64)
        da, db = ((v - cb[j, codes_h[i, j]]) ** 2).sum(), ((v - cb[j, ref_codes[i, j]]) ** 2).sum()
        assert abs(da - db) <= RTOL * db
    own = O.search_flat(xq, cb, codes_h, ht, k)
    same = np.all(O.query_codes(O.build_lut(xq, cb)) == qc, axis=1)
    assert same.mean() >= 0.95
    fin = np.isfinite(own["dists"][same])
    assert np.allclose(d[same][fin], own["dists"][same][fin], rtol=RTOL)
    assert np.array_equal(np.isfinite(d[same]), fin)
    truth = O.exact_knn(xb, xq, 1)[0][:, 0]
    r_gpu, r_orc = O.recall_at(ids, truth, 10), O.recall_at(ref["ids"], truth, 10)
    print(f"tiny: recall@10 gpu {r_gpu:.3f} oracle {r_orc:.3f}, survivors/query {ref['nsurv'].mean():.0f}", flush=True)
    assert r_gpu == r_orc


@pytest.mark.parametrize("m,spread,sigma", [(8, 3000.0, 10.0), (16, 30000.0, 2.0), (8, 100.0, 15.0)])
def test_tables_when_centroids_lie_far_apart(m, spread, sigma):
    """The table kernel's expansion |q'|^2 - 2 q'.c' + |c'|^2 cancels badly for a centroid close to
    the query when the centroids are spread far wider than that distance; such entries are redone
    by direct differences, so every entry -- small ones included -- is within 1e-5 of its own
    value, on clustered centroids 30 to 10000 times farther apart than the query is from the
    nearest one, and the query code is the oracle's except on near-ties."""
    import paper_1609_01882_amd as psc
    rng = np.random.default_rng(int(spread) + m)
    dsub = 128 // m
    centres = rng.random((40, 128)) * spread
    cb = np.empty((m, 256, dsub), np.float32)
    for j in range(m):   # centroids scattered around the 40 cluster centres of each sub-space
        cb[j] = centres[rng.integers(0, 40, size=256), j * dsub:(j + 1) * dsub] + rng.normal(0, sigma, size=(256, dsub))
    xq = (centres[rng.integers(0, 40, size=300)] + rng.normal(0, sigma, size=(300, 128))).astype(np.float32)
    idx = psc.Index(128, m)
    idx.set_codebook(cb)
    lut, qc = idx.build_lut(_dev(xq))
    torch.cuda.synchronize()
    lut, qc = lut.cpu().numpy(), qc.cpu().numpy()
    ref = O.build_lut(xq, cb)
    err = np.abs(lut - ref) / np.maximum(ref, 1e-30)
    print(f"tables m={m} spread={spread}: max rel err {err.max():.2e}, row max/min up to "
          f"{(ref.max(axis=2) / ref.min(axis=2)).max():.1e}", flush=True)
    assert err.max() <= RTOL
    assert np.array_equal(qc, lut.argmin(axis=2).astype(np.uint8))
    pick = np.take_along_axis(ref, qc[:, :, None].astype(np.int64), axis=2)[:, :, 0]
    assert np.all(pick <= ref.min(axis=2) * (1 + 2 * RTOL))
