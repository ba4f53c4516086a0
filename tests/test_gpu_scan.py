"""Parity of the fused HIP scan with the CPU oracle, through the C ABI (needs an MI355X)."""
import numpy as np
import pytest
import torch

import oracle as O
import workloads as W
from gpu_util import RTOL, assert_topk_matches

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def psc():
    import paper_1609_01882_amd as p
    assert torch.cuda.is_available()
    return p


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _rand_problem(m, n, nq, seed, lut_kind):
    rng = np.random.default_rng(seed)
    codes = W.random_codes(n, m, seed=seed)
    # query codes near some database codes so that low thresholds still see survivors
    qcodes = codes[rng.integers(0, max(n, 1), size=nq)].copy() if n > 0 else W.random_codes(nq, m, seed + 1)
    flip = rng.integers(0, 256, size=qcodes.shape).astype(np.uint8) & rng.integers(0, 256, size=qcodes.shape).astype(np.uint8)
    qcodes ^= flip
    if lut_kind == "int":      # few small integers: sums exact in float32, many exact ties
        lut = rng.integers(0, 4, size=(nq, m, 256)).astype(np.float32)
    else:
        lut = (rng.random(size=(nq, m, 256)) * 1000.0).astype(np.float32)
    return codes, qcodes, lut


def _run(psc, lut, qcodes, codes, ht, k):
    ids, d = psc.scan(_dev(lut), _dev(qcodes), _dev(codes), ht, k)
    torch.cuda.synchronize()
    return ids.cpu().numpy(), d.cpu().numpy()


def _took(psc, route, m, nq, ht, k=1):
    """The kernel a forced route launches (None: automatic, which also knows the pool)."""
    took = psc.last_scan_route().split()[0]
    dense_from = 30 if m == 8 else 62
    if ht >= 8 * m:
        want = "adc_kernel"
    elif ht >= dense_from:
        want = "adc_kernel+filter"
    else:  # (k past the largest that fits its tile of 16 queries, 8 at 128 bits: the narrower tiles of the other)
        want = "scan_mfma_kernel" if route == "mfma" and nq >= 9 and k <= (136 if m == 8 else 272) else "scan_kernel"
    assert route == "auto" or took == want, (route, took, want)


@pytest.mark.parametrize("route", ["auto", "mfma", "popcount"])
@pytest.mark.parametrize("m,n,nq,k,lut_kind", [
    (8, 100_003, 37, 10, "float"),      # ragged tail (odd n), ragged query tile
    (8, 100_003, 37, 100, "int"),       # exact ties: ids must match exactly
    (8, 4096, 16, 100, "float"),
    (8, 70_001, 5, 1, "float"),
    (16, 50_001, 19, 10, "float"),
    (16, 50_001, 19, 100, "int"),
    (8, 30_000, 3, 300, "int"),         # k > 128: smaller query tile
    (16, 20_000, 9, 1024, "float"),     # maximum k
    (8, 60_001, 1, 100, "float"),       # small batches take narrower query tiles
    (8, 45_003, 8, 10, "int"),
    (16, 33_001, 2, 100, "int"),
    (16, 40_001, 7, 10, "float"),
])
def test_scan_random_codes(psc, force_route, route, m, n, nq, k, lut_kind):
    force_route(route)
    codes, qcodes, lut = _rand_problem(m, n, nq, seed=100 + m + k, lut_kind=lut_kind)
    nb = 8 * m
    for ht in sorted({0, nb // 4, nb * 3 // 8, nb // 2 - 4, nb // 2, nb, nb + 50}):
        print(f"case m={m} n={n} nq={nq} k={k} lut={lut_kind} ht={ht}", flush=True)
        got_ids, got_d = _run(psc, lut, qcodes, codes, ht, k)
        _took(psc, route, m, nq, ht, k)
        ref = O.scan(lut.astype(np.float64), qcodes, codes, ht, k)
        nd = assert_topk_matches(got_ids, got_d, ref, lut.astype(np.float64), qcodes, codes, min(ht, nb),
                                 what=f"m={m} ht={ht} k={k}")
        if lut_kind == "int":
            assert nd == 0 and np.array_equal(got_d[ref["ids"] >= 0], ref["dists"][ref["ids"] >= 0])


@pytest.mark.parametrize("route", ["mfma", "popcount"])
@pytest.mark.parametrize("m,n,nq,k,lut_kind", [
    (8, 100_003, 37, 10, "float"),     # ragged last block (n % 128 = 35), ragged query tile (37 = 2 * 16 + 5)
    (8, 100_003, 37, 100, "int"),      # exact ties: ids must match exactly
    (8, 65_536 + 127, 160, 136, "int"),  # the largest k of the 16-query tile
    (8, 9_000, 17, 5, "float"),        # barely more than one tile of queries, one slice
    (8, 300_001, 9, 10, "int"),        # the fewest queries the matrix-core route takes: many slices
    (8, 50_000, 16, 100, "float"),     # exactly one full tile
    (8, 1_000_001, 48, 20, "float"),   # several slices per query tile
    (16, 100_003, 37, 10, "float"),    # 128 bits: blocks of 256 codes, tiles of 8 queries (37 = 4 * 8 + 5)
    (16, 100_003, 37, 100, "int"),
    (16, 65_536 + 255, 80, 272, "int"),  # the largest k of the 8-query tile
    (16, 300_001, 9, 10, "int"),
    (16, 500_001, 48, 20, "float"),
])
def test_both_filter_routes(psc, force_route, route, m, n, nq, k, lut_kind):
    """The Hamming test runs either as xor/popcount or on the matrix cores; the library picks by
    shape and threshold.  Here each route is forced in turn (psc_set_filter_route) on batches
    of 9 queries or more and must give the oracle's result at every threshold, including
    those the rule would hand to the other route."""
    force_route(route)
    codes, qcodes, lut = _rand_problem(m, n, nq, seed=900 + k, lut_kind=lut_kind)
    for ht in (0, 9, 16, 22, 24, 27, 29, 30, 33) if m == 8 else (0, 20, 40, 48, 54, 59, 61, 62, 66):
        print(f"case route={route} m={m} n={n} nq={nq} k={k} ht={ht}", flush=True)
        got_ids, got_d = _run(psc, lut, qcodes, codes, ht, k)
        # the library says which kernel it launched: the forced filter below the dense route's thresholds
        _took(psc, route, m, nq, ht, k)
        ref = O.scan(lut.astype(np.float64), qcodes, codes, ht, k)
        nd = assert_topk_matches(got_ids, got_d, ref, lut.astype(np.float64), qcodes, codes, ht,
                                 what=f"route={route} ht={ht} k={k}")
        if lut_kind == "int":
            assert nd == 0 and np.array_equal(got_d[ref["ids"] >= 0], ref["dists"][ref["ids"] >= 0])


@pytest.mark.parametrize("m,hts", [(8, (17, 18, 19, 20)), (16, (39, 41, 43, 44))])
def test_survivor_set_on_the_matrix_cores(psc, force_route, m, hts):
    """k above the number of survivors: the matrix-core route lists exactly the survivor set."""
    force_route("mfma")
    k = 136
    codes, qcodes, lut = _rand_problem(m, 40_000, 33, seed=77, lut_kind="float")
    for ht in hts:
        ref = O.scan(lut.astype(np.float64), qcodes, codes, ht, k, want_bitmap=True)
        got_ids, _ = _run(psc, lut, qcodes, codes, ht, k)
        _took(psc, "mfma", m, 33, ht, k)
        assert (ref["nsurv"] <= k).any()
        for q in range(33):
            if ref["nsurv"][q] <= k:
                assert sorted(got_ids[q][got_ids[q] >= 0].tolist()) == np.flatnonzero(ref["bitmap"][q]).tolist()


@pytest.mark.parametrize("m", [8, 16])
def test_pairs_at_the_threshold(psc, force_route, m):
    """Codes at distance ht and ht + 1 of a query, the differing bits drawn anywhere, at every threshold of the
    matrix-core filter: the fields of its results hold ht + 8 m - distance in 7 (8) bits, whose
    verdict changes between these two.  Every query slot, place in a block and result register has some."""
    force_route("mfma")
    nq, per, k = 24, 96, 100
    rng = np.random.default_rng(m)
    for ht in range(0, 30 if m == 8 else 62):
        qcodes = W.random_codes(nq, m, seed=ht)
        owner = rng.permutation(np.repeat(np.arange(nq), per))
        bits = np.unpackbits(qcodes[owner], axis=1)
        far = rng.integers(0, 2, size=len(owner))
        order = rng.random(bits.shape).argsort(axis=1)
        bits ^= (order < (ht + far)[:, None]).astype(np.uint8)
        codes = np.packbits(bits, axis=1)
        lut = rng.integers(0, 4, size=(nq, m, 256)).astype(np.float32)
        got_ids, got_d = _run(psc, lut, qcodes, codes, ht, k)
        _took(psc, "mfma", m, nq, ht, k)
        ref = O.scan(lut.astype(np.float64), qcodes, codes, ht, k)
        assert np.array_equal(got_ids, ref["ids"]), (m, ht)
        assert np.array_equal(got_d[ref["ids"] >= 0], ref["dists"][ref["ids"] >= 0])


@pytest.mark.parametrize("m,nq", [(8, 9), (8, 16), (8, 33), (16, 9), (16, 16), (16, 17)])
def test_matrix_core_filter_at_block_edges(psc, force_route, m, nq):
    """Database sizes around the matrix-core kernel's blocks (128 codes at 64 bits, 256 at 128), its 64-code
    loads and the stride of its 16 waves; extreme codes (all zeros, all ones, a query's own code and
    its complement) among the random ones; thresholds up to the last before the dense route.  Integer
    tables: sums are exact in float32, so ids and distances equal the oracle's."""
    force_route("mfma")
    stride = 16 * (128 if m == 8 else 256)
    for n in (1, 15, 16, 17, 63, 65, 127, 128, 129, 255, 256, 257, stride - 1, stride + 1, 2 * stride + 130, 5 * stride - 3):
        codes, qcodes, lut = _rand_problem(m, n, nq, seed=7 * n + nq, lut_kind="int")
        for i, c in enumerate((np.zeros(m, np.uint8), np.full(m, 255, np.uint8), qcodes[0], ~qcodes[nq - 1])):
            codes[(n - 1 - 5 * i) % n] = c
        qcodes[1], qcodes[2] = 0, 255
        for ht in (0, 1, 3 * m, 29 if m == 8 else 60):
            print(f"case m={m} nq={nq} n={n} ht={ht}", flush=True)
            got_ids, got_d = _run(psc, lut, qcodes, codes, ht, 50)
            assert psc.last_scan_route().startswith("scan_mfma_kernel ")
            ref = O.scan(lut.astype(np.float64), qcodes, codes, ht, 50)
            nd = assert_topk_matches(got_ids, got_d, ref, lut.astype(np.float64), qcodes, codes, ht, what=f"n={n} ht={ht}")
            assert nd == 0 and np.array_equal(got_d[ref["ids"] >= 0], ref["dists"][ref["ids"] >= 0])


@pytest.mark.parametrize("m,n,nq,k,lut_kind", [
    (8, 63, 3, 100, "int"), (8, 513, 2, 100, "int"),          # fewer codes than a wave's turn, one more
    (8, 8_191, 5, 100, "int"), (16, 8_193, 5, 100, "int"),    # around the workgroup's turn of 8192 codes
    (8, 100_003, 1, 100, "int"), (16, 40_001, 7, 100, "float"),  # several slices per query, merged
    (8, 50_000, 150, 64, "int"), (16, 50_001, 150, 200, "int"),  # one slice; many exact ties
    (8, 60_000, 4, 1024, "float"), (16, 60_000, 130, 1024, "int"),  # the largest k
])
def test_pool_scan(psc, m, n, nq, k, lut_kind):
    """Small scans: survivors' keys pooled and selected.  Thresholds on both sides of the dense route (where
    every code enters a pool of 4096 until the first selection), exact ties and the ends of the sizes."""
    codes, qcodes, lut = _rand_problem(m, n, nq, seed=31 * m + n, lut_kind=lut_kind)
    for ht in (0, 3 * m, 29 if m == 8 else 60, 4 * m, 8 * m):
        print(f"case m={m} n={n} nq={nq} k={k} ht={ht}", flush=True)
        got_ids, got_d = _run(psc, lut, qcodes, codes, ht, k)
        assert psc.last_scan_route().startswith("scan_pool_kernel"), psc.last_scan_route()
        ref = O.scan(lut.astype(np.float64), qcodes, codes, ht, k)
        nd = assert_topk_matches(got_ids, got_d, ref, lut.astype(np.float64), qcodes, codes, ht, what=f"n={n} ht={ht}")
        if lut_kind == "int":
            assert nd == 0 and np.array_equal(got_d[ref["ids"] >= 0], ref["dists"][ref["ids"] >= 0])


@pytest.mark.parametrize("m,n,nq,k,ht,kernel", [
    (8, 650_403, 273, 100, 0, "scan_mfma_kernel"), (16, 3_942_775, 22, 100, 32, "scan_mfma_kernel"),
    (8, 160_602, 2384, 100, 0, "scan_mfma_kernel"), (8, 54_554, 4300, 1, 28, "scan_kernel"), (8, 12_123, 4200, 10, 29, "scan_kernel")])
def test_few_survivors_and_small_lists_take_the_tiled_kernels(psc, force_route, m, n, nq, k, ht, kernel):
    """Sizes at which the pool (hardly anything survives: the lists cost nothing) or the matrix-core filter (many
    survive few pairs) takes 1.5 to 3 times as long as the kernel named; the answer is that of the others."""
    codes, qcodes, lut = (_dev(a) for a in _rand_problem(m, n, nq, seed=n % 1000, lut_kind="float"))
    got = psc.scan(lut, qcodes, codes, ht, k)
    assert psc.last_scan_route().split()[0] == kernel, psc.last_scan_route()
    force_route("popcount" if kernel == "scan_mfma_kernel" else "mfma")
    want = psc.scan(lut, qcodes, codes, ht, k)
    torch.cuda.synchronize()
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])


@pytest.mark.parametrize("m,n,nq,k", [(8, 20_000, 12, 40), (8, 100_003, 40, 300), (16, 20_000, 12, 300),
                                      (16, 40_001, 1, 1024), (8, 40_001, 2, 50), (8, 1_200_000, 2, 600)])
def test_small_scans_answer_tables_that_are_not_finite_as_the_tiled_kernels_do(psc, force_route, m, n, nq, k):
    """Table entries that are not numbers (of a query that is not) or infinite: the fused tiled kernels put a
    survivor at distance +inf where the sum over the first 3 m / 8 sub-quantizers is not a number and leave
    it out where only a later entry makes it so; codes at +inf come after all others in order of their ids,
    except that the merge for a handful of queries and 64 results or more leaves them out.  Small scans, pooled
    in one slice or several, answer the same."""
    codes, qcodes, lut = _rand_problem(m, n, nq, seed=5 * m + nq, lut_kind="int")
    early = 3 * m // 8
    lut[0, early - 1, ::2] = np.nan       # some codes, in an early sub-quantizer
    lut[0, early - 1, 1::4] = np.inf      # not finite, but a number
    if nq > 1:
        lut[1] = np.nan                   # a query that is no vector
    if nq > 2:
        lut[2, m - 1, ::3] = np.nan       # a late sub-quantizer
        lut[3, 0, :] = np.inf
    for ht in (3 * m, 3 * m + 2, 4 * m, 8 * m):
        print(f"case m={m} n={n} nq={nq} k={k} ht={ht}", flush=True)
        got_ids, got_d = _run(psc, lut, qcodes, codes, ht, k)
        assert psc.last_scan_route().startswith("scan_pool_kernel"), psc.last_scan_route()
        for route in ("popcount", "mfma") if nq >= 9 else ("popcount",):
            force_route(route)
            want_ids, want_d = _run(psc, lut, qcodes, codes, ht, k)
            force_route("auto")
            assert np.array_equal(got_ids, want_ids) and np.array_equal(got_d, want_d), (m, ht, route)
        if k >= 64 or ht >= 4 * m:
            continue
        near = O.hamming_matrix(qcodes, codes) <= ht  # by the rule as stated
        for q in range(nq):
            rows = np.flatnonzero(near[q])
            entry = np.stack([lut[q, j, codes[rows, j]] for j in range(m)], 1).astype(np.float64)
            d = entry.sum(1)
            d[np.isnan(entry[:, :early].sum(1))] = np.inf
            rows, d = rows[~np.isnan(d)], d[~np.isnan(d)]
            order = np.lexsort((rows, d))[:k]
            assert np.array_equal(got_ids[q][: len(order)], rows[order]) and np.all(got_ids[q][len(order):] == -1), (q, ht)
            assert np.array_equal(got_d[q][: len(order)], d[order].astype(np.float32))


@pytest.mark.parametrize("m", [8, 16])
@pytest.mark.parametrize("route", ["mfma", "popcount"])
def test_nested_prefix_patterns_at_every_threshold(psc, force_route, route, m):
    """Database row r = the first r bits set (r = 0..8m, repeated to fill several blocks), query q =
    the first 3q (128 bits: 6q) bits set: their Hamming distance is |r - 3q| exactly, so the survivor set
    at every threshold is known in closed form.  Both filters at every threshold they serve, and the dense
    route, which tests only the pairs that beat the k-th best, at the thresholds above (30, 62 and
    more); the table makes the distance itself the score."""
    force_route(route)
    reps, nq = 7, 20
    def prefix(r):
        c = np.zeros(m, np.uint8)
        full, rem = divmod(r, 8)
        c[:full] = 0xFF
        if rem:
            c[full] = (1 << rem) - 1
        return c
    rows = np.array([r for _ in range(reps) for r in range(8 * m + 1)])
    codes = np.stack([prefix(r) for r in rows])
    qbits = np.array([3 * m // 8 * q for q in range(nq)])
    qc = np.stack([prefix(b) for b in qbits])
    lut = np.zeros((nq, m, 256), np.float32)
    pc = np.array([bin(v).count("1") for v in range(256)], np.float32)
    for q in range(nq):  # score = Hamming distance to the query code: sum over bytes of popcount(byte xor query byte)
        for j in range(m):
            lut[q, j] = pc[np.arange(256) ^ int(qc[q, j])]
    k = 136
    for ht in range(0, 36 if m == 8 else 67):
        ids, d = _run(psc, lut, qc, codes, ht, k)
        _took(psc, route, m, nq, ht, k)
        for q in range(nq):
            want = np.flatnonzero(np.abs(rows - qbits[q]) <= ht)
            got = ids[q][ids[q] >= 0]
            if len(want) <= k:
                assert sorted(got.tolist()) == want.tolist(), (route, ht, q)
            else:
                assert len(got) == k
            assert np.array_equal(d[q][: len(got)], np.abs(rows[got] - qbits[q]).astype(np.float32)), (route, ht, q)


@pytest.mark.parametrize("m,nq,hts", [(8, 4100 + 13, (14, 22)), (16, 2048 + 13, (30, 44))])
@pytest.mark.parametrize("route", ["mfma", "popcount"])
def test_whole_and_sliced_query_tiles_in_one_launch(psc, force_route, route, m, nq, hts):
    """More query tiles than workgroups run at a time: the tiles of the whole rounds scan the
    database in one piece, those of the last partial round in slices.  Queries from both regions
    (and the last, ragged tile) against the oracle."""
    force_route(route)
    n, k = 150_011, 20
    codes, qcodes, lut = _rand_problem(m, n, nq, seed=4242, lut_kind="float")
    sel = np.array([0, 1, 7, 8, 15, 16, nq // 2, nq - 34, nq - 33, nq - 18, nq - 17, nq - 16, nq - 13, nq - 6, nq - 5, nq - 2, nq - 1])
    for ht in hts:
        got_ids, got_d = _run(psc, lut, qcodes, codes, ht, k)
        _took(psc, route, m, nq, ht, k)
        took = dict(f.split("=") for f in psc.last_scan_route().split()[1:])
        whole = int(took["tiles"]) < -(-nq // int(took["tq"])) * int(took["slices"])
        assert whole, psc.last_scan_route()  # (some tiles in one piece, others in slices)
        ref = O.scan(lut[sel].astype(np.float64), qcodes[sel], codes, ht, k)
        assert_topk_matches(got_ids[sel], got_d[sel], ref, lut[sel].astype(np.float64), qcodes[sel], codes, ht,
                            what=f"two regions route={route} ht={ht}")
        # all queries: as many results as the (separately tested) filter counts survivors, up to k
        ns = psc.hamming_filter(_dev(qcodes), _dev(codes), ht)
        torch.cuda.synchronize()
        assert got_ids.max() < n
        assert np.array_equal((got_ids >= 0).sum(axis=1), np.minimum(ns.cpu().numpy(), k))


@pytest.mark.parametrize("m,nq", [(16, 2051), (8, 4099)])
def test_whole_tiles_over_more_than_2_to_the_25_codes(psc, force_route, m, nq):
    """Enough query tiles to scan 34M codes in one piece: positions past 2^25 come through the matrix-core
    filter's queue entries whole.  Rows near both ends and past 2^25 repeat query codes (distance 0); the rest
    against the popcount kernel's answer."""
    n, k, ht = (1 << 25) + 70_003, 5, 8 * m // 4
    g = torch.Generator(device="cuda")
    g.manual_seed(17 + m)
    codes = torch.randint(0, 256, (n, m), generator=g, device="cuda", dtype=torch.uint8)
    qcodes = torch.randint(0, 256, (nq, m), generator=g, device="cuda", dtype=torch.uint8)
    rows = torch.tensor([3, (1 << 25) - 1, 1 << 25, (1 << 25) + 16, (1 << 25) + 65_537, n - 1], device="cuda")
    owner = torch.tensor([0, 15, 16, 1000, 2047, nq - 1], device="cuda")
    codes[rows] = qcodes[owner]
    lut = torch.empty((nq, m, 256), device="cuda").uniform_(1.0, 1000.0, generator=g)
    lut.scatter_(2, qcodes.long()[:, :, None], 0.0)  # the query's own code: distance 0
    out = {}
    for route in ("mfma", "popcount"):
        force_route(route)
        out[route] = psc.scan(lut, qcodes, codes, ht, k)
        torch.cuda.synchronize()
        assert psc.last_scan_route().startswith("scan_mfma_kernel " if route == "mfma" else "scan_kernel ")
    assert torch.equal(out["mfma"][0][owner, 0], rows) and torch.all(out["mfma"][1][owner, 0] == 0)
    assert torch.equal(out["mfma"][0], out["popcount"][0]) and torch.equal(out["mfma"][1], out["popcount"][1])


@pytest.mark.parametrize("m,nq,ht,fewer", [(8, 2721, 28, True), (16, 1000, 56, False)])
def test_a_workspace_for_the_popcount_plan_is_enough(psc, force_route, m, nq, ht, fewer):
    """A caller's fixed workspace that holds the xor/popcount kernel's partial lists but not the matrix-core
    kernel's is taken, by the former (128-bit codes: the two plans are the same); one byte less is refused."""
    n, k = 1_000_001, 100
    codes, qcodes, lut = (_dev(a) for a in _rand_problem(m, n, nq, seed=3, lut_kind="float"))
    slices = {}
    for route in ("popcount", "mfma"):
        force_route(route)
        want = psc.scan(lut, qcodes, codes, ht, k)
        slices[route] = int(psc.last_scan_route().split("slices=")[1].split()[0])
    force_route("auto")
    words = lambda s: min(s, 64) if s >= 4 else 1
    r = lambda b: -(-b // 256) * 256
    need = 256 + r(4 * nq * words(slices["popcount"])) + r(4 * nq * k * slices["popcount"]) + 8 * nq * k * slices["popcount"]
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    got = psc.scan(lut, qcodes, codes, ht, k, workspace=ws)
    torch.cuda.synchronize()
    print(f"m={m}: slices {slices}, {psc.last_scan_route()}", flush=True)
    assert (slices["mfma"] > slices["popcount"]) == fewer
    assert psc.last_scan_route().startswith("scan_kernel " if fewer else "scan_mfma_kernel ")
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
    with pytest.raises(psc.PscError, match="workspace too small"):
        psc.scan(lut, qcodes, codes, ht, k, workspace=ws[:-1])


@pytest.mark.parametrize("route", ["auto", "popcount"])
def test_many_slices_for_few_queries(psc, force_route, route):
    """Two queries over 3M codes: 256 database slices, whose partial lists the merge takes four to a lane (without
    the pool, which a forced route excludes)."""
    force_route(route)
    codes, qcodes, lut = _rand_problem(8, 3_000_001, 2, seed=321, lut_kind="float")
    for ht, k in ((22, 10), (64, 3)):
        got_ids, got_d = _run(psc, lut, qcodes, codes, ht, k)
        _took(psc, route, 8, 2, ht, k)
        assert route == "auto" or int(psc.last_scan_route().split("slices=")[1].split()[0]) > 128
        ref = O.scan(lut.astype(np.float64), qcodes, codes, ht, k)
        assert_topk_matches(got_ids, got_d, ref, lut.astype(np.float64), qcodes, codes, ht, what=f"many slices ht={ht}")


@pytest.mark.parametrize("case", ["all tied", "best in one slice", "wide range"])
@pytest.mark.parametrize("route", ["auto", "popcount"])
@pytest.mark.parametrize("nq,k,m", [(1, 100, 8), (3, 7, 8), (12, 1, 8), (5, 640, 8), (3, 100, 16)])
def test_what_the_slices_tell_each_other_costs_no_result(psc, force_route, route, case, nq, k, m):
    """Queries cut into many slices prune with a bound taken from the other slices' lists (the
    r-th best of each, and the value enough of them have reached).  Where that bound equals the
    k-th distance (everything tied), where one slice holds the whole answer, and where distances
    span sixty binary orders of magnitude (the bound is rounded up in the float's bits), the result
    is still the oracle's."""
    force_route(route)
    n = 1_200_007
    rng = np.random.default_rng(900 + k)
    codes, qcodes, lut = _rand_problem(m, n, nq, seed=901 + k, lut_kind="int")
    if case == "all tied":
        lut[:] = 2.0
    elif case == "best in one slice":
        # the last 2000 codes are the only ones with small distances: byte 0 below 16 there only
        codes[:, 0] |= 16
        codes[-2000:, 0] &= 15
        lut[:, 0, :16] = 0.0
        lut[:, 0, 16:] = 50.0
    else:
        lut = np.exp2(rng.uniform(-30.0, 30.0, size=(nq, m, 256))).astype(np.float32)
    for ht in (26, 64) if m == 8 else (56, 128):
        got_ids, got_d = _run(psc, lut, qcodes, codes, ht, k)
        _took(psc, route, m, nq, ht, k)
        assert route == "auto" or int(psc.last_scan_route().split("slices=")[1].split()[0]) >= 64
        ref = O.scan(lut.astype(np.float64), qcodes, codes, ht, k)
        nd = assert_topk_matches(got_ids, got_d, ref, lut.astype(np.float64), qcodes, codes, ht,
                                 what=f"{case} nq={nq} k={k} ht={ht}")
        if case != "wide range":
            assert nd == 0


@pytest.mark.parametrize("route", ["auto", "popcount"])
@pytest.mark.parametrize("nq,n,k,lut_kind", [(1, 3_000_001, 100, "int"), (3, 1_000_003, 64, "int"),
                                             (8, 400_009, 128, "float"), (2, 70_001, 1024, "int"),
                                             (1, 300, 500, "int")])
def test_selecting_merge_for_a_handful_of_queries(psc, force_route, route, nq, n, k, lut_kind):
    """A handful of queries (up to 32, or 512 with many lists each) and k >= 64: the partial lists of the slices are merged by a workgroup that
    selects the k smallest (distance, id) pairs.  Integer tables put hundreds of entries at the
    k-th distance, so the last place is decided by the id; short databases leave padding."""
    force_route(route)
    codes, qcodes, lut = _rand_problem(8, n, nq, seed=77 + k, lut_kind=lut_kind)
    for ht in (24, 64):
        got_ids, got_d = _run(psc, lut, qcodes, codes, ht, k)
        _took(psc, route, 8, nq, ht, k)
        ref = O.scan(lut.astype(np.float64), qcodes, codes, ht, k)
        nd = assert_topk_matches(got_ids, got_d, ref, lut.astype(np.float64), qcodes, codes, ht, what=f"nq={nq} k={k} ht={ht}")
        if lut_kind == "int":
            assert nd == 0  # exact sums: ties must resolve exactly as in the oracle


@pytest.mark.parametrize("route", ["auto", "popcount"])
@pytest.mark.parametrize("m,n,k,lut_kind", [(8, 2_000_003, 100, "int"), (8, 2_000_003, 130, "int"), (8, 900, 100, "float"),
                                            (8, 5_000_001, 1, "float"), (16, 700_001, 100, "int"), (8, 300_001, 64, "int"),
                                            (16, 200_003, 200, "float")])
def test_a_single_query_spreads_its_candidates_over_four_lists(psc, force_route, route, m, n, k, lut_kind):
    """One query: the three empty slots of the tile hold copies of its tables, every wave feeds the
    list of slot wave % 4 and the four lists are merged when the slice ends (one slice for small
    databases, 256 for large ones).  Exact ties (small-integer tables) must come out in id order."""
    force_route(route)
    codes, qcodes, lut = _rand_problem(m, n, 1, seed=400 + k, lut_kind=lut_kind)
    nb = 8 * m
    for ht in (nb // 4, nb * 3 // 8, nb // 2 - 3):
        print(f"single query m={m} n={n} k={k} ht={ht}", flush=True)
        got_ids, got_d = _run(psc, lut, qcodes, codes, ht, k)
        _took(psc, route, m, 1, ht, k)
        ref = O.scan(lut.astype(np.float64), qcodes, codes, ht, k)
        nd = assert_topk_matches(got_ids, got_d, ref, lut.astype(np.float64), qcodes, codes, ht, what=f"single m={m} ht={ht}")
        if lut_kind == "int":
            assert nd == 0


@pytest.mark.parametrize("m", [8, 16])
def test_hamming_filter_is_bit_exact(psc, m):
    codes, qcodes, _ = _rand_problem(m, 20_011, 23, seed=7 + m, lut_kind="int")
    want = O.hamming_matrix(qcodes, codes)
    for ht in (0, 2 * m, 3 * m, 4 * m, 8 * m):
        ns, hd = psc.hamming_filter(_dev(qcodes), _dev(codes), ht, want_distances=True)
        torch.cuda.synchronize()
        assert np.array_equal(hd.cpu().numpy().astype(np.int32), want)
        assert np.array_equal(ns.cpu().numpy(), (want <= ht).sum(axis=1))
        ref = O.scan(np.zeros((23, m, 256)), qcodes, codes, ht, 1)
        assert np.array_equal(ns.cpu().numpy(), ref["nsurv"])


@pytest.mark.parametrize("route", ["auto", "mfma", "popcount"])
@pytest.mark.parametrize("m", [8, 16])
def test_survivor_set_through_the_fused_scan(psc, force_route, route, m):
    """With k above the number of survivors the result lists exactly the survivor set."""
    force_route(route)
    codes, qcodes, lut = _rand_problem(m, 60_000, 11, seed=50 + m, lut_kind="float")
    ht = 2 * m + 2
    ref = O.scan(lut.astype(np.float64), qcodes, codes, ht, 1024, want_bitmap=True)
    assert ref["nsurv"].max() < 1024 and ref["nsurv"].max() > 0
    got_ids, got_d = _run(psc, lut, qcodes, codes, ht, 1024)
    for q in range(11):
        surv = np.flatnonzero(ref["bitmap"][q])
        assert sorted(got_ids[q][got_ids[q] >= 0].tolist()) == surv.tolist()


def test_hand_built_patterns_through_the_scan(psc):
    """Row r of the database has exactly r bits set; the query code is zero; table = first byte."""
    for m in (8, 16):
        nb = 8 * m
        codes = np.zeros((nb + 1, m), np.uint8)
        for r in range(nb + 1):
            full, rem = divmod(r, 8)
            codes[r, :full] = 0xFF
            if rem:
                codes[r, full] = (1 << rem) - 1
        lut = np.zeros((1, m, 256), np.float32)
        lut[0, m - 1, :] = 1.0 + np.arange(256)
        qc = np.zeros((1, m), np.uint8)
        for ht in (0, 1, 7, 8, 9, nb // 2, nb - 1, nb):
            got_ids, got_d = _run(psc, lut, qc, codes, ht, nb + 5)
            ref = O.scan(lut.astype(np.float64), qc, codes, ht, nb + 5)
            assert np.array_equal(got_ids, ref["ids"]) and (got_ids[0] >= 0).sum() == ht + 1
            assert np.array_equal(got_d[got_ids >= 0], ref["dists"][ref["ids"] >= 0])


def test_edge_sizes(psc):
    m, k = 8, 5
    lut = np.ones((3, m, 256), np.float32)
    qc = np.zeros((3, m), np.uint8)
    # empty database: all padding
    ids, d = _run(psc, lut, qc, np.zeros((0, m), np.uint8), 64, k)
    assert np.all(ids == -1) and np.all(np.isinf(d))
    # no queries
    ids, d = psc.scan(_dev(lut[:0]), _dev(qc[:0]), _dev(np.zeros((10, m), np.uint8)), 64, k)
    assert ids.shape == (0, k)
    # tiny databases
    for n in (1, 2, 63, 64, 65, 127, 129):
        codes = W.random_codes(n, m, seed=n)
        ids, d = _run(psc, lut, qc, codes, 64, k)
        ref = O.scan(lut.astype(np.float64), qc, codes, 64, k)
        assert np.array_equal(ids, ref["ids"]), n
    # bad arguments are errors, not crashes
    with pytest.raises(psc.PscError):
        psc.scan(_dev(lut), _dev(qc), _dev(W.random_codes(10, m, 1)), 64, 0)
    with pytest.raises(psc.PscError):
        psc.scan(_dev(lut), _dev(qc), _dev(W.random_codes(10, m, 1)), -1, 5)


def test_scan_is_deterministic(psc):
    codes, qcodes, lut = _rand_problem(8, 200_000, 64, seed=9, lut_kind="float")
    a = _run(psc, lut, qcodes, codes, 26, 100)
    b = _run(psc, lut, qcodes, codes, 26, 100)
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])


@pytest.mark.parametrize("m", [8, 16])
def test_hamming_histogram_is_bit_exact(psc, m):
    """Threshold adjustment (Section 4.2): the pair histogram equals the oracle's, count for count,
    and both sides pick the same threshold for a 95 % filter."""
    codes, qcodes, _ = _rand_problem(m, 300_007, 29, seed=40 + m, lut_kind="int")
    got = psc.hamming_histogram(_dev(qcodes), _dev(codes))
    torch.cuda.synchronize()
    want = O.hamming_histogram(qcodes, codes)
    assert np.array_equal(got.cpu().numpy(), want)
    assert psc.threshold_for_rate(got, 0.05) == O.threshold_for_rate(want, 0.05)
    empty = psc.hamming_histogram(_dev(qcodes), torch.empty((0, m), dtype=torch.uint8, device="cuda"))
    assert int(empty.sum()) == 0


@pytest.mark.parametrize("route", ["auto", "mfma", "popcount"])
@pytest.mark.parametrize("m,n,nq,k", [
    (8, 60_001, 37, 1), (8, 60_001, 37, 64), (8, 60_001, 20, 100), (8, 60_001, 9, 129), (8, 60_001, 1, 100),
    (8, 40_003, 3, 300), (16, 40_003, 19, 100), (16, 40_003, 2, 65), (16, 40_003, 9, 272),
])
def test_thousands_of_codes_at_the_kth_distance(psc, force_route, route, m, n, nq, k):
    """Six distinct codes share every database: each list fills with copies of a few of them, everything
    else at the k-th distance ties and is told apart by its id alone.  Whole-number tables: ids are exact."""
    force_route(route)
    rng = np.random.default_rng(77 + k)
    few = W.random_codes(6, m, seed=5)
    codes = np.ascontiguousarray(few[rng.integers(0, 6, size=n)])
    qcodes = np.ascontiguousarray(few[rng.integers(0, 6, size=nq)])
    lut = rng.integers(0, 50, size=(nq, m, 256)).astype(np.float32)
    for ht in (0, 7 * m // 2, 8 * m):
        got_ids, got_d = _run(psc, lut, qcodes, codes, ht, k)
        _took(psc, route, m, nq, ht, k)
        ref = O.scan(lut.astype(np.float64), qcodes, codes, ht, k)
        assert np.array_equal(got_ids, ref["ids"]) and np.array_equal(got_d, ref["dists"]), (m, n, nq, k, ht)


@pytest.mark.parametrize("nq", [1, 3, 64, 128, 129])
@pytest.mark.parametrize("m,n,ht", [(8, 200_003, 24), (16, 100_001, 64), (8, 65_536, 64)])
def test_slices_put_together_by_the_last_workgroup(psc, m, n, nq, ht):
    """Small scans of up to 128 queries are cut into slices whose keys the query's last workgroup selects from, or
    a merge launch where they do not fit its pool (8 slices of 513 or more) or are many for few results: the same
    workspace call after call."""
    codes, qcodes, lut = _rand_problem(m, n, nq, seed=41 + nq, lut_kind="int")
    ws = torch.full((psc.scan_workspace_bytes(m, nq, n, 1024),), 0xa5, dtype=torch.uint8, device="cuda")
    args = _dev(lut), _dev(qcodes), _dev(codes)
    fit = []
    for k in (1, 10, 512, 513, 1024, 10):
        ids, d = psc.scan(*args, ht, k, workspace=ws)
        torch.cuda.synchronize()
        if k > 1:  # (for k = 1 some of these sizes take the tiles)
            kernel, slices = _route(psc)
            assert kernel.startswith("scan_pool_kernel") and (slices > 1) == (nq <= 128), (k, kernel, slices)
            fit.append(slices * k <= (256 if k <= 16 else 4096))
        ref = O.scan(lut.astype(np.float64), qcodes, codes, ht, k)
        assert np.array_equal(ids.cpu().numpy(), ref["ids"]) and np.array_equal(d.cpu().numpy(), ref["dists"]), k
    assert sum(fit) >= 3 and all(fit) == (nq > 3), fit


def _route(psc):
    words = psc.last_scan_route().split()
    return words[0], int([w for w in words if w.startswith("slices=")][0][7:])


@pytest.mark.parametrize("nq,k", [(1, 100), (1, 64), (2, 1024)])
def test_slices_whose_keys_do_not_fit_one_pool(psc, nq, k):
    """More than 4096 keys of a query's slices: a merge launch (64 places: the last number of slices that fits)."""
    codes, qcodes, lut = _rand_problem(8, 5_000_001, nq, seed=60 + k, lut_kind="int")
    ws = torch.full((psc.scan_workspace_bytes(8, nq, 5_000_001, k),), 0xa5, dtype=torch.uint8, device="cuda")
    for _ in range(2):
        ids, d = psc.scan(_dev(lut), _dev(qcodes), _dev(codes), 24, k, workspace=ws)
        torch.cuda.synchronize()
        kernel, slices = _route(psc)
        assert kernel == "scan_pool_kernel" and (slices * k > 4096) == (k != 64), (kernel, slices)
        ref = O.scan(lut.astype(np.float64), qcodes, codes, 24, k)
        assert np.array_equal(ids.cpu().numpy(), ref["ids"]) and np.array_equal(d.cpu().numpy(), ref["dists"])
