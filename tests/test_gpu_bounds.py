"""The flat search by bounds on the matrix cores: the same answer as the kernels it stands in for, to the bit, over the
sizes, thresholds and data that its rule and its tiles distinguish (needs an MI355X)."""
import numpy as np
import pytest
import torch

import oracle as O
import workloads as W
from gpu_util import assert_topk_matches

pytestmark = pytest.mark.gpu


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _mixture(n, dim, seed, clusters=40):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    centres = torch.rand((clusters, dim), generator=torch.Generator(device="cuda").manual_seed(7), device="cuda") * 100.0
    comp = torch.randint(0, clusters, (n,), generator=g, device="cuda")
    return (torch.randn((n, dim), generator=g, device="cuda") * 15.0 + centres[comp]).round_(), comp


@pytest.fixture(scope="module")
def trained():
    """Indexes by (dim, m), trained once; codes of 400 003 vectors."""
    import paper_1609_01882_amd as psc
    made = {}

    def get(dim, m):
        if (dim, m) not in made:
            idx = psc.Index(dim, m)
            idx.train_pq_device(_mixture(8_000, dim, 1)[0], iters=4, seed=1)
            idx.optimize_index_assignment(n_iter=30_000, seed=2)
            made[dim, m] = (idx, idx.encode(_mixture(400_003, dim, 2)[0]))
        return made[dim, m]
    return get


def _both(psc, idx, q, codes, ht, k, ws=None):
    """(route, ids, dists) taken by the rule, and by the tiled kernels."""
    out = []
    for route in ("auto", "mfma"):
        psc.set_filter_route(route)
        ids, d = idx.search(q, codes, ht, k, workspace=ws if route == "auto" else None)
        torch.cuda.synchronize()
        out.append((psc.last_scan_route().split()[0], ids, d))
    psc.set_filter_route("auto")
    return out


# every padded length of a sub-vector and step count; queries at the edges of groups of 32 and tiles; codes at the edges
# of blocks of 128 and turns of 32; k from 1 to the largest the route takes; thresholds from filtering to none
@pytest.mark.parametrize("dim,m,n,nq,ht,k", [
    (128, 8, 400_003, 1025, 64, 10), (128, 8, 262_144, 1500, 24, 100), (128, 8, 262_145, 1537, 28, 256),
    (96, 8, 399_999, 700, 30, 1), (64, 8, 400_000, 801, 29, 37), (48, 8, 300_031, 1000, 64, 100),
    (256, 8, 400_003, 600, 32, 100), (192, 8, 200_033, 700, 64, 10),
    (128, 16, 400_003, 999, 56, 100), (96, 16, 262_143, 1500, 128, 200), (64, 16, 300_097, 640, 128, 10),
    (256, 16, 400_003, 513, 64, 100), (192, 16, 200_001, 700, 128, 37),
])
def test_bounds_and_tiled_kernels_agree(trained, force_route, dim, m, n, nq, ht, k):
    import paper_1609_01882_amd as psc
    idx, codes = trained(dim, m)
    q = _mixture(nq, dim, 3)[0]
    print(f"dim={dim} m={m} n={n} nq={nq} ht={ht} k={k}", flush=True)
    (route, ids, d), (other, want_ids, want_d) = _both(psc, idx, q, codes[:n].contiguous(), ht, k)
    assert route == "bound_scan_kernel" and other != route, (route, other)
    assert torch.equal(ids, want_ids) and torch.equal(d, want_d)


@pytest.mark.parametrize("m,ht", [(8, 64), (8, 26), (16, 128)])
def test_search_by_bounds_matches_oracle(trained, m, ht):
    import paper_1609_01882_amd as psc
    idx, codes = trained(128, m)
    n, nq, k = 200_007, 600, 20
    c = codes[:n].contiguous()
    q = _mixture(nq, 128, 4)[0]
    ids, d = idx.search(q, c, ht, k)
    assert psc.last_scan_route().startswith("bound_scan_kernel ")
    lut, qc = idx.build_lut(q[:60].contiguous())
    torch.cuda.synchronize()
    lut64, qc_h, c_h = lut.cpu().numpy().astype(np.float64), qc.cpu().numpy(), c.cpu().numpy()
    ref = O.scan(lut64, qc_h, c_h, ht, k)
    assert_topk_matches(ids[:60].cpu().numpy(), d[:60].cpu().numpy(), ref, lut64, qc_h, c_h, ht, what=f"bounds m={m} ht={ht}")


@pytest.mark.parametrize("data", ["sorted", "few distinct", "one code", "random codes", "far queries", "near the mean"])
def test_data_that_the_rounds_do_not_expect(trained, force_route, data):
    """Databases in the order of their clusters, with thousands of equal codes, of one code; codes and numberings
    that say nothing about distance; queries far from every code, and at the mean: marked or not, the same answer."""
    import paper_1609_01882_amd as psc
    idx, codes = trained(128, 8)
    n, nq, k, ht = 300_007, 600, 50, 24
    q = _mixture(nq, 128, 5)[0]
    c = codes[:n]
    if data == "sorted":
        c = c[torch.sort(c[:, 0].to(torch.int64) * 256 + c[:, 1].to(torch.int64)).indices]
    elif data == "few distinct":
        c = c[:300].repeat((n + 299) // 300, 1)[:n]
    elif data == "one code":
        c = c[:1].repeat(n, 1)
        ht = 64
    elif data == "random codes":
        c = _dev(W.random_codes(n, 8, seed=5))
    elif data == "far queries":
        q = q * 50.0 + 3000.0
        ht = 64
    elif data == "near the mean":
        q = q * 1e-3 + q.mean(0, keepdim=True)
        ht = 64
    print(data, flush=True)
    (route, ids, d), (_, want_ids, want_d) = _both(psc, idx, q.contiguous(), c.contiguous(), ht, k)
    assert route == "bound_scan_kernel", route
    assert torch.equal(ids, want_ids) and torch.equal(d, want_d)


# the shapes whose waves hold four groups of queries (256 dimensions), whose queue is drained in the middle of a group, and one
# of 8 coordinates a sub-vector; rows of a turn of 32 apart: those of result registers 6 .. 8 far, the others near, and the reverse
@pytest.mark.parametrize("dim,m,ht", [(256, 8, 64), (256, 8, 30), (256, 16, 128), (256, 16, 60), (64, 8, 64)])
@pytest.mark.parametrize("data", ["sorted", "few distinct", "one code", "mostly one code", "half one code", "six rows of 32 far",
                                  "six rows of 32 near"])
def test_data_that_the_rounds_do_not_expect_at_other_lengths(trained, force_route, dim, m, ht, data):
    import paper_1609_01882_amd as psc
    idx, codes = trained(dim, m)
    n, nq, k = 300_007, 330, 50
    q = _mixture(nq, dim, 5)[0]
    c = codes[:n].clone()
    common = codes[123].clone()
    six = torch.isin(torch.arange(n, device="cuda") % 32, torch.tensor([10, 11, 14, 15, 16, 20], device="cuda"))
    if data == "sorted":
        c = c[torch.sort(c[:, 0].to(torch.int64) * 256 + c[:, 1].to(torch.int64)).indices]
    elif data == "few distinct":
        c = c[:300].repeat((n + 299) // 300, 1)[:n]
    elif data == "one code":
        c[:] = common
    else:
        if data in ("mostly one code", "half one code"):
            share = 0.7 if data == "mostly one code" else 0.5
            c[torch.rand((n,), generator=torch.Generator(device="cuda").manual_seed(11), device="cuda") < share] = common
        else:
            c[~six if data == "six rows of 32 far" else six] = common
        # queries at the common code's vector and a little off it, and some of the mixture
        vector = torch.from_numpy(idx.get_codebook()).cuda()[torch.arange(m, device="cuda"), common.long()].reshape(1, dim)
        q[:300] = vector + (torch.arange(300, device="cuda") % 5)[:, None] * 0.02 * (q[:300] - vector)
    print(f"dim={dim} m={m} ht={ht} {data}", flush=True)
    (route, ids, d), (other, want_ids, want_d) = _both(psc, idx, q.contiguous(), c.contiguous(), ht, k)
    assert route == "bound_scan_kernel" and other != route, (route, other)
    assert torch.equal(ids, want_ids) and torch.equal(d, want_d)


def test_queries_that_are_not_finite_are_left_to_the_other_scan(trained, force_route):
    import paper_1609_01882_amd as psc
    idx, codes = trained(128, 8)
    q = _mixture(700, 128, 6)[0]
    q[3, 5], q[40, 0], q[41, 127], q[699, 64], q[100], q[200] = float("nan"), float("inf"), -float("inf"), 3e38, 1e25, 1e19
    (route, ids, d), (_, want_ids, want_d) = _both(psc, idx, q, codes[:250_000].contiguous(), 64, 10)
    assert route == "bound_scan_kernel", route
    assert torch.equal(ids, want_ids) and torch.equal(d.view(torch.int32), want_d.view(torch.int32))


def test_fewer_codes_within_the_threshold_than_asked_for(trained, force_route):
    """Queries whose own code is far from every other: some have fewer than k codes within the threshold."""
    import paper_1609_01882_amd as psc
    idx, codes = trained(128, 16)
    q = _mixture(1200, 128, 8)[0]
    q[::3] = 100.0 - q[::3]
    (route, ids, d), (_, want_ids, want_d) = _both(psc, idx, q, codes[:300_000].contiguous(), 48, 256)
    assert route == "bound_scan_kernel", route
    assert torch.equal(ids, want_ids) and torch.equal(d, want_d)


def test_workspaces_and_codebooks_without_the_bounds(trained, force_route):
    """A workspace with room for the plain search only, one full of another call's words, and a codebook that has no
    scale."""
    import paper_1609_01882_amd as psc
    idx, codes = trained(128, 8)
    n, nq, k, ht = 300_000, 700, 10, 64
    c, q = codes[:n].contiguous(), _mixture(nq, 128, 9)[0]
    full = idx.search_workspace_bytes(nq, n, k)
    plain = (psc.scan_workspace_bytes(8, nq, n, k) + 255) // 256 * 256 + nq * 8 * 1024 + (nq * 8 + 255) // 256 * 256
    assert plain < full
    ws = torch.full((full,), 0xa5, dtype=torch.uint8, device="cuda")
    ids, d = idx.search(q, c, ht, k, workspace=ws)
    assert psc.last_scan_route().startswith("bound_scan_kernel ")
    ids2, d2 = idx.search(q, c, ht, k, workspace=ws[:plain])
    assert not psc.last_scan_route().startswith("bound_scan_kernel ")
    torch.cuda.synchronize()
    assert torch.equal(ids, ids2) and torch.equal(d, d2)
    flat = psc.Index(128, 8)
    flat.set_codebook(np.zeros((8, 256, 16), np.float32))
    ids3, d3 = flat.search(q, c, ht, k)
    torch.cuda.synchronize()
    assert not psc.last_scan_route().startswith("bound_scan_kernel ")
    assert torch.equal(ids3.cpu(), torch.arange(k).repeat(nq, 1))


def test_replays_of_a_recorded_search_by_bounds(trained):
    import paper_1609_01882_amd as psc
    idx, codes = trained(128, 8)
    n, nq, k, ht = 250_000, 700, 10, 64
    c, q = codes[:n].contiguous(), _mixture(nq, 128, 10)[0].clone()
    ws = torch.empty(idx.search_workspace_bytes(nq, n, k), dtype=torch.uint8, device="cuda")
    out = (torch.empty((nq, k), dtype=torch.int64, device="cuda"), torch.empty((nq, k), dtype=torch.float32, device="cuda"))
    idx.search(q, c, ht, k, workspace=ws, out=out)
    assert psc.last_scan_route().startswith("bound_scan_kernel ")
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        idx.search(q, c, ht, k, workspace=ws, out=out)
    for turn in range(4):
        q.copy_(_mixture(nq, 128, 20 + turn)[0])
        out[0].fill_(-7)
        print(f"replay {turn}", flush=True)
        graph.replay()
        torch.cuda.synchronize()
        got = out[0].clone(), out[1].clone()
        want = idx.search(q, c, ht, k)
        torch.cuda.synchronize()
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1]), turn


@pytest.mark.parametrize("marked", ["none", "few", "a sixteenth", "one more", "many"])
def test_marked_queries_side_by_side(trained, force_route, marked):
    """A search long enough for few marks to be scanned by themselves: none, some scattered ones (the first and
    the last query among them), as many as are few, one more, and a third of all (marks by queries that are not finite)."""
    import paper_1609_01882_amd as psc
    idx, codes = trained(128, 8)
    codes = codes.repeat(3, 1).contiguous()
    nq = 3001
    q = _mixture(nq, 128, 5)[0]
    few = (nq + 15) // 16
    rows = {"none": [], "few": [0, 17, 255, 256, 1000, nq - 1], "a sixteenth": list(range(0, nq, 16))[:few],
            "one more": list(range(0, 7 * (few + 1), 7)), "many": list(range(0, nq, 3))}[marked]
    if rows:
        q[torch.tensor(rows, device="cuda"), 5] = float("inf")
    (route, ids, d), (other, ids2, d2) = _both(psc, idx, q, codes, 64, 20)
    assert route == "bound_scan_kernel" and other != route, (route, other)
    assert torch.equal(ids, ids2)
    assert torch.equal(d.view(torch.int32), d2.view(torch.int32))


@pytest.mark.parametrize("m,nq,k", [(8, 400, 100), (16, 300, 64), (8, 520, 256)])
def test_few_marked_queries_whose_distances_are_infinite(trained, force_route, m, nq, k):
    """Which codes at distance +infinity are listed goes by the size of the whole batch (the kernel that merges its lists),
    not by that of the few marked queries that are scanned by themselves."""
    import paper_1609_01882_amd as psc
    idx, codes = trained(128, m)
    codes = codes.repeat(10, 1).contiguous()
    q = _mixture(nq, 128, 12)[0]
    q[3, 5], q[77], q[nq - 1, 0], q[nq - 1, 127] = float("inf"), 1e25, 1.5e19, 1.5e19
    print(f"m={m} nq={nq} k={k}", flush=True)
    (route, ids, d), (other, want_ids, want_d) = _both(psc, idx, q, codes, 8 * m, k)
    assert route == "bound_scan_kernel" and other != route, (route, other)
    assert torch.equal(ids, want_ids) and torch.equal(d.view(torch.int32), want_d.view(torch.int32))


@pytest.mark.parametrize("m,n,nq,ht,k", [(8, 200_003, 3000, 24, 100), (8, 100_003, 2000, 64, 10), (8, 400_003, 100, 64, 10),
                                         (16, 200_003, 1500, 56, 37), (16, 300_001, 100, 128, 100)])
@pytest.mark.parametrize("share", [1.0, 0.3])
def test_batches_that_are_left_to_the_scan(trained, m, n, nq, ht, k, share):
    """All queries marked, and a third of them: the scan of the former route answers them, the small scan (whose results
    those of `scan` on ready tables are) where that is its route."""
    import paper_1609_01882_amd as psc
    idx, codes = trained(128, m)
    c = codes[:n].contiguous() if share < 1.0 else _dev(W.random_codes(n, m, seed=6))
    q = _mixture(nq, 128, 13)[0]
    if share < 1.0:
        q[torch.arange(nq, device="cuda") % 10 < 3, 7] = float("inf")
    print(f"m={m} n={n} nq={nq} ht={ht} k={k} {share}", flush=True)
    ids, d = idx.search(q, c, ht, k)
    assert psc.last_scan_route().startswith("bound_scan_kernel ")
    lut, qc = idx.build_lut(q)
    want_ids, want_d = psc.scan(lut, qc, c, ht, k)
    torch.cuda.synchronize()
    assert torch.equal(ids, want_ids) and torch.equal(d.view(torch.int32), want_d.view(torch.int32))


@pytest.mark.parametrize("dim,m,n,nq", [(128, 8, 3_200_024, 600), (256, 16, 1_200_009, 300)])
def test_lists_that_run_over_in_the_first_of_several_rounds(trained, force_route, dim, m, n, nq):
    """A database of one code but for some rows: every query is marked before the later rounds."""
    import paper_1609_01882_amd as psc
    idx, codes = trained(dim, m)
    c = codes[:1].repeat(n, 1)
    c[::1001] = codes[1]
    q = _mixture(nq, dim, 14)[0]
    print(f"dim={dim} m={m} n={n} nq={nq}", flush=True)
    (route, ids, d), (other, want_ids, want_d) = _both(psc, idx, q, c, 8 * m, 10)
    assert route == "bound_scan_kernel" and other != route, (route, other)
    assert torch.equal(ids, want_ids) and torch.equal(d, want_d)


@pytest.mark.parametrize("m,ht,kinds", [(16, 48, 1000), (16, 50, 400), (8, 22, 300)])
def test_batches_of_which_a_part_is_marked_at_the_sample(trained, m, ht, kinds):
    """Codes of few kinds under a strict threshold: the sample finds no bound for a part of the queries, more than are
    answered by themselves and fewer than most; the batch is given up or not, the results are those of the scan."""
    import paper_1609_01882_amd as psc
    idx, codes = trained(128, m)
    n, nq, k = 200_003, 3000, 100
    c = codes[:kinds].repeat((n + kinds - 1) // kinds, 1)[:n].contiguous()
    q = _mixture(nq, 128, 15)[0]
    print(f"m={m} ht={ht} kinds={kinds}", flush=True)
    ids, d = idx.search(q, c, ht, k)
    assert psc.last_scan_route().startswith("bound_scan_kernel ")
    lut, qc = idx.build_lut(q)
    want_ids, want_d = psc.scan(lut, qc, c, ht, k)
    torch.cuda.synchronize()
    assert torch.equal(ids, want_ids) and torch.equal(d.view(torch.int32), want_d.view(torch.int32))
