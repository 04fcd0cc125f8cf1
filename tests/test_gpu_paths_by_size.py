"""Kernel variants that a rule on sizes selects, at the sizes where they can go wrong."""
import time

import numpy as np
import pytest
import torch

import oracle as O
import paper_2502_20969_amd as P
from parity import check_topk, stored

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def streams():
    assert torch.cuda.is_available()
    return torch.cuda.Stream(), torch.cuda.Stream()


@pytest.mark.parametrize("k", [57, 64, 112])
@pytest.mark.parametrize("n,layout", [(130, "random"), (9000, "random"), (60000, "random"), (60000, "best_first"),
                                      (60000, "best_in_two_lists"), (60000, "equal")])
def test_merge_of_wide_lists(streams, k, n, layout):
    """More than 56 results: the merge cuts by the heads of the wavefronts' lists.  best_first and
    best_in_two_lists put all good rows into few lists, so that the first cut lets more pass than
    the pool holds; with masses of equal scores no cut helps and the radix select takes over."""
    rng = np.random.default_rng(k + n)
    d, nlist = 16, 70                       # more than 64 lists: contiguous shares per wavefront
    score = rng.permutation(n).astype(np.float32) / n
    if layout == "best_first":
        score = -np.sort(-score)
    elif layout == "best_in_two_lists":
        score[n // 2:n // 2 + 6000] += 2.0
    elif layout == "equal":
        score[rng.permutation(n)[:30000]] = 2.0
    rows = np.zeros((n, d), np.float32)
    rows[:, 0] = score
    assign = (np.arange(n) * nlist // n).astype(np.int32)
    cent = 0.01 * rng.standard_normal((nlist, d)).astype(np.float32)
    ids = rng.permutation(n).astype(np.int64) * 3
    index = P.ivf_build_layout(rows, "f32", cent, assign, ids=ids, compute_stream=streams[0], copy_stream=streams[1])
    off, perm = O.build_layout(assign, nlist)
    q = np.zeros((1, d), np.float32)
    q[0, 0] = 1.0
    gi, gd = index.ivf_search(q, nlist, k)
    oi, osc = O.search(rows[perm], O.F32, off, ids[perm], cent, q[0], nlist, k, O.IP)
    assert list(gi[0]) == list(oi)
    np.testing.assert_array_equal(gd[0], osc.astype(np.float32))
    index.close()


@pytest.mark.parametrize("B,d,micro", [(2, 64, 2), (16, 65, 3), (17, 128, 16), (511, 64, 9), (512, 3, 512), (513, 130, 8),
                                       (1025, 64, 600), (4096, 4, 17)])
def test_scheduler_walks_sorted_lists(streams, B, d, micro):
    """Edges of the scheduler's tiles (16 queries, 64 components), of its sorted lists (a power of
    two, steps of 512 entries) and groups that need more than one step; half the queries are
    duplicates of others, so that equal distances are common."""
    rng = np.random.default_rng(B + d)
    q = rng.standard_normal((B, d)).astype(np.float32)
    q[rng.permutation(B)[:B // 2]] = q[rng.integers(0, B, B // 2)]
    rows = torch.zeros(1, d, device="cuda")
    index = P.ivf_adopt_layout(rows, "f32", np.array([0, 1]), np.zeros((1, d), np.float32), compute_stream=streams[0],
                               copy_stream=streams[1])
    assert list(index.ivf_schedule(q, micro)) == list(O.schedule(q, micro))
    index.close()


def test_scheduler_calls_of_changing_size(streams):
    """Batches whose workspace is kept, replaced by a larger one's or made for one call, in turn."""
    rng = np.random.default_rng(7)
    index = P.ivf_adopt_layout(torch.zeros(1, 20, device="cuda"), "f32", np.array([0, 1]), np.zeros((1, 20), np.float32),
                               compute_stream=streams[0], copy_stream=streams[1])
    for B in (100, 1024, 1025, 300, 2100, 1024):
        q = rng.standard_normal((B, 20)).astype(np.float32)
        assert list(index.ivf_schedule(q, 7)) == list(O.schedule(q, 7))
    index.close()


@pytest.mark.parametrize("value", [np.nan, np.inf])
@pytest.mark.parametrize("B", [40, 700])
def test_scheduler_distances_that_are_no_numbers(streams, B, value):
    """A distance that is no number is farther than any other, an infinite one farther than any finite."""
    rng = np.random.default_rng(B)
    q = rng.standard_normal((B, 24)).astype(np.float32)
    q[rng.permutation(B)[:B // 5], 3] = value
    index = P.ivf_adopt_layout(torch.zeros(1, 24, device="cuda"), "f32", np.array([0, 1]), np.zeros((1, 24), np.float32),
                               compute_stream=streams[0], copy_stream=streams[1])
    order = list(index.ivf_schedule(q, 9))
    index.close()
    with np.errstate(invalid="ignore"):
        dist = ((q.astype(np.float64)[:, None] - q.astype(np.float64)[None]) ** 2).sum(2)
    left, want = list(range(B)), []
    while left:
        seed = left.pop(0)
        near = sorted(left, key=lambda j: (np.isnan(dist[seed, j]), 0.0 if np.isnan(dist[seed, j]) else dist[seed, j], j))[:8]
        want += [seed] + near
        left = [j for j in left if j not in near]
    assert order == want


@pytest.mark.parametrize("metric", ["ip", "l2"])
@pytest.mark.parametrize("nq,nlist,d", [(2, 40, 64), (3, 15, 4), (3, 129, 768), (15, 17, 36), (16, 1, 260), (17, 33, 1028),
                                        (33, 6200, 20), (130, 1100, 96), (1, 9, 3), (2, 30, 257), (4, 33, 1), (5, 70, 2), (17, 40, 31),
                                        (20, 300, 295), (40, 2000, 1023), (200, 50, 37),
                                        (3, 2048, 768), (4, 2049, 1024), (4, 31, 1028), (16, 13000, 33), (64, 16384, 64), (250, 8200, 100),
                                        (250, 8200, 67)])
def test_coarse_scores_by_batch_size(streams, nq, nlist, d, metric):
    """Row kernel, small and large matrix-core tiles: ragged in queries, centroids and elements (a
    row's blocks of 32 elements are dealt to 1, 4 or 8 wavefronts), two XCD groups and more."""
    rng = np.random.default_rng(nq * nlist + d)
    cent = rng.standard_normal((nlist, d)).astype(np.float32)
    q = rng.standard_normal((nq, d)).astype(np.float32)
    rows = torch.zeros(nlist, d, device="cuda")
    index = P.ivf_adopt_layout(rows, "f32", np.arange(nlist + 1), cent, metric=P.IVF_IP if metric == "ip" else P.IVF_L2,
                               compute_stream=streams[0], copy_stream=streams[1])
    got = index.ivf_coarse_scores(q)
    x, y = q.astype(np.float64), cent.astype(np.float64)
    want = x @ y.T if metric == "ip" else np.stack([((one - y) ** 2).sum(1) for one in x])
    # a sum of d products rounded d times: d 2^-53 times the sum of the magnitudes, with room for the three norms form
    bound = 8 * d * 2.0 ** -53 * (np.abs(x) @ np.abs(y).T + (x * x).sum(1)[:, None] + (y * y).sum(1)[None])
    assert (np.abs(got - want) <= bound).all()
    index.close()


@pytest.mark.parametrize("nlist,nq,nprobe,k,d", [(8192, 5, 40, 3, 64), (8193, 5, 40, 3, 64), (9000, 70, 33, 100, 64), (8193, 211, 39, 3, 64),
                                                 (20000, 33, 250, 10, 64), (8192, 211, 39, 3, 64), (3, 2, 3, 1, 128),
                                                 (40, 300, 7, 20, 64), (700, 33, 512, 112, 128)])
def test_front_of_a_list_major_batch(streams, nlist, nq, nprobe, k, d):
    """The map from clusters to queries in LDS, in global memory and counted by launches of its own, samples of fewer rows than k, one
    and several steps of the sample per workgroup: list-major equals query by query bit for bit."""
    rng = np.random.default_rng(nlist + nq)
    n = nlist * 9
    assign = rng.integers(0, nlist, n).astype(np.int32)
    assign[:n // 3] = 0                              # one large cluster, some empty ones
    cent = rng.standard_normal((nlist, d)).astype(np.float32)
    rows = (cent[assign] + 0.5 * rng.standard_normal((n, d))).astype(np.float16)
    index = P.ivf_build_layout(rows, "f16", cent, assign, compute_stream=streams[0], copy_stream=streams[1])
    q = (cent[rng.integers(0, nlist, nq)] + 0.3 * rng.standard_normal((nq, d))).astype(np.float32)
    q[0] = cent[0]
    index.ivf_set_batch_mode(2)
    bi, bd = index.ivf_search(q, nprobe, k)
    index.ivf_set_batch_mode(1)
    pi, pd = index.ivf_search(q, nprobe, k)
    assert np.array_equal(bi, pi) and np.array_equal(bd, pd)
    index.close()


@pytest.mark.parametrize("dtype,metric,k", [("bf16", "ip", 112), ("f16", "l2", 10), ("f32", "ip", 100)])
@pytest.mark.parametrize("band", [3, 120, 700, 4500])
def test_survivors_of_a_list_major_batch(streams, dtype, metric, k, band):
    """`band` rows per query score within the filter's error of each other, a third of them exact
    copies: fewer survivors than k, one look, two looks, and more than the merge holds (the query is
    searched again).  List-major equals query by query bit for bit."""
    rng = np.random.default_rng(band + k)
    d, nlist, nq = 128, 6, 9
    cent = rng.standard_normal((nlist, d)).astype(np.float32)
    rows = 0.2 * rng.standard_normal((nlist * 5000, d)).astype(np.float32)
    assign = (np.arange(rows.shape[0]) % nlist).astype(np.int32)
    for c in range(nlist):
        at = np.nonzero(assign == c)[0][rng.permutation(5000)[:band]]
        rows[at] = cent[c] + 1e-4 * rng.standard_normal((band, d)).astype(np.float32)
        rows[at[:band // 3]] = rows[at[0]]
    st, _ = stored(rows, dtype)
    index = P.ivf_build_layout(st, dtype, cent, assign, metric=P.IVF_IP if metric == "ip" else P.IVF_L2,
                               compute_stream=streams[0], copy_stream=streams[1])
    q = (cent[np.arange(nq) % nlist] + 1e-3 * rng.standard_normal((nq, d))).astype(np.float32)
    index.ivf_set_batch_mode(2)
    bi, bd = index.ivf_search(q, 4, k)
    index.ivf_set_batch_mode(1)
    pi, pd = index.ivf_search(q, 4, k)
    assert np.array_equal(bi, pi) and np.array_equal(bd, pd)
    index.close()


@pytest.mark.parametrize("metric", ["ip", "l2"])
@pytest.mark.parametrize("nlist,nprobe", [(65, 65), (1000, 257), (1024, 1024), (2049, 512), (8191, 65), (8193, 512), (16500, 300), (4097, 3)])
@pytest.mark.parametrize("kind", ["random", "one_side", "ties", "pairs", "near", "many_equal", "infinite", "nan"])
def test_select_of_many_clusters(streams, nlist, nprobe, kind, metric):
    """Selections through the pooled path: scores around zero, scores far from zero, masses of equal
    scores (the pool overflows: the exact path), scores that are equal in pairs, that differ in the low
    bits of their keys only or that are equal by the hundred (prefixes tie inside the pool and across
    the cut), and infinite ones; order and content are the oracle's."""
    rng = np.random.default_rng(nlist + nprobe)
    d = 8
    cent = rng.standard_normal((nlist, d)).astype(np.float32)
    q = rng.standard_normal((3, d)).astype(np.float32)
    if kind == "one_side":
        cent, q = np.abs(cent) + 3.0, np.abs(q) + 1.0
    elif kind == "ties":
        cent = np.round(cent)
        cent[rng.permutation(nlist)[:nlist // 2]] = cent[0]
    elif kind == "pairs":
        cent[nlist // 2:nlist // 2 * 2] = cent[:nlist // 2]
    elif kind == "near":
        # one large element of one value, the small one decides: relative differences of 1e-11 and less
        cent[:, 1:] = 0.0
        cent[:, 0] = 1.0
        cent[:, 3] = 1e-10 * rng.permutation(nlist) / nlist
        q[:, 0], q[:, 3] = 100.0, 1.0
        if metric == "l2":
            cent[:, 3] *= 1e2
    elif kind == "many_equal":
        best = rng.permutation(nlist)[:min(nprobe + 40, 700)]
        cent[best] = 4.0 * np.sign(q[0])
    elif kind == "infinite":
        cent[rng.permutation(nlist)[:nprobe // 2]] *= np.float32(1e30)
        q *= np.float32(1e30)
    elif kind == "nan":
        cent[nlist // 2, 3] = np.nan            # one score that is none: the same choice in every path
    rows = torch.zeros(nlist, d, device="cuda")
    index = P.ivf_adopt_layout(rows, "f32", np.arange(nlist + 1), cent, metric=P.IVF_IP if metric == "ip" else P.IVF_L2,
                               compute_stream=streams[0], copy_stream=streams[1])
    pr = index.ivf_probe(q, nprobe)
    if kind == "nan":
        # the oracle's sort has no place for it: the exact selection of all lists does
        full = index.ivf_probe(q, nlist)
        assert np.array_equal(pr, full[:, :nprobe])
    else:
        for b in range(3):
            assert list(pr[b]) == list(O.probe(cent, q[b], nprobe, O.IP if metric == "ip" else O.L2))
    index.close()


@pytest.mark.parametrize("metric", ["ip", "l2"])
@pytest.mark.parametrize("dtype,d", [("f32", 3), ("f32", 5), ("f32", 63), ("f32", 65), ("f32", 129), ("f32", 333), ("f32", 770), ("f32", 2047),
                                     ("f16", 7), ("f16", 9), ("f16", 127), ("f16", 129), ("f16", 300), ("f16", 513), ("bf16", 31),
                                     ("bf16", 767), ("bf16", 1030), ("bf16", 4095)])
def test_rows_that_are_not_whole_chunks(streams, dtype, d, metric):
    """Every scan shape with a partial last chunk, rows at every alignment; the last row ends where the
    buffer does.  The oracle's results.  Then an infinite element in the part of a row that two
    lanes load: counted once it makes the row the nearest (inner product) or the farthest (L2), and
    multiplied by the zero that the second lane has for it the row would be no number and lost."""
    rng = np.random.default_rng(d)
    n, nlist, k = 331, 5, 12
    om = O.IP if metric == "ip" else O.L2
    cent = rng.standard_normal((nlist, d)).astype(np.float32)
    assign = rng.integers(0, nlist, n).astype(np.int32)
    rows = (cent[assign] + rng.standard_normal((n, d))).astype(np.float32)
    q = np.abs(rng.standard_normal((4, d))).astype(np.float32) + 0.1

    def search(rows, k):
        st, odt = stored(rows, dtype)
        index = P.ivf_build_layout(st, dtype, cent, assign, metric=P.IVF_IP if metric == "ip" else P.IVF_L2,
                                   compute_stream=streams[0], copy_stream=streams[1])
        out = index.ivf_search(q, nlist, k)
        index.close()
        return st, odt, out

    st, odt, (gi, gd) = search(rows, k)
    off, perm = O.build_layout(assign, nlist)
    for b in range(4):
        assert check_topk(gi[b], gd[b], st[perm], odt, off, perm.astype(np.int64), cent, q[b], nlist, k, om) == 0
    per_chunk = 4 if dtype == "f32" else 8
    odd = int(gi[0][2])                                     # a row that is among the nearest
    rows[odd, max(d - per_chunk, 0)] = np.inf               # the first element of the 16 bytes that end the row
    assert d < per_chunk or max(d - per_chunk, 0) < d // per_chunk * per_chunk
    _, _, (hi, hd) = search(rows, k)
    for b in range(4):
        others = [(i, x) for i, x in zip(gi[b], gd[b]) if i != odd]
        got = list(zip(hi[b], hd[b]))
        if metric == "ip":
            assert got == [(odd, np.inf)] + others[:k - 1]
        else:
            assert odd not in hi[b] and got[:len(others)] == others


@pytest.mark.parametrize("dtype,d,per_batch", [("f32", 64, 24), ("f16", 90, 24), ("f32", 128, 12), ("f32", 101, 12), ("bf16", 512, 6), ("f32", 255, 6)])
@pytest.mark.parametrize("windows", [1, 511, 512, 513, 1100])
def test_scan_of_few_rows(streams, dtype, d, per_batch, windows):
    """Calls of few rows take smaller batches than the search on the fixed scratch area, which keeps
    the usual ones: the results are the same bit for bit on both sides of the rule, and the oracle's
    is found for the smallest."""
    rng = np.random.default_rng(windows + d)
    nlist, n = 7, windows * per_batch + 5
    cent = rng.standard_normal((nlist, d)).astype(np.float32)
    assign = rng.integers(0, nlist, n).astype(np.int32)
    rows = (cent[assign] + 0.5 * rng.standard_normal((n, d))).astype(np.float32)
    st, odt = stored(rows, dtype)
    index = P.ivf_build_layout(st, dtype, cent, assign, compute_stream=streams[0], copy_stream=streams[1])
    index.ivf_set_batch_mode(1)
    for nq in (1, 3):
        q = torch.from_numpy((cent[:nq] + 0.3 * rng.standard_normal((nq, d))).astype(np.float32)).cuda()
        out = []
        for call in (index.ivf_search_device, index.ivf_search_device_noalloc):
            ids, dists = torch.empty(nq, 9, dtype=torch.int64, device="cuda"), torch.empty(nq, 9, device="cuda")
            torch.cuda.synchronize()
            call(q, nlist, 9, ids, dists)
            torch.cuda.synchronize()
            out.append((ids.cpu().numpy(), dists.cpu().numpy()))
        assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])
    if windows == 1:
        off, perm = O.build_layout(assign, nlist)
        for b in range(3):
            assert check_topk(out[0][0][b], out[0][1][b], st[perm], odt, off, perm.astype(np.int64), cent, q[b].cpu().numpy(), nlist, 9, O.IP) == 0
    index.close()


def _copies(streams, copies, ids, nq=4, d=64, per=5000, nlist=6):
    """An index whose best rows for queries at the centres are `copies` equal ones per cluster."""
    rng = np.random.default_rng(copies)
    cent = rng.standard_normal((nlist, d)).astype(np.float32)
    assign = np.repeat(np.arange(nlist, dtype=np.int32), per)
    rows = (cent[assign] + 0.5 * rng.standard_normal((nlist * per, d))).astype(np.float32)
    for c in range(nlist):
        rows[c * per + rng.permutation(per)[:copies]] = 1.5 * cent[c]
    index = P.ivf_build_layout(rows.astype(np.float16), "f16", cent, assign, ids=ids, compute_stream=streams[0], copy_stream=streams[1])
    return index, (cent[np.arange(nq) % nlist] + 0.01 * rng.standard_normal((nq, d))).astype(np.float32)


@pytest.mark.parametrize("copies", [2, 40, 600, 3500])
@pytest.mark.parametrize("kind", ["none", "small", "large"])
def test_equal_scores_in_a_list_major_batch(streams, copies, kind):
    """Scores that several survivors share, fewer and more than k, around the 512 from which the
    edge of the k best is cut by ids, with ids of 32 and 63 bits: equal to query by query."""
    ids = None if kind == "none" else np.random.default_rng(1).permutation(30000).astype(np.int64) * (3 if kind == "small" else 1 << 48)
    index, q = _copies(streams, copies, ids)
    for k in (1, 39, 41, 112):
        index.ivf_set_batch_mode(2)
        bi, bd = index.ivf_search(q, 3, k)
        index.ivf_set_batch_mode(1)
        pi, pd = index.ivf_search(q, 3, k)
        assert np.array_equal(bi, pi) and np.array_equal(bd, pd)
    index.close()


def test_equal_scores_do_not_stall_a_list_major_batch(streams):
    """3500 copies of the best row cost a batch some hundred microseconds, no multiple of that: not
    every survivor asks memory for the id of every other (which took over 100 times a plain batch)."""
    took = []
    for copies in (1, 3500):
        index, q = _copies(streams, copies, None, nq=32)
        index.ivf_set_batch_mode(2)
        times = []
        for _ in range(9):
            t0 = time.perf_counter()
            index.ivf_search(q, 3, 10)
            times.append(time.perf_counter() - t0)
        took.append(sorted(times)[4])
        index.close()
    # measured 5 to 8 times a plain batch; 25 leaves room for a busy host
    assert took[1] < 25 * took[0], took


@pytest.mark.parametrize("nq", [1, 32])
def test_filter_scores_do_not_depend_on_earlier_searches(streams, nq):
    """ivf_batched_scores leaves the launches it shares with a search what a selection would have
    left: the same scores and bounds on a fresh index, after searches of other shapes, and for clusters
    of one row and of many."""
    rng = np.random.default_rng(nq)
    nlist, d = 9, 128
    assign = np.concatenate([[0], np.full(3000, 1), rng.integers(2, nlist, 4000)]).astype(np.int32)
    cent = rng.standard_normal((nlist, d)).astype(np.float32)
    rows = (cent[assign] + rng.standard_normal((assign.size, d))).astype(np.float16)
    q = rng.standard_normal((nq, d)).astype(np.float32)
    index = P.ivf_build_layout(rows, "f16", cent, assign, compute_stream=streams[0], copy_stream=streams[1])
    sizes = (1, 3000)
    fresh = [index.ivf_batched_scores(q, c, sizes[c]) for c in (0, 1)]
    index.ivf_search(rng.standard_normal((40, d)).astype(np.float32), 7, 5)
    for c in (0, 1):
        for want, got in zip(fresh[c], index.ivf_batched_scores(q, c, sizes[c])):
            np.testing.assert_array_equal(got, want)
        s64 = q.astype(np.float64) @ rows[assign == c].astype(np.float64).T
        assert (np.abs(fresh[c][0] - s64) <= fresh[c][1][:, None]).all()
    index.close()


@pytest.mark.parametrize("nq,nlist,d", [(3, 4096, 4), (3, 4097, 5), (4, 3073, 7), (5, 2460, 255), (15, 820, 256), (15, 819, 257), (15, 5000, 1028),
                                        (16, 769, 259), (63, 200, 513), (130, 1037, 102), (300, 9001, 30)])
def test_coarse_scores_four_by_four(streams, nq, nlist, d):
    """Squared L2 that the matrix cores do not take: from 12,288 pairs of query and centroid on, four by
    four.  The scores are sums of squared differences in fp64, the same bit for bit as of single queries (which
    are never taken four by four); edges of the tiles, of the chunks and of rows that are no multiple of 4."""
    rng = np.random.default_rng(nq + d)
    cent = rng.standard_normal((nlist, d)).astype(np.float32)
    q = rng.standard_normal((nq, d)).astype(np.float32)
    q[nq // 2] = cent[nlist // 3]
    index = P.ivf_adopt_layout(torch.zeros(nlist, d, device="cuda"), "f32", np.arange(nlist + 1), cent, metric=P.IVF_L2,
                               compute_stream=streams[0], copy_stream=streams[1])
    got = index.ivf_coarse_scores(q)
    for b in {0, 1, nq // 2, nq - 1}:
        assert np.array_equal(got[b], index.ivf_coarse_scores(q[b:b + 1])[0])
        want = ((q[b].astype(np.float64) - cent.astype(np.float64)) ** 2).sum(1)
        np.testing.assert_allclose(got[b], want, rtol=1e-12)
    index.close()
