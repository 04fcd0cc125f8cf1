"""GPU parity of the list-major batched search (Sec. 4.2 'Batching': the GPU part becomes a
matrix-matrix product) against the oracle and against the query-by-query path."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2502_20969_amd as P
import workloads as W
from parity import check_topk

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def streams():
    assert torch.cuda.is_available()
    return torch.cuda.Stream(), torch.cuda.Stream()


def _stored_numpy(ds):
    if ds.dtype == "f32":
        return ds.rows.cpu().numpy(), O.F32
    if ds.dtype == "f16":
        return ds.rows.cpu().numpy(), O.F16
    return ds.rows.cpu().view(torch.int16).numpy().view(np.uint16), O.BF16


@pytest.mark.parametrize("dtype,d,nq,k,nprobe,metric", [
    ("f16", 768, 32, 10, 24, "ip"), ("bf16", 1024, 37, 10, 16, "ip"), ("f16", 128, 5, 100, 40, "ip"),
    ("bf16", 256, 64, 1, 7, "ip"),
    ("f32", 768, 8, 3, 24, "ip"), ("f32", 128, 37, 100, 40, "ip"), ("f32", 1024, 16, 10, 7, "l2"), ("f32", 64, 70, 1, 30, "l2"),
    ("f16", 768, 32, 10, 24, "l2"), ("bf16", 256, 64, 5, 7, "l2"),
])
def test_list_major_equals_oracle_and_per_query(streams, dtype, d, nq, k, nprobe, metric):
    pm, om = (P.IVF_IP, O.IP) if metric == "ip" else (P.IVF_L2, O.L2)
    esz = 4 if dtype == "f32" else 2
    nlist = 96
    sizes = W.zipf_sizes(60000 if d <= 256 else 30000, nlist, 1.1, 3)
    sizes[5] += sizes[7]; sizes[7] = 0                  # an empty cluster
    ds = W.cluster_major_datastore(sizes, d, 0.3, 4, dtype=dtype, device="cuda")
    q = W.shared_batch_queries(ds, nq, max(2, nq // 8), 5).cpu().numpy()
    lists, odt = _stored_numpy(ds)
    off = ds.offsets.numpy()
    cent = ds.centroids.cpu().numpy()
    ids = (np.random.default_rng(1).permutation(ds.n) * 2 + 3).astype(np.int64)
    index = P.ivf_adopt_layout(ds.rows, dtype, off, cent, ids=ids, metric=pm,
                               compute_stream=streams[0], copy_stream=streams[1])
    index.ivf_set_batch_mode(2)
    bi, bd, st = index.ivf_search(q, nprobe, k, with_stats=True)
    index.ivf_set_batch_mode(1)
    pi, pd = index.ivf_search(q, nprobe, k)
    assert np.array_equal(bi, pi) and np.array_equal(bd, pd)
    exempt = 0
    for b in range(nq):
        exempt += check_topk(bi[b], bd[b], lists, odt, off, ids, cent, q[b], nprobe, k, om)
    assert exempt == 0
    # bytes reported: the union of the selected clusters, each once
    union = set()
    for b in range(nq):
        union |= set(O.probe(cent, q[b], nprobe, om))
    assert st.bytes_gpu == sum(int(off[c + 1] - off[c]) for c in union) * d * esz
    # device-pointer entry point, automatic mode (nq >= 4 goes list-major)
    index.ivf_set_batch_mode(0)
    q_dev = torch.from_numpy(q).cuda()
    ids_dev = torch.empty(nq, k, dtype=torch.int64, device="cuda")
    d_dev = torch.empty(nq, k, dtype=torch.float32, device="cuda")
    torch.cuda.synchronize()
    index.ivf_search_device(q_dev, nprobe, k, ids_dev, d_dev)
    index.ivf_synchronize()
    assert np.array_equal(ids_dev.cpu().numpy(), pi) and np.array_equal(d_dev.cpu().numpy(), pd)
    index.close()


def test_candidate_overflow_falls_back(streams):
    """Identical rows make every row a candidate: the per-query redo must give the oracle's answer."""
    n, d, nlist = 40000, 64, 4
    rows = torch.full((n, d), 0.125, dtype=torch.float16, device="cuda")
    off = np.array([0, 10000, 20000, 30000, 40000], dtype=np.int64)
    cent = np.eye(nlist, d, dtype=np.float32)
    index = P.ivf_adopt_layout(rows, "f16", off, cent, metric=P.IVF_IP, compute_stream=streams[0], copy_stream=streams[1])
    index.ivf_set_batch_mode(2)
    q = np.abs(np.random.default_rng(2).standard_normal((4, d))).astype(np.float32)
    gi, gd = index.ivf_search(q, 3, 5)
    lists = rows.cpu().numpy()
    for b in range(4):
        oi, osc = O.search(lists, O.F16, off, None, cent, q[b], 3, 5, O.IP)
        assert list(gi[b]) == list(oi)
        np.testing.assert_allclose(gd[b], osc, rtol=2e-3)
    index.close()


@pytest.mark.parametrize("depth", [1, 2, 3])
def test_batches_in_flight_are_finished_by_synchronize(streams, depth):
    """ivf_search_device does not wait for a list-major batch: the queries whose candidate lists
    overflowed are searched again when the batch's stream is next needed or in ivf_synchronize.
    Six batches in a row over `depth` streams, every second one on identical rows in cluster 0
    (all of them overflow), each with its own outputs: all equal the oracle afterwards."""
    n, d, nlist = 24000, 64, 6
    rng = np.random.default_rng(11)
    rows_np = rng.standard_normal((n, d)).astype(np.float16)
    rows_np[:8000] = np.float16(0.125)                         # cluster 0 and 1: identical rows
    off = np.arange(0, n + 1, 4000, dtype=np.int64)
    cent = rng.standard_normal((nlist, d)).astype(np.float32)
    cent[0] = 1.0; cent[1] = 0.9                               # positive queries select them first
    rows = torch.from_numpy(rows_np).cuda()
    index = P.ivf_adopt_layout(rows, "f16", off, cent, metric=P.IVF_IP, compute_stream=streams[0], copy_stream=streams[1])
    index.ivf_set_batch_mode(2)
    index.ivf_set_pipeline_depth(depth)
    nq, k, nprobe = 6, 5, 2
    qs, outs = [], []
    for j in range(6):
        q = rng.standard_normal((nq, d)).astype(np.float32)
        if j % 2 == 0:
            q = np.abs(q)                                      # nearest clusters: the two of identical rows
        qs.append(torch.from_numpy(q).cuda())
        outs.append((torch.empty(nq, k, dtype=torch.int64, device="cuda"), torch.empty(nq, k, device="cuda")))
    torch.cuda.synchronize()
    for j in range(6):
        index.ivf_search_device(qs[j], nprobe, k, outs[j][0], outs[j][1])
    index.ivf_synchronize()
    for j in range(6):
        gi, gd = outs[j][0].cpu().numpy(), outs[j][1].cpu().numpy()
        q = qs[j].cpu().numpy()
        for b in range(nq):
            assert check_topk(gi[b], gd[b], rows_np, O.F16, off, None, cent, q[b], nprobe, k, O.IP) == 0, f"batch {j} query {b}"
    index.close()


@pytest.mark.parametrize("dtype,d,nq", [("f16", 128, 256), ("bf16", 256, 200), ("f16", 768, 32), ("bf16", 64, 77),
                                        ("f32", 128, 200), ("f32", 768, 17), ("f32", 64, 77)])
def test_list_major_finds_every_row_by_its_own_query(streams, dtype, d, nq):
    """Coverage of the batched scan: with every list selected, each stored row is the nearest
    neighbour of its own values (normalised, distinct rows), whichever tile of 256 rows and group of
    queries it falls into.  All rows are asked, nq queries per call; lists are ragged (Zipf sizes
    from thousands of rows down to a handful) and one is empty.  A row's query is its stored values,
    so the rounding of the query to the storage type changes nothing."""
    nlist = 12
    sizes = W.zipf_sizes(7000, nlist, 1.2, 9)
    sizes[3] += sizes[8]; sizes[8] = 0
    ds = W.cluster_major_datastore(sizes, d, 0.3, 10, dtype=dtype, device="cuda")
    wide = ds.rows.to(torch.float64).cpu().numpy()
    n = ds.n
    for lo in range(0, n, 1000):                      # the case is what it claims
        assert np.array_equal(np.argmax(wide[lo:lo + 1000] @ wide.T, axis=1), np.arange(lo, min(lo + 1000, n)))
    ids = (np.random.default_rng(2).permutation(n) * 5 + 2).astype(np.int64)
    index = P.ivf_adopt_layout(ds.rows, dtype, ds.offsets.numpy(), ds.centroids.cpu().numpy(), ids=ids, metric=P.IVF_IP,
                               compute_stream=streams[0], copy_stream=streams[1])
    index.ivf_set_batch_mode(2)
    q = wide.astype(np.float32)
    for lo in range(0, n, nq):
        hi = min(lo + nq, n)
        if hi - lo < 2:                               # a single query is never list-major
            break
        gi, gd = index.ivf_search(q[lo:hi], nlist, 1)
        assert np.array_equal(gi[:, 0], ids[lo:hi]), f"rows {np.flatnonzero(gi[:, 0] != ids[lo:hi])[:8] + lo}"
    index.close()


@pytest.mark.parametrize("dtype,d,metric", [("f16", 1920, "ip"), ("bf16", 1920, "ip"), ("f16", 768, "ip"), ("bf16", 1024, "ip"),
                                            ("f32", 768, "ip"), ("f32", 1920, "ip"), ("f32", 1024, "l2"), ("f16", 1920, "l2"),
                                            ("bf16", 768, "l2")])
def test_filter_scores_stay_within_the_assumed_bound(streams, dtype, d, metric):
    """The list-major scan prunes with MFMA scores and a bound eps of their error (query rounded to
    the storage type, fp32 accumulation inside the matrix cores; for squared L2 also the rounded
    norms).  The scores of every row of a cluster are read back and compared with fp64 values from
    the unrounded query, for sign patterns that make the rounding add up: all-positive operands,
    alternating signs on both sides (every product positive), and random signs.  d = 1920 is the
    longest row this path takes."""
    _check_filter_scores(streams, dtype, d, metric, 12)


# rows that are not whole blocks of 64 elements, and not whole 16-byte chunks; fp32: up to 8 queries go to the vector
# units, in walks of 1, 2, 4 and 8; 16 bytes are the narrowest rows, 1920 elements the longest
@pytest.mark.parametrize("dtype,d,metric,nq", [
    ("f32", 768, "ip", 1), ("f32", 768, "l2", 2), ("f32", 1920, "ip", 3), ("f32", 128, "l2", 8), ("f32", 4, "ip", 12), ("f32", 5, "l2", 12),
    ("f32", 31, "ip", 1), ("f32", 33, "l2", 2), ("f32", 100, "ip", 4), ("f32", 100, "l2", 12), ("f32", 255, "ip", 7), ("f32", 415, "l2", 12),
    ("f32", 1001, "ip", 5), ("f32", 1001, "l2", 17), ("f32", 1917, "ip", 8), ("f32", 1919, "l2", 32), ("f16", 8, "ip", 12), ("f16", 9, "l2", 12),
    ("f16", 63, "ip", 12), ("f16", 65, "l2", 1), ("f16", 300, "ip", 5), ("f16", 511, "l2", 12), ("f16", 1003, "ip", 32), ("f16", 1919, "l2", 12),
    ("bf16", 10, "l2", 12), ("bf16", 71, "ip", 12), ("bf16", 250, "l2", 9), ("bf16", 513, "ip", 12), ("bf16", 760, "l2", 12), ("bf16", 1917, "ip", 12),
])
def test_filter_scores_of_any_width_stay_within_the_assumed_bound(streams, dtype, d, metric, nq):
    _check_filter_scores(streams, dtype, d, metric, nq)


def _check_filter_scores(streams, dtype, d, metric, nq):
    rng = np.random.default_rng(21)
    n = 3000
    mag = np.abs(rng.standard_normal((n, d))) + 0.05
    signs_alt = np.where(np.arange(d) % 2 == 0, 1.0, -1.0)
    rows = np.concatenate([mag[:1000], mag[1000:2000] * signs_alt, mag[2000:] * rng.choice([-1.0, 1.0], (1000, d))])
    rows /= np.linalg.norm(rows, axis=1, keepdims=True)
    tdt = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}[dtype]
    t = torch.from_numpy(rows.astype(np.float32)).to(tdt).cuda()
    off = np.array([0, n], dtype=np.int64)
    cent = np.ones((1, d), dtype=np.float32)
    index = P.ivf_adopt_layout(t, dtype, off, cent, metric=P.IVF_IP if metric == "ip" else P.IVF_L2,
                               compute_stream=streams[0], copy_stream=streams[1])
    q = np.abs(rng.standard_normal((nq, d))) + 0.05
    third = nq // 3                                  # (fewer than three queries: random signs only)
    q[third:2 * third] *= signs_alt
    q[2 * third:] *= rng.choice([-1.0, 1.0], (nq - 2 * third, d))
    q = (q / np.linalg.norm(q, axis=1, keepdims=True)).astype(np.float32)
    approx, eps = index.ivf_batched_scores(q, 0, n)
    y = t.to(torch.float64).cpu().numpy()
    q64 = q.astype(np.float64)
    if metric == "ip":
        exact = q64 @ y.T
    else:
        exact = -((q64[:, None, :] - y[None, :, :]) ** 2).sum(axis=2)
    err = np.abs(approx.astype(np.float64) - exact).max(axis=1)
    print(f"{dtype} {metric} d {d}: largest |filter score - exact| / eps per query: {np.round(err / eps, 3)}")
    assert np.all(eps > 0) and np.all(err <= eps), (err, eps)
    # the bound is not vacuous: it is within two orders of magnitude of the largest error seen
    # (fp32 rows: within three, the accumulation order inside the matrix cores is not known)
    if nq == 12 and d % 64 == 0:
        assert (err / eps).max() > (0.001 if dtype == "f32" else 0.01)
    index.close()


@pytest.mark.parametrize("nq", [2, 3, 4, 5, 8, 9, 16, 17, 33])
@pytest.mark.parametrize("dtype,d,metric", [("f32", 64, "ip"), ("f32", 256, "l2"), ("f32", 320, "ip"), ("f32", 832, "l2"),
                                            ("f16", 512, "ip"), ("bf16", 576, "l2")])
def test_groups_of_every_size(streams, dtype, d, nq, metric):
    """The scan of fp32 rows walks groups of 1, 2, 4, 8 and more queries in code of their own, and the
    queries of narrow rows (up to 1 KB) stay in LDS for the whole scan: clusters that all nq queries,
    or only some of them, select, in lists that end inside a tile."""
    nlist, n, k, nprobe = 7, 3700, 9, 3
    rng = np.random.default_rng(nq * 100 + d)
    cent = rng.standard_normal((nlist, d)).astype(np.float32)
    off = np.array([0, 1, 258, 514, 900, 2000, 2000, n], dtype=np.int64)
    rows = (np.repeat(cent, np.diff(off), 0) + 0.5 * rng.standard_normal((n, d))).astype(np.float32)
    q = (cent[[3] * (nq - nq // 3) + [6] * (nq // 3)] + 0.3 * rng.standard_normal((nq, d))).astype(np.float32)
    dev = torch.from_numpy(rows).to({"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}[dtype]).cuda()
    index = P.ivf_adopt_layout(dev, dtype, off, cent, metric=P.IVF_IP if metric == "ip" else P.IVF_L2,
                               compute_stream=streams[0], copy_stream=streams[1])
    index.ivf_set_batch_mode(2)
    for m in (nprobe, nlist):
        gi, gd = index.ivf_search(q, m, k)
        index.ivf_set_batch_mode(1)
        pi, pd = index.ivf_search(q, m, k)
        index.ivf_set_batch_mode(2)
        assert np.array_equal(gi, pi) and np.array_equal(gd, pd)
    index.close()
