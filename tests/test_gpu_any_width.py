"""List-major batches over rows of any width (automatic mode, rows that are not whole blocks of 64
elements): bit-equal to the query-by-query path, complete in stream order."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2502_20969_amd as P
from parity import check_topk, stored

pytestmark = pytest.mark.gpu
TORCH = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
METRIC = {"ip": (P.IVF_IP, O.IP), "l2": (P.IVF_L2, O.L2)}


def _problem(seed, dtype, n, d, nlist, nq, spread, scale=1.0):
    """Rows around nlist centres in uneven lists (one of them empty), queries around `spread` of the centres."""
    rng = np.random.default_rng(seed)
    cent = rng.standard_normal((nlist, d)).astype(np.float32)
    w = rng.uniform(0.3, 1.7, nlist)
    w[nlist // 2] = 0.0
    sizes = np.floor(w / w.sum() * n).astype(np.int64)
    sizes[0] += n - sizes.sum()
    off = np.concatenate([[0], np.cumsum(sizes)])
    rows = np.repeat(cent, sizes, 0) + 0.5 * rng.standard_normal((n, d)).astype(np.float32)
    q = cent[rng.integers(0, spread, nq)] + 0.3 * rng.standard_normal((nq, d)).astype(np.float32)
    dev = torch.from_numpy((rows * scale).astype(np.float32)).to(TORCH[dtype]).cuda()
    return dev, off, (cent * scale).astype(np.float32), (q * scale).astype(np.float32)


def _adopt(rows, dtype, off, cent, metric, ids=None):
    return P.ivf_adopt_layout(rows, dtype, off, cent, ids=ids, metric=METRIC[metric][0],
                              compute_stream=torch.cuda.Stream(), copy_stream=torch.cuda.Stream())


def _rows_scanned(index, q, nprobe, k):
    """Results of a host call, and the rows its scan read (list-major: each selected cluster once)."""
    index.ivf_profile_enable(True)
    index.ivf_profile_reset()
    out = index.ivf_search(q, nprobe, k)
    read = index.ivf_profile_read().scan_rows
    index.ivf_profile_enable(False)
    return out, read


# widths around the pieces (32 fp32, 64 two-byte elements), the 16-byte chunks, the two stages in flight and the
# width up to which the queries of the whole batch stay in LDS; groups of 1 to more than 32 queries per cluster
@pytest.mark.parametrize("dtype,d,nq,spread,metric,k", [
    ("f32", 4, 40, 7, "ip", 5), ("f32", 5, 48, 2, "l2", 3), ("f32", 31, 40, 7, "ip", 10), ("f32", 33, 43, 1, "l2", 7),
    ("f32", 95, 40, 3, "ip", 1), ("f32", 97, 64, 7, "ip", 33), ("f32", 100, 40, 7, "l2", 20), ("f32", 200, 70, 1, "ip", 100),
    ("f32", 255, 40, 4, "ip", 8), ("f32", 257, 40, 7, "l2", 8), ("f32", 415, 41, 2, "ip", 10), ("f32", 1001, 40, 7, "ip", 4),
    ("f16", 8, 40, 7, "ip", 5), ("f16", 9, 50, 1, "l2", 3), ("f16", 63, 40, 7, "ip", 10), ("f16", 65, 75, 2, "l2", 12),
    ("f16", 129, 40, 1, "ip", 112), ("f16", 300, 48, 7, "l2", 10), ("f16", 511, 40, 3, "ip", 9), ("f16", 1003, 40, 7, "ip", 2),
    ("bf16", 10, 64, 7, "ip", 6), ("bf16", 71, 40, 1, "ip", 56), ("bf16", 104, 44, 7, "l2", 10), ("bf16", 250, 90, 2, "ip", 30),
    ("bf16", 513, 40, 7, "l2", 5), ("bf16", 760, 40, 5, "ip", 10),
])
def test_list_major_of_any_width_equals_query_by_query(dtype, d, nq, spread, metric, k):
    n, nlist, nprobe = 24000, 8, 5
    rows, off, cent, q = _problem(d * 7 + nq, dtype, n, d, nlist, nq, spread)
    ids = np.random.default_rng(d).permutation(n).astype(np.int64) * 3 + 1
    index = _adopt(rows, dtype, off, cent, metric, ids)
    (gi, gd), read = _rows_scanned(index, q, nprobe, k)
    assert 0 < read <= n                                     # list-major: no cluster more than once
    q_dev = torch.from_numpy(q).cuda()
    di, dd = torch.empty(nq, k, dtype=torch.int64, device="cuda"), torch.empty(nq, k, device="cuda")
    torch.cuda.synchronize()
    index.ivf_search_device(q_dev, nprobe, k, di, dd)
    torch.cuda.synchronize()                                 # stream order is enough: no ivf_synchronize
    index.ivf_set_batch_mode(1)
    (pi, pd), read = _rows_scanned(index, q, nprobe, k)
    assert read > n
    assert np.array_equal(gi, pi) and np.array_equal(gd, pd)
    assert np.array_equal(di.cpu().numpy(), pi) and np.array_equal(dd.cpu().numpy(), pd)
    lists = rows.cpu().numpy() if dtype != "bf16" else rows.cpu().view(torch.int16).numpy().view(np.uint16)
    odt = {"f32": O.F32, "f16": O.F16, "bf16": O.BF16}[dtype]
    for b in (0, nq - 1):
        assert check_topk(gi[b], gd[b], lists, odt, off, ids, cent, q[b], nprobe, k, METRIC[metric][1]) == 0
    # the second mode is still refused for such rows
    with pytest.raises(P.IvfError):
        index.ivf_set_batch_mode(2)
    index.close()


@pytest.mark.parametrize("dtype,d", [("f32", 100), ("f32", 128), ("f16", 100), ("f16", 128), ("bf16", 72), ("bf16", 128)])
@pytest.mark.parametrize("kind", ["inf", "nan", "beyond", "tiny", "zero"])
@pytest.mark.parametrize("metric", ["ip", "l2"])
def test_values_without_an_error_bound(dtype, d, kind, metric):
    """Infinities, no numbers, queries beyond the storage type, squares that underflow: the filter's bound
    says nothing there, the results are those of the query-by-query path all the same."""
    nq, nprobe, k, n = 64, 5, 10, 24000
    scale = {"tiny": {"f16": 1e-6, "bf16": 1e-19, "f32": 1e-19}[dtype]}.get(kind, 1.0)
    rows, off, cent, q = _problem(3, dtype, n, d, 8, nq, 7, scale)
    if kind == "inf":
        rows[5, d - 1] = float("inf"); rows[17, 0] = float("-inf"); rows[n - 1, d // 2] = float("inf")
    elif kind == "nan":
        rows[6, d - 1] = float("nan"); rows[7, 0] = float("nan"); rows[n - 1, d - 1] = float("nan")
    elif kind == "beyond":
        q[3] *= 1e6; q[5] *= 1e19
    elif kind == "zero":
        q[0] = 0.0; q[9] = 0.0; rows[::3] = 0
    index = _adopt(rows, dtype, off, cent, metric)
    gi, gd = index.ivf_search(q, nprobe, k)
    q_dev = torch.from_numpy(q).cuda()
    di, dd = torch.empty(nq, k, dtype=torch.int64, device="cuda"), torch.empty(nq, k, device="cuda")
    torch.cuda.synchronize()
    index.ivf_search_device(q_dev, nprobe, k, di, dd)
    if d % 64 == 0:
        index.ivf_synchronize()
    torch.cuda.synchronize()
    index.ivf_set_batch_mode(1)
    pi, pd = index.ivf_search(q, nprobe, k)
    assert np.array_equal(gi, pi) and np.array_equal(gd, pd, equal_nan=True)
    assert np.array_equal(di.cpu().numpy(), pi) and np.array_equal(dd.cpu().numpy(), pd, equal_nan=True)
    index.close()


@pytest.mark.parametrize("depth", [1, 3])
def test_overflowing_queries_are_finished_on_the_stream(depth):
    """More identical rows than a candidate list holds: the exact pass behind the merge answers, on the
    same stream (depth 1: without ivf_synchronize), for every batch in flight."""
    n, d, nlist, nq, nprobe, k = 120000, 72, 4, 12, 3, 7
    rng = np.random.default_rng(5)
    rows_np = rng.standard_normal((n, d)).astype(np.float16)
    rows_np[:90000] = np.float16(0.125)
    off = np.arange(0, n + 1, n // nlist, dtype=np.int64)
    cent = rng.standard_normal((nlist, d)).astype(np.float32)
    cent[0], cent[1], cent[2] = 1.0, 0.9, 0.8
    ids = rng.permutation(n).astype(np.int64)
    index = _adopt(torch.from_numpy(rows_np).cuda(), "f16", off, cent, "ip", ids)
    index.ivf_set_pipeline_depth(depth)
    qs = [torch.from_numpy(np.abs(rng.standard_normal((nq, d))).astype(np.float32)).cuda() for _ in range(4)]
    for q in qs[1::2]:
        q[::2] *= -1.0                                       # these select the list of different rows first
    outs = [(torch.empty(nq, k, dtype=torch.int64, device="cuda"), torch.empty(nq, k, device="cuda")) for _ in qs]
    torch.cuda.synchronize()
    for q, (i, s) in zip(qs, outs):
        index.ivf_search_device(q, nprobe, k, i, s)
    if depth > 1:
        index.ivf_synchronize()
    torch.cuda.synchronize()
    index.ivf_set_pipeline_depth(1)
    index.ivf_set_batch_mode(1)
    for q, (i, s) in zip(qs, outs):
        pi, pd = index.ivf_search(q.cpu().numpy(), nprobe, k)
        assert np.array_equal(i.cpu().numpy(), pi) and np.array_equal(s.cpu().numpy(), pd)
    index.close()


def test_reserved_batch_can_be_captured():
    """After ivf_reserve a batch allocates nothing and can be captured; every replay gives the eager result."""
    n, d, nq, nprobe, k = 24000, 100, 48, 5, 10
    rows, off, cent, q = _problem(8, "f32", n, d, 8, nq, 7)
    stream = torch.cuda.Stream()
    index = P.ivf_adopt_layout(rows, "f32", off, cent, metric=P.IVF_IP, compute_stream=stream, copy_stream=torch.cuda.Stream())
    index.ivf_reserve(nq, nprobe, k)
    want_i, want_d = index.ivf_search(q, nprobe, k)
    q_dev = torch.from_numpy(q).cuda()
    di, dd = torch.empty(nq, k, dtype=torch.int64, device="cuda"), torch.empty(nq, k, device="cuda")
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        index.ivf_search_device(q_dev, nprobe, k, di, dd)
    for _ in range(3):
        di.zero_(); dd.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(di.cpu().numpy(), want_i) and np.array_equal(dd.cpu().numpy(), want_d)
        index.ivf_search(q, nprobe, k)                       # eager work between the replays
    index.close()


@pytest.mark.parametrize("dtype,d,nq,nprobe,k", [("f32", 64, 4, 3, 5), ("f16", 256, 16, 6, 20), ("bf16", 128, 60, 2, 3)])
def test_small_batches_of_automatic_mode(dtype, d, nq, nprobe, k):
    """Whole blocks of elements, but too few rows for a list-major scan to pay: query by query, with the
    results and the reported bytes (each cluster once) of the list-major mode."""
    rows, off, cent, q = _problem(d + nq, dtype, 6000, d, 30, nq, 5)
    index = _adopt(rows, dtype, off, cent, "ip")
    (gi, gd), read = _rows_scanned(index, q, nprobe, k)
    _, _, st = index.ivf_search(q, nprobe, k, with_stats=True)
    q_dev = torch.from_numpy(q).cuda()
    di, dd = torch.empty(nq, k, dtype=torch.int64, device="cuda"), torch.empty(nq, k, device="cuda")
    torch.cuda.synchronize()
    index.ivf_search_device(q_dev, nprobe, k, di, dd)
    index.ivf_synchronize()
    index.ivf_set_batch_mode(2)
    (mi, md), once = _rows_scanned(index, q, nprobe, k)
    _, _, mst = index.ivf_search(q, nprobe, k, with_stats=True)
    assert read > once
    assert np.array_equal(gi, mi) and np.array_equal(gd, md)
    assert np.array_equal(di.cpu().numpy(), mi) and np.array_equal(dd.cpu().numpy(), md)
    assert st.bytes_gpu == mst.bytes_gpu and st.n_probed == mst.n_probed and st.hit_rate == mst.hit_rate
    index.close()


@pytest.mark.parametrize("dtype,d,n,nlist,nq,nprobe,k,list_major", [
    ("f16", 20, 200000, 2000, 4096, 2, 5, False),         # a list-major call pays for its queries: 0.57 against 0.26 ms
    ("f32", 109, 24600, 249, 2772, 3, 12, False),         # 0.35 / 0.18
    ("f32", 100, 100000, 1000, 64, 200, 20, True),
    ("f16", 300, 60000, 70, 512, 20, 10, True),
    ("bf16", 64, 100000, 100, 10, 6, 50, True),           # the query-by-query merge overflows: 97 us against 64
    ("f32", 64, 30000, 80, 13, 3, 45, True),
    ("bf16", 64, 100000, 100, 10, 6, 10, False),
    ("bf16", 256, 30000, 100, 10, 6, 50, False),
])
def test_the_faster_way_is_taken(dtype, d, n, nlist, nq, nprobe, k, list_major):
    rows, off, cent, q = _problem(nq, dtype, n, d, nlist, nq, nlist)
    index = _adopt(rows, dtype, off, cent, "ip")
    (gi, gd), read = _rows_scanned(index, q, nprobe, k)
    index.ivf_set_batch_mode(1)
    (pi, pd), each = _rows_scanned(index, q, nprobe, k)
    assert np.array_equal(gi, pi) and np.array_equal(gd, pd)
    assert read < each if list_major else read == each
    index.close()


def test_a_reserved_size_covers_every_smaller_batch():
    """A batch of the reserved size is searched query by query, smaller ones list-major: their workspace is there."""
    n, d, nlist, nprobe, k = 120000, 40, 300, 30, 5
    rows, off, cent, q = _problem(2, "f16", n, d, nlist, 3000, nlist)
    index = _adopt(rows, "f16", off, cent, "ip")
    index.ivf_reserve(3000, nprobe, k)
    torch.cuda.synchronize()
    free, routes = torch.cuda.mem_get_info()[0], set()
    for nq in (3000, 1000, 300, 150, 60, 4):
        (gi, gd), read = _rows_scanned(index, q[:nq], nprobe, k)
        routes.add(read <= n)
        index.ivf_set_batch_mode(1)
        pi, pd = index.ivf_search(q[:nq], nprobe, k)
        index.ivf_set_batch_mode(0)
        assert np.array_equal(gi, pi) and np.array_equal(gd, pd)
    assert routes == {True, False}
    assert torch.cuda.mem_get_info()[0] == free
    index.close()


NO_LIMIT = (1 << 64) - 1


def _device_search(index, q, nprobe, k):
    """Complete in stream order, without ivf_synchronize."""
    q_dev = torch.from_numpy(q).cuda()
    ids, dists = torch.empty(q.shape[0], k, dtype=torch.int64, device="cuda"), torch.empty(q.shape[0], k, device="cuda")
    torch.cuda.synchronize()
    index.ivf_search_device(q_dev, nprobe, k, ids, dists)
    torch.cuda.synchronize()
    return ids.cpu().numpy(), dists.cpu().numpy()


@pytest.mark.parametrize("dtype,d", [("f32", 200), ("f32", 201), ("f16", 301), ("bf16", 75)])       # slices start at any element
def test_batches_that_do_not_fit_their_memory(dtype, d):
    """What the list-major workspace did get is given back when the rest of it is refused; the batch is searched
    in slices, or query by query when nothing fits, and smaller batches stay list-major."""
    n, nlist, nq, nprobe, k = 24000, 8, 300, 5, 10
    rows, off, cent, q = _problem(4, dtype, n, d, nlist, nq, 7)
    index = _adopt(rows, dtype, off, cent, "ip")
    index.ivf_set_batch_mode(1)
    (wi, wd), each = _rows_scanned(index, q, nprobe, k)            # sizes the rest of the workspace
    index.ivf_set_batch_mode(0)
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    for limit, low, high in ((0, each, each), (1 << 20, each, each), (44 << 20, n + 1, each // 4), (NO_LIMIT, 1, n),
                             (9 << 20, each, each)):        # room for nine queries, which share too little
        index.ivf_limit_batch_memory(limit)
        for _ in range(2):                                          # a refusal is not asked for again
            (gi, gd), read = _rows_scanned(index, q, nprobe, k)
            assert low <= read <= high, (limit, read)
            assert np.array_equal(gi, wi) and np.array_equal(gd, wd)
        di, dd = _device_search(index, q, nprobe, k)
        assert np.array_equal(di, wi) and np.array_equal(dd, wd)
        held = free - torch.cuda.mem_get_info()[0]
        assert held <= min(limit, 300 * (600 << 10)) + (16 << 20), (limit, held)
        if limit >= 44 << 20:                                       # a batch of which the slices hold all
            (si, sd), read = _rows_scanned(index, q[:40], nprobe, k)
            assert 0 < read <= n and np.array_equal(si, wi[:40]) and np.array_equal(sd, wd[:40])
    index.close()


def test_slices_finish_their_own_queries():
    """Batches searched in slices: every slice's tied queries get the exact pass before the next slice takes the
    workspace, on the stream, and are counted."""
    n, d, nlist, nq, nprobe, k = 24000, 72, 4, 90, 3, 7
    rng = np.random.default_rng(6)
    rows_np = rng.standard_normal((n, d)).astype(np.float16)
    rows_np[:18000] = np.float16(0.125)
    off = np.arange(0, n + 1, n // nlist, dtype=np.int64)
    cent = rng.standard_normal((nlist, d)).astype(np.float32)
    cent[0], cent[1], cent[2] = 1.0, 0.9, 0.8
    index = _adopt(torch.from_numpy(rows_np).cuda(), "f16", off, cent, "ip", rng.permutation(n).astype(np.int64))
    q = np.abs(rng.standard_normal((nq, d))).astype(np.float32)
    q[::3] *= -1.0                                                  # these select the list of different rows first
    (oi, od, ost), (ti, td) = index.ivf_search(q, nprobe, k, with_stats=True), _device_search(index, q, nprobe, k)
    index.ivf_limit_batch_memory(20 << 20)
    (gi, gd, st), (di, dd) = index.ivf_search(q, nprobe, k, with_stats=True), _device_search(index, q, nprobe, k)
    index.ivf_set_batch_mode(1)
    pi, pd, pst = index.ivf_search(q, nprobe, k, with_stats=True)
    for i, s in ((oi, od), (ti, td), (gi, gd), (di, dd)):
        assert np.array_equal(i, pi) and np.array_equal(s, pd)
    assert st.n_exact_gpu == ost.n_exact_gpu >= nq // 2
    assert st.bytes_gpu == ost.bytes_gpu == pst.bytes_gpu and st.n_probed == pst.n_probed
    index.close()


def test_more_queries_than_a_slice_holds():
    n, d, nlist, nq, nprobe, k = 24000, 60, 8, 4103, 5, 3
    rows, off, cent, q = _problem(9, "f16", n, d, nlist, nq, 7)
    index = _adopt(rows, "f16", off, cent, "l2")
    (gi, gd), read = _rows_scanned(index, q, nprobe, k)
    assert 0 < read <= 2 * n
    index.ivf_set_batch_mode(1)
    pi, pd = index.ivf_search(q, nprobe, k)
    assert np.array_equal(gi, pi) and np.array_equal(gd, pd)
    index.close()
