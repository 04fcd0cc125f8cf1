"""A search while the prefetched lists are still on their way: the host scans the missed clusters beside the fetch."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2502_20969_amd as P
from parity import check_topk

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nq,nprobe,cache", [(1, 20, False), (3, 40, True), (2, 96, True)])
def test_search_beside_a_fetch_equals_one_behind_it(nq, nprobe, cache):
    rng = np.random.default_rng(nq)
    n, d, nlist, k = 60000, 768, 96, 10
    rows = rng.standard_normal((n, d)).astype(np.float16)
    off = np.linspace(0, n, nlist + 1).astype(np.int64)
    cent = np.stack([rows[off[c]:off[c + 1]].astype(np.float32).mean(0) for c in range(nlist)])
    q = rng.standard_normal((nq, d)).astype(np.float32)
    results = []
    for wait in (False, True):
        index = P.ivf_adopt_layout(torch.from_numpy(rows).pin_memory(), "f16", off, cent, metric=P.IVF_IP, placement=P.IVF_PLACE_HOST,
                                   device_buffer_bytes=rows.nbytes, compute_stream=torch.cuda.Stream(), copy_stream=torch.cuda.Stream())
        if cache:
            index.ivf_cache_configure(1.0, 1.0, 2.0, 1.0)
        for turn in range(2):              # half of what the queries want; then more of it, beside what is there
            index.ivf_prefetch(q, nprobe, rows.nbytes // nlist * nprobe * nq // (2 if turn == 0 else 3), P.IVF_PREFETCH_RESET if turn == 0 else 0)
            if wait:
                torch.cuda.synchronize()
            ids, dists, st = index.ivf_search(q, nprobe, k, with_stats=True)
            results.append((wait, turn, ids, dists, (st.n_probed, st.n_overlap, st.n_miss, st.bytes_gpu, st.bytes_host, st.hit_rate)))
            if cache:
                index.ivf_cache_end_round()
                results.append((wait, turn, index.ivf_cache_hotness()))
        index.close()
    half = len(results) // 2
    for a, b in zip(results[:half], results[half:]):
        assert a[1] == b[1]
        for x, y in zip(a[2:], b[2:]):
            np.testing.assert_array_equal(x, y)
    gid = np.arange(n, dtype=np.int64)
    for b in range(nq):
        assert check_topk(results[0][2][b], results[0][3][b], rows, O.F16, off, gid, cent, q[b], nprobe, k, O.IP) == 0


@pytest.mark.parametrize("nq,cache", [(1, False), (4, True)])
def test_clusters_are_selected_while_the_fetch_waits(nq, cache):
    """Other work holds the copy stream up, so that the fetch cannot have ended when the search is called: the host knows the
    clusters long before the search is over, and the lists are found where the fetch has put them."""
    rng = np.random.default_rng(nq)
    n, d, nlist, nprobe, k = 60000, 256, 96, 40, 10
    rows = rng.standard_normal((n, d)).astype(np.float16)
    off = np.linspace(0, n, nlist + 1).astype(np.int64)
    cent = np.stack([rows[off[c]:off[c + 1]].astype(np.float32).mean(0) for c in range(nlist)])
    q = rng.standard_normal((nq, d)).astype(np.float32)
    copy = torch.cuda.Stream()
    index = P.ivf_adopt_layout(torch.from_numpy(rows).pin_memory(), "f16", off, cent, metric=P.IVF_IP, placement=P.IVF_PLACE_HOST,
                               device_buffer_bytes=rows.nbytes, compute_stream=torch.cuda.Stream(), copy_stream=copy)
    if cache:
        index.ivf_cache_configure(1.0, 1.0, 2.0, 1.0)
    a, b = torch.ones(4096, 4096, device="cuda"), torch.empty(4096, 4096, device="cuda")
    torch.mm(a, a, out=b)
    index.ivf_search(q, nprobe, k)                       # the host's threads are there
    torch.cuda.synchronize()
    gid = np.arange(n, dtype=np.int64)
    index.ivf_profile_enable(True)
    index.ivf_profile_reset()
    for turn in range(2):              # a part of what the queries want; then more of it, beside what is there
        with torch.cuda.stream(copy):
            for _ in range(60):                          # 130 GFLOP each
                torch.mm(a, a, out=b)
        index.ivf_prefetch(q, nprobe, rows.nbytes // nlist * nprobe * nq // (4 if turn == 0 else 6), P.IVF_PREFETCH_RESET if turn == 0 else 0)
        assert not copy.query()
        ids, dists, st = index.ivf_search(q, nprobe, k, with_stats=True)
        assert copy.query()
        assert st.ms_probe < 0.5 * st.ms_total, (st.ms_probe, st.ms_total)
        assert st.n_miss > 0 and st.n_overlap > 0
        for i in range(nq):
            assert check_topk(ids[i], dists[i], rows, O.F16, off, gid, cent, q[i], nprobe, k, O.IP) == 0
        if cache:
            index.ivf_cache_end_round()
            torch.cuda.synchronize()
    p = index.ivf_profile_read()
    assert p.calls == 2 and min(p.ms_coarse, p.ms_select, p.ms_scan, p.ms_merge) > 0
    index.close()
