"""Selection of up to 64 clusters: as a kernel of its own and inside the scan of a search, at the edges of its sizes and
with scores that its cut does not separate."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2502_20969_amd as P

pytestmark = pytest.mark.gpu


def _centroids(kind, nlist, d, rng):
    c = (0.01 * rng.standard_normal((nlist, d))).astype(np.float32)
    i = np.arange(nlist)
    if kind == "random":
        return rng.standard_normal((nlist, d)).astype(np.float32)
    if kind == "rising":
        c[:, 0] = 1 + i * 1e-3
    elif kind == "one_group":                            # the best ones are all of the same group
        c[:, 0] = np.where(i % 128 == 5, 2 + i * 1e-3, i * 1e-5)
    elif kind == "few_values":
        c[:] = 0
        c[:, 0] = i % 3
    elif kind == "last_bits":                            # scores that differ in their low words only
        c[:] = 0
        c[:, 0] = 1
        c[:, 1] = rng.permutation(nlist) * np.float32(2.0 ** -35)
    else:                                                # all the same
        c[:] = 0.25
    return c


@pytest.mark.parametrize("metric", ["ip", "l2"])
@pytest.mark.parametrize("kind", ["random", "rising", "one_group", "few_values", "last_bits", "equal"])
@pytest.mark.parametrize("nlist", [1, 63, 64, 130, 1024, 1025, 4096])
def test_clusters_and_results(nlist, kind, metric):
    rng = np.random.default_rng(nlist + len(kind))
    d, per, k = 8, 3, 7
    pm, om = (P.IVF_IP, O.IP) if metric == "ip" else (P.IVF_L2, O.L2)
    cent = _centroids(kind, nlist, d, rng)
    n = nlist * per
    rows = rng.standard_normal((n, d)).astype(np.float32)
    off = np.arange(0, n + 1, per).astype(np.int64)
    index = P.ivf_adopt_layout(torch.from_numpy(rows).cuda(), "f32", off, cent, metric=pm,
                               compute_stream=torch.cuda.Stream(), copy_stream=torch.cuda.Stream())
    q = np.zeros((2, d), np.float32)
    q[:, 0] = 1.0
    q[:, 1] = 1.0
    q[1] = 0 if kind == "equal" else rng.standard_normal(d)
    gid = np.arange(n, dtype=np.int64)
    for nprobe in sorted({1, min(nlist, 32), min(nlist, 33), min(nlist, 64)}):
        want = [list(O.probe(cent, x, nprobe, om)) for x in q]
        pr = index.ivf_probe(q, nprobe)
        for b in range(2):
            assert list(pr[b]) == want[b], (nprobe, b)
            ids, dists = index.ivf_search(q[b], nprobe, k)                        # the scan selects (up to 1024 clusters)
            other, again, _ = index.ivf_search(q[b], nprobe, k, with_stats=True)   # a kernel of its own does
            oi, _ = O.search(rows, O.F32, off, gid, cent, q[b], nprobe, k, om)
            assert list(ids[0]) == list(oi) == list(other[0]), (nprobe, b)
            np.testing.assert_array_equal(dists, again)
    index.close()


@pytest.mark.parametrize("nlist", [64, 1024, 1025])
def test_profile_times_the_kernels_that_a_search_launches(nlist):
    """With up to 1024 clusters the scan of a single query selects, and the time of its selection is the scan's."""
    rng = np.random.default_rng(nlist)
    d, per, k, nprobe = 32, 20, 5, 16
    cent = rng.standard_normal((nlist, d)).astype(np.float32)
    rows = rng.standard_normal((nlist * per, d)).astype(np.float32)
    off = np.arange(0, nlist * per + 1, per).astype(np.int64)
    index = P.ivf_adopt_layout(torch.from_numpy(rows).cuda(), "f32", off, cent, metric=P.IVF_IP, compute_stream=torch.cuda.Stream(),
                               copy_stream=torch.cuda.Stream())
    q = torch.from_numpy(rng.standard_normal((1, d)).astype(np.float32)).cuda()
    ids, dists = torch.empty(1, k, dtype=torch.int64, device="cuda"), torch.empty(1, k, device="cuda")
    torch.cuda.synchronize()
    index.ivf_profile_enable(True)
    index.ivf_profile_reset()
    for _ in range(3):
        index.ivf_search_device(q, nprobe, k, ids, dists)
    p = index.ivf_profile_read()
    index.ivf_profile_enable(False)
    assert p.calls == 3 and p.scan_rows == 3 * nprobe * per
    assert (p.ms_select > 0) == (nlist > 1024)
    assert min(p.ms_coarse, p.ms_scan, p.ms_merge) > 0
    oi, _ = O.search(rows, O.F32, off, np.arange(nlist * per, dtype=np.int64), cent, q[0].cpu().numpy(), nprobe, k, O.IP)
    assert list(ids[0].cpu().numpy()) == list(oi)
    index.close()
