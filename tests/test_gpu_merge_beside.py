"""Searches with others in flight: the merge then has half the wavefronts (up to 40 results; single queries and large batches), and its
rare ways give what a search by itself gives."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2502_20969_amd as P
from parity import check_topk, stored
from test_gpu_merge_pools import _rows

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["random", "falling", "steps", "mass", "equal"])
@pytest.mark.parametrize("dtype,d", [("f32", 32), ("f16", 30)])
def test_pools_of_every_size_beside_others(kind, dtype, d):
    n, nlist = 30000, 16
    rng = np.random.default_rng(d + len(kind))
    q = np.zeros(d, np.float32)
    q[3] = 1.0                                           # scores are one element of the row: the same for equal rows, whatever the sums
    rows, odt = stored(_rows(kind, n, d, q, rng), dtype)
    off = np.linspace(0, n, nlist + 1).astype(np.int64)
    cent = rng.standard_normal((nlist, d)).astype(np.float32)
    index = P.ivf_adopt_layout(torch.from_numpy(rows).cuda(), dtype, off, cent, metric=P.IVF_IP, compute_stream=torch.cuda.Stream(),
                               copy_stream=torch.cuda.Stream())
    index.ivf_set_pipeline_depth(3)
    gid = np.arange(n, dtype=np.int64)
    q_dev = torch.from_numpy(q).cuda()[None]
    for k in (1, 3, 10, 24, 40, 41):
        ids, dists = index.ivf_search(q[None], nlist, k)
        assert check_topk(ids[0], dists[0], rows, odt, off, gid, cent, q, nlist, k, O.IP) == 0, k
        out = [(torch.empty(1, k, dtype=torch.int64, device="cuda"), torch.empty(1, k, device="cuda")) for _ in range(6)]
        torch.cuda.synchronize()
        for i, x in out:
            index.ivf_search_device(q_dev, nlist, k, i, x)
        index.ivf_synchronize()
        for i, x in out:
            np.testing.assert_array_equal(i.cpu().numpy(), ids)
            np.testing.assert_array_equal(x.cpu().numpy(), dists)
    index.close()


def test_batch_of_large_scans_beside_others():
    """Eight queries over 320 MB in all, one by one (mode 1): their merges have half the wavefronts too."""
    n, nlist, d, k = 80000, 8, 128, 20
    gen = torch.Generator(device="cuda").manual_seed(5)
    rows = torch.randn(n, d, generator=gen, device="cuda")
    rows[::40] = rows[7]                                 # 2000 copies of one row, the best of query 0
    q = torch.randn(8, d, generator=gen, device="cuda")
    q[0] = rows[7]
    off = np.linspace(0, n, nlist + 1).astype(np.int64)
    index = P.ivf_adopt_layout(rows, "f32", off, np.random.default_rng(1).standard_normal((nlist, d)).astype(np.float32), metric=P.IVF_IP,
                               compute_stream=torch.cuda.Stream(), copy_stream=torch.cuda.Stream())
    index.ivf_set_batch_mode(1)
    results = []
    for depth in (1, 4):
        index.ivf_set_pipeline_depth(depth)
        out = [(torch.empty(8, k, dtype=torch.int64, device="cuda"), torch.empty(8, k, device="cuda")) for _ in range(depth)]
        torch.cuda.synchronize()
        for i, x in out:
            index.ivf_search_device(q, nlist, k, i, x)
        index.ivf_synchronize()
        results += [(i.cpu(), x.cpu()) for i, x in out]
    index.close()
    for i, x in results[1:]:
        assert torch.equal(i, results[0][0]) and torch.equal(x, results[0][1])
    s = q.double().cpu() @ rows.double().cpu().T
    s[:, ::40] = s[:, 7:8]                               # the same score, whatever the order of the sums
    assert torch.equal(results[0][0], (-s).argsort(dim=1, stable=True)[:, :k])


@pytest.mark.parametrize("k,nprobe", [(10, 28), (10, 64), (56, 8), (56, 28)])
def test_selection_beside_others(k, nprobe):
    """Single queries over 22 to 178 MB of lists: with others in flight the scan selects the clusters up to 112 MB (56 for more than 40
    results), and a kernel of its own above."""
    nlist, per, d = 64, 1450, 480
    gen = torch.Generator(device="cuda").manual_seed(nprobe)
    rows = torch.randn(nlist * per, d, generator=gen, device="cuda")
    cent = torch.randn(nlist, d, generator=gen, device="cuda")
    q = torch.randn(9, d, generator=gen, device="cuda")
    index = P.ivf_adopt_layout(rows, "f32", np.arange(nlist + 1) * per, cent.cpu().numpy(), metric=P.IVF_IP, compute_stream=torch.cuda.Stream(),
                               copy_stream=torch.cuda.Stream())
    results = []
    for depth in (1, 3):
        index.ivf_set_pipeline_depth(depth)
        ids, dists = torch.empty(9, k, dtype=torch.int64, device="cuda"), torch.empty(9, k, device="cuda")
        torch.cuda.synchronize()
        for b in range(9):
            index.ivf_search_device(q[b:b + 1], nprobe, k, ids[b:b + 1], dists[b:b + 1])
        index.ivf_synchronize()
        results.append((ids.cpu(), dists.cpu()))
    index.close()
    assert torch.equal(results[0][0], results[1][0]) and torch.equal(results[0][1], results[1][1])
    picked = (q.double() @ cent.double().T).topk(nprobe, dim=1).indices
    for b in range(9):
        at = (picked[b][:, None] * per + torch.arange(per, device="cuda")).flatten()
        best = (rows[at].double() @ q[b].double()).topk(k)
        assert torch.equal(results[0][0][b], at[best.indices].cpu())
