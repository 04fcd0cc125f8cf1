"""The merge of up to 56 results at the sizes of its pool: candidates that are all re-scored (up to 32), ranked by ballots
(up to 64), by counting (up to 384) or in sorted runs (more), cut again (from 512 on) and left to the radix select (more than
4096 that no cut thins out)."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2502_20969_amd as P
from parity import check_topk, stored

pytestmark = pytest.mark.gpu


def _rows(kind, n, d, q, rng):
    """Rows whose inner product with q is: unrelated to their place; falling along the rows, so that the best of them
    share few scan wavefronts; one of 40 values; the same for 6000 of them; the same for all."""
    rows = rng.standard_normal((n, d)).astype(np.float32)
    if kind == "random":
        return rows
    rows -= np.outer(rows @ q, q) / (q @ q)              # nothing along q but what is added here
    score = {"falling": np.linspace(1.0, 0.1, n), "steps": rng.integers(0, 40, n) / 40.0 + 0.5,
             "mass": np.where(np.arange(n) % 5 == 0, 0.75, np.linspace(0.7, 0.1, n)), "equal": np.full(n, 0.5)}[kind]
    if kind in ("steps", "mass", "equal"):               # rows of one score are the same row
        rows[:] = 0
    return (rows + np.outer(score, q / (q @ q))).astype(np.float32)


@pytest.mark.parametrize("place", ["device", "host"])
@pytest.mark.parametrize("kind", ["random", "falling", "steps", "mass", "equal"])
@pytest.mark.parametrize("dtype,d", [("f32", 32), ("f16", 30)])
def test_pools_of_every_size(place, kind, dtype, d):
    n, nlist = 30000, 16
    rng = np.random.default_rng(d + len(kind))
    q = np.zeros(d, np.float32)
    q[3] = 1.0                                           # scores are one element of the row: the same for equal rows, whatever the sums
    rows, odt = stored(_rows(kind, n, d, q, rng), dtype)
    off = np.linspace(0, n, nlist + 1).astype(np.int64)
    cent = rng.standard_normal((nlist, d)).astype(np.float32)
    t = torch.from_numpy(rows.view(np.int16) if odt == O.BF16 else rows)
    compute, copy = torch.cuda.Stream(), torch.cuda.Stream()
    if place == "device":
        index = P.ivf_adopt_layout(t.cuda(), dtype, off, cent, metric=P.IVF_IP, compute_stream=compute, copy_stream=copy)
    else:
        index = P.ivf_adopt_layout(t.pin_memory(), dtype, off, cent, metric=P.IVF_IP, placement=P.IVF_PLACE_HOST,
                                   device_buffer_bytes=rows.nbytes // 2, compute_stream=compute, copy_stream=copy)
        index.ivf_prefetch(q[None], nlist, rows.nbytes // 2, P.IVF_PREFETCH_RESET)
    gid = np.arange(n, dtype=np.int64)
    for k in (1, 3, 10, 24, 40, 56):
        ids, dists = index.ivf_search(q[None], nlist, k)
        assert check_topk(ids[0], dists[0], rows, odt, off, gid, cent, q, nlist, k, O.IP) == 0, (k, place)
    index.close()


@pytest.mark.parametrize("depth", [1, 2])                # alone, and beside other searches
@pytest.mark.parametrize("copies", [21, 22, 53, 54, 373, 374, 501, 502, 1013, 1014, 2500, 4085, 4086])
def test_pools_that_no_cut_thins_out(copies, depth):
    """Eleven rows that differ and, behind them, copies of one row: the pool of k = 10 holds them all, and the result is proven
    without the exact pass."""
    n, nlist, d, best = 30000, 16, 32, 11
    rng = np.random.default_rng(copies)
    rows = rng.uniform(-1, 0, (n, d)).astype(np.float32)
    at = rng.permutation(n)[:best + copies]
    rows[at] = 1.0
    rows[at[:best]] += np.arange(best, 0, -1, dtype=np.float32)[:, None] / 16
    off = np.linspace(0, n, nlist + 1).astype(np.int64)
    cent = rng.standard_normal((nlist, d)).astype(np.float32)
    index = P.ivf_adopt_layout(torch.from_numpy(rows).cuda(), "f32", off, cent, metric=P.IVF_IP, compute_stream=torch.cuda.Stream(),
                               copy_stream=torch.cuda.Stream())
    index.ivf_set_pipeline_depth(depth)
    q = np.ones((1, d), np.float32)
    want = np.concatenate([at[:best], np.sort(at[best:])])       # equal scores come by number
    for k in (1, 10, 24, 32):
        ids, dists, st = index.ivf_search(q, nlist, k, with_stats=True)
        np.testing.assert_array_equal(ids[0], want[:k])
        np.testing.assert_array_equal(dists[0], rows[want[:k]].sum(1))
        assert k != 10 or st.n_exact_gpu == 0
    index.close()
