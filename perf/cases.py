"""The searches that a user of this library runs, as cases that can be timed and compared.

A case is a dict of plain values; `op` says which entry points it goes through:

  search     one call with device-resident queries and outputs (`ivf_search_device`; a batch is
             followed by `ivf_synchronize`, which completes a list-major call), or, with
             entry = "host", one call with host buffers (`ivf_search`)
  stream     nq single queries submitted one after the other with `depth` searches in flight
             (`ivf_set_pipeline_depth`), completed by one `ivf_synchronize`
  lookahead  lists in pinned host memory: `ivf_prefetch` for the predicted queries, `ivf_search`
             for the final ones over the resident and the missed clusters; with cache = True two
             rounds of it, the second one on what the cluster cache kept, each closed by
             `ivf_cache_end_round`
  schedule   `ivf_schedule`: a global batch of queries grouped into micro-batches
"""
import math
import os

import numpy as np
import torch

import paper_2502_20969_amd as P

SIGMA = 0.3                      # spread of a list's rows around its centre, as in the synthetic datastores
TORCH = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
METRIC = {"ip": P.IVF_IP, "l2": P.IVF_L2}


def listed():
    return [
        # the smallest call: a 20,000-row datastore, one query; launches and latency are all there is
        dict(name="tiny_query", op="search", entry="device", dtype="f32", metric="ip", n=20000, d=128, nlist=64,
             skew=0.0, nprobe=8, k=10, nq=1, groups=1),
        # single-query retrieval over a million 768-d embeddings, one search at a time
        dict(name="single_query", op="search", entry="device", dtype="f32", metric="ip", n=1_000_000, d=768, nlist=1024,
             skew=0.0, nprobe=32, k=10, nq=1, groups=1),
        # the same datastore served at full rate: 16 searches in flight
        dict(name="query_stream", op="stream", dtype="f32", metric="ip", n=1_000_000, d=768, nlist=1024, skew=0.0,
             nprobe=32, k=10, nq=64, groups=64, depth=16),
        # a re-ranker's call: a hundred results from many clusters of a skewed fp16 datastore
        dict(name="single_k100_f16", op="search", entry="device", dtype="f16", metric="ip", n=4_000_000, d=768, nlist=4096,
             skew=1.1, nprobe=256, k=100, nq=1, groups=1),
        # word-vector-like data: a row of 600 bytes is no whole number of 16-byte chunks; host buffers, squared L2
        dict(name="single_d300_l2", op="search", entry="host", dtype="f16", metric="l2", n=600_000, d=300, nlist=700,
             skew=0.5, nprobe=48, k=10, nq=1, groups=1),
        # a micro-batch of the paper's set-up (fp32, Zipf lists, top 3), scaled to 12 GB
        dict(name="batch8_f32", op="search", entry="device", dtype="f32", metric="ip", n=4_000_000, d=768, nlist=2048,
             skew=1.1, nprobe=128, k=3, nq=8, groups=8),
        # 32 queries that share lists, fp16 rows, Zipf lists
        dict(name="batch32_f16", op="search", entry="device", dtype="f16", metric="ip", n=4_000_000, d=768, nlist=4096,
             skew=1.1, nprobe=128, k=10, nq=32, groups=24),
        # 32 queries in squared L2 over the million-row datastore, host buffers
        dict(name="batch32_l2", op="search", entry="host", dtype="f32", metric="l2", n=1_000_000, d=768, nlist=1024,
             skew=0.0, nprobe=32, k=10, nq=32, groups=24),
        # a batch over rows of a width that is not a multiple of 64
        dict(name="batch48_d100", op="search", entry="device", dtype="f32", metric="l2", n=1_000_000, d=100, nlist=1000,
             skew=0.5, nprobe=24, k=20, nq=48, groups=48),
        # the largest: 256 distinct queries, bf16 rows, a hundred results, Zipf lists down to a few rows
        dict(name="batch256_bf16", op="search", entry="device", dtype="bf16", metric="ip", n=6_000_000, d=1024, nlist=8192,
             skew=1.2, nprobe=512, k=100, nq=256, groups=256),
        # lookahead retrieval with the cluster cache: two rounds of a micro-batch of four
        dict(name="lookahead_cache", op="lookahead", dtype="f16", metric="ip", n=400_000, d=768, nlist=1600, skew=0.1,
             nprobe=128, k=10, nq=4, groups=4, budget=0.6, cache=True),
        # the prefetching scheduler over a global batch
        dict(name="schedule_512", op="schedule", d=768, nq=512, micro=8, groups=40),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(max(lo, hi))))))


def draw(rng):
    op = rng.choice(["search"] * 8 + ["stream", "lookahead", "schedule"])
    if op == "schedule":
        nq = _log_int(rng, 16, 600)
        return dict(op=op, d=rng.choice([100, 128, 384, 768, 1024]), nq=nq, micro=_log_int(rng, 2, 32), groups=max(1, nq // rng.randint(2, 16)))
    dtype = rng.choice(["f32", "f16", "bf16"])
    metric = rng.choice(["ip", "ip", "l2"])
    # widths: half of them the usual embedding sizes, half anything
    d = rng.choice([64, 128, 256, 384, 512, 768, 1024]) if rng.random() < 0.5 else _log_int(rng, 40, 1024)
    row = d * (4 if dtype == "f32" else 2)
    batch = op == "search" and rng.random() < 0.6
    nq = _log_int(rng, 2, 256) if batch else 1
    top = 6e8 if op == "lookahead" else 1.2e10
    n = int(min(8e6, math.exp(rng.uniform(math.log(5e6), math.log(top))) / row))
    nlist = min(8192, max(16, int(n / math.exp(rng.uniform(math.log(100), math.log(2500))))))
    nprobe = _log_int(rng, 4, min(512, nlist // 2))
    if op == "stream":
        nq = rng.choice([16, 32, 64])
    if op == "lookahead":
        nq = rng.choice([1, 1, 2, 4])
    # a pass does no more than the largest listed case: its scores, and 6 GB read query by query
    mean = n / nlist
    most = min(1.9e11 / (2.0 * d), 6e9 / row if d % 64 or op != "search" or nq < 4 else 1e30)
    nprobe = max(1, min(nprobe, int(most / (mean * nq))))
    case = dict(op=op, dtype=dtype, metric=metric, n=n, d=d, nlist=nlist, skew=rng.choice([0.0, 0.5, 1.1, 1.2]), nprobe=nprobe,
                k=_log_int(rng, 1, 112), nq=nq, groups=max(1, int(nq * rng.uniform(0.3, 1.0))))
    if op == "search":
        case["entry"] = rng.choice(["device", "host"])
    elif op == "stream":
        case["depth"] = rng.choice([2, 4, 8, 16])
    else:
        case.update(budget=rng.uniform(0.2, 1.2), cache=rng.random() < 0.5)
    return case


# ---- inputs -----------------------------------------------------------------------------------
_shared = {}


def _streams():
    """One compute and one copy stream for the whole program, as a serving process has them."""
    if not _shared:
        _shared["s"] = (torch.cuda.Stream(), torch.cuda.Stream())
    return _shared["s"]


def _unit(x):
    return x / x.norm(dim=-1, keepdim=True).clamp_min(1e-30)


def _sizes(case, gen):
    """List sizes: the list of rank r gets a share r^-skew of the rows, in shuffled order, ragged."""
    nlist, n = case["nlist"], case["n"]
    w = torch.arange(1, nlist + 1, dtype=torch.float64) ** (-float(case["skew"]))
    w = w * (0.6 + 0.8 * torch.rand(nlist, generator=gen, dtype=torch.float64))
    sizes = torch.floor(w / w.sum() * (n - nlist)).to(torch.int64) + 1
    sizes[0] += n - int(sizes.sum())
    return sizes[torch.randperm(nlist, generator=gen)]


def _noisy(x, alpha, gen):
    return _unit(x + alpha * x.shape[1] ** -0.5 * torch.randn(x.shape, generator=gen, device=x.device))


def _data(case, seed):
    """Rows (cluster-major, on the GPU), offsets, centroids and the queries q_in, q_out."""
    cpu = torch.Generator().manual_seed(int(seed))
    gen = torch.Generator(device="cuda").manual_seed(int(seed) + 1)
    n, d, nlist, nq = case["n"], case["d"], case["nlist"], case["nq"]
    sizes = _sizes(case, cpu)
    off = torch.zeros(nlist + 1, dtype=torch.int64)
    off[1:] = torch.cumsum(sizes, 0)
    centres = torch.randn(nlist, d, generator=gen, device="cuda")
    of_row = torch.repeat_interleave(torch.arange(nlist, device="cuda"), sizes.cuda())
    rows = torch.empty(n, d, dtype=TORCH[case["dtype"]], device="cuda")
    step = max(1, (1 << 28) // d)
    for s in range(0, n, step):
        e = min(n, s + step)
        x = torch.randn(e - s, d, generator=gen, device="cuda")
        x.mul_(SIGMA).add_(centres[of_row[s:e]])
        x.div_(x.norm(dim=1, keepdim=True))
        rows[s:e] = x
    cent = _unit(centres) / math.sqrt(1 + SIGMA * SIGMA)
    if nq == 1 or case["op"] != "search":      # questions near stored rows
        at = torch.randint(0, n, (case["groups"],), generator=cpu)[torch.arange(nq) % case["groups"]].cuda()
        q_in = _noisy(rows[at].float(), 0.1, gen)
        q_out = _noisy(q_in, 0.3, gen)
    else:                                      # a batch drawn around some of the centres: its queries share lists
        at = torch.randperm(nlist, generator=cpu)[torch.arange(nq) % min(nlist, case["groups"])].cuda()
        q_in = q_out = _noisy(_unit(centres[at]), 0.5, gen)
    return rows, off.numpy(), cent.cpu().numpy(), q_in.contiguous(), q_out.contiguous()


def _global_batch(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    centres = torch.randn(case["groups"], case["d"], generator=gen, device="cuda")
    which = torch.randint(0, case["groups"], (case["nq"],), generator=gen, device="cuda")
    return _noisy(_unit(centres)[which], 0.3, gen).cpu().numpy()


def prepare(case, seed):
    compute, copy = _streams()
    if case["op"] == "schedule":
        q = _global_batch(case, seed)
        d = case["d"]
        one = torch.zeros(1, d, device="cuda")
        index = P.ivf_adopt_layout(one, "f32", np.array([0, 1]), np.zeros((1, d), np.float32), compute_stream=compute,
                                   copy_stream=copy)
        return dict(case=case, index=index, q=q)
    rows, off, cent, q_in, q_out = _data(case, seed)
    row_bytes = rows.element_size() * case["d"]
    kw = {}
    if case["op"] == "lookahead":
        # room for what the queries of a pass select, and a budget that covers part of it
        want = case["nq"] * case["nprobe"] * (case["n"] / case["nlist"]) * row_bytes
        host = torch.empty(rows.shape, dtype=rows.dtype, pin_memory=True)
        host.copy_(rows)
        rows = host
        kw = dict(placement=P.IVF_PLACE_HOST, device_buffer_bytes=int(min(2 * want, case["n"] * row_bytes)) + 4096)
    torch.cuda.synchronize()
    index = P.ivf_adopt_layout(rows, case["dtype"], off, cent, metric=METRIC[case["metric"]], compute_stream=compute,
                               copy_stream=copy, **kw)
    nq, k = case["nq"], case["k"]
    st = dict(case=case, index=index, q=q_out, ids=torch.empty(nq, k, dtype=torch.int64, device="cuda"),
              dists=torch.empty(nq, k, dtype=torch.float32, device="cuda"))
    if case["op"] == "lookahead":
        index.ivf_set_host_threads(min(16, os.cpu_count() or 1))
        st["budget"] = int(case["budget"] * want)
        st["q_in"], st["q"] = q_in.cpu().numpy(), q_out.cpu().numpy()
        # the second round's queries: the next step of the same conversations
        gen = torch.Generator(device="cuda").manual_seed(int(seed) + 2)
        q_in2 = _noisy(q_out, 0.3, gen)
        st["q_in2"], st["q2"] = q_in2.cpu().numpy(), _noisy(q_in2, 0.3, gen).cpu().numpy()
        if case["cache"]:
            index.ivf_cache_configure(0.5, 1.0, 2.0, 1.0)
    elif case["op"] == "stream":
        st["q"] = [one.clone() for one in q_out]          # queries arrive one by one
        index.ivf_set_pipeline_depth(case["depth"])
        index.ivf_reserve(1, case["nprobe"], k)
    else:
        index.ivf_reserve(nq, case["nprobe"], k)
        if case["entry"] == "host":
            st["q"] = q_out.cpu().numpy()
    return st


def run(state):
    case, index = state["case"], state["index"]
    op = case["op"]
    if op == "schedule":
        return index.ivf_schedule(state["q"], case["micro"])
    nprobe, k = case["nprobe"], case["k"]
    if op == "lookahead":
        index.ivf_prefetch(state["q_in"], nprobe, state["budget"], P.IVF_PREFETCH_RESET)
        out = list(index.ivf_search(state["q"], nprobe, k))
        if case["cache"]:
            index.ivf_cache_end_round()
            index.ivf_prefetch(state["q_in2"], nprobe, state["budget"])
            out += index.ivf_search(state["q2"], nprobe, k)
            index.ivf_cache_end_round()
            cached = np.zeros(case["nlist"], np.int32)
            cached[index.ivf_resident()] = 1
            out += [index.ivf_cache_hotness(), cached]
        return out
    if op == "stream":
        q, ids, dists = state["q"], state["ids"], state["dists"]
        for i in range(case["nq"]):
            index.ivf_search_device(q[i], nprobe, k, ids[i], dists[i])
        index.ivf_synchronize()
        return [ids, dists]
    if case["entry"] == "host":
        return list(index.ivf_search(state["q"], nprobe, k))
    index.ivf_search_device(state["q"], nprobe, k, state["ids"], state["dists"])
    if case["nq"] > 1:
        index.ivf_synchronize()
    return [state["ids"], state["dists"]]


# ---- what a pass cannot do without ---------------------------------------------------------------
def work(case):
    d, nq = case["d"], case["nq"]
    if case["op"] == "schedule":
        return {"bytes": 4.0 * nq * d + 4.0 * nq, "flops": 1.5 * d * nq * (nq - 1)}
    row = d * (4 if case["dtype"] == "f32" else 2)
    share = min(1.0, case["nprobe"] / case["nlist"])
    centroids = 4.0 * case["nlist"] * d
    io = nq * (4.0 * d + 12.0 * case["k"])
    flops = 2.0 * d * nq * (case["n"] * share + case["nlist"])
    if case["op"] == "stream":          # independent calls: each reads its own lists and the centroids
        return {"bytes": nq * (case["n"] * share * row + centroids) + io, "flops": flops}
    union = case["n"] * (1.0 - (1.0 - share) ** min(nq, case["groups"]))
    if case["op"] == "lookahead":
        rounds = 2 if case["cache"] else 1
        moved = min(case["budget"], 1.0) * union * row          # read from the host, written to the buffer, scanned
        return {"bytes": rounds * (2 * moved + union * row + 2 * centroids + 2 * io), "flops": 2 * rounds * flops}
    return {"bytes": union * row + centroids + io, "flops": flops}


def tolerance(case):
    """Results are the exact ranking by 64-bit scores, and distances are those scores rounded once to 32 bits
    (3e-8 relative in the mean): four times that, and whole numbers as they are."""
    return "exact" if case["op"] == "schedule" else {"rel": 1.2e-7, "max": 1e-6, "differ": 0.0}


# ---- the same results in 64 bits ------------------------------------------------------------------
def _scores(q, y, metric):
    s = q @ y.T
    if metric == "ip":
        return s
    return 2 * s - (q * q).sum(1)[:, None] - (y * y).sum(1)[None]


def _search64(case, rows, off, cent, q):
    """Coarse scores, the nprobe nearest lists and the k best of their rows, in float64."""
    metric, nprobe, k = case["metric"], min(case["nprobe"], case["nlist"]), case["k"]
    q = torch.as_tensor(q).cuda().double()
    coarse = _scores(q, torch.from_numpy(cent).cuda().double(), metric)
    picked = torch.zeros(q.shape[0], case["nlist"], dtype=torch.bool, device="cuda")
    picked.scatter_(1, coarse.topk(nprobe, dim=1).indices, True)
    off_dev = torch.from_numpy(off).cuda()
    best = torch.full((q.shape[0], k), -math.inf, dtype=torch.float64, device="cuda")
    ids = torch.full((q.shape[0], k), -1, dtype=torch.int64, device="cuda")
    wanted = torch.repeat_interleave(picked.any(0), off_dev[1:] - off_dev[:-1]).nonzero()[:, 0]     # rows of any picked list
    step = max(1, (1 << 26) // case["d"])
    for s in range(0, wanted.numel(), step):
        at = wanted[s:s + step]
        y = rows[at.to(rows.device)].cuda().double()
        sc = _scores(q, y, metric)
        sc[~picked[:, torch.searchsorted(off_dev, at, right=True) - 1]] = -math.inf
        both = torch.cat([best, sc], 1)
        best, pos = both.topk(k, dim=1)
        ids = torch.cat([ids, at[None].expand(q.shape[0], -1)], 1).gather(1, pos)
    none = torch.isinf(best)
    return torch.where(none, torch.full_like(ids, -1), ids), (best if metric == "ip" else -best)


def _greedy64(q, micro):
    """While queries remain, the one of lowest index seeds a group and the nearest remaining ones follow."""
    x = torch.from_numpy(q).cuda().double()
    dist = torch.stack([((x - y) ** 2).sum(1) for y in x]).cpu().numpy()
    left = np.ones(len(q), bool)
    order = []
    while left.any():
        seed = int(np.argmax(left))
        left[seed] = False
        order.append(seed)
        near = np.argsort(np.where(left, dist[seed], np.inf), kind="stable")[:min(micro - 1, int(left.sum()))]
        left[near] = False
        order += [int(i) for i in near]
    return np.array(order, np.int32)


def exact(case, seed):
    if case["op"] == "schedule":
        return _greedy64(_global_batch(case, seed), case["micro"])
    rows, off, cent, _, q_out = _data(case, seed)
    out = list(_search64(case, rows, off, cent, q_out))
    if case["op"] == "lookahead" and case["cache"]:
        gen = torch.Generator(device="cuda").manual_seed(int(seed) + 2)
        q2 = _noisy(_noisy(q_out, 0.3, gen), 0.3, gen)
        out += list(_search64(case, rows, off, cent, q2)) + [None, None]
    return out
