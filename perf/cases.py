"""The calls whose speed counts: query routing, residual-PQ search, k-means, assignment, inverted
lists, PQ training and encoding, and the candidate-restricted construction, each through the
package's public entry points, from one small batch of queries to millions of base rows.

Inputs come from the case's seed alone. Two kinds of vectors stand for the datasets this path
serves: "u8", integer values 0..255 around uniform means (SIFT- and SPACEV-like), and "f32",
unit-norm anisotropic floats (DEEP-like). Queries, centroids and residuals of "u8" data are fp32
arrays, base and training rows are uint8; everything is fp32 for "f32".
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2608_08751_amd as ivf

DEV = "cuda:0"
K = 256  # codewords per PQ subspace


# ------------------------------------------------------------------ the cases

def listed():
    return [
        # A small table and a batch of a thousand queries: launches and latency.
        dict(name="route_tiny", kind="route", data="u8", queries=1000, lists=1024, dim=128, nprobe=16),
        # Routing of SIFT-like queries against a 65,536-list index.
        dict(name="route_u8", kind="route", data="u8", queries=10000, lists=65536, dim=128, nprobe=64),
        # Routing of DEEP-like queries against a large table, the widest probe set.
        dict(name="route_f32", kind="route", data="f32", queries=10000, lists=262144, dim=96, nprobe=128),
        # Online search with the smallest batch: route, then the ADC scan of the probed lists.
        dict(name="search_b8", kind="search", data="u8", queries=8, rows=10_000_000, lists=65536, dim=128,
             nprobe=64, subspaces=16, handoff=512),
        # Throughput search, the largest batch.
        dict(name="search_b2048", kind="search", data="u8", queries=2048, rows=10_000_000, lists=65536, dim=128,
             nprobe=96, subspaces=16, handoff=512),
        # The second Lloyd iteration of the training of a 65,536-list index, hinted by the first one's labels.
        dict(name="kmeans_u8", kind="kmeans", data="u8", rows=5_000_000, lists=65536, dim=128, close=False, hints=True),
        # A Lloyd iteration on fp32 rows.
        dict(name="kmeans_f32", kind="kmeans", data="f32", rows=500_000, lists=16384, dim=96, close=False, hints=False),
        # Full assignment of one batch of base rows to more than 65,536 lists, rows of 100 bytes, and its lists;
        # centroids so close to each other that many rows lie between two or more of them, as in real datasets.
        dict(name="assign_u8_d100", kind="assign", data="u8", rows=1_000_003, lists=131072, dim=100, close=True),
        # The inverted lists alone, skewed list sizes.
        dict(name="lists_50m", kind="lists", rows=50_000_000, lists=65536, skew=1.0),
        # One batch of the base laid out list by list, its residuals, and their PQ codes.
        dict(name="encode_2m", kind="encode", data="u8", rows=2_000_000, lists=16384, dim=128, subspaces=16),
        # A Lloyd iteration of the PQ codebooks.
        dict(name="pq_train_1m", kind="pq_train", rows=1 << 20, dim=128, subspaces=16),
        # Fast construction: coarse cells, first choice and walk, then one iteration on the neighbours of the label.
        dict(name="fast_2m", kind="fast", data="u8", rows=2_000_000, lists=16384, dim=128, cells=256, degree=8,
             hops=8),
    ]


def _between(rng, lo, hi):
    """A whole number from lo to hi, spread over its logarithm."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _dim(rng):
    return rng.choice([128, 96, 100, 64, 4 * rng.randint(8, 64)])


def draw(rng):
    kind = rng.choice(["route", "route", "search", "kmeans", "kmeans", "assign", "lists", "encode", "pq_train",
                       "fast"])
    data = rng.choice(["u8", "f32"])
    if kind == "route":
        q, c, d = _between(rng, 1, 10000), _between(rng, 1000, 262144), _dim(rng)
        while 2.0 * q * c * d > 5e11:
            q = max(1, q // 2)
        return dict(kind=kind, data=data, queries=q, lists=c, dim=d, nprobe=_between(rng, 1, 256))
    if kind == "search":
        dsub = rng.choice([4, 8, 8, 16])
        d = rng.choice([128, 96, 64, 160])
        return dict(kind=kind, data=data, queries=_between(rng, 1, 2048), rows=_between(rng, 200_000, 8_000_000),
                    lists=_between(rng, 1024, 65536), dim=d, nprobe=_between(rng, 4, 96), subspaces=d // dsub,
                    handoff=_between(rng, 10, 512))
    if kind in ("kmeans", "assign"):
        d, c = _dim(rng), _between(rng, 256, 131072)
        cap = 1e12 if data == "f32" else 2e13 if d <= 128 else 8e12
        while 2.0 * (4 * c) * c * d > cap:
            c //= 2
        n = _between(rng, 4 * c, min(4_000_000, cap / (2.0 * c * d)))
        close = rng.random() < 0.5
        if kind == "assign":
            return dict(kind=kind, data=data, rows=n, lists=c, dim=d, close=close)
        return dict(kind=kind, data=data, rows=n, lists=c, dim=d, close=close, hints=rng.random() < 0.5)
    if kind == "lists":
        return dict(kind=kind, rows=_between(rng, 100_000, 40_000_000), lists=_between(rng, 1000, 524288),
                    skew=rng.choice([0.0, 0.5, 1.0]))
    dsub = rng.choice([4, 8, 8, 16])
    d = rng.choice([128, 96, 64, 160])
    if kind == "encode":
        return dict(kind=kind, data=data, rows=_between(rng, 20_000, 2_000_000), lists=_between(rng, 256, 16384),
                    dim=d, subspaces=d // dsub)
    if kind == "pq_train":
        return dict(kind=kind, rows=_between(rng, 20_000, 1 << 20), dim=d, subspaces=d // dsub)
    c = _between(rng, 2048, 16384)
    return dict(kind="fast", data=data, rows=_between(rng, 50_000, 2_000_000), lists=c, dim=_dim(rng),
                cells=max(16, c // rng.choice([32, 64, 100])), degree=rng.choice([4, 8, 16]), hops=rng.choice([2, 8]))


# ------------------------------------------------------------------ inputs

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(0x5EED0000 + int(seed))
    return g


def _randint(g, high, n):
    return torch.randint(0, int(high), (int(n),), generator=g, device=DEV)


def _means(g, data, n, d):
    """Component means: uniform in [0, 255], or anisotropic with unit norm."""
    if data == "u8":
        return torch.rand((n, d), generator=g, device=DEV) * 255.0
    s = torch.rand(d, generator=g, device=DEV) * 0.8 + 0.2
    m = torch.randn((n, d), generator=g, device=DEV) * s
    return (m / m.norm(dim=1, keepdim=True)).contiguous()


def _rows(g, data, means, comp, dtype):
    """A row around the mean of each component: rounded and clipped, or normalised."""
    out = torch.empty((comp.numel(), means.shape[1]), dtype=dtype, device=DEV)
    for a in range(0, comp.numel(), 1 << 20):
        m = means[comp[a:a + (1 << 20)]]
        z = torch.randn(m.shape, generator=g, device=DEV)
        if data == "u8":
            v = (m + 20.0 * z).round_().clamp_(0, 255)
        else:
            v = m + 0.05 * z
            v /= v.norm(dim=1, keepdim=True)
        out[a:a + (1 << 20)] = v.to(dtype)
    return out


def _row_type(data):
    return torch.uint8 if data == "u8" else torch.float32


def _close(g, data, means, n_cent):
    """Centroids that are means of eight rows of a component each: some components hold several, some none.
    Returns (centroids, one centroid of each component or -1)."""
    comp = _randint(g, means.shape[0], n_cent)
    z = torch.randn((n_cent, means.shape[1]), generator=g, device=DEV) / math.sqrt(8.0)
    if data == "u8":
        cent = (means[comp] + 20.0 * z).clamp_(0, 255)
    else:
        cent = means[comp] + 0.05 * z
        cent /= cent.norm(dim=1, keepdim=True) * 1.05
    owner = torch.full((means.shape[0],), -1, dtype=torch.int64, device=DEV)
    owner[comp] = torch.arange(n_cent, device=DEV)
    return cent.contiguous(), owner


def _nearest(x, c, dtype=torch.float32):
    """argmin of the squared distance, a block of rows at a time."""
    c = c.to(dtype)
    n2 = (c * c).sum(1)
    out = torch.empty(x.shape[0], dtype=torch.int64, device=DEV)
    step = max(1, (1 << 30) // c.shape[0])
    for a in range(0, x.shape[0], step):
        out[a:a + step] = torch.addmm(n2, x[a:a + step].to(dtype), c.t(), alpha=-2.0).argmin(1)
    return out


def _zipf_labels(g, n, lists, skew):
    if skew <= 0:
        return _randint(g, lists, n).to(torch.int32)
    w = 1.0 / torch.arange(1, lists + 1, device=DEV, dtype=torch.float64) ** skew
    cdf = (w / w.sum()).cumsum(0)
    names = torch.randperm(lists, generator=g, device=DEV)
    out = torch.empty(n, dtype=torch.int32, device=DEV)
    for a in range(0, n, 1 << 24):
        u = torch.rand(min(1 << 24, n - a), generator=g, device=DEV, dtype=torch.float64)
        out[a:a + (1 << 24)] = names[torch.searchsorted(cdf, u).clamp_(max=lists - 1)].to(torch.int32)
    return out


def _lists_of(labels, lists):
    """offsets int64 [lists + 1] and the stable permutation of labels."""
    off = torch.zeros(lists + 1, dtype=torch.int64, device=DEV)
    off[1:] = torch.bincount(labels.long(), minlength=lists).cumsum(0)
    perm = torch.sort(labels, stable=True)[1]
    return off, perm.to(torch.int32)


def _residuals(g, data, n, d):
    """Residuals of rows to their list's centroid: noise around it, wider in some dims."""
    r = torch.randn((n, d), generator=g, device=DEV) * (20.0 if data == "u8" else 0.05)
    r *= 0.75 + 0.5 * ((torch.arange(d, device=DEV) * 7) % 13) / 12.0
    return r


def _codebooks(g, data, d, m):
    """Codewords as means of a few residual sub-vectors, [m, 256, d / m]."""
    r = _residuals(g, data, K * 4, d).view(K, 4, m, d // m).mean(1) * 1.6
    return r.permute(1, 0, 2).contiguous()


def _codes(g, data, n, cb):
    """PQ codes of n residuals, [n, m] uint8."""
    m, _, ds = cb.shape
    n2 = (cb * cb).sum(2)[:, None, :]
    cbt = cb.transpose(1, 2).contiguous()
    out = torch.empty((n, m), dtype=torch.uint8, device=DEV)
    for a in range(0, n, 1 << 18):
        r = _residuals(g, data, min(1 << 18, n - a), m * ds).view(-1, m, ds).transpose(0, 1).contiguous()
        key = torch.baddbmm(n2, r, cbt, alpha=-2.0)
        out[a:a + (1 << 18)] = key.argmin(2).t().to(torch.uint8)
    return out


def prepare(case, seed):
    g = _gen(seed)
    st = dict(case=case, ctx=ivf.Context(0), seed=int(seed) & 0xFFFF)
    kind, data = case["kind"], case.get("data", "u8")
    if kind in ("route", "search"):
        cent = _means(g, data, case["lists"], case["dim"])
        st["centroids"] = cent
        st["queries"] = _rows(g, data, cent, _randint(g, case["lists"], case["queries"]), torch.float32)
    if kind == "search":
        lab = _zipf_labels(g, case["rows"], case["lists"], 0.4)
        st["offsets"], st["perm"] = _lists_of(lab, case["lists"])
        st["codebooks"] = _codebooks(g, data, case["dim"], case["subspaces"])
        st["codes"] = _codes(g, data, case["rows"], st["codebooks"])
    elif kind in ("kmeans", "assign"):
        means = _means(g, data, case["lists"], case["dim"])
        comp = _randint(g, case["lists"], case["rows"])
        x = st["rows"] = _rows(g, data, means, comp, _row_type(data))
        if case["close"]:
            st["centroids"], owner = _close(g, data, means, case["lists"])
            # labels of an earlier iteration: rows of a component without a centroid went anywhere
            hints = torch.where(owner[comp] >= 0, owner[comp], _randint(g, case["lists"], case["rows"])).to(torch.int32)
        else:  # the training so far: sampled rows, then one iteration
            start = x[torch.randperm(case["rows"], generator=g, device=DEV)[:case["lists"]]].float()
            hints, st["centroids"], _, _ = ivf.ivf_kmeans_step(st["ctx"], x, start, seed=st["seed"], it=0)
        if case.get("hints"):
            st["hints"] = hints
    elif kind == "lists":
        st["labels"] = _zipf_labels(g, case["rows"], case["lists"], case["skew"])
    elif kind == "encode":
        st["centroids"] = _means(g, data, case["lists"], case["dim"])
        lab = _randint(g, case["lists"], case["rows"]).to(torch.int32)
        st["rows"] = _rows(g, data, st["centroids"], lab.long(), _row_type(data))
        st["offsets"], st["perm"] = _lists_of(lab, case["lists"])
        st["codebooks"] = _codebooks(g, data, case["dim"], case["subspaces"])
    elif kind == "pq_train":
        st["residuals"] = _residuals(g, data, case["rows"], case["dim"])
        st["codebooks"] = _codebooks(g, data, case["dim"], case["subspaces"])
    elif kind == "fast":
        c, s = case["lists"], case["degree"]
        cent = _means(g, data, c, case["dim"])
        st["rows"] = _rows(g, data, cent, _randint(g, c, case["rows"]), _row_type(data))
        coarse = cent[_randint(g, c, case["cells"])].contiguous()
        own = _nearest(cent, coarse)
        for _ in range(2):  # the coarse table: two Lloyd iterations over the centroids
            n = torch.bincount(own, minlength=case["cells"]).clamp_(min=1)
            order = torch.sort(own, stable=True)[1]
            run = torch.zeros((c + 1, case["dim"]), dtype=torch.float64, device=DEV)
            run[1:] = cent[order].double().cumsum(0)
            end = torch.bincount(own, minlength=case["cells"]).cumsum(0)
            sums = run[end] - run[end - torch.bincount(own, minlength=case["cells"])]
            coarse = (sums / n[:, None]).float().contiguous()
            own = _nearest(cent, coarse)
        coarse = coarse[torch.bincount(own, minlength=case["cells"]) > 0].contiguous()  # every cell has a member
        own = _nearest(cent, coarse)
        st["centroids"], st["coarse"] = cent, coarse
        st["cell_offsets"], st["cell_members"] = _lists_of(own.to(torch.int32), coarse.shape[0])
        n2 = (cent * cent).sum(1)
        st["graph"] = torch.cat([torch.addmm(n2, cent[a:a + 4096], cent.t(), alpha=-2.0).topk(s, 1, largest=False)[1]
                                 for a in range(0, c, 4096)]).to(torch.int32).contiguous()
        # the centroids after the update that follows: the graph stays the one they had
        st["updated"] = (cent + (3.0 if data == "u8" else 0.008) * torch.randn(cent.shape, generator=g, device=DEV))
        if data == "u8":
            st["updated"].clamp_(0, 255)
    return st


# ------------------------------------------------------------------ one pass

def run(st):
    case, ctx, kind = st["case"], st["ctx"], st["case"]["kind"]
    if kind == "route":
        ids, dist = ivf.ivf_route(ctx, st["queries"], st["centroids"], case["nprobe"])
        return dict(ids=ids, dist=dist)
    if kind == "search":
        probes, _ = ivf.ivf_route(ctx, st["queries"], st["centroids"], case["nprobe"], want_dist=False)
        ids, dist = ivf.ivf_adc_scan(ctx, st["queries"], st["centroids"], probes, st["offsets"], st["perm"],
                                     st["codes"], st["codebooks"], case["handoff"])
        return dict(probes=probes, ids=ids, dist=dist)
    if kind == "kmeans":
        lab, cen, cnt, obj = ivf.ivf_kmeans_step(ctx, st["rows"], st["centroids"], seed=st["seed"], it=1,
                                                 hint_labels=st.get("hints"))
        return dict(labels=lab, centroids=cen, counts=cnt, objective=obj[:1])
    if kind == "assign":
        lab, cnt, off, perm = ivf.ivf_assign_build(ctx, st["rows"], st["centroids"])
        return dict(labels=lab, counts=cnt, offsets=off, perm=perm)
    if kind == "lists":
        cnt, off, perm = ivf.ivf_build_lists(ctx, st["labels"], case["lists"])
        return dict(counts=cnt, offsets=off, perm=perm)
    if kind == "encode":
        rows, res = ivf.ivf_list_major(ctx, st["rows"], st["centroids"], st["offsets"], st["perm"])
        return dict(rows=rows, residuals=res, codes=ivf.ivf_pq_encode(ctx, res, st["codebooks"]))
    if kind == "pq_train":
        cb, cnt, obj = ivf.ivf_pq_train_step(ctx, st["residuals"], st["codebooks"], seed=st["seed"], it=1)
        return dict(codebooks=cb, counts=cnt, objective=obj)
    cell, _, _, by_cell = ivf.ivf_assign_build(ctx, st["rows"], st["coarse"])
    first, d0 = ivf.ivf_assign_cells(ctx, st["rows"], st["centroids"], cell, st["cell_offsets"], st["cell_members"],
                                     st["graph"], case["hops"], order=by_cell)
    _, _, by_label = ivf.ivf_build_lists(ctx, first, case["lists"])
    lab, d1 = ivf.ivf_assign_graph(ctx, st["rows"], st["updated"], st["graph"], first, order=by_label)
    return dict(cell=cell, first=first, first_dist=d0, labels=lab, dist=d1)


# ------------------------------------------------------------------ what a pass cannot do without

def work(case):
    kind, d = case["kind"], case.get("dim", 0)
    c, n, q = case.get("lists", 0), case.get("rows", 0), case.get("queries", 0)
    width = d * (1 if case.get("data", "u8") == "u8" else 4)  # bytes of a base or training row
    if kind == "route":
        return dict(bytes=4.0 * d * (q + c) + 8.0 * q * case["nprobe"], flops=2.0 * q * c * d)
    if kind == "search":
        p, m = case["nprobe"], case["subspaces"]
        scanned = float(q) * p * n / c
        return dict(bytes=4.0 * d * (q + c) + min(scanned, float(n)) * (m + 4) + 1024.0 * d
                    + q * (4.0 * p + 8.0 * case["handoff"]),
                    flops=2.0 * q * c * d + 3.0 * K * d * q * p + m * scanned)
    if kind == "kmeans":
        return dict(bytes=float(n) * (width + 4 + (4 if case["hints"] else 0)) + 8.0 * c * d + 8.0 * c,
                    flops=2.0 * n * c * d + 4.0 * n * d)
    if kind == "assign":
        return dict(bytes=float(n) * (width + 8) + 4.0 * c * d + 16.0 * c, flops=2.0 * n * c * d)
    if kind == "lists":
        return dict(bytes=8.0 * n + 16.0 * c, flops=0.0)
    if kind == "encode":
        return dict(bytes=float(n) * (2 * width + 4 + 4 * d + case["subspaces"]) + 4.0 * c * d + 1024.0 * d,
                    flops=(2.0 * K + 1.0) * n * d)
    if kind == "pq_train":
        return dict(bytes=4.0 * n * d + 2048.0 * d, flops=2.0 * K * n * d + 4.0 * n * d)
    g, s = case["cells"], case["degree"]
    return dict(bytes=float(n) * (2 * width + 28) + 4.0 * d * (2 * c + g) + 4.0 * c * s,
                flops=2.0 * n * d * (g + c / g + 2 * s + s))


def tolerance(case):
    # Ids, labels, counts, permutations and codes are defined to the bit, and so are distances (one fp64
    # evaluation in a stated order, rounded once) and ADC sums (a stated order in fp32). The objective is an fp64
    # sum in any order, and a mean of fp32 rows may round the other way where its fp64 sum is taken in another order.
    if case["kind"] in ("kmeans", "pq_train"):
        return {"rel": 1e-9, "max": 2.5e-7}
    return "exact"


# ------------------------------------------------------------------ in 64 bits

_M64 = (1 << 64) - 1


def _splitmix(seed, n):
    """Output n of SplitMix64 seeded with `seed`."""
    z = (seed + n * 0x9E3779B97F4A7C15) & _M64
    z = ((z ^ (z >> 30)) * 0xBF58476D1CE4E5B9) & _M64
    z = ((z ^ (z >> 27)) * 0x94D049BB133111EB) & _M64
    return z ^ (z >> 31)


def _dist64(x, c, cand):
    """Squared distances of rows x to candidates c[cand], [n, s] in fp64."""
    out = torch.empty(cand.shape, dtype=torch.float64, device=DEV)
    step = max(1, (1 << 28) // (cand.shape[1] * x.shape[1]))
    for a in range(0, x.shape[0], step):
        t = x[a:a + step, None, :].double() - c[cand[a:a + step].long()].double()
        out[a:a + step] = (t * t).sum(2)
    return out


def _lloyd64(x, cent, lab, seed, it):
    """New centroids and the objective of an iteration with labels lab."""
    c = cent.shape[0]
    cnt = torch.bincount(lab, minlength=c)
    end = cnt.cumsum(0)
    order = torch.sort(lab, stable=True)[1]
    sums = torch.empty(cent.shape, dtype=torch.float64, device=DEV)
    for a in range(0, cent.shape[1], 16):  # sums of sorted rows per list, some columns at a time
        v = x[:, a:a + 16].double()[order]
        sums[:, a:a + 16] = torch.segment_reduce(v, "sum", lengths=cnt, axis=0, unsafe=True, initial=0.0)
    new = sums / cnt.clamp(min=1)[:, None]
    for j in torch.nonzero(end - (end - cnt) == 0).flatten().tolist():
        new[j] = x[_splitmix(seed, ((it << 32) | j) + 1) % x.shape[0]].double()
    return new, _dist64(x, cent, lab[:, None]).sum().reshape(1)


def exact(case, seed):
    st = prepare(case, seed)
    kind = case["kind"]
    if kind in ("route", "search"):
        q, cent, p = st["queries"], st["centroids"], case["nprobe"]
        c64 = cent.double()
        n2, step = (c64 * c64).sum(1), max(1, (1 << 28) // cent.shape[0])
        ids = torch.cat([torch.addmm(n2, q[a:a + step].double(), c64.t(), alpha=-2.0).topk(p, 1, largest=False)[1]
                         for a in range(0, q.shape[0], step)])
        dist = _dist64(q, cent, ids).sort(1)[0]
        if kind == "route":
            return dict(ids=None, dist=dist)
        off, codes, cb = st["offsets"], st["codes"], st["codebooks"].double()
        m, k = cb.shape[0], case["handoff"]
        out = torch.full((q.shape[0], k), math.inf, dtype=torch.float64, device=DEV)
        for i in range(q.shape[0]):
            n = (off[ids[i] + 1] - off[ids[i]])
            total = int(n.sum())
            if total == 0:
                continue
            which = torch.repeat_interleave(torch.arange(p, device=DEV), n, output_size=total)
            pos = off[ids[i]][which] + torch.arange(total, device=DEV) - (n.cumsum(0) - n)[which]
            r = (q[i].double() - cent[ids[i]].double()).view(p, m, 1, -1)
            lut = (r - cb).square().sum(3).view(p * m, K)
            at = (which[:, None] * m + torch.arange(m, device=DEV)) * K + codes[pos].long()
            d = lut.view(-1)[at].sum(1)
            best = d.topk(min(k, total), largest=False, sorted=True)[0]
            out[i, :best.numel()] = best
        return dict(probes=None, ids=None, dist=out)
    if kind == "kmeans":
        lab = _nearest(st["rows"], st["centroids"], torch.float64)
        cen, obj = _lloyd64(st["rows"], st["centroids"], lab, st["seed"], 1)
        return dict(labels=None, centroids=cen, counts=None, objective=obj)
    if kind == "encode":
        lab = torch.repeat_interleave(torch.arange(case["lists"], device=DEV), st["offsets"].diff())
        rows = st["rows"][st["perm"].long()].double()
        return dict(rows=rows if st["rows"].dtype == torch.float32 else None,
                    residuals=rows - st["centroids"][lab].double(), codes=None)
    if kind == "pq_train":
        cb, ds = st["codebooks"], case["dim"] // case["subspaces"]
        new, obj = [], []
        for m in range(case["subspaces"]):
            x = st["residuals"][:, m * ds:(m + 1) * ds].contiguous()
            a, b = _lloyd64(x, cb[m], _nearest(x, cb[m], torch.float64), st["seed"] + m, 1)
            new.append(a)
            obj.append(b)
        return dict(codebooks=torch.stack(new), counts=None, objective=torch.cat(obj))
    if kind == "fast":
        x, cent, graph = st["rows"], st["centroids"], st["graph"].long()
        cell = _nearest(x, st["coarse"], torch.float64)
        cells, off = st["coarse"].shape[0], st["cell_offsets"].tolist()
        best = torch.zeros(x.shape[0], dtype=torch.int64, device=DEV)
        d0 = torch.full((x.shape[0],), math.inf, dtype=torch.float64, device=DEV)
        by_cell = torch.sort(cell, stable=True)[1]
        end = torch.bincount(cell, minlength=cells).cumsum(0).tolist()
        for j in range(cells):
            rows, mem = by_cell[end[j - 1] if j else 0:end[j]], st["cell_members"][off[j]:off[j + 1]].long().sort()[0]
            if rows.numel() and mem.numel():
                d, at = _dist64(x[rows], cent, mem.expand(rows.numel(), -1)).min(1)
                d0[rows], best[rows] = d, mem[at]
        live = torch.isfinite(d0)
        for _ in range(case["hops"]):
            d, at = _dist64(x, cent, graph[best]).min(1)
            move = live & (d < d0)
            best = torch.where(move, graph[best].gather(1, at[:, None])[:, 0], best)
            d0 = torch.where(move, d, d0)
        d1 = _dist64(x, st["updated"], graph[best]).min(1)[0]
        d1 = torch.where(live, d1, torch.full_like(d1, math.inf))
        return dict(cell=None, first=None, first_dist=d0, labels=None, dist=d1)
    return None  # assign, lists: whole numbers only
