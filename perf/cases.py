"""Timed cases of the library's public entry points.

Each case is one call (or one short chain of calls) as a program makes it:
device tensors in, device tensors out.  Builds take integer points (or a
dissimilarity matrix) and return every edge and triangle of the filtration;
the pairs cases go on from points to the persistence pairs of each dimension,
from which the bars are read off; the column order and the F2 product are the
sparse steps that stand on their own.

Inputs are noisy circles, spheres and tori for surface samples, Gaussian
mixtures for high-dimensional data, uniform points for odd types and sizes,
and Hamming distances of binary sequences for matrix input.  A case fixes one
such data set; the seed puts its points in another order and moves them by an
isometry (coordinates swapped and reflected), and thresholds given as a number
or share of the edges never part edges of one length.  So another seed gives
other bytes in and out, and filtrations of the same size.
"""
from __future__ import annotations

import math

import torch

import paper_1809_04424_amd as vr

DTYPES = {"int8": torch.int8, "int16": torch.int16, "int32": torch.int32}


def listed():
    return [
        # the smallest call: a few dozen points of the plane at the infinite
        # threshold, where the fixed cost of a build counts
        {"name": "plain64", "kind": "build", "shape": "uniform", "n": 64, "d": 2, "dtype": "int32", "thr": "full",
         "bp": 10000},
        # an ordinary surface-like sample at a percentile of the distances
        {"name": "circle1000", "kind": "build", "shape": "circle", "n": 1000, "d": 3, "dtype": "int8",
         "thr": "fraction", "bp": 2000},
        # an odd size and dimension in 16-bit coordinates, a given number of edges
        {"name": "ragged777", "kind": "build", "shape": "uniform", "n": 777, "d": 37, "dtype": "int16",
         "thr": "count", "bp": 3000},
        # clustered high-dimensional data
        {"name": "mixture4000", "kind": "build", "shape": "mixture", "n": 4000, "d": 64, "dtype": "int8",
         "thr": "fraction", "bp": 1000},
        # the most points a build takes, 16-bit coordinates, an upper distance
        {"name": "torus8192", "kind": "build", "shape": "torus", "n": 8192, "d": 3, "dtype": "int16", "thr": "sqdist",
         "bp": 300},
        # Hamming distances of sequences at the default infinite threshold
        {"name": "hamming1088", "kind": "matrix", "n": 1088, "bits": 96, "thr": "full", "bp": 10000},
        # many clouds of uneven sizes in one call
        {"name": "batch32", "kind": "batch", "clouds": 32, "nmin": 50, "nmax": 2000, "lo": 500, "hi": 2500},
        # points to the persistence pairs of dimensions 0 and 1: a cloud with
        # one long bar, and clustered data with many short ones
        {"name": "pairs_circle1000", "kind": "pairs", "shape": "circle", "n": 1000, "d": 3, "dtype": "int8",
         "thr": "fraction", "bp": 2000, "maxdim": 2},
        {"name": "pairs_mixture4000", "kind": "pairs", "shape": "mixture", "n": 4000, "d": 64, "dtype": "int8",
         "thr": "fraction", "bp": 1000, "maxdim": 2},
        # the same with the tetrahedra and the pairs of dimension 2
        {"name": "pairs3_sphere400", "kind": "pairs", "shape": "sphere", "n": 400, "d": 3, "dtype": "int8",
         "thr": "fraction", "bp": 1500, "maxdim": 3},
        # the columns of a complete graph's rank matrix, put in order
        {"name": "columns2000", "kind": "columns", "ncols": 2000, "mean": 1999, "ragged": False, "maxvalue": 1999000},
        # one sparse product and sum over F2
        {"name": "schur16384", "kind": "schur", "m": 16384, "c": 32, "e": 8},
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["build", "build", "build", "torus", "matrix", "batch", "pairs", "pairs", "pairs3", "columns",
                       "schur"])
    if kind == "build":
        n = _logint(rng, 40, 5000)
        shape = rng.choice(["circle", "sphere", "mixture", "uniform"])
        d = {"circle": rng.choice([2, 3]), "sphere": 3, "mixture": rng.choice([16, 64]),
             "uniform": rng.choice([2, 5, 37])}[shape]
        dtype = rng.choice(["int16", "int32"]) if shape == "uniform" else "int8"
        thr = "full" if n <= 400 else rng.choice(["fraction", "count"])
        bp = 10000 if thr == "full" else rng.randint(500, 2000)
        bp = min(bp, int(10000 * 590000 / (n * (n - 1) / 2)))  # at most the triangles of the largest listed
        return {"kind": "build", "shape": shape, "n": n, "d": d, "dtype": dtype, "thr": thr, "bp": bp}
    if kind == "torus":
        return {"kind": "build", "shape": "torus", "n": _logint(rng, 500, 8192), "d": 3, "dtype": "int16",
                "thr": "sqdist", "bp": rng.randint(50, 300)}
    if kind == "matrix":
        n = _logint(rng, 60, 1088)
        return {"kind": "matrix", "n": n, "bits": rng.choice([33, 64, 96]), "thr": rng.choice(["full", "fraction"]),
                "bp": rng.randint(3000, 9000)}
    if kind == "batch":
        return {"kind": "batch", "clouds": _logint(rng, 4, 32), "nmin": 50, "nmax": rng.randint(300, 2000), "lo": 500,
                "hi": 2500}
    if kind == "pairs":
        shape = rng.choice(["circle", "mixture"])
        n = _logint(rng, 60, 1000 if shape == "circle" else 4000)
        return {"kind": "pairs", "shape": shape, "n": n, "d": 3 if shape == "circle" else 64, "dtype": "int8",
                "thr": "fraction", "bp": rng.randint(500, 1000) if shape == "mixture" else rng.randint(800, 2000),
                "maxdim": 2}
    if kind == "pairs3":
        return {"kind": "pairs", "shape": "sphere", "n": _logint(rng, 40, 400), "d": 3, "dtype": "int8",
                "thr": "fraction", "bp": rng.randint(800, 1500), "maxdim": 3}
    if kind == "columns":
        ncols, mean = _logint(rng, 10, 4000), _logint(rng, 4, 2000)
        mean = min(mean, 4000000 // ncols)
        return {"kind": "columns", "ncols": ncols, "mean": mean, "ragged": rng.random() < 0.5,
                "maxvalue": _logint(rng, 10, 2000000)}
    return {"kind": "schur", "m": _logint(rng, 300, 16384), "c": rng.randint(4, 32), "e": rng.randint(2, 8)}


# ------------------------------------------------------------------ inputs ----
def _gen(device, seed):
    g = torch.Generator(device=device)
    g.manual_seed(int(seed))
    return g


def _points(shape, n, d, dtype, g, device):
    def normal(*s):
        return torch.randn(*s, generator=g, device=device, dtype=torch.float64)

    def uniform(*s):
        return torch.rand(*s, generator=g, device=device, dtype=torch.float64)

    if shape == "uniform":
        return torch.randint(0, 1024, (n, d), generator=g, device=device).to(DTYPES[dtype])
    if shape == "mixture":
        mu = torch.randint(-80, 81, (8, d), generator=g, device=device).double()
        comp = torch.randint(0, 8, (n,), generator=g, device=device)
        x = mu[comp] + 12.0 * normal(n, d)
    elif shape == "circle":
        t = 2 * math.pi * uniform(n)
        x = torch.zeros(n, d, dtype=torch.float64, device=device)
        x[:, 0], x[:, 1] = 100 * torch.cos(t), 100 * torch.sin(t)
        x += 5.0 * normal(n, d)
    elif shape == "sphere":
        v = normal(n, 3)
        x = 100 * v / v.norm(dim=1, keepdim=True).clamp_min(1e-12) + 3.0 * normal(n, 3)
    else:  # torus
        scale = 100.0 if dtype != "int8" else 1.0
        u, w = 2 * math.pi * uniform(n), 2 * math.pi * uniform(n)
        ring = 80.0 + 30.0 * torch.cos(w)
        x = torch.stack([ring * torch.cos(u), ring * torch.sin(u), 30.0 * torch.sin(w)], 1) + 3.0 * normal(n, 3)
        x *= scale
    lim = 127 if dtype == "int8" else 32767
    return x.round().clamp(-lim, lim).to(DTYPES[dtype]).contiguous()


def _moved(x, g, device):
    """The points in another order, coordinates swapped and reflected."""
    n, d = x.shape
    x = x[torch.randperm(n, generator=g, device=device)][:, torch.randperm(d, generator=g, device=device)]
    flip = torch.randint(0, 2, (d,), generator=g, device=device)
    return torch.where(flip.bool(), -x, x).contiguous()


def _sqdist(pts):
    x = pts.double()  # whole numbers below 2^53: exact
    s = (x * x).sum(1)
    return (s[:, None] + s[None, :] - 2 * (x @ x.T)).round().long()


def _threshold(case, bp, dist_of):
    """Threshold of a cloud: about bp / 10000 of the edges, all or none of one length."""
    if case.get("thr") == "full":
        return ("full", 0, 1)
    if case.get("thr") == "sqdist":
        # the disc of radius sqrt(tau) holds bp / 10000 of the torus' area
        return ("sqdist", int(bp / 10000 * 4 * math.pi * 8000.0 * 3000.0), 0)
    dist = dist_of()
    n = dist.shape[0]
    q = torch.sort(dist[tuple(torch.triu_indices(n, n, 1, device=dist.device))]).values
    pairs = q.numel()
    want = bp * pairs // 10000
    k = int((q <= q[want - 1]).sum()) if want else 0
    return ("count", k, 1) if case.get("thr") == "count" else ("fraction", k, pairs)


def _hamming(n, bits, g, h, device):
    centres = torch.randint(0, 2, (6, bits), generator=g, device=device)
    seqs = centres[torch.randint(0, 6, (n,), generator=g, device=device)]
    seqs = seqs ^ (torch.rand(n, bits, generator=g, device=device) < 0.1).long()
    s = seqs[torch.randperm(n, generator=h, device=device)].float()
    both = (s @ s.T).round().int()  # whole numbers below 2^24: exact
    ones = s.sum(1).int()
    return (ones[:, None] + ones[None, :] - 2 * both).contiguous()


def _cloud_sizes(case):
    """Sizes and thresholds of a batch: spread over the range by a fixed sequence."""
    out = []
    for c in range(case["clouds"]):
        u, w = (0.5 + 0.6180339887498949 * c) % 1.0, (0.5 + 0.7548776662466927 * c) % 1.0
        n = int(math.exp(math.log(case["nmin"]) + u * math.log(case["nmax"] / case["nmin"])))
        out.append((n, case["lo"] + int(w * (case["hi"] - case["lo"]))))
    return out


def _columns(ncols, mean, ragged, hi, g, device):
    """A CSC array: columns of `mean` entries (ragged: geometric lengths of
    that mean, at most hi), values in 0 .. hi - 1."""
    lens = torch.full((ncols,), mean, dtype=torch.int64, device=device)
    if ragged:
        u = torch.rand(ncols, generator=g, device=device, dtype=torch.float64)
        lens = (-torch.log1p(-u) * mean).long().clamp_max(hi)
    cp = torch.zeros(ncols + 1, dtype=torch.int64, device=device)
    cp[1:] = torch.cumsum(lens, 0)
    return cp, torch.randint(0, hi, (int(cp[-1]),), generator=g, device=device, dtype=torch.int64).to(torch.int32)


def _columns_in(order, cp, v):
    """The columns of a CSC array in another order."""
    lens = (cp[1:] - cp[:-1])[order]
    to = torch.zeros_like(cp)
    to[1:] = torch.cumsum(lens, 0)
    at = torch.repeat_interleave(cp[:-1][order] - to[:-1], lens) + torch.arange(v.numel(), device=v.device)
    return to, v[at].contiguous()


def _inputs(case, seed, device):
    g, h = _gen(device, 1), _gen(device, seed)  # the data set, and its order
    kind = case["kind"]
    if kind in ("build", "pairs"):
        pts = _moved(_points(case["shape"], case["n"], case["d"], case["dtype"], g, device), h, device)
        return {"pts": pts, "thr": _threshold(case, case["bp"], lambda: _sqdist(pts))}
    if kind == "matrix":
        dist = _hamming(case["n"], case["bits"], g, h, device)
        return {"dist": dist, "thr": _threshold(case, case["bp"], lambda: dist)}
    if kind == "batch":
        pts, thr = [], []
        for c, (n, bp) in enumerate(_cloud_sizes(case)):
            pts.append(_moved(_points(("circle", "sphere", "torus")[c % 3], n, 3, "int8", g, device), h, device))
            thr.append(_threshold(case, bp, lambda: _sqdist(pts[-1])))
        return {"pts": pts, "thr": thr}
    if kind == "columns":
        cp, v = _columns(case["ncols"], case["mean"], case["ragged"], case["maxvalue"] + 1, g, device)
        cp, v = _columns_in(torch.randperm(case["ncols"], generator=h, device=device), cp, v)
        return {"colptr": cp, "v": v}
    m = case["m"]
    C, E, D = (_columns(m, k, True, m, g, device) for k in (case["c"], case["e"], case["e"]))
    rows, inner, cols = (torch.randperm(m, generator=h, device=device) for _ in range(3))
    back = torch.empty_like(inner)
    back[inner] = torch.arange(m, device=device)
    C = _columns_in(inner, C[0], rows[C[1].long()].int())  # column x of C moves to where E's rows now say
    E = _columns_in(cols, E[0], back[E[1].long()].int())
    D = _columns_in(cols, D[0], rows[D[1].long()].int())
    return {"mats": [C, E, D]}


def prepare(case, seed):
    state = _inputs(case, seed, torch.device("cuda"))
    state["case"] = case
    return state


# -------------------------------------------------------------------- pass ----
def _filtration(r):
    return {"edge_ij": r.edge_ij(), "edge_q": r.edge_q(), "tri_key": r.tri_key()}


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "build":
        return _filtration(vr.build(state["pts"], state["thr"]))
    if kind == "matrix":
        return _filtration(vr.build_matrix(state["dist"], state["thr"]))
    if kind == "batch":
        return [(r.edge_ij(), r.tri_key()) for r in vr.build_batch(state["pts"], state["thr"])]
    if kind == "pairs":
        r = vr.build(state["pts"], state["thr"], maxdim=case["maxdim"])
        e_low, death = vr.pairs_dim0(r)
        tri_of_edge = vr.pairs_dim1(r, e_low)
        out = {"e_low": e_low, "death": death, "tri_of_edge": tri_of_edge}
        if case["maxdim"] == 3:
            out["tri_tet"] = vr.pairs_dim2(r, tri_of_edge)
        return out
    if kind == "columns":
        return vr.column_order(state["colptr"], state["v"])
    C, E, D = state["mats"]
    colptr, rows = vr.blockprodsum(case["m"], C, E, D)
    return {"colptr": colptr, "rows": rows}


# ------------------------------------------------- the same in plain torch ----
def _sorted_pairs(q_of_row, n, device):
    """All pairs i < j by (q, i, j): q, i, j."""
    i, j = torch.triu_indices(n, n, 1, device=device)
    q = q_of_row[i, j]
    order = torch.sort(q, stable=True).indices
    return q[order], i[order], j[order]


def _kept(thr, q, n):
    kind, num, den = thr
    pairs = n * (n - 1) // 2
    if kind == "full":
        return pairs
    if kind == "count":
        return num
    if kind == "fraction":
        return num * pairs // den
    return int((q < num).sum())


def _plain_filtration(dist, thr):
    n, device = dist.shape[0], dist.device
    q, i, j = _sorted_pairs(dist, n, device)
    k = _kept(thr, q, n)
    q, i, j = q[:k], i[:k], j[:k]
    far = torch.iinfo(torch.int32).max
    rank = torch.full((n, n), far, dtype=torch.int32, device=device)
    r = torch.arange(k, dtype=torch.int32, device=device)
    rank[i, j] = r
    rank[j, i] = r
    keys = []
    step = max(1, (1 << 26) // n)
    for lo in range(0, k, step):
        a, b, v = i[lo:lo + step], j[lo:lo + step], r[lo:lo + step]
        e, c = torch.nonzero((rank[a] < v[:, None]) & (rank[b] < v[:, None]), as_tuple=True)
        tri = torch.sort(torch.stack([a[e], b[e], c], 1), 1).values
        keys.append((v[e].long() << 39) | (tri[:, 0] << 26) | (tri[:, 1] << 13) | tri[:, 2])
    return {"edge_ij": torch.stack([i, j], 1).int(), "edge_q": q,
            "tri_key": torch.cat(keys) if keys else torch.zeros(0, dtype=torch.int64, device=device)}


def exact(case, seed):
    kind = case["kind"]
    if kind == "pairs":  # whole numbers; a plain column reduction takes minutes
        return None
    x = _inputs(case, seed, torch.device("cuda"))
    if kind == "build":
        return _plain_filtration(_sqdist(x["pts"]), x["thr"])
    if kind == "matrix":
        return _plain_filtration(x["dist"].long(), x["thr"])
    if kind == "batch":
        each = [_plain_filtration(_sqdist(p), t) for p, t in zip(x["pts"], x["thr"])]
        return [(f["edge_ij"], f["tri_key"]) for f in each]
    if kind == "columns":
        cp, v = x["colptr"], x["v"]
        col = torch.repeat_interleave(torch.arange(case["ncols"], device=cp.device), cp[1:] - cp[:-1])
        order = torch.sort(col * (int(v.max()) + 1 if v.numel() else 1) + v.long(), stable=True).indices
        z = torch.empty_like(order)
        z[order] = torch.arange(order.numel(), device=cp.device)
        return z
    m = case["m"]

    def dense(cp, rows):
        a = torch.zeros(m * m, dtype=torch.float64, device=cp.device)
        col = torch.repeat_interleave(torch.arange(m, device=cp.device), cp[1:] - cp[:-1])
        a.index_add_(0, col * m + rows.long(), torch.ones(rows.numel(), dtype=torch.float64, device=cp.device))
        return a.view(m, m)  # [column, row]

    C, E, D = (dense(*mat) for mat in x["mats"])
    s = torch.remainder(D + E @ C, 2.0) > 0.5
    colptr = torch.zeros(m + 1, dtype=torch.int64, device=s.device)
    colptr[1:] = torch.cumsum(s.sum(1), 0)
    return {"colptr": colptr, "rows": torch.nonzero(s)[:, 1].int()}


# -------------------------------------------------------------------- cost ----
def _count_complex(dist, thr):
    """(K, T) of a cloud, from the trace of the cubed adjacency matrix."""
    n = dist.shape[0]
    q = _sorted_pairs(dist, n, dist.device)[0]
    k = _kept(thr, q, n)
    if k == 0:
        return 0, 0
    adj = (dist <= q[k - 1]).double()  # ties at the last edge: a few more than kept
    adj.fill_diagonal_(0)
    return k, int(((adj @ adj) * adj).sum().item() / 6)


def work(case):
    """Input read once, output written once; arithmetic of the distances (for
    the F2 product, of its row additions)."""
    kind = case["kind"]
    x = _inputs(case, 0, torch.device("cuda" if torch.cuda.is_available() else "cpu"))
    if kind == "columns":
        nnz = x["v"].numel()
        return {"bytes": 12 * nnz + 8 * (case["ncols"] + 1), "flops": nnz}
    if kind == "schur":
        (cpc, rc), (cpe, re_), (_, rd) = x["mats"]
        lens = (cpc[1:] - cpc[:-1])[re_.long()].sum().item()
        return {"bytes": 4 * (rc.numel() + re_.numel() + rd.numel() + lens) + 32 * case["m"], "flops": lens}
    if kind == "matrix":
        n = case["n"]
        k, t = _count_complex(x["dist"].long(), x["thr"])
        return {"bytes": 2 * n * n + 16 * k + 8 * t, "flops": n * n}
    clouds = list(zip(x["pts"], x["thr"])) if kind == "batch" else [(x["pts"], x["thr"])]
    b = f = 0
    for p, thr in clouds:
        n, d = p.shape
        f += 3 * d * n * (n - 1) // 2
        b += p.numel() * p.element_size()
        k, t = _count_complex(_sqdist(p), thr)
        if kind == "pairs":  # a partner for each point and edge (with tetrahedra, each triangle)
            b += 4 * n + 8 * k + (8 * t if case["maxdim"] == 3 else 0)
            continue
        b += 16 * k + 8 * t
    return {"bytes": b, "flops": f}
