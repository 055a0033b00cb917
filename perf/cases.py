"""The work that users of the clustering library have it do, as measurable cases.

Each case is one call (or one short sequence of calls) through the package's
public entry points: Context.run, Context.batch, Context.rmsd and Server.
Input matrices are made on the GPU from the seed alone, with the workloads'
distributions: Gaussian mixtures, RMSD-like matrices (anisotropic clusters,
scaled to [0, 20] and rounded to 1e-3, so with many exact ties) and chain
conformations.  Ward and centroid linkage get squared distances, for which
Table 1 gives their usual meaning.

A program that clusters more than one matrix keeps one context (and one
server), so these are made once per process.  Inputs are preserved
(`preserve=True`) where a pass starts from a given matrix; the pipeline case
clusters in place the matrix that its first half has just produced.
"""
import math
import time

import numpy as np
import torch

import paper_1709_06816_amd as hac

DIMS = 16
MAX_SERVED = 4096
_kept = {}


def _context():
    if "ctx" not in _kept:
        _kept["ctx"] = hac.Context(0)
    return _kept["ctx"]


def _server():
    if "srv" not in _kept:
        _kept["srv"] = hac.Server(_context(), budget_bytes=4 << 30, max_jobs=1024, max_n=MAX_SERVED)
    return _kept["srv"]


# ---------------------------------------------------------------------------
# The cases
# ---------------------------------------------------------------------------

def listed():
    return [
        # The smallest calls: one matrix of a few dozen items, where launches
        # and the dependent chain of merges count.
        {"name": "run_100_average", "kind": "run", "n": 100, "linkage": "average", "data": "mixture"},
        # The n=512 workload: one workgroup.
        {"name": "run_512_complete", "kind": "run", "n": 512, "linkage": "complete", "data": "mixture"},
        # The paper's own setting: complete linkage of about 1968
        # conformations (Section 6), here an odd number of them.
        {"name": "run_1967_complete", "kind": "run", "n": 1967, "linkage": "complete", "data": "rmsd"},
        # Ward's criterion on an ordinary, ragged size.
        {"name": "run_3001_ward", "kind": "run", "n": 3001, "linkage": "ward", "data": "mixture"},
        # The n=8192 workload, single and average linkage.
        {"name": "run_8192_single", "kind": "run", "n": 8192, "linkage": "single", "data": "mixture"},
        {"name": "run_8192_average", "kind": "run", "n": 8192, "linkage": "average", "data": "mixture"},
        # The benchmark's dendrogram: n=32768 RMSD-like, complete linkage.
        {"name": "run_32768_complete", "kind": "run", "n": 32768, "linkage": "complete", "data": "rmsd"},
        # The largest instance the library takes: 16 GiB, average linkage.
        {"name": "run_65536_average", "kind": "run", "n": 65536, "linkage": "average", "data": "mixture"},
        # The whole path of the paper: conformations to RMSD matrix to
        # dendrogram, the matrix clustered in place.
        {"name": "pipeline_2500", "kind": "pipeline", "n": 2500, "atoms": 128, "linkage": "complete"},
        # The input producer at the benchmark's size.
        {"name": "rmsd_32768", "kind": "rmsd", "n": 32768, "atoms": 128},
        # The 1024-instance ragged batch, four linkages.
        {"name": "batch_1024", "kind": "batch", "count": 1024, "n_lo": 64, "n_hi": 4096, "sizes": 4},
        # A burst of requests to the server, from page-locked host memory.
        {"name": "serve_48", "kind": "serve", "count": 48, "n_lo": 256, "n_hi": 4096, "sizes": 5},
    ]


def _log_int(rng, lo, hi):
    return int(math.floor(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))


def draw(rng):
    kind = rng.choice(["run", "run", "run", "run", "run", "pipeline", "rmsd", "batch", "serve"])
    if kind == "run":
        n = _log_int(rng, 48, 24000)
        if n % 2 == 0 and rng.random() < 0.4:
            n += 1
        return {"kind": kind, "n": n, "linkage": rng.choice(sorted(hac.LINKAGES)),
                "data": rng.choice(["mixture", "rmsd"])}
    if kind == "pipeline":
        return {"kind": kind, "n": _log_int(rng, 64, 12000), "atoms": _log_int(rng, 10, 400),
                "linkage": rng.choice(sorted(hac.LINKAGES))}
    if kind == "rmsd":
        return {"kind": kind, "n": _log_int(rng, 200, 20000), "atoms": _log_int(rng, 4, 300)}
    if kind == "batch":
        lo = _log_int(rng, 16, 512)
        return {"kind": kind, "count": _log_int(rng, 4, 600), "n_lo": lo,
                "n_hi": _log_int(rng, 2 * lo, 4096), "sizes": rng.randrange(1 << 20)}
    return {"kind": kind, "count": rng.randrange(4, 48), "n_lo": 128, "n_hi": _log_int(rng, 512, MAX_SERVED),
            "sizes": rng.randrange(1 << 20)}


def _sizes(case):
    """Sizes and linkages of a batch or of a burst of requests: log-uniform,
    the four linkages in equal parts, fixed by the case (a program's next
    batch has the same shape and other matrices)."""
    rng = np.random.default_rng(170906816 * 100 + case["sizes"])
    ns = np.exp(rng.uniform(math.log(case["n_lo"]), math.log(case["n_hi"] + 1), size=case["count"]))
    ns = np.clip(np.floor(ns).astype(np.int64), case["n_lo"], case["n_hi"])
    links = rng.integers(0, 4, size=case["count"]).astype(np.int32)
    return ns, links


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------

def _points(n, seed, rmsd):
    """Points of a Gaussian mixture (float32, on the GPU): in R^16 with one
    sigma per cluster, or (RMSD-like) in R^30 with anisotropic clusters."""
    rng = np.random.default_rng(seed)
    dim = 30 if rmsd else DIMS
    k = 64 if rmsd else int(rng.integers(2, 33)) if n < 4096 else 32
    centres = rng.uniform(-10.0, 10.0, size=(k, dim))
    labels = rng.integers(0, k, size=n)
    z = rng.standard_normal((n, dim))
    if rmsd:
        pts = np.empty((n, dim))
        for c in range(k):
            q, r = np.linalg.qr(rng.standard_normal((dim, dim)))
            s = rng.uniform(0.3, 3.0, size=dim)
            at = labels == c
            pts[at] = centres[c] + (z[at] * s) @ (q * np.sign(np.diag(r))).T
    else:
        sigma = rng.uniform(0.5, 2.0, size=k) if n != 512 else np.ones(k)
        pts = centres[labels] + z * sigma[labels, None]
    return torch.from_numpy(pts.astype(np.float32)).cuda()


def _matrix(x, squared, rmsd, out=None):
    """Euclidean (or squared Euclidean) distances of the rows of x."""
    n, dim = x.shape
    d = torch.empty((n, n), dtype=torch.float32, device=x.device) if out is None else out
    rows = max(1, min(n, (1 << 28) // n))
    for a in range(0, n, rows):
        acc = torch.zeros((min(rows, n - a), n), dtype=torch.float32, device=x.device)
        for q in range(dim):
            t = x[a:a + rows, q, None] - x[None, :, q]
            acc.addcmul_(t, t)
        d[a:a + rows] = acc
    if not squared:
        d.sqrt_()
    if rmsd:
        d.mul_(20.0 / float(d.max()))
        if not squared:
            for a in range(0, n, rows):
                d[a:a + rows] = torch.round(d[a:a + rows].double() * 1000.0).div_(1000.0).float()
    return d


def _dist(n, linkage, data, seed, out=None):
    rmsd = data == "rmsd"
    return _matrix(_points(n, seed, rmsd), linkage in ("ward", "centroid"), rmsd, out)


def _conformations(n, atoms, seed):
    """n conformations of one chain (angstrom): a persistent random walk with
    3.8 A steps, 32 folding states (a smooth displacement each), noise per
    atom, and a random placement of each conformation."""
    rng = np.random.default_rng(seed)
    step = rng.standard_normal((atoms, 3))
    for i in range(1, atoms):
        step[i] += 0.6 * step[i - 1]
    base = np.cumsum(step * 3.8 / np.maximum(np.linalg.norm(step, axis=1, keepdims=True), 1e-12), axis=0)
    pos = np.arange(atoms, dtype=np.float64)[:, None]
    fields = np.zeros((32, atoms, 3))
    for c in range(32):
        for _ in range(3):
            way = rng.standard_normal(3)
            fields[c] += rng.uniform(1.0, 4.0) / 3.0 * np.sin(
                rng.uniform(0.01, 0.2) * pos + rng.uniform(0, 2 * np.pi, size=3)) * way / np.linalg.norm(way)
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)
    label = torch.from_numpy(rng.integers(0, 32, size=n)).to(dev)
    sigma = torch.from_numpy(rng.uniform(0.2, 1.0, size=n).astype(np.float32)).to(dev)
    x = torch.from_numpy((base - base.mean(0) + fields).astype(np.float32)).to(dev)[label]
    x = x + sigma[:, None, None] * torch.randn(x.shape, generator=gen, device=dev)
    q = rng.standard_normal((n, 4))
    w, a, b, c = (q / np.linalg.norm(q, axis=1, keepdims=True)).T
    rot = np.stack([1 - 2 * (b * b + c * c), 2 * (a * b - c * w), 2 * (a * c + b * w),
                    2 * (a * b + c * w), 1 - 2 * (a * a + c * c), 2 * (b * c - a * w),
                    2 * (a * c - b * w), 2 * (b * c + a * w), 1 - 2 * (a * a + b * b)], axis=1)
    rot = torch.from_numpy(rot.astype(np.float32)).to(dev).view(n, 1, 3, 3)
    x = (rot * x[:, :, None, :]).sum(-1)
    return (x + torch.from_numpy(rng.uniform(-50, 50, size=(n, 1, 3)).astype(np.float32)).to(dev)).contiguous()


def prepare(case, seed):
    kind = case["kind"]
    state = {"kind": kind, "ctx": _context()}
    if kind == "run":
        state["dist"] = _dist(case["n"], case["linkage"], case["data"], seed)
        state["linkage"] = case["linkage"]
    elif kind in ("rmsd", "pipeline"):
        n = case["n"]
        state["coords"] = _conformations(n, case["atoms"], seed)
        state["dist"] = torch.zeros((n, n), dtype=torch.float32, device="cuda")
        state["linkage"] = case.get("linkage")
    elif kind == "batch":
        ns, links = _sizes(case)
        offs = np.zeros(len(ns), np.int64)
        offs[1:] = np.cumsum((ns * ns + 63) // 64 * 64)[:-1]
        packed = torch.empty(int(offs[-1] + ns[-1] * ns[-1]), dtype=torch.float32, device="cuda")
        for k, n in enumerate(ns):
            n = int(n)
            view = packed[int(offs[k]):int(offs[k]) + n * n].view(n, n)
            _matrix(_points(n, seed * 4099 + k, False), links[k] == 3, False, view)
        state.update(packed=packed, offs=offs, ns=ns, links=[int(v) for v in links])
    else:
        ns, links = _sizes(case)
        # Requests are blocks of two page-locked matrices.
        pool = []
        for p in range(2):
            d = _dist(int(ns.max()), "average", "mixture", seed * 2 + p)
            h = torch.empty(d.shape, dtype=torch.float32, pin_memory=True)
            h.copy_(d)
            pool.append(h)
        torch.cuda.synchronize()
        state.update(jobs=[(pool[k % 2][:int(n), :int(n)], int(links[k])) for k, n in enumerate(ns)], srv=_server())
    return state


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------

def _records(rec):
    """The merge records (i, j, height, size) as plain arrays."""
    ints = rec.view(np.int32).reshape(-1, 4)
    return {"pairs": ints[:, :2], "size": ints[:, 3], "height": rec["h"]}


def run(state):
    kind, ctx = state["kind"], state["ctx"]
    if kind == "run":
        return _records(ctx.run(state["dist"], state["linkage"], preserve=True))
    if kind == "rmsd":
        return ctx.rmsd(state["coords"], out=state["dist"])
    if kind == "pipeline":
        return _records(ctx.run(ctx.rmsd(state["coords"], out=state["dist"]), state["linkage"]))
    if kind == "batch":
        return _records(ctx.batch(state["packed"], state["offs"], state["ns"], state["links"], preserve=True))
    srv = state["srv"]
    tickets = [srv.submit(d, link) for d, link in state["jobs"]]
    got = [None] * len(tickets)
    left = list(range(len(tickets)))
    while left:
        for k in list(left):
            got[k] = srv.poll(tickets[k])
            if got[k] is not None:
                left.remove(k)
        if left:
            time.sleep(0.0002)
    return _records(np.concatenate(got))


# ---------------------------------------------------------------------------
# What a pass cannot do without, and what it should return
# ---------------------------------------------------------------------------

_FLOPS = {"single": 1, "complete": 1, "average": 3, "weighted": 3, "centroid": 5, "ward": 11,
          0: 1, 1: 1, 2: 3, 3: 11}


def _cluster_work(n, linkage):
    # The strict upper triangle read once, a record per merge written; one
    # Table 1 update per live cluster and merge.
    return 2.0 * n * (n - 1) + 16.0 * (n - 1), _FLOPS[linkage] * 0.5 * n * n


def work(case):
    kind = case["kind"]
    if kind == "run":
        b, f = _cluster_work(case["n"], case["linkage"])
    elif kind in ("rmsd", "pipeline"):
        n, m = case["n"], case["atoms"]
        b, f = 12.0 * n * m + 2.0 * n * (n + 1), 9.0 * m * n * (n - 1)
        if kind == "pipeline":
            # The matrix in between need not reach memory, the records do.
            b, f = 12.0 * n * m + 16.0 * (n - 1), f + _cluster_work(n, case["linkage"])[1]
    else:
        b = f = 0.0
        for n, link in zip(*_sizes(case)):
            x, y = _cluster_work(int(n), int(link))
            b, f = b + x, f + y
    return {"bytes": b, "flops": f}


def _heights64(d, linkage):
    """Merge heights in 64 bits: the closest pair merged n-1 times, cached
    row minima over the symmetric matrix."""
    n = d.shape[0]
    d = np.triu(d.astype(np.float64), 1)
    d += d.T
    np.fill_diagonal(d, np.inf)
    size = np.ones(n)
    near = d.argmin(1)
    best = d[np.arange(n), near]
    live = np.ones(n, bool)
    out = np.empty(n - 1)
    for s in range(n - 1):
        i = int(best.argmin())
        j = int(near[i])
        i, j = min(i, j), max(i, j)
        h, ni, nj = d[i, j], size[i], size[j]
        out[s] = h
        x, y = d[i], d[j]
        if linkage == "single":
            v = np.minimum(x, y)
        elif linkage == "complete":
            v = np.maximum(x, y)
        elif linkage == "average":
            v = (ni * x + nj * y) / (ni + nj)
        elif linkage == "weighted":
            v = 0.5 * x + 0.5 * y
        elif linkage == "centroid":
            v = (ni * x + nj * y) / (ni + nj) - ni * nj / (ni + nj) ** 2 * h
        else:
            v = ((ni + size) * x + (nj + size) * y - size * h) / (ni + nj + size)
        live[j] = False
        v[~live] = np.inf
        v[i] = np.inf
        d[i] = v
        d[:, i] = v
        d[:, j] = np.inf
        size[i] += nj
        best[j] = np.inf
        again = live & ((near == i) | (near == j))
        again[i] = True
        lower = live & (v < best) & ~again
        near[lower] = i
        best[lower] = v[lower]
        at = np.nonzero(again)[0]
        rows = d[at]
        near[at] = rows.argmin(1)
        best[at] = rows[np.arange(len(at)), near[at]]
    return out


def _rmsd64(x):
    """Superposed RMSD of every pair in 64 bits: the largest eigenvalue of
    the 4 x 4 quaternion matrix by Newton's method on its characteristic
    polynomial, from the upper bound (G_a + G_b) / 2."""
    n, m, _ = x.shape
    x = x.double()
    x = x - x.mean(1, keepdim=True)
    g = x.square().sum((1, 2))
    planes = [x[:, :, p].contiguous() for p in range(3)]
    out = torch.zeros((n, n), dtype=torch.float64, device=x.device)
    rows = max(1, min(n, (1 << 25) // n))
    for a in range(0, n, rows):
        c = [[planes[p][a:a + rows] @ planes[q].t() for q in range(3)] for p in range(3)]
        (xx, xy, xz), (yx, yy, yz), (zx, zy, zz) = c
        k = [[xx + yy + zz, yz - zy, zx - xz, xy - yx], [None, xx - yy - zz, xy + yx, zx + xz],
             [None, None, -xx + yy - zz, yz + zy], [None, None, None, -xx - yy + zz]]
        for p in range(4):
            for q in range(p):
                k[p][q] = k[q][p]

        def minor(r, p, q):
            return k[r][p] * k[r + 1][q] - k[r][q] * k[r + 1][p]

        c0 = (minor(0, 0, 1) * minor(2, 2, 3) - minor(0, 0, 2) * minor(2, 1, 3) + minor(0, 0, 3) * minor(2, 1, 2) +
              minor(0, 1, 2) * minor(2, 0, 3) - minor(0, 1, 3) * minor(2, 0, 2) + minor(0, 2, 3) * minor(2, 0, 1))
        c1 = -8.0 * (xx * (yy * zz - yz * zy) - xy * (yx * zz - yz * zx) + xz * (yx * zy - yy * zx))
        c2 = -2.0 * (xx * xx + xy * xy + xz * xz + yx * yx + yy * yy + yz * yz + zx * zx + zy * zy + zz * zz)
        del k
        lam = 0.5 * (g[a:a + rows, None] + g[None, :])
        total = lam * 2.0
        for _ in range(40):
            sq = lam * lam
            slope = (4.0 * sq + 2.0 * c2) * lam + c1
            delta = ((sq + c2) * sq + c1 * lam + c0) / slope
            lam = torch.where(slope > 0, lam - delta, lam)
        out[a:a + rows] = ((total - 2.0 * lam).clamp_min_(0.0) / m).sqrt_()
    return out.triu_(1)


def exact(case, seed):
    kind, n = case["kind"], case.get("n", 0)
    if kind == "run" and n <= 8192:
        d = _dist(n, case["linkage"], case["data"], seed).cpu().numpy()
        return {"pairs": None, "size": None, "height": _heights64(d, case["linkage"])}
    if kind == "rmsd":
        return _rmsd64(_conformations(n, case["atoms"], seed))
    if kind == "pipeline" and n <= 8192:
        d = _rmsd64(_conformations(n, case["atoms"], seed)).cpu().numpy()
        return {"pairs": None, "size": None, "height": _heights64(d, case["linkage"])}
    return None
