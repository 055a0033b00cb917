"""The ordered-round engine's rule, checked on the CPU: sorted by (D, i, j),
the pairs whose distance is below every row's second smallest entry (less the
rounding margin) are the next merges of the sequential loop, also when the
second entries are only lower bounds.  A plain model of the rule, with its own
fp32 updates, gives the oracle's merge list byte for byte."""
import numpy as np
import pytest

import oracle
import synth

F = np.float32


def _update(link, x, y, h, ni, nj, nk):
    if link == "average":
        return F(float(ni) / (ni + nj)) * x + F(float(nj) / (ni + nj)) * y
    if link == "weighted":
        return F(0.5) * x + F(0.5) * y
    t = (ni + nj + nk).astype(np.float64)
    wi, wj, wb = ((ni + nk) / t).astype(F), ((nj + nk) / t).astype(F), (-nk / t).astype(F)
    return (wi * x + wj * y) + wb * F(h)


def _model(d, link, bounds):
    """Merge records by ordered rounds.  bounds: second entries whose column
    merges are kept as lower bounds instead of being recomputed."""
    n = d.shape[0]
    d = np.triu(d, 1)
    d = d + d.T
    np.fill_diagonal(d, np.inf)
    live, size = np.ones(n, bool), np.ones(n, np.int64)
    out, largest = [], 0
    bound = np.full(n, np.inf, F)  # of rows not recomputed
    lazy = np.zeros(n, bool)
    while len(out) < n - 1:
        order = np.argsort(d, axis=1, kind="stable")
        near = order[:, 0]
        m1 = d[np.arange(n), near]
        m2 = np.where(lazy, np.minimum(bound, d[np.arange(n), order[:, 1]]), d[np.arange(n), order[:, 1]])
        T = m2[live].min()
        lim = F(T * F(1 - 2.0 ** -18)) if T >= 2.0 ** -100 else F(-np.inf)
        take = [(m1[a], a, int(near[a])) for a in np.nonzero(live)[0] if a < near[a] and m1[a] < lim]
        if not take:
            a = min(np.nonzero(live)[0], key=lambda q: (m1[q], min(q, near[q]), max(q, near[q])))
            take = [(m1[a], min(a, int(near[a])), max(a, int(near[a])))]
        take.sort()
        members = {q for _, i, j in take for q in (i, j)}
        assert len(members) == 2 * len(take)  # reciprocal pairs: disjoint
        if bounds:
            hit = live & np.isin(order[:, 1], list(members)) & ~np.isin(near, list(members))
            bound = np.where(hit, np.where(lazy, np.minimum(bound, m2), m2), bound)
            lazy = (lazy | hit) & ~np.isin(near, list(members))
        largest = max(largest, len(take))
        for h, i, j in take:
            assert d[i, j] == h
            out.append((i, j, h, size[i] + size[j]))
            k = np.nonzero(live)[0]
            k = k[(k != i) & (k != j)]
            v = _update(link, d[k, i], d[k, j], h, size[i], size[j], size[k]).astype(F)
            v[v == 0] = 0
            d[i, k] = d[k, i] = v
            live[j] = False
            d[j, :] = d[:, j] = np.inf
            size[i] += size[j]
            lazy[i] = False
            bound = np.where(lazy & live, np.minimum(bound, d[:, i]), np.where(lazy, bound, np.inf))
    return np.array(out, dtype=[("i", "<i4"), ("j", "<i4"), ("h", "<f4"), ("size", "<i4")]), largest


@pytest.mark.parametrize("link", ["average", "weighted", "ward"])
@pytest.mark.parametrize("bounds", [False, True])
def test_rounds_of_ordered_merges_give_the_sequential_list(link, bounds):
    for name, d in (("mixture", synth.mixture_8192(seed=1, n=150)), ("rmsd_like", synth.rmsd_like(seed=2, n=150)),
                    ("quantized", synth.quantized_matrix(90, 3, levels=4)), ("uniform", synth.uniform_matrix(120, 4))):
        got, largest = _model(d, link, bounds)
        assert got.tobytes() == oracle.run_f32(d, link).tobytes(), name
        if name == "mixture" and not bounds:
            assert largest > 3
