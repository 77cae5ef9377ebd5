"""CPU check of the rule by which the bounded general kernel leaves sources out: with hi and lo
the largest and least R[i][.] over a set of targets, a source with fl(C[i] + lo[i]) >
min_i fl(C[i] + hi[i]) is neither the minimum of any of them nor its lowest index.  Also counts
how many sources stay per 64-row tile, the figures that the kernel's thresholds go by."""
import numpy as np
import pytest

from paper_2504_21411_amd.workloads import random_tables

INF = np.float32(np.inf)


def _fronts(T, O, R, r_index, E, group):
    """Per front: mean number of sources that a 64-row tile lists, after checking the rule against
    the scan of all sources for every row.  group: targets that share a bound (None: all)."""
    L, S = T.shape
    e = np.arange(E + 1)
    low = np.cumsum(O.min(1))
    top = np.cumsum(O.min(1)[::-1])[::-1]
    C = np.where(e[None] >= O[0][:, None], T[0][:, None], INF).astype(np.float32)
    out = []
    for l in range(1, L):
        Rk = R[r_index[l]]
        idle = (e < low[l - 1]) | (e > E - top[l])
        counts = []
        best = np.empty((S, E + 1), np.float32)
        for j0 in range(0, S, group or S):
            js = np.arange(j0, min(S, j0 + (group or S)))
            bound = (C + Rk[:, js].max(1)[:, None]).min(0)
            listed = C + Rk[:, js].min(1)[:, None] <= bound[None]
            for j in js:
                sums = C + Rk[:, j][:, None]
                best[j] = sums.min(0)
                some = np.where(listed, sums, INF)
                assert np.array_equal(some.min(0), best[j])
                full = np.isfinite(best[j])  # (index 0 is the rule where nothing is finite)
                assert np.array_equal(some.argmin(0)[full], sums.argmin(0)[full])
            listed &= ~idle[None]
            counts += [listed[:, t:t + 64].any(1).sum() for t in range(0, E + 1, 64)
                       if t <= E - top[l] and t + 64 > low[l - 1]]
        out.append(np.mean(counts) if counts else 0.0)
        nxt = np.full_like(C, INF)
        for j in range(S):
            o = O[l][j]
            if o <= E:
                nxt[j, o:] = best[j, :E + 1 - o] + T[l][j]
        C = nxt
    return out


@pytest.mark.parametrize("S,group", [(30, None), (44, None), (96, None), (130, 16)])
@pytest.mark.parametrize("kind", ["cheap", "even", "dear", "ties", "forbidden", "subnormal", "huge"])
def test_left_out_sources_never_win(S, group, kind):
    w = random_tables(f"{kind}{S}", 1, 5, S, 260, K=2, seed=S)
    T, O, R = w.T[0], w.O[0], w.R
    g = np.random.RandomState(S)
    if kind in ("cheap", "dear"):
        R = R * np.float32(0.25 if kind == "cheap" else 20.0)
    elif kind == "ties":
        T, R = np.ceil(T), np.floor(R)
    elif kind == "forbidden":
        R = np.where(g.rand(*R.shape) < 0.3, INF, R)
    elif kind == "subnormal":
        tiny = np.float32(2.0 ** -149)
        T, R = g.randint(0, 1 << 20, T.shape) * tiny, g.randint(0, 200, R.shape) * tiny
    elif kind == "huge":
        T, R = T * np.float32(2e37), R * np.float32(1e36)
    with np.errstate(over="ignore"):
        left = _fronts(T.astype(np.float32), O, R.astype(np.float32), w.r_index[0], 260, group)
    if kind == "forbidden" and group is None:  # every source has a forbidden target somewhere
        assert min(left) > 0.6 * S             # (less the ones with no finite cost yet)
    if kind == "cheap":
        assert max(left) < 0.25 * S


@pytest.mark.parametrize("S,group,r,lo,hi", [(44, None, 1.0, 3, 8), (44, None, 2.0, 5, 13),
                                             (44, None, 4.0, 11, 24), (96, None, 1.0, 7, 14),
                                             (96, None, 2.0, 13, 26), (96, None, 4.0, 28, 46),
                                             (242, 16, 1.0, 13, 26), (242, 16, 2.0, 28, 48)])
def test_sources_left_by_cost_ratio(S, group, r, lo, hi):
    """Layer times of 1 to 10, transition costs of up to r: mean number of sources left per tile
    over six fronts (three with bounds per wave)."""
    L = 7 if group is None else 4
    w = random_tables(f"left{S}", 1, L, S, 500, seed=S, o_hi=83)
    left = _fronts(w.T[0], w.O[0], (w.R * np.float32(r / 2.0)).astype(np.float32), w.r_index[0],
                   500, group)
    assert lo <= np.mean(left) <= hi, left
