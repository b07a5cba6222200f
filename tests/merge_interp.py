"""A plain interpreter of the merge program, one scenario at a time."""
import numpy as np

VISIT, MAX, RELEASE, LOAD, FORCE, DRAIN = range(6)
INF = 1 << 62


def interpret(program, n_res, dur, gap=None, delay=None):
    """Finish time of every op (by row) for one duration column, and the
    number of deferred ops each instruction ran."""
    head, ins, defs, chains = program
    slots, zero = int(head[3]), int(head[5])
    S = [0] * slots
    at = [int(c[0]) for c in chains]
    ends = [int(c[0]) for c in chains[1:]] + [len(defs)]
    ready = [INF] * len(defs)
    d_of = [None] * len(defs)
    fin = np.full(len(dur), -1, np.int64)
    ran = []
    gap = [0] * n_res if gap is None else gap
    delay = [0] * n_res if delay is None else delay
    defs = defs.tolist()

    def first(c0, c1):
        return min(((ready[at[c]], defs[at[c]][1], c) for c in range(c0, c1) if at[c] < ends[c]), default=(INF, 0, -1))

    def commit(row, r, t, d):
        assert fin[row] < 0
        f = max(t, S[r]) + d
        fin[row] = f
        S[r] = f + int(gap[r])
        return f + int(delay[r])

    def go(c):
        x = at[c]
        row, _, _, y = defs[x]
        ready[x] = commit(row, int(chains[c][1]), ready[x], d_of[x])  # its arrival from now on
        at[c] = x + 1
        if y >= 0:
            assert ready[y] == INF and d_of[y] is not None
            ready[y] = ready[x]

    for kind, row, r, out, p0, p1, p2, p3, c0, c1, x, vid, nxt in ins.tolist():
        assert S[zero] == 0
        t = S[r] if nxt else max(S[p0], S[p1], S[p2], S[p3])
        k = 0
        if kind == VISIT:
            while first(c0, c1)[:2] < (t, vid):
                go(first(c0, c1)[2])
                k += 1
            S[out] = commit(row, r, t, int(dur[row]))
        elif kind == MAX:
            S[out] = t
        elif kind == RELEASE:
            assert ready[x] == INF
            ready[x], d_of[x] = t, int(dur[row])
        elif kind == LOAD:
            d_of[x] = int(dur[row])
        elif kind == FORCE:
            while at[defs[x][2]] <= x:
                go(first(c0, c1)[2])
                k += 1
            S[out] = ready[x]
        else:
            while first(c0, c1)[0] < INF:
                go(first(c0, c1)[2])
                k += 1
        ran.append(k)
    return fin, ran
