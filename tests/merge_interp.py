"""A plain interpreter of the merge program, one scenario at a time, with the
state that the kernel keeps: of each deferred chain its first waiting op's
ready time, duration and partner's duration, and how many of its ops have been
released and have run; ops released while others of their chain wait queue up
by their deferred index."""
import numpy as np

VISIT, MAX, RELEASE, LOAD, FORCE, DRAIN = range(6)
INF = 1 << 62


def interpret(program, n_res, dur, gap=None, delay=None):
    """Finish time of every op (by row) for one duration column, and the
    number of deferred ops each instruction ran."""
    head, ins, defs, chains = program
    slots, zero = int(head[3]), int(head[5])
    S = [0] * slots
    defs, chains = defs.tolist(), chains.tolist()
    ends = [c[0] for c in chains[1:]] + [len(defs)]
    at, rel = [0] * len(chains), [0] * len(chains)
    first, first_dur, first_aux = ([INF] * len(chains) for _ in range(3))
    queue, queue_dur = [None] * len(defs), [None] * len(defs)
    arrival = [None] * len(defs)
    aux = None  # the duration a load has handed over for the next release
    fin = np.full(len(dur), -1, np.int64)
    ran = []
    gap = [0] * n_res if gap is None else gap
    delay = [0] * n_res if delay is None else delay

    def smallest(c0, c1):
        return min(((first[c], defs[chains[c][0] + at[c]][1], c) for c in range(c0, c1) if first[c] < INF),
                   default=(INF, 0, -1))

    def commit(row, r, t, d):
        assert fin[row] < 0
        f = max(t, S[r]) + d
        fin[row] = f
        S[r] = f + int(gap[r])
        return f + int(delay[r])

    def go(c):
        beg, r, follow, lead = chains[c]
        pos = at[c]
        x = beg + pos
        assert x < ends[c]
        arrival[x] = commit(defs[x][0], r, first[c], first_dur[c])
        at[c] = pos + 1
        if follow >= 0:  # the op at the same place of the following chain is ready
            y = chains[follow][0] + pos
            assert y < ends[follow]
            if at[follow] == pos:
                first[follow], first_dur[follow] = arrival[x], first_aux[c]
            else:
                queue[y], queue_dur[y] = arrival[x], first_aux[c]
        first[c] = INF
        if pos + 1 < (at[lead] if lead >= 0 else rel[c]):
            first[c], first_dur[c] = queue[x + 1], queue_dur[x + 1]
            assert first[c] is not None
            if follow >= 0:
                first_aux[c] = queue_dur[chains[follow][0] + pos + 1]

    for kind, row, r, out, p0, p1, p2, p3, c0, c1, x, vid, nxt in ins.tolist():
        assert S[zero] == 0
        t = S[r] if nxt else max(S[p0], S[p1], S[p2], S[p3])
        k = 0
        assert aux is None or kind == RELEASE, "a load stands right before its release"
        if kind == VISIT:
            while smallest(c0, c1)[:2] < (t, vid):
                go(smallest(c0, c1)[2])
                k += 1
            S[out] = commit(row, r, t, int(dur[row]))
        elif kind == MAX:
            S[out] = t
        elif kind == RELEASE:
            c = defs[x][2]
            beg, _, follow, lead = chains[c]
            place = x - beg
            assert lead < 0, "an op of a following chain is released by its leader only"
            assert (aux is not None) == (follow >= 0), "every op of a leading chain has a partner"
            assert rel[c] == place, "a chain's ops are released in its order"
            rel[c] = place + 1
            if at[c] == place:
                first[c], first_dur[c], first_aux[c] = t, int(dur[row]), aux
            else:
                queue[x], queue_dur[x] = t, int(dur[row])
                if follow >= 0:
                    queue_dur[chains[follow][0] + place] = aux
            aux = None
        elif kind == LOAD:
            aux = int(dur[row])
        elif kind == FORCE:
            while at[defs[x][2]] <= x - chains[defs[x][2]][0]:
                go(smallest(c0, c1)[2])
                k += 1
            S[out] = arrival[x]
        else:
            while smallest(c0, c1)[0] < INF:
                go(smallest(c0, c1)[2])
                k += 1
        ran.append(k)
    return fin, ran
