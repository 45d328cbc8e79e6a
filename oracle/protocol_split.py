"""Step-level models of two protocols in which many workgroups act as one
endpoint, with the exhaustive explorer of ``protocol_kernels``.

TEST INFRASTRUCTURE ONLY (paper Sec. 4.3, the Channels frontend; Sec. 5, Test
Case 1).  Explored under sequential consistency, like the models beside it.

* ``explore_split`` -- a ring with one producer whose two ends are each split
  over A teams of B members.  Messages are cut into groups (at most `most` of
  them and `lim` bytes, unless the first is larger); group g belongs to team
  g mod A of either end, and the members of a team move a share of its bytes
  each; a member without a share leaves the group alone.  A producer member
  waits for room only, a consumer member for the group's publication only.  The
  first member of a team writes the entries, waits for the words in which the
  others tell of their shares, then for the groups before, and publishes the
  group (or releases its room, both counters in one unit).  The first producer
  member also tells where the ring's byte counter stood.
* ``explore_tree`` -- ping-pong between two groups of W members, in which a
  stripe is counted in a counter of its G neighbours, the last of them counts
  the neighbourhood in the channel's counter, and who completes that raises
  the flag of every waiting member, one by one; a member polls its own flags.

Checked in every reachable state: no read of a byte, entry or stripe that does
not hold the expected message, no overwrite of one not yet read, entry and byte
capacity, order of publication, and no deadlock while work remains.  ``Bug``
flags plant one mistake each.
"""
from dataclasses import dataclass

from .protocol_kernels import Violation, _dfs, _set


@dataclass(frozen=True)
class Bug:
    publish_without_others: bool = False   # split: the first member does not wait for the shares
    release_without_others: bool = False   # split: the same at the consumer
    publish_out_of_turn: bool = False      # split: not after the groups before
    release_out_of_turn: bool = False
    waits_without_share: bool = False      # split: a member waits for groups it has no share of
    entries_only: bool = False             # split: room is checked in entries, not in bytes
    stale_base: bool = False               # split: the byte counter is told after publication
    flags_by_neighbours: bool = False      # tree: a complete neighbourhood raises the flags
    count_before_copy: bool = False        # tree: a stripe is counted before it is copied


def groups_of(sizes, E, most, lim):
    """[(first message, end message)], as every member cuts them."""
    out, m = [], 0
    while m < len(sizes):
        e, b = m + 1, sizes[m]
        while e < len(sizes) and e - m < min(most, E) and b + sizes[e] <= lim:
            b += sizes[e]
            e += 1
        out.append((m, e))
        m = e
    return out


def explore_split(P, E, sizes, A, B, most, lim, base_b=0, bug=Bug(), max_states=3_000_000):
    """One stream of messages ``sizes`` through a ring of P bytes and E entries
    whose byte counter stands at base_b.  Returns the number of states."""
    n = len(sizes)
    offs = [sum(sizes[:i]) for i in range(n + 1)]
    groups = groups_of(sizes, E, most, lim)
    NG = len(groups)

    def share(g, b):
        """Stream bytes [lo, hi) of group g that member b moves; None: no share."""
        lo, hi = offs[groups[g][0]], offs[groups[g][1]]
        part = max(1, -(-(hi - lo) // B))
        if b and b * part >= hi - lo:
            return None
        return min(lo + b * part, hi), min(lo + (b + 1) * part, hi)

    def sharers(g):
        return [b for b in range(1, B) if share(g, b) is not None]

    def first_group(g, b, end):
        """The member's next group from g on."""
        while g < NG and share(g, b) is None and not (bug.waits_without_share and end == 0):
            g += A
        return g

    marker = {}
    for m in range(n):
        for k in range(sizes[m]):
            marker[offs[m] + k] = (m, k)

    # shared: cells, ents, tm, hm, hb, base word (0: not told), words of either
    # end ([team][member] -> groups finished), read markers
    # member: (phase, group, byte, hm_seen)
    sh0 = (tuple([None] * P), tuple([None] * E), 0, 0, base_b, 0,
           tuple([0] * (A * B)), tuple([0] * (A * B)), frozenset())
    NAMES = ("cells", "ents", "tm", "hm", "hb", "base", "pw", "cw", "rset")
    prods = tuple(("base", first_group(t // B, t % B, 0), 0, 0) for t in range(A * B))
    cons = tuple(("wait", first_group(t // B, t % B, 1), 0) for t in range(A * B))
    start = (sh0, prods, cons)

    def succ(st):
        sh, prs, cos = st
        cells, ents, tm, hm, hb, base, pw, cw, rset = sh

        def SH(**kw):
            v = list(sh)
            for a, x in kw.items():
                v[NAMES.index(a)] = x
            return tuple(v)

        for t in range(A * B):
            ph, g, at, seen = prs[t]
            b = t % B

            def PR(ph, g=g, at=at, seen=seen):
                return _set(prs, t, (ph, g, at, seen))

            def after(g):
                ng = first_group(g + A, b, 0)
                return PR("rd_hm" if ng < NG else "end", ng, 0)

            if ph == "base":
                if t == 0 and not bug.stale_base:
                    yield SH(base=hb + 1), PR("rd_hm" if g < NG else "end"), cos
                elif base or bug.stale_base:
                    yield sh, PR("rd_hm" if g < NG else "end"), cos
                continue
            if ph == "end":
                continue
            m0, m1 = groups[g]
            mine = share(g, b)
            if ph == "rd_hm":
                yield sh, PR("rd_hb", seen=hm), cos
            elif ph == "rd_hb":
                # (differences are unsigned: a group already released looks as
                # if it had no room ever)
                fits = 0 <= m1 - seen <= E and (bug.entries_only or base_b + offs[m1] - hb <= P)
                if fits and mine is None:
                    yield sh, after(g), cos
                elif fits:
                    yield sh, PR("ents" if b == 0 else "pay", at=mine[0]), cos
                elif hm != seen:
                    yield sh, PR("rd_hm"), cos
            elif ph == "ents":
                ne = ents
                for m in range(m0, m1):
                    ne = _set(ne, m % E, m)
                yield SH(ents=ne), PR("pay"), cos
            elif ph == "pay":
                if at < mine[1]:
                    pos = (base_b + at) % P
                    if cells[pos] is not None and cells[pos] not in rset:
                        raise Violation(f"producer overwrote unread byte {cells[pos]}")
                    yield SH(cells=_set(cells, pos, marker[at])), PR("pay", at=at + 1), cos
                elif b:
                    yield SH(pw=_set(pw, t, g + 1)), after(g), cos
                else:
                    yield sh, PR("gather"), cos
            elif ph == "gather":
                if bug.publish_without_others or all(pw[t + k] > g for k in sharers(g)):
                    yield sh, PR("turn"), cos
            elif ph == "turn":
                if tm == m0 or bug.publish_out_of_turn:
                    yield SH(tm=m1), after(g), cos
        for t in range(A * B):
            ph, g, at = cos[t]
            b = t % B

            def CO(ph, g=g, at=at):
                return _set(cos, t, (ph, g, at))

            if g >= NG:
                continue
            m0, m1 = groups[g]
            mine = share(g, b)
            if ph == "wait":
                if tm >= m1:
                    yield sh, prs, CO("ents", at=mine[0])
            elif ph == "ents":
                if not base:
                    raise Violation("the ring's byte counter is not known yet")
                for m in range(m0, m1):
                    if ents[m % E] != m:
                        raise Violation(f"consumer read entry {ents[m % E]} for message {m}")
                yield sh, prs, CO("pay")
            elif ph == "pay":
                if at < mine[1]:
                    pos = (base - 1 + at) % P
                    if cells[pos] != marker[at]:
                        raise Violation(f"consumer read {cells[pos]} expecting {marker[at]}")
                    yield SH(rset=rset | {marker[at]}), prs, CO("pay", at=at + 1)
                elif b:
                    yield SH(cw=_set(cw, t, g + 1)), prs, CO("wait", first_group(g + A, b, 1))
                else:
                    yield sh, prs, CO("gather")
            elif ph == "gather":
                if bug.release_without_others or all(cw[t + k] > g for k in sharers(g)):
                    yield sh, prs, CO("turn")
            elif ph == "turn":
                if hm == m0 or bug.release_out_of_turn:
                    yield SH(hm=m1, hb=base - 1 + offs[m1]), prs, \
                        CO("wait", first_group(g + A, b, 1))

    def done(st):
        sh, prs, cos = st
        return sh[3] == n and len(sh[8]) == offs[n] and \
            all(p[0] == "end" for p in prs) and all(c[1] >= NG for c in cos)

    def checked(st):
        sh = st[0]
        tm, hm, hb = sh[2], sh[3], sh[4]
        if not 0 <= tm - hm <= E or base_b + offs[tm] - hb > P:
            raise Violation("capacity exceeded")
        return succ(st)

    return _dfs(start, checked, done, max_states)


def explore_tree(W, G, reps, bug=Bug(), max_states=3_000_000):
    """Ping-pong of ``reps`` messages; members i of [jG, jG + G) are
    neighbours.  Channels' counters: A arrived, A freed, B arrived, B freed.
    Returns the number of states."""
    NGR = -(-W // G)
    size = [min(G, W - j * G) for j in range(NGR)]

    # shared: rings A and B, buffer, neighbourhood counters [4][NGR], channel
    # counters [4], flags [4][W] (of the end that waits for the counter), read
    # stripes of A and of B
    # member: (k, step, j): j counts the flags it has raised
    start = (tuple([None] * W), tuple([None] * W), tuple([None] * W),
             tuple(tuple([0] * NGR) for _ in range(4)), (0,) * 4,
             tuple(tuple([0] * W) for _ in range(4)),
             tuple((0, 0, 0) for _ in range(W)), tuple((0, 0, 0) for _ in range(W)),
             frozenset(), frozenset())
    # an end's round: wait for counter c to show k + x messages; copy; count c
    PING = [("wait", 1, 0), ("put", 0), ("count", 0), ("wait", 2, 1), ("get", 1), ("count", 3)]
    PONG = [("wait", 0, 1), ("get", 0), ("count", 1), ("wait", 3, 0), ("put", 1), ("count", 2)]

    def program(steps):
        out = []
        for i, s in enumerate(steps):
            if s[0] == "count":
                out += [("nb", s[1]), ("ch", s[1]), ("raise", s[1])]
            else:
                out.append(s)
        if bug.count_before_copy:
            out = [x for s in range(0, len(out), 5) for x in
                   [out[s], out[s + 2], out[s + 3], out[s + 4], out[s + 1]]]
        return out

    progs = (program(PING), program(PONG))

    def succ(st):
        A, Bq, buf, nb, ch, fl, pi, po, rA, rB = st
        rings = (A, Bq)
        rsets = (rA, rB)
        for end in (0, 1):
            for i in range(W):
                k, s, j = (pi, po)[end][i]
                if k == reps:
                    continue
                prog = progs[end]

                def step(ns, nj=0, rings=rings, buf=buf, nb=nb, ch=ch, fl=fl, rsets=rsets):
                    nk = k
                    if ns == len(prog):
                        nk, ns = k + 1, 0
                    mem = _set((pi, po)[end], i, (nk, ns, nj))
                    ends = (mem, po) if end == 0 else (pi, mem)
                    return (rings[0], rings[1], buf, nb, ch, fl, ends[0], ends[1], rsets[0],
                            rsets[1])

                op = prog[s]
                if op[0] == "wait":
                    if fl[op[1]][i] >= k + op[2]:
                        yield step(s + 1)
                elif op[0] == "put":
                    r = op[1]
                    old = rings[r][i]
                    if old is not None and old not in rsets[r]:
                        raise Violation(f"unread stripe {old} of ring {r} overwritten")
                    what = (k, i) if end == 0 else buf[i]
                    yield step(s + 1, rings=_set(rings, r, _set(rings[r], i, what)))
                elif op[0] == "get":
                    r = op[1]
                    if rings[r][i] != (k, i):
                        raise Violation(f"read {rings[r][i]} of ring {r} expecting {(k, i)}")
                    yield step(s + 1, rsets=_set(rsets, r, rsets[r] | {(k, i)}),
                               buf=_set(buf, i, (k, i)) if end else buf)
                elif op[0] == "nb":
                    c, q = op[1], i // G
                    v = nb[c][q] + 1
                    last = v == (k + 1) * size[q]
                    if last and bug.flags_by_neighbours:
                        yield step(s + 2, nb=_set(nb, c, _set(nb[c], q, v)))
                    else:
                        yield step(s + 1 if last else s + 3, nb=_set(nb, c, _set(nb[c], q, v)))
                elif op[0] == "ch":
                    c = op[1]
                    v = ch[c] + 1
                    yield step(s + 1 if v == (k + 1) * NGR else s + 2, ch=_set(ch, c, v))
                elif op[0] == "raise":
                    c = op[1]
                    yield step(s if j + 1 < W else s + 1, j + 1 if j + 1 < W else 0,
                               fl=_set(fl, c, _set(fl[c], j, k + 1)))

    def done(st):
        return all(m[0] == reps for m in st[6]) and all(m[0] == reps for m in st[7])

    return _dfs(start, succ, done, max_states)
