"""The notification rule of in-place sweeps (AND) with support counting.
CPU only.

In place, a member of an s-clique may read another's value before or after it
fell in the same sweep.  An r-clique R' that keeps its value c' may go on
counting an s-clique S only while somebody tells it when S falls below c': of
the members of S that fall in one sweep at least one has to notify R'.  Lists
kept by a wave or a lane notify from the values their update gathered, before
their own write; a workgroup's list gathers again, ahead of its own write, with
the same test.  Both are modelled here step by step, next to the order in which
a workgroup writes first and then tests h <= tau(Q): sound where every member
does so, unsound beside the other lists.
"""
import itertools
import random

import pytest


def _tells(hub, early, h, told, first, now, c):
    """Does a faller (told -> h) notify R' (value c)?  first / now: the other
    fallers' values at its update and at its own notification."""
    if not hub:  # R' holds the minimum gathered by the update
        return h < c <= told and all(c <= v for v in first)
    if early:    # the same test on a gather ahead of the write
        return h < c <= told and all(c <= v for v in now)
    return h < c <= told and all(h <= v for v in now)


def _missed(k, hubs, early, news, c=2, told=3):
    """Interleavings of the k fallers' three steps after which R' lost the
    s-clique and nobody told it."""
    bad = 0
    for order in set(itertools.permutations(sorted(list(range(k)) * 3))):
        tau, step, first = [told] * k, [0] * k, [None] * k
        heard = False
        for r in order:
            step[r] += 1
            others = [tau[q] for q in range(k) if q != r]
            if step[r] == 1:
                first[r] = others
            elif (step[r] == 2) == (hubs[r] and early):
                heard |= _tells(hubs[r], early, news[r], told, first[r], others, c)
            else:
                tau[r] = news[r]
        bad += min(tau) < c and not heard
    return bad


@pytest.mark.parametrize("early", [True, False])
def test_two_fallers_every_interleaving(early):
    for hubs in itertools.product((False, True), repeat=2):
        missed = sum(_missed(2, hubs, early, news)
                     for news in itertools.product((0, 1, 2), repeat=2))
        # writing first fails exactly where both kinds of list meet
        assert (missed > 0) == (not early and hubs[0] != hubs[1]), hubs


def test_three_fallers_every_interleaving():
    orders = list(set(itertools.permutations((0, 0, 1, 1, 2, 2))))
    # hubs move as (gather, tell) and then write, the others as gather, then
    # write: the update's gather of a hub and a telling that reads nothing
    # anew do not matter
    for hubs in itertools.product((False, True), repeat=3):
        for news in itertools.product((0, 1), repeat=3):
            for order in orders:
                tau, seen = [3, 3, 3], [None] * 3
                for r in order:
                    if seen[r] is None:
                        seen[r] = [tau[q] for q in range(3) if q != r]
                    else:
                        tau[r] = news[r]
                heard = any(_tells(hubs[r], True, news[r], 3, seen[r], seen[r], 2)
                            for r in range(3))
                assert heard, (hubs, news, order)


def _h_index(vals):
    h = 0
    for i, x in enumerate(sorted(vals, reverse=True), 1):
        h = i if x >= i else h
    return h


def _decompose(seed, k, n, m, early):
    """AND with support counting on a random set system of m (k+1)-sets, the
    r-cliques' gather, write and telling interleaved at random (tellings that
    come after the write tend to come late); lists above the mean length are
    hubs.  Returns (slack words found too high, values, their fixed point)."""
    rng = random.Random(seed)
    sets = set()
    while len(sets) < m:
        sets.add(tuple(sorted(rng.sample(range(n), k + 1))))
    inc = [[tuple(q for q in s if q != r) for s in sorted(sets) if r in s]
           for r in range(n)]
    hub = [len(x) > m * (k + 1) // n for x in inc]
    tau = [len(x) for x in inc]
    slack, lost = [0] * n, [0] * n
    high = 0
    while True:
        step = {r: 0 for r in range(n) if slack[r] <= lost[r]}
        for r in range(n):
            if r not in step:
                slack[r] -= lost[r]
        lost = [0] * n
        start, read = tau[:], {}
        while step:
            late = [r for r in step if hub[r] and step[r] == 2]
            rest = [r for r in step if not (hub[r] and step[r] == 2)]
            r = rng.choice(rest if rest and (not late or rng.random() < 0.95) else late)
            step[r] += 1
            if step[r] == 1:
                rho = [min(tau[q] for q in o) for o in inc[r]]
                hold = [[q for q in o if tau[q] == x] for o, x in zip(inc[r], rho)]
                cnt = sum(x >= tau[r] for x in rho)
                h = tau[r] if cnt >= tau[r] else min(tau[r], _h_index(rho))
                read[r] = (rho, hold, tau[r], h, cnt)
                continue
            rho, hold, told, h, cnt = read[r]
            if (step[r] == 2) != (hub[r] and early):  # writes
                tau[r] = h
                slack[r] = 0 if h != told else cnt - told + 1
            elif h != told and not hub[r]:
                for x, who in zip(rho, hold):
                    for q in who if h < x <= told else ():
                        lost[q] += 1
            elif h != told:
                for o in inc[r]:
                    for q in o:
                        v = tau[q]
                        rest_ok = all((v if early else h) <= tau[y] for y in o if y != q)
                        lost[q] += h < v <= told and rest_ok
            if step[r] == 3:
                del step[r]
        for r in range(n):
            if slack[r] and tau[r] == start[r]:
                true = sum(min(tau[q] for q in o) >= tau[r] for o in inc[r]) - tau[r]
                high += slack[r] - 1 - lost[r] > true
        if tau == start:
            break
    want = [len(x) for x in inc]
    while True:
        nxt = [min(want[r], _h_index([min(want[q] for q in o) for o in inc[r]]))
               for r in range(n)]
        if nxt == want:
            return high, tau, want
        want = nxt


# seeds at which writing first leaves a slack word too high
@pytest.mark.parametrize("k,n,m,seeds", [(2, 9, 26, (419, 3195)), (2, 8, 20, (1910, 1916)),
                                         (2, 12, 60, (2019, 2517))])
def test_slack_never_too_high(k, n, m, seeds):
    for seed in seeds:
        assert _decompose(seed, k, n, m, early=False)[0] > 0
    for seed in list(seeds) + list(range(400)):
        high, tau, want = _decompose(seed, k, n, m, early=True)
        assert high == 0 and tau == want, seed
