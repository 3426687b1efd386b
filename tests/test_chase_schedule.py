"""The bulge chase's parallel schedule, on a model of its memory accesses: each
step's loads, body and tail, ordered by program order and by the progress
counters.  Every conflicting pair of accesses to one band entry must be
ordered as in the sequential reduction; with one step less of distance
anywhere it is not (the check can fail)."""
import pytest


def steps(n, b, s):
    return 0 if s < 0 else (n - s - 2 + b - 1) // b


def unordered(n, b, slack=0):
    index, reads, writes, before = {}, [], [], []

    def add(op, r, w, deps):
        anc = 0
        for d in deps:
            if d in index:
                anc |= before[index[d]] | 1 << index[d]
        index[op] = len(reads)
        reads.append(r)
        writes.append(w)
        before.append(anc)

    for s in range(n - 2):
        S, Sp = steps(n, b, s), steps(n, b, s - 1)
        # stage s-1's counter: stored behind the body, in its last step behind the tail
        done = [("body" if q + 1 < Sp else "tail", s - 1, q) for q in range(Sp)]
        for j in range(S):
            r0 = s + 1 + j * b
            ln = min(b, n - r0)
            nr = min(b, n - r0 - ln)
            c = s if j == 0 else r0 - b
            last, corner = j + 1 == S, ln == b and nr == b
            diag = {(i, k) for k in range(r0, r0 + ln) for i in range(k, r0 + ln)}
            right = {(i, k) for k in range(r0, r0 + ln) for i in range(r0 + ln, r0 + ln + nr)}
            crow = {x for x in right if corner and x[0] == r0 + 2 * b - 1}
            centry = {x for x in crow if x[1] == r0 + b - 1}
            left = {(i, k) for k in range(c, r0 if j else c + 1) for i in range(r0, r0 + ln)}
            add(("load", s, j), diag | (right - centry) | (left if j == 0 else set()), set(),
                done[:2 - slack] if j == 0 else [("wait", s, j - 1)])
            # the right block stays in registers: the next step's left block
            add(("body", s, j), set(), left | diag | (right - crow if last else set()),
                [("load", s, j), ("tail", s, j - 1)])
            add(("wait", s, j), set(), set(), [("body", s, j)] + done[:j + 3 - slack])
            add(("tail", s, j), centry, crow if last else set(), [("wait", s, j)])
    touched = {}
    for i, (r, w) in enumerate(zip(reads, writes)):
        for x in r | w:
            touched.setdefault(x, []).append((i, x in w))
    return sum((wa or wb) and not before[ib] >> ia & 1
               for t in touched.values() for p, (ia, wa) in enumerate(t) for ib, wb in t[p + 1:])


@pytest.mark.parametrize("b", [2, 3, 4, 7])
def test_every_conflict_is_ordered(b):
    for n in (3, 4, 5, 2 * b + 1, 3 * b + 2, 4 * b + 3, 5 * b + 1, 6 * b + 2):
        assert unordered(n, b) == 0, n
    assert unordered(6 * b + 2, b, slack=1) > 0
