"""The self records of the exchange solve's one-block form (paper_2511_11514_amd/csrc/mesh.hip),
run on the CPU under random interleavings of the waves that finish a self sweep.

More than 64 rows are finished by two waves without a barrier between them.  A row whose lagged
sum is unusable walks every key record of the sweep twice (maximum, then sum).  Every row has to
see the records that were swept (a Jacobi update), so the new ones may be written only after the
next barrier; written at once, it must break.  That the kernel keeps them, and between which
barriers it writes them, is read from mesh.hip."""
import math
import os
import random
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2511_11514_amd", "csrc")


def _iteration():
    """The steps of one iteration as the kernel orders them: finish and put of the self rows,
    sweeps over the self records, barriers."""
    src = open(os.path.join(CSRC, "mesh.hip")).read()
    finish = src[src.index("void finish_rows("):src.index("void put_rows(")]
    writes = re.findall(r"(.*)\br\[3\] = ", finish)
    assert writes and all("if (!avg)" in w for w in writes), "self rows write at once"
    body = src[src.index("for (int k = 0; k < A.iters; ++k) {"):]
    body = body[:body.index("// store the own rows")]
    steps = []
    for m in re.finditer(r"__syncthreads\(\)|finish_rows<D, NT, LOCAL>\(A, ., 2, \w+, true, r([pq])"
                         r"|put_rows\(A, ., 2, lds \+ 4 \* A\.o_r([pq])|sweep_rows<D, NT>\(A, ., r([pq]),", body):
        if m.group(1):
            steps.append(("finish", m.group(1)))
        elif m.group(2):
            steps.append(("put", m.group(2)))
        elif m.group(3):
            steps.append(("sweep", m.group(3)))
        else:
            steps.append(("barrier", ""))
    return steps


@pytest.mark.parametrize("pot", ["p", "q"])
def test_barriers_separate_the_self_records(pot):
    """sweep | finish | put | next sweep: a barrier between each two of them."""
    steps = _iteration()
    # without what follows the loop: a barrier, the last finish of q, a barrier
    assert steps[-3:] == [("barrier", ""), ("finish", "q"), ("barrier", "")]
    seen = [k for k, p in steps[:-3] * 3 if k == "barrier" or p == pot]
    order = [k for k in seen if k != "barrier"]
    assert order.count("put") == 3 and order.count("finish") == 3 and order.count("sweep") == 3
    for a, b in zip(range(len(seen)), range(1, len(seen))):
        assert seen[a] == "barrier" or seen[b] == "barrier", seen
    nxt = {"sweep": "finish", "finish": "put", "put": "sweep"}
    assert all(nxt[a] == b for a, b in zip(order, order[1:])), order


def _wave(rows, rescued, read, write):
    """A wave's rows in lockstep, one record access of the whole wave at a time."""
    m = -math.inf
    if rescued:
        for j in range(len(read)):
            m = max(m, read[j])
            yield
        s = 0.0
        for j in range(len(read)):
            s += 2.0 ** (read[j] - m)
            yield
        m += math.log2(s)
    for i in rows:
        write[i] = m if rescued else float(i)
        yield


def _finish(n, kept, rescued, rng):
    """One finish step: the new records of n rows, by two waves of at most 64 rows, kept apart
    until both are done or written at once."""
    rec = [-4.0 - (i % 7) for i in range(n)]
    out = list(rec) if kept else rec
    waves = [_wave(range(w * 64, min(n, (w + 1) * 64)), rescued[w], rec, out) for w in range(2)]
    live = [0, 1]
    while live:
        w = rng.choice(live)
        for _ in range(rng.randint(1, 3 * n)):
            if next(waves[w], "end") == "end":
                live.remove(w)
                break
    return out


def _wrong(n, kept, rescued):
    want = math.log2(sum(2.0 ** (-4.0 - (j % 7)) for j in range(n)))
    for seed in range(30):
        got = _finish(n, kept, rescued, random.Random(seed))
        for i in range(n):
            if abs(got[i] - (want if rescued[i // 64] else i)) > 1e-9:
                return True
    return False


@pytest.mark.parametrize("n", [65, 100, 128])
@pytest.mark.parametrize("rescued", [(True, True), (True, False), (False, True)])
def test_rescued_self_rows_see_the_swept_records(n, rescued):
    assert not _wrong(n, True, rescued)


def test_writing_at_once_breaks_it():
    assert _wrong(128, False, (True, False)) and _wrong(128, False, (False, True))
