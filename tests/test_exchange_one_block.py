"""The self records of the exchange solve's one-block form (paper_2511_11514_amd/csrc/mesh.hip),
run on the CPU under random interleavings of the waves that finish a self sweep.

More than 64 rows are finished by two waves without a barrier between them.  A row whose lagged
sum is unusable walks every key record of the sweep twice (maximum, then sum), while the other
wave may already write its rows' new records.  Every row has to see the sweep's records: a Jacobi
update.  The number of copies is read from the plan in mesh.hip; with one copy it must break."""
import math
import os
import random
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2511_11514_amd", "csrc")


def _copies():
    src = open(os.path.join(CSRC, "mesh.hip")).read()
    n = int(re.search(r"copies = A\.local \? (\d) : 1;", src).group(1))
    assert re.search(r"o_rp = r4; r4 \+= debias \? copies \* T", src)
    assert re.search(r"o_rq = r4; r4 \+= ref_iter \? copies \* M", src)
    return n


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


def _finish(n, copies, rescued, rng):
    """One finish step: the new records of n rows, by two waves of at most 64 rows."""
    rec = [[-4.0 - (i % 7) for i in range(n)] for _ in range(copies)]
    half = 64
    waves = [_wave(range(w * half, min(n, (w + 1) * half)), rescued[w], rec[0], rec[copies - 1])
             for w in range(2)]
    live = [0, 1]
    while live:
        w = rng.choice(live)
        for _ in range(rng.randint(1, 3 * n)):
            if next(waves[w], "end") == "end":
                live.remove(w)
                break
    return rec[copies - 1]


def _wrong(n, copies, rescued):
    want = math.log2(sum(2.0 ** (-4.0 - (j % 7)) for j in range(n)))
    for seed in range(30):
        got = _finish(n, copies, rescued, random.Random(seed))
        for i in range(n):
            if abs(got[i] - (want if rescued[i // 64] else i)) > 1e-9:
                return True
    return False


@pytest.mark.parametrize("n", [65, 100, 128])
@pytest.mark.parametrize("rescued", [(True, True), (True, False), (False, True)])
def test_rescued_self_rows_see_the_swept_records(n, rescued):
    assert not _wrong(n, _copies(), rescued)


def test_one_copy_breaks_it():
    assert _wrong(128, 1, (True, False)) and _wrong(128, 1, (False, True))
