"""The order in which the exchange solve (paper_2511_11514_amd/csrc/mesh.hip) gathers and
publishes its rows' potentials, run on the CPU under random interleavings of its blocks,
also where blocks own no rows of one point set.

Per iteration k a block: gathers g(k), p(k); publishes q(k) (from k = 1 on); publishes
f(k+1); gathers f(k+1), q(k); publishes p(k+1), then g(k+1).  Version v lives in buffer
v mod 2.  No read may find a later version than the one awaited, and every interleaving
has to end; with one buffer the first property must break."""
import random

import pytest


def _own(n, G, b):
    c = -(-n // G)
    return range(min(n, b * c), min(n, b * c + c))


def _run(G, T, M, K, debias, ref, buffers, seed):
    rng = random.Random(seed)
    n = {"f": T, "p": T, "g": M, "q": M}
    used = ["f", "g"] + ["p"] * debias + ["q"] * ref
    mem = {k: [[-1] * n[k] for _ in range(buffers)] for k in used}

    def program(b):
        pub = lambda k, v: [("pub", k, r, v) for r in _own(n[k], G, b)] if k in used else []
        get = lambda *kv: [("get", [(k, v, i) for k, v in kv if k in used for i in range(n[k])])]
        acts = pub("p", 0) + pub("g", 0) + pub("q", 0)
        for k in range(K):
            acts += get(("g", k), ("p", k)) + (pub("q", k) if k else []) + pub("f", k + 1)
            acts += get(("f", k + 1), ("q", k)) + pub("p", k + 1) + pub("g", k + 1)
        return acts + pub("q", K)

    progs = [program(b) for b in range(G)]
    pc, pending = [0] * G, [None] * G
    while any(pc[b] < len(progs[b]) for b in range(G)):
        ready = []
        for b in range(G):
            if pc[b] == len(progs[b]):
                continue
            act = progs[b][pc[b]]
            if act[0] == "pub":
                ready.append(b)
                continue
            if pending[b] is None:
                pending[b] = rng.sample(act[1], len(act[1]))
            for k, v, i in pending[b]:
                if mem[k][v % buffers][i] > v:
                    return f"block {b} awaited {k}[{i}] version {v}"
            if not pending[b] or any(mem[k][v % buffers][i] == v for k, v, i in pending[b]):
                ready.append(b)
        if not ready:
            return "no block can proceed"
        b = rng.choice(ready)
        act = progs[b][pc[b]]
        if act[0] == "pub":
            mem[act[1]][act[3] % buffers][act[2]] = act[3]
            pc[b] += 1
        else:
            for e in [e for e in pending[b] if mem[e[0]][e[1] % buffers][e[2]] == e[1]][:2]:
                pending[b].remove(e)
            if not pending[b]:
                pending[b] = None
                pc[b] += 1
    return None


@pytest.mark.parametrize("G,T,M", [(2, 4, 4), (3, 6, 1), (4, 2, 8), (1, 2, 2)])
@pytest.mark.parametrize("debias,ref", [(True, True), (True, False), (False, False)])
def test_no_word_is_overwritten_before_it_is_read(G, T, M, debias, ref):
    for seed in range(8):
        assert _run(G, T, M, 5, debias, ref, 2, seed) is None


def test_one_buffer_breaks_it():
    assert any(_run(3, 6, 6, 5, True, True, 1, seed) for seed in range(20))
