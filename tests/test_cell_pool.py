"""Places of a batch's moments in their common pool (paper_2511_11514_amd/csrc/cell_pool.h), compiled
for the host: rows beyond 32 bits, against exact integers."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2511_11514_amd", "csrc")
MAIN = r"""
#include <cstdio>
#include <vector>
#include "cell_pool.h"
// stdin: room, problems, then per problem cells and chunks of x and y and the four sweeps
int main() {
    long long room;
    int n;
    if (std::scanf("%lld %d", &room, &n) != 2) return 1;
    std::vector<long long> rows(n), at(n);
    for (int b = 0; b < n; ++b) {
        int c[4], s[4];
        for (int& v : c) if (std::scanf("%d", &v) != 1) return 1;
        for (int& v : s) if (std::scanf("%d", &v) != 1) return 1;
        const bool on[4] = {s[0] != 0, s[1] != 0, s[2] != 0, s[3] != 0};
        rows[b] = ct::pool_rows(c[0], c[1], c[2], c[3], on).all();
    }
    ct::pool_places(rows.data(), n, room, at.data());
    for (int b = 0; b < n; ++b) std::printf("%lld %lld\n", rows[b], at[b]);
}
"""


@pytest.fixture(scope="module")
def places(tmp_path_factory):
    d = tmp_path_factory.mktemp("pool")
    src, exe = d / "pool.cpp", d / "pool"
    src.write_text(MAIN)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                           "-I", CSRC, str(src), "-o", str(exe)])

    def run(room, problems):
        text = f"{room} {len(problems)}\n" + "\n".join(" ".join(map(str, p)) for p in problems)
        out = subprocess.run([str(exe)], input=text, capture_output=True, text=True, check=True).stdout
        return [tuple(int(v) for v in line.split()) for line in out.splitlines()]
    return run


def _rows(cx, hx, cy, hy, f, g, p, q):
    return max(cx * hy * f, cy * hx * g) + cx * hx * p + cy * hy * q


def _apart(got, room):
    """Placed problems lie in the pool and do not overlap."""
    end = 0
    for rows, at in got:
        if at < 0:
            continue
        assert end <= at and at + rows <= room
        end = at + rows


@pytest.mark.parametrize("n", [42, 43, 86, 341])
def test_rows_beyond_32_bits_have_no_place(places, n):
    """Problems of 4096 cells a side: 5e7 rows each, more than the whole pool; 43 of them pass
    2^31, 86 pass 2^32."""
    room = (256 << 20) // 192
    big = (4096, 4096 + 600, 4096, 4096 + 600, 1, 1, 1, 1)
    got = places(room, [big] * n)
    assert all(g == (_rows(*big), -1) for g in got)


def test_places_are_disjoint_and_in_the_pool(places):
    room = 100000
    probs = [(i % 90 + 1, i % 70 + 2, i % 110 + 3, i % 60 + 1, i % 2, 1, int(i % 3 > 0), int(i % 5 > 1))
             for i in range(200)]
    got = places(room, probs)
    assert [r for r, _ in got] == [_rows(*p) for p in probs]
    assert any(a >= 0 for _, a in got) and any(a < 0 for _, a in got)
    _apart(got, room)


def test_a_problem_without_a_place_takes_none(places):
    """One that does not fit leaves the pool to those after it."""
    small, big = (10, 20, 30, 40, 1, 1, 0, 0), (4096, 9000, 4096, 9000, 1, 1, 1, 1)
    got = places(1300, [big, small, big, small, small])
    assert [a for _, a in got] == [-1, 0, -1, 600, -1] and got[1][0] == 600
    got = places(1800, [big, small, big, small, small])
    assert [a for _, a in got] == [-1, 0, -1, 600, 1200]


def test_batch_without_a_reference_solve_reserves_less():
    """The pool has no rows for sweeps that the batch does not make."""
    import ctypes
    from paper_2511_11514_amd import _lib
    off = lambda n: (ctypes.c_int64 * 13)(*[n * i for i in range(13)])
    size = lambda flags: _lib.lib().ct_sinkhorn_batched_workspace_size(
        12, off(3000), off(9000), ctypes.byref(_lib.SinkhornOpts(2, 100, 0.01, flags)))
    direct = lambda flags: size(flags | _lib.CT_UNFUSED)
    room = [size(f) - direct(f) for f in (0, _lib.CT_DEBIAS, _lib.CT_DEBIAS | _lib.CT_VALUE)]
    # moments of 64 floats a row and their exponents: x-x and y-y rows of 12 problems
    row = 4 * 65
    x, y = (3000 // 24 + 1), (9000 // 24 + 1)
    assert room[1] - room[0] == pytest.approx(12 * row * x * (x + 3000 // 512), rel=0.02)
    assert room[2] - room[1] == pytest.approx(12 * row * y * (y + 9000 // 512), rel=0.02)
