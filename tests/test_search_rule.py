"""The launch rules of the search (host arithmetic, compiled by itself)."""
import os
import subprocess
import tempfile

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CUS = 256
PROGRAM = r"""
#include <cstdio>
#include "search_rule.h"
int main() {
  char what;
  long long a, b, c, d, e, f;
  while (scanf(" %c %lld %lld %lld %lld %lld %lld", &what, &a, &b, &c, &d, &e, &f) == 7)
    printf("%d\n", what == 'w' ? (int)finger::wide_passes(a, b, c, d, e, f) : finger::resident_blocks(a, b, c, d));
}
"""


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    d = tmp_path_factory.mktemp("rule")
    (d / "rule.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-I", os.path.join(ROOT, "paper_2206_11408_amd", "csrc"),
                    str(d / "rule.cpp"), "-o", str(d / "rule")], check=True)

    def run(rows):
        text = "".join(" ".join(map(str, r + (0,) * (7 - len(r)))) + "\n" for r in rows)
        out = subprocess.run([str(d / "rule")], input=text, capture_output=True, text=True, check=True).stdout
        return [int(x) for x in out.split()]
    return run


# (plain, lanes per vector, float4 per lane): waves per CU of the wide instance
SHAPES = {(0, 32, 2): 12, (1, 32, 2): 16, (0, 32, 4): 8, (1, 32, 4): 8, (0, 64, 4): 8, (1, 64, 4): 8, (0, 64, 8): 8,
          (1, 64, 8): 8}


def wide(ask, shape, nqs, per_cu=16):
    return ask([("w", *shape, nq, min(nq, per_cu * CUS), CUS) for nq in nqs])


@pytest.mark.parametrize("shape,waves", SHAPES.items())
def test_wide_while_every_query_is_resident(ask, shape, waves):
    fit = waves * CUS
    assert wide(ask, shape, [1, 33, fit - 1, fit]) == [1, 1, 1, 1]
    # one more query is a second round of waves
    assert wide(ask, shape, [fit + 1, fit + fit // 4, 2 * fit - 1 if waves < 16 else fit + 1]) == [0, 0, 0]


@pytest.mark.parametrize("shape", SHAPES)
def test_wide_again_for_many_queries(ask, shape):
    again = shape in ((0, 32, 2), (0, 64, 4), (1, 64, 4))
    assert wide(ask, shape, [36 * CUS - 1, 36 * CUS, 100_000]) == [0, again, again]


@pytest.mark.parametrize("shape", SHAPES)
def test_wide_where_registers_do_not_bind(ask, shape):
    """LDS or the caller holds the launch to eight waves a CU or fewer."""
    assert wide(ask, shape, [1000, 5000, 50_000], per_cu=8) == [1, 1, 1]


def test_never_wide_for_short_vectors(ask):
    assert ask([("w", p, 8, t, nq, min(nq, 4096), CUS) for p in (0, 1) for t in (1, 2, 3, 4)
                for nq in (1, 5000, 100_000)]) == [0] * 24


def test_static_grid_is_what_is_resident(ask):
    # several queries to a workgroup: no partial round of workgroups
    assert ask([("r", 4096, 20_000, 12, CUS), ("r", 3584, 20_000, 8, CUS), ("r", 4096, 4097, 8, CUS)]) == [3072, 2048, 2048]
    # a workgroup per query, or all of them resident
    assert ask([("r", 4096, 4096, 8, CUS), ("r", 1000, 1000, 2, CUS), ("r", 3072, 20_000, 16, CUS),
                ("r", 3072, 20_000, 0, CUS)]) == [4096, 1000, 3072, 3072]


@pytest.mark.parametrize("shape", SHAPES)
def test_queue_of_mixed_ef(ask, shape):
    src = PROGRAM.replace("(a, b, c, d, e, f)", "(a, b, c, d, e, f, true)")
    assert src != PROGRAM
    many = shape in ((0, 32, 2), (0, 64, 4), (1, 64, 4))
    with tempfile.TemporaryDirectory() as d:
        with open(os.path.join(d, "rule.cpp"), "w") as fh:
            fh.write(src)
        subprocess.run(["g++", "-std=c++17", "-I", os.path.join(ROOT, "paper_2206_11408_amd", "csrc"),
                        os.path.join(d, "rule.cpp"), "-o", os.path.join(d, "rule")], check=True)
        text = "".join(f"w {shape[0]} {shape[1]} {shape[2]} {nq} {min(nq, 4096)} {CUS}\n" for nq in (33, 12 * CUS, 12 * CUS + 1, 8000, 100_000))
        out = subprocess.run([os.path.join(d, "rule")], input=text, capture_output=True, text=True, check=True).stdout
    always, resident = shape == (0, 32, 2), shape == (1, 32, 2)
    assert [int(v) for v in out.split()] == [1, many or resident, always or resident, always, always]
