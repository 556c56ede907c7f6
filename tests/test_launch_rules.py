"""Host-side launch rules (csrc/eq_rules.h), compiled with the host compiler:
their choices at shapes where one choice measured far slower than the other,
and the Python copies that GPU tests use to name their paths."""
import os
import random
import subprocess

import pytest

import launch_rules
from paper_2601_22787_amd import _build

PROG = r"""
#include <cstdio>
#include "eq_rules.h"
int main() {
  unsigned a, b, c, d, e;
  while (scanf("%u %u %u %u %u", &a, &b, &c, &d, &e) == 5)
    printf("%d\n", int(eq_detail::ragged_fused(a, b, c, d, e)));
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    src, exe = os.path.join(d, "rules.cpp"), os.path.join(d, "rules")
    with open(src, "w") as f:
        f.write(PROG)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", _build.CSRC, src, "-o", exe], check=True)

    def run(rows):
        text = "\n".join(" ".join(map(str, r)) for r in rows)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True)
        return [list(map(int, line.split())) for line in out.stdout.splitlines()]
    return run


# chunks, columns, chunk symbols, batch: the faster way by 1.5 and more
RAGGED = [
    (1024, 200, 4096, 1, True),  # 24 against 57 us
    (16384, 3000, 4096, 1, True),  # 53 against 142 us
    (640, 100, 16384, 1, True),  # 99 against 253 us
    (16, 65, 16384, 1, False),  # 31 against 120 us
    (96, 100, 16384, 1, False),  # 68 against 123 us
    (128, 200, 16384, 1, False),  # 47 against 76 us
    (4096, 6001, 16384, 2, True),  # 51 against 162 us
    (1024, 150, 16384, 2, True),  # 123 against 277 us
    (1024, 1999, 65536, 2, True),  # 147 against 249 us
    (64, 1000, 65536, 2, False),  # 78 against 158 us
    (4, 600, 65536, 2, False),  # 65 against 208 us
    (64, 300, 16384, 2, False),  # 32 against 77 us
    (1024, 200, 4096, 3, True),  # 34 against 58 us
    (1024, 1999, 16384, 3, True),  # 42 against 68 us
    (1200, 65, 1024, 3, True),  # 21 against 48 us
    (64, 100, 65536, 3, False),  # 158 against 524 us
    (96, 400, 16384, 3, False),  # 33 against 78 us
    (16, 200, 65536, 3, False),  # 115 against 416 us
    (4096, 600, 4096, 5, True),  # 43 against 96 us
    (1024, 65, 16384, 5, True),  # 326 against 596 us
    (4096, 300, 16384, 5, True),  # 181 against 526 us
    (16, 1000, 16384, 5, False),  # 27 against 63 us
    (96, 200, 16384, 5, False),  # 42 against 142 us
    (64, 100, 16384, 5, False),  # 56 against 222 us
    (16384, 100, 4096, 8, True),  # 341 against 1461 us
    (1023, 6001, 4096, 8, True),  # 19 against 43 us
    (255, 6001, 4096, 8, True),  # 20 against 42 us
    (16, 150, 65536, 8, False),  # 119 against 717 us
    (64, 600, 16384, 8, False),  # 39 against 79 us
    (96, 100, 1024, 8, False),  # 12 against 25 us
]


def test_ragged_gemv(rules):
    got = rules([r[:4] + (launch_rules.CUS,) for r in RAGGED])
    assert [bool(g[0]) for g in got] == [r[4] for r in RAGGED]


def test_ragged_gemv_python_copy(rules):
    rng = random.Random(5)
    pts = [(int(2 ** rng.uniform(0, 15)), int(2 ** rng.uniform(6, 14)),
            64 * int(2 ** rng.uniform(0, 10)), rng.randint(1, 8), 256) for _ in range(2000)]
    assert [bool(g[0]) for g in rules(pts)] == [launch_rules.ragged_fused(*p) for p in pts]
