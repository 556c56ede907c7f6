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
  char rule;
  while (scanf(" %c", &rule) == 1) {
    unsigned long v[6];
    const int n = rule == 's' ? 6 : 5;
    for (int i = 0; i < n; ++i)
      if (scanf("%lu", &v[i]) != 1) return 1;
    if (rule == 'r') {
      printf("%d\n", int(eq_detail::ragged_fused(v[0], v[1], v[2], v[3], v[4])));
    } else if (rule == 'w') {  // tiles, most wavefronts, table bytes, bytes per wavefront
      const unsigned t = v[0];
      const auto c = eq_detail::choose_waves(&t, 1, v[1], v[2], v[3], 160 * 1024, v[4]);
      printf("%u %lu\n", c.waves, (unsigned long)c.cost);
    } else {
      printf("%d\n", int(eq_detail::long_segments(v[0], v[1], v[2], v[3], v[4], v[5])));
    }
  }
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
        text = "\n".join(f"{r[0]} " + " ".join(str(int(v)) for v in r[1:]) for r in rows)
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
    got = rules([("r",) + r[:4] + (launch_rules.CUS,) for r in RAGGED])
    assert [bool(g[0]) for g in got] == [r[4] for r in RAGGED]


def test_ragged_gemv_python_copy(rules):
    rng = random.Random(5)
    pts = [(int(2 ** rng.uniform(0, 15)), int(2 ** rng.uniform(6, 14)),
            64 * int(2 ** rng.uniform(0, 10)), rng.randint(1, 8), 256) for _ in range(2000)]
    assert [bool(g[0]) for g in rules([("r",) + p for p in pts])] == [launch_rules.ragged_fused(*p) for p in pts]


# LDS of a version-2 block: the table, and a wavefront's window, rings and list
# (codes, BF16) or activations (GEMV)
PACKED, SPLIT = 32784, 65552


def out_lds(TR, seg):
    small = TR == 256 and seg == 64
    return (1024 if small else 2048) + TR * (seg + (4 if small else 8))


def gemv_lds(TC, nb):
    if nb == 1:
        return 2048 + (8 * (TC + 4) + 15) // 16 * 16 + 1024
    return 2048 + 4 * nb * (TC + 8)


def waves(rules, tiles, wmax, table, per_wave):
    return tuple(rules([("w", tiles, wmax, table, per_wave, launch_rules.CUS)])[0])


@pytest.mark.parametrize("tiles,TC,nb,want", [
    # several blocks fit a compute unit: their number counts, not one block's rounds
    (4970, 64, 4, 5),    # 25.6 us; 7 wavefronts 30.9
    (6162, 64, 4, 5),    # 31.9 us; 7: 38.5
    (10920, 64, 4, 5),   # 48.5 us; 8: 56.0
    # the fewest rounds before the evenest ones
    (10920, 64, 8, 8),   # 71.5 us; 4: 109.2
    (4970, 128, 8, 7),   # 81.4 us; 5: 99.1
    (10952, 128, 1, 15),
])
def test_gemv_waves(rules, tiles, TC, nb, want):
    wmax = 8 if nb >= 4 else 16
    assert waves(rules, tiles, wmax, SPLIT, gemv_lds(TC, nb))[0] == want


@pytest.mark.parametrize("TR,TC,tiles,bits,bf16,want", [
    # at the same rounds 64-code segments (0.90 to 0.97 of the time)
    (64, 128, 8192, 2.5, False, (64, 16)), (128, 128, 2550, 2.5, True, (64, 10)),
    (256, 256, 3584, 2.0, True, (64, 7)),
    # one round of 32-code segments against two: 24, 39, 43, 49 us against 37, 61, 62, 73
    (128, 64, 2888, 2.5, False, (32, 12)), (128, 128, 2862, 2.5, False, (32, 12)),
    (128, 128, 4096, 2.5, False, (32, 16)), (128, 128, 4096, 2.5, True, (32, 16)),
    (64, 64, 4970, 2.5, False, (32, 10)),                 # 21 against 27
    (64, 256, 12544, 2.0, False, (32, 10)), (64, 128, 14792, 3.5, True, (32, 10)),
    # 128-row tiles, two rounds against three: 75 against 94, 140 against 165 us
    (128, 128, 6162, 2.5, False, (32, 13)), (128, 256, 7168, 2.0, False, (32, 14)),
    # but stores beyond the memory-side cache at few bits: 229 -> 191, 194 -> 171 us
    (128, 256, 7168, 2.0, True, (64, 10)), (128, 256, 8192, 2.0, False, (64, 11)),
    (128, 256, 7168, 3.5, True, (32, 14)),                # 269 against 290
    (128, 256, 8192, 3.5, False, (32, 16)),               # 235 against 256
    (128, 256, 8192, 3.0, False, (32, 16)),               # 238 against 250
    (128, 128, 12544, 4.0, True, (64, 10)),               # 244 -> 232
    (64, 256, 14336, 2.0, True, (64, 14)), (64, 256, 14336, 4.0, True, (64, 14)),
    # 256-row tiles: 304 against 347 us
    (256, 256, 4096, 2.5, True, (32, 8)),
])
def test_output_segments(rules, TR, TC, tiles, bits, bf16, want):
    w = {seg: waves(rules, tiles, 16, PACKED, out_lds(TR, seg)) for seg in (32, 64)}
    codes = TR * TC * tiles
    long = rules([("s", w[32][1], w[64][1], TR, codes * (2 if bf16 else 1), codes * bits / 16,
                   codes)])[0][0]
    seg = 64 if long else 32
    assert (seg, w[seg][0]) == want


def test_waves_fit(rules):
    """Whatever the sizes: no more wavefronts than the limit or than LDS holds,
    none only where not one fits."""
    rng = random.Random(6)
    pts = [("w", int(2 ** rng.uniform(0, 20)), rng.randint(1, 16), rng.choice([PACKED, SPLIT]),
            int(2 ** rng.uniform(10, 18)), 256) for _ in range(2000)]
    for (_, n, wmax, tb, wl, _), (w, cost) in zip(pts, rules(pts)):
        assert w <= wmax and tb + w * wl <= 160 * 1024
        assert (w == 0) == (tb + wl > 160 * 1024)
