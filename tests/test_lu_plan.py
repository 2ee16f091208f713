"""The plan of the product beside the panels (bm_lu_rules.h, compiled with the host
compiler) against the same search without its short cuts, and its cost on the host."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2512_14193_amd", "csrc")
MAIN = r"""
#include <stdio.h>
#include <chrono>
#include "bm_lu_rules.h"
int main() {
  int n, gs, nseg;
  long w;
  sp_seg seg[SP_MAXSEG];
  while (scanf("%d %d %ld", &n, &gs, &w) == 3) {
    int on = 0;
    double us = 1e9;
    for (int i = 0; i < 50; ++i) {
      const auto t0 = std::chrono::steady_clock::now();
      on = sp_plan(n, 2 * n, 256, gs, (size_t)w, seg, &nseg);
      const double t = std::chrono::duration<double, std::micro>(std::chrono::steady_clock::now() - t0).count();
      us = (t < us) ? t : us;
    }
    printf("%f", us);
    for (int i = 0; on && i < nseg; ++i) printf(" %d %d %d", seg[i].b0, seg[i].b1, seg[i].ks);
    printf("\n");
  }
  return 0;
}
"""


def ksplit(tiles, slots, k, w):
    ks = min(slots // tiles if tiles <= slots else 1, max(k // 256, 1), 16)
    while ks > 1 and ks * tiles * 4096 > w:
        ks -= 1
    return max(ks, 1)


def time(tiles, ks, slots, k, per_k):
    kc = -(-(-(-k // ks)) // 16) * 16
    return -(-tiles * ks // slots) * per_k * kc + (0.006 if ks > 1 else 0.0)


def plan_at(beta, k1, k2, n, k, gs, w):
    nb = -(-n // 64)
    ks0 = ksplit(nb, 512, k, w)
    t0 = time(nb, ks0, 512, k, k2)
    segs, end, f = [(0, 1, ks0)], t0, 1
    while f < nb:
        best = 1
        for b in range(2, nb - f + 1):
            fin = end + time(nb * b, ksplit(nb * b, gs, k, w), gs, k, k1)
            late = min(max(int((fin - t0) / beta), 0), f - 1)
            if fin + late * (0.012 + 8.0 * n * (64.0 * b) * 64.0 / 25e9) <= t0 + beta * f - 0.03:
                best = b
        if nb - f - best == 1 and len(segs) >= 2:
            best = nb - f
        ks = ksplit(nb * best, gs, k, w)
        segs.append((f, f + best, ks))
        end += time(nb * best, ks, gs, k, k1)
        f += best
    return segs if len(segs) <= 10 and end <= t0 + beta * nb - 0.03 else None


def plan(n, gs, w):
    for count, k1, k2 in ((5, 0.49, 0.84), (8, 0.43, 0.74)):
        for i in range(count):
            s = plan_at(0.09 + 0.015 * i, k1 / 4096, k2 / 4096, n, 2 * n, gs, w)
            if s:
                return s
    return []


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    d = tmp_path_factory.mktemp("lu_plan")
    (d / "main.cpp").write_text(MAIN)
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, "-o", str(d / "plan"),
                           str(d / "main.cpp")])
    ns = [8, 64, 128, 130, 512, 700, 1024, 1500, 1728, 1732, 2048, 2112, 2114, 2178, 2368, 2430, 2496, 2688, 3000, 4096]
    q = [(n, 208, max(16 * n * 64, 256 * 4096)) for n in ns]
    out = subprocess.run([str(d / "plan")], input="\n".join("%d %d %d" % x for x in q), capture_output=True, text=True,
                         check=True).stdout.splitlines()
    return q, [x.split() for x in out]


def test_same_plan_as_the_whole_search(plans):
    for q, line in zip(*plans):
        v = [int(x) for x in line[1:]]
        assert [tuple(v[i:i + 3]) for i in range(0, len(v), 3)] == plan(*q), q
    found = {q[0]: len(line) > 1 for q, line in zip(*plans)}
    assert all(found[n] == (n <= 2430) for n in found)


def test_cost(plans):
    """Best of 50: under a few us; the whole search takes 50 us at n = 2430 and 110 at 4096."""
    assert max(float(line[0]) for line in plans[1]) < 25.0
