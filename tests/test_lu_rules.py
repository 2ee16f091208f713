"""The LU's host rules (bm_lu_rules.h, compiled with the host compiler): the workgroups
that a panel needs resident, and what batches and server lanes are allowed by them."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2512_14193_amd", "csrc")
MAIN = r"""
#include <stdio.h>
#include "bm_lu_rules.h"
int main() {
  char op;
  int a, b, c, d;
  while (scanf(" %c %d %d %d %d", &op, &a, &b, &c, &d) == 5) {
    int v = 0;
    if (op == 'w') v = lu_panel_wgs(a, b);
    if (op == 'f') v = lu_batch_fit(a, b, c);
    if (op == 'o') v = srv_lanes_ok(a, b, c);
    if (op == 's') v = srv_small_lanes(a, b, c);
    if (op == 'b') v = srv_batch_limit(a, b, c, d);
    printf("%d\n", v);
  }
  return 0;
}
"""


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    d = tmp_path_factory.mktemp("lu_rules")
    (d / "main.cpp").write_text(MAIN)
    subprocess.check_call(["g++", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, "-o", str(d / "rules"),
                           str(d / "main.cpp")])

    def call(queries):
        text = "\n".join(" ".join(str(x) for x in q + (0,) * (5 - len(q))) for q in queries)
        out = subprocess.run([str(d / "rules")], input=text, capture_output=True, text=True, check=True).stdout
        return [int(x) for x in out.split()]
    return call


def test_panel_workgroups(ask):
    want = {8: 1, 63: 8, 64: 8, 65: 16, 128: 16, 1024: 16, 2048: 16, 2688: 16, 2689: 22, 8192: 64, 16384: 128}
    assert ask([("w", n, 256) for n in want]) == list(want.values())


def units(n):  # the count by which orders and batches are taken or refused
    return -(-n // 128) if n > 2048 else -(-n // 64)


@pytest.mark.parametrize("ncu", [32, 64, 256])
def test_batches_stay_resident(ask, ncu):
    qs = [(n, c) for n in (8, 64, 65, 128, 512, 1024, 2048, 2049, 2688, 2689, 4000, 8192) for c in (1, 2, 3, 4)]
    wgs = ask([("w", n, ncu) for n, _ in qs])
    fit = ask([("f", n, c, ncu) for n, c in qs])
    for (n, c), w, f in zip(qs, wgs, fit):
        if c * units(n) > ncu:
            assert f == 0, (n, c)
        else:
            assert 1 <= f <= c and f * w <= ncu, (n, c, w, f)
            assert f == c or (f + 1) * w > ncu
    if ncu == 256:
        assert all(f == c for (n, c), f in zip(qs, fit) if f)


@pytest.mark.parametrize("ncu", [32, 64, 256])
def test_server_panels_within_half_the_cus(ask, ncu):
    cfg = [(lanes, cmax) for lanes in range(1, 17) for cmax in (64, 128, 256, 512, 1024, 2048, 4096)]
    ok = ask([("o", lanes, cmax, ncu) for lanes, cmax in cfg])
    assert ok == [int(lanes == 1 or (cmax <= 2048 and lanes * -(-cmax // 64) <= ncu // 2)) for lanes, cmax in cfg]
    cfg = [c for c, o in zip(cfg, ok) if o and c[0] > 1]
    small = ask([("s", lanes, cmax, ncu) for lanes, cmax in cfg])
    for (lanes, cmax), sl in zip(cfg, small):
        assert 1 <= sl <= lanes
        ns = [n for n in (8, 64, 66, 128, 256, 512, 1024, 2048) if n <= cmax]
        wgs = ask([("w", n, ncu) for n in ns])
        for bm in (1, 2, 4):
            lim = ask([("b", n, bm, sl, ncu) for n in ns])
            for n, w, b in zip(ns, wgs, lim):
                assert 1 <= b <= bm
                assert sl * b * w <= ncu // 2 or (sl == 1 and b == 1), (lanes, cmax, n, sl, b, w)
    if ncu == 256:
        assert all(sl == min(lanes, 8 if cmax > 64 else 16) for (lanes, cmax), sl in zip(cfg, small))
        assert ask([("b", n, 4, 4, 256) for n in (64, 128, 1024, 2048)]) == [4, 2, 2, 2]
