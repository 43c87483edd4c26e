"""The sizes of the product tests against the rule that picks the tiles: every kernel there is must be among them."""
import subprocess

import pytest

pytest.importorskip("torch")

from paper_2101_07706_amd import build
from test_gpu_launch_shapes import GRAD_W_SIZES, PRODUCT_SHAPES

ASK = """
#include <cstdio>
#include "gemm_rules.hpp"
int main()
{
    char what[4];
    long M, K, N;
    while (scanf("%3s %ld %ld %ld", what, &M, &K, &N) == 4) {
        csgs::Shape s;
        int parts = 0;
        if (what[1] == 'W') csgs::dw_split((int)M, K, N, &s, &parts);
        else s = what[0] == 'H' ? csgs::pick_shape(M, N, 1, false) : csgs::pick_shape(M, K, 1, true);
        printf("%d %d %d\\n", s.rt, s.nt, parts);
    }
}
"""


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    (d / "ask.cpp").write_text(ASK)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", build.CSRC, "-o", str(d / "ask"), str(d / "ask.cpp")], check=True)

    def run(sizes):
        out = subprocess.run([str(d / "ask")], input="\n".join(f"{w} {m} {k} {n}" for w, m, k, n in sizes), stdout=subprocess.PIPE, text=True,
                             check=True).stdout
        return [tuple(map(int, line.split())) for line in out.splitlines()]
    return run


def test_products_run_every_tile_and_tail(ask):
    got = ask([(what, M, K, N) for what, _, _, _, M, K, N in PRODUCT_SHAPES])
    assert [(rt, nt) for rt, nt, _ in got] == [(rt, nt) for _, rt, nt, _, _, _, _ in PRODUCT_SHAPES]
    for what, _, _, tail, _, K, N in PRODUCT_SHAPES:
        left = (K if what == "H" else N) % 32
        assert tail == (0 if left == 0 else 8 if left <= 8 else 32)
    tiles = [(2, 4), (2, 3), (2, 2), (1, 4), (1, 3), (1, 2), (2, 1), (1, 1)]
    assert {c[:4] for c in PRODUCT_SHAPES} == {(w, rt, nt, t) for w in ("H", "dZ") for rt, nt in tiles for t in (0, 8, 32)}


def test_weight_gradient_runs_every_tile(ask):
    got = ask([("dW", M, K, N) for M, K, N in GRAD_W_SIZES])
    assert {(rt, nt) for rt, nt, _ in got} == {(2, 2), (2, 4), (2, 3), (1, 4), (1, 2), (2, 1), (1, 1)}
    assert any(p == 1 for _, _, p in got) and any(p > 1 for _, _, p in got)
