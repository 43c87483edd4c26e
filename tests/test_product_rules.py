"""The sizes of the product tests against the rule that picks the tiles: every kernel there is must be among them."""
import subprocess

import numpy as np

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


ASK_DIGITS = """
#include <cstdio>
#include "gemm_rules.hpp"
int main()
{
    long M, K, N, n;
    int z;
    while (scanf("%ld %ld %ld %ld %d", &M, &K, &N, &n, &z) == 5) {
        const csgs::DigitsPlan d = csgs::digits_plan(M, N, K, K, z ? K : N, N, n, z);
        printf("%d %d %d %d %d %lld\\n", d.use, d.kc, d.cgs, d.wcs, d.rgs, (long long)d.few);
    }
}
"""


def test_digit_products_run_every_kernel(tmp_path):
    from test_gpu_digits import SHAPES
    (tmp_path / "ask.cpp").write_text(ASK_DIGITS)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", build.CSRC, "-o", str(tmp_path / "ask"), str(tmp_path / "ask.cpp")], check=True)

    def ask(sizes):
        out = subprocess.run([str(tmp_path / "ask")], input="\n".join(" ".join(map(str, s)) for s in sizes), stdout=subprocess.PIPE, text=True, check=True)
        return [tuple(map(int, line.split())) for line in out.stdout.splitlines()]
    got = ask([(M, K, N, 1, z) for K, N, M in SHAPES for z in (0, 1)] + [(65_536, 256, 100, 1, 0), (8_000, 100, 256, 8, 0), (32_000, 256, 256, 1, 0)])
    assert all(use for use, *_ in got), got
    assert {kc for _, kc, *_ in got} == {1, 2, 3, 4, 5, 8}
    assert {w for _, _, _, w, *_ in got} >= {4, 8} and any(c > 1 for _, _, c, *_ in got)
    # every step of rows has a block, every column a wavefront, and few enough rows on the device are done in double
    rng = np.random.default_rng(0)
    sizes = [(int(2 ** rng.uniform(4, 21)), int(rng.integers(1, 700)), int(rng.integers(1, 700)), int(rng.choice([1, 2, 8])), int(rng.integers(2)))
             for _ in range(2000)]
    for (M, K, N, n, _), (use, kc, cgs, wcs, rgs, few) in zip(sizes, ask(sizes)):
        if use:
            cols = 16 if kc > 4 else 32
            assert 64 * kc >= K and cgs * wcs * cols >= N > (cgs - 1) * wcs * cols and wcs <= 8 and 1 <= rgs and 0 < few < M * n


ASK_TILES = """
#include <cstdio>
#include "gemm_rules.hpp"
int main()
{
    for (int kc : {1, 2, 3, 4, 5, 8})
        for (long M = 1; M < 600; ++M)
            for (long s0 = 0; s0 < M + 2 * csgs::digit_rows(kc); s0 += csgs::digit_rows(kc))
                printf("%d %ld %ld %d\\n", csgs::digit_rows(kc), M, s0, csgs::row_tiles(M - s0, csgs::digit_rows(kc)));
}
"""


def test_step_has_no_tile_past_the_last_row(tmp_path):
    """The row offset of a tile's lanes is formed from its first row before that is compared with the count: it has to exist."""
    (tmp_path / "ask.cpp").write_text(ASK_TILES)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", build.CSRC, "-o", str(tmp_path / "ask"), str(tmp_path / "ask.cpp")], check=True)
    out = subprocess.run([str(tmp_path / "ask")], stdout=subprocess.PIPE, text=True, check=True).stdout
    for rs, M, s0, tiles in np.array(out.split(), dtype=np.int64).reshape(-1, 4):
        assert tiles == len([m0 for m0 in range(s0, s0 + rs, 16) if m0 < M])


ASK_LIST = """
#include <cstdio>
#include "gemm_rules.hpp"
int main()
{
    for (int kc : {1, 2, 3, 4, 5, 8})
        printf("%d %d %d %d %d\\n", kc, csgs::digit_rows(kc), csgs::digit_tile_list(kc), csgs::digit_step_list(kc), csgs::digit_list(kc));
}
"""


def test_list_has_room_for_a_step(tmp_path):
    """What a block sums again: whatever the operands, a step finds room for all that it lists, however many steps a call has, in the LDS there is."""
    (tmp_path / "ask.cpp").write_text(ASK_LIST)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", build.CSRC, "-o", str(tmp_path / "ask"), str(tmp_path / "ask.cpp")], check=True)
    out = subprocess.run([str(tmp_path / "ask")], stdout=subprocess.PIPE, text=True, check=True).stdout
    for kc, rows, tile, step, room in np.array(out.split(), dtype=np.int64).reshape(-1, 5):
        nt = 1 if kc > 4 else 2
        assert step == rows // 16 * 8 * nt * tile     # every wavefront, each of its tiles
        # it is worked off after a step that left less than the next may take, and in one with more than half of that in every step so far
        assert 2 * step <= room < 2 ** 15 and tile <= 16
        lds = 2 * rows // 16 * 5 * kc * 1088 + 8 * kc * nt * 1024 + 2 * rows * 8 + 4 * room + 16
        assert lds <= 160 * 1024


def test_digit_forms_are_compared_with_calls_in_double(tmp_path):
    """The products that the tests compare go by digits, and the calls of 512 rows that they are compared with never do."""
    from test_gpu_digits import SHAPES
    (tmp_path / "ask.cpp").write_text(ASK_DIGITS)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", build.CSRC, "-o", str(tmp_path / "ask"), str(tmp_path / "ask.cpp")], check=True)
    by_digits = [(M, K, N, 1, z) for K, N, M in SHAPES + [(64, 256, 131_069), (256, 256, 32_033), (512, 512, 8_191), (256, 256, 65_537), (128, 256, 100_003), (100, 256, 600_005),
                                                         (260, 256, 200_009)] for z in (0, 1)]
    by_digits += [(M, K, 256, n, 0) for K in (100, 256) for M, n in ((16_000, 8), (16_000, 4), (27_000, 3), (2_100, 64))]
    in_double = [(512, K, N, 1, z) for K in range(16, 513, 3) for N in (16, 100, 256, 512, 700) for z in (0, 1)]
    sent = "\n".join(" ".join(map(str, s)) for s in by_digits + in_double)
    out = subprocess.run([str(tmp_path / "ask")], input=sent, stdout=subprocess.PIPE, text=True, check=True).stdout
    use = [int(line.split()[0]) for line in out.splitlines()]
    assert use == [1] * len(by_digits) + [0] * len(in_double), [s for s, u in zip(by_digits + in_double, use) if u != (s in by_digits)]
