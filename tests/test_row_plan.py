"""Choice of the row tile (csrc/row_plan.h, host code): compiled on its own and asked about sizes."""
import os
import subprocess

import pytest

from paper_2505_11432_amd import build

MAIN = r'''
#include <cstdio>
#include "row_plan.h"
int main() {
  int swiglu, store, across, M, E, N, K, esz;
  while (scanf("%d %d %d %d %d %d %d %d", &swiglu, &store, &across, &M, &E, &N, &K, &esz) == 8) {
    const moe::RowPlan p = moe::plan_rows({swiglu != 0, store != 0, across != 0}, M, E, N, K, esz);
    printf("%s %d\n", p.tile == moe::RowTile::FEW ? "few" : p.tile == moe::RowTile::MID ? "mid" : "full", (int)p.split);
  }
}
'''


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("plan")
    src, exe = tmp / "main.cpp", tmp / "main"
    src.write_text(MAIN)
    subprocess.run([build.CXX, "-std=c++17", "-I", build.CSRC, str(src), "-o", str(exe)], check=True)

    def ask(rows):
        text = "\n".join(" ".join(map(str, r)) for r in rows)
        out = subprocess.run([str(exe)], input=text, capture_output=True, text=True, check=True).stdout.split("\n")
        return [(l.split()[0], l.split()[1] == "1") for l in out if l]
    return ask


FC1, FC2, DGRAD2, DGRAD1 = (1, 0, 0), (0, 1, 0), (0, 0, 1), (0, 1, 1)


def gemms(M, E, d, f):
    return [FC1 + (M, E, f, d, 2), FC2 + (M, E, d, f, 2), DGRAD2 + (M, E, f, d, 2), DGRAD1 + (M, E, d, 2 * f, 2)]


def test_few_rows_stream_the_weights(plan):
    """A handful of rows: the 64-row tile for all four products (a round of it lasts less than one of the large tile)."""
    for M, E, d, f in ((1, 1, 16, 16), (32, 8, 4096, 14336), (64, 64, 2048, 1408), (512, 16, 4096, 1536), (576, 24, 1040, 1424)):
        assert [t for t, _ in plan(gemms(M, E, d, f))] == ["few"] * 4, (M, E, d, f)
    assert [t for t, _ in plan(gemms(2056, 64, 2048, 1408))[:2]] == ["few"] * 2


def test_no_small_tile_where_gathered_rows_would_be_slow(plan):
    """Averages of 32 rows and less whose sum, gathered on one expert, keeps the 64-row tile busy for several rounds of which
    the large tile needs one."""
    for M, E, d, f in ((8192, 256, 1024, 1024), (8192, 256, 2048, 1408), (4096, 128, 2048, 2048), (512, 16, 4096, 14336)):
        assert plan([FC1 + (M, E, f, d, 2)])[0][0] == "mid", (M, E, d, f)
    for M in range(64, 33000, 64):
        E = (M + 31) // 32
        if E <= 256:
            (t, _), = plan([FC1 + (M, E, 2048, 2048, 2)])
            # rounds of 64 x 64 outputs in 17.8 us each against rounds of 256 x 128 in 72.6
            few, full = -(-(M // 64 * 32) // 256) * 17.8, -(-(-(-M // 256) * 16) // 256) * 72.6
            assert (t == "few") == (few <= full + 1e-6), (M, t, few, full)


def test_ordinary_sizes(plan):
    assert [t for t, _ in plan(gemms(16384, 8, 4096, 14336))] == ["full"] * 4
    assert [t for t, _ in plan(gemms(131072, 64, 2048, 1408))] == ["full"] * 4
    assert plan([FC1 + (8000, 8, 6160, 1040, 2), FC1 + (4096, 8, 10368, 4096, 2)]) == [("full", False)] * 2
    assert [t for t, _ in plan(gemms(4593, 24, 1040, 1424))] == ["mid", "mid", "full", "mid"]
    assert plan([FC2 + (16384, 8, 4096, 14336, 2)]) == [("full", True)]
    assert not any(s for _, s in plan([k + (M, 8, 4096, 4096, 2) for k in (FC1, DGRAD2) for M in (16, 600, 9000)]))


GROUPS = r'''
#include <cstdio>
#include "row_plan.h"
int main() {
  int M, E, d, f;
  while (scanf("%d %d %d %d", &M, &E, &d, &f) == 4) {
    auto up = [](long a, long b) { return (a + b - 1) / b; };
    const int steps = (int)up(up(M, 128) + E, E);
    const moe::RowPlan plan = moe::plan_rows({true, false, false}, M, E, f, d, 1), bf16 = moe::plan_rows({true, false, false}, M, E, f, d, 2);
    const moe::Stagger s[] = {plan.stagger, moe::wgrad_stagger(d, f, E * up(d, 256) * up(f, 256), steps),
                              moe::wgrad_stagger(2 * f, d, E * up(2 * f, 256) * up(d, 256), steps)};
    for (const auto& q : s) printf("%dx%d ", q.groups, q.lag);
    printf("%s %d\n", plan.tile == moe::RowTile::FULL ? "full" : "other", bf16.stagger.groups);
  }
}
'''


def test_groups_that_start_one_after_another(tmp_path):
    """e4m3 FC1, d_w2, d_w1: number of groups and steps between them; none in short launches, short tiles and tall gradients of many
    steps, none in bf16."""
    (tmp_path / "m.cpp").write_text(GROUPS)
    subprocess.run([build.CXX, "-std=c++17", "-I", build.CSRC, str(tmp_path / "m.cpp"), "-o", str(tmp_path / "m")], check=True)
    sizes = {(16384, 8, 4096, 14336): "8x2 8x1 8x1", (4096, 8, 4096, 14336): "8x2 8x1 8x1", (32768, 8, 4096, 14336): "8x2 8x1 0x0",
             (16384, 8, 2048, 8192): "8x1 4x1 8x1", (16384, 16, 1024, 8192): "8x1 4x1 4x1", (131072, 64, 2048, 1408): "8x1 4x1 8x1",
             (8000, 8, 2048, 8192): "8x1 4x1 8x1",
             (32768, 8, 512, 14336): "4x1 0x0 0x0", (32768, 8, 256, 14336): "0x0 0x0 0x0", (2000, 8, 1024, 2816): "0x0 0x0 0x0",
             (8000, 8, 1040, 6160): "8x1 0x0 4x1", (2048, 8, 4096, 14336): "0x0 0x0 0x0"}
    out = subprocess.run([str(tmp_path / "m")], input="\n".join(" ".join(map(str, k)) for k in sizes), capture_output=True, text=True, check=True)
    got = out.stdout.split("\n")[:-1]
    assert [" ".join(l.split()[:3]) for l in got] == list(sizes.values())
    assert all(l.split()[4] == "0" for l in got)


PAIRS = r'''
#include <cstdio>
#include "row_plan.h"
int main() {
  int M, E, d, f;
  while (scanf("%d %d %d %d", &M, &E, &d, &f) == 4)
    printf("%d %d %d %d\n", (int)moe::plan_rows({true, false, false}, M, E, f, d, 2).pair, (int)moe::plan_rows({false, false, true}, M, E, f, d, 2).pair,
           (int)moe::wgrad_in_pairs(M, E, d, f), (int)moe::wgrad_in_pairs(M, E, 2 * f, d));
}
'''


def test_pairs_of_workgroups(tmp_path):
    """FC1, dgrad2, d_w2, d_w1 on 128 x 128 tiles with two workgroups per CU: where the large tile would leave CUs idle."""
    (tmp_path / "m.cpp").write_text(PAIRS)
    subprocess.run([build.CXX, "-std=c++17", "-I", build.CSRC, str(tmp_path / "m.cpp"), "-o", str(tmp_path / "m")], check=True)
    sizes = {(4593, 24, 1040, 1424): "1 0 0 0", (2000, 8, 1024, 2816): "1 1 0 0", (4096, 8, 512, 512): "1 0 1 1", (6000, 8, 1024, 1024): "0 1 1 0",
             (512, 8, 4096, 14336): "0 0 0 0", (16384, 8, 4096, 14336): "0 0 0 0", (131072, 64, 2048, 1408): "0 0 0 0", (0, 8, 16, 16): "0 0 1 1",
             (1222, 6, 272, 336): "1 0 1 1", (4096, 16, 1024, 1024): "1 1 0 0",
             (8000, 8, 1040, 6160): "0 0 0 0", (4096, 8, 4096, 10368): "0 0 0 0"}
    out = subprocess.run([str(tmp_path / "m")], input="\n".join(" ".join(map(str, k)) for k in sizes), capture_output=True, text=True, check=True)
    assert out.stdout.split("\n")[:-1] == list(sizes.values())


DEAL = r'''
#include <cstdio>
#include "row_plan.h"
int main() {
  int items, window, pair;
  while (scanf("%d %d %d", &items, &window, &pair) == 3) {
    long n = 0, sum = 0;
    int last = 0;
    for (int first = 0; first < items; first += 8 * window) {
      last = moe::tiles_per_xcd(items, items - first, window, pair != 0);
      for (int xcd = 0; xcd < 8; ++xcd)
        for (int i = 0; i < window; ++i) {
          const int l = first + xcd * last + i;
          if (i < last && l < items) { ++n; sum += l; }
        }
    }
    printf("%d %d %d\n", last, (int)(n == items && sum == (long)items * (items - 1) / 2), last <= window);
  }
}
'''


def test_last_round_is_dealt_evenly_in_short_lists(tmp_path):
    """Every tile once, whatever the count; an eighth of the last round to every XCD up to three rounds (pairs of workgroups: four), whole
    windows in longer lists."""
    (tmp_path / "m.cpp").write_text(DEAL)
    subprocess.run([build.CXX, "-std=c++17", "-I", build.CSRC, str(tmp_path / "m.cpp"), "-o", str(tmp_path / "m")], check=True)
    cases = [(n, w, p) for w in (1, 4, 32, 64) for p in (0, 1) for n in [*range(1, 40), *range(8 * w - 9, 8 * w + 10), *range(24 * w - 9, 24 * w + 10), *range(32 * w - 9, 32 * w + 10)] if n > 0]
    out = subprocess.run([str(tmp_path / "m")], input="\n".join("%d %d %d" % c for c in cases), capture_output=True, text=True, check=True)
    got = [tuple(map(int, l.split())) for l in out.stdout.split("\n") if l]
    assert len(got) == len(cases)
    for (n, w, p), (last, each, fits) in zip(cases, got):
        assert each and fits, (n, w, p)
        left = n % (8 * w) or 8 * w
        assert last == (-(-left // 8) if n < (4 if p else 3) * 8 * w else w), (n, w, p, last)
    # 8 experts, 1024 x 2816: d_w2, d_w1; weight gradients of 24 experts, 3072 x 2400; FC1 of 19 row tiles in pairs
    sizes = [(352, 32, 0, 12), (704, 32, 0, 24), (2880, 32, 0, 32), (5760, 32, 0, 32), (836, 64, 1, 41)]
    out = subprocess.run([str(tmp_path / "m")], input="\n".join("%d %d %d" % c[:3] for c in sizes), capture_output=True, text=True, check=True)
    assert [int(l.split()[0]) for l in out.stdout.split("\n") if l] == [c[3] for c in sizes]


F32 = r'''
#include <cstdio>
#include "row_plan.h"
int main() {
  int M, E, d, f;
  while (scanf("%d %d %d %d", &M, &E, &d, &f) == 4) {
    const moe::F32Product p[] = {{true, M, 2 * f, d, E}, {true, M, d, f, E}, {true, M, f, d, E}, {true, M, d, 2 * f, E}, {false, d, f, M, E}, {false, 2 * f, d, M, E}};
    // results that fit behind A in the full workspace (FC2), in A and dA (dgrad1)
    const long a = ((long)M * f * 4 + 255) / 256 * 64, dh = ((long)M * 2 * f * 4 + 255) / 256 * 64, out = (long)M * d;
    const long room[] = {0, (a + dh) / out, 0, 2 * a / out, 0, 0};
    for (int i = 0; i < 6; ++i) {
      const moe::F32Plan q = moe::f32_plan(p[i], room[i]);
      if (!moe::f32_split_pays(p[i])) printf("- ");
      else printf(q.parts > 1 ? "%s/%d " : "%s ", q.tile == moe::F32_128 ? "128" : q.tile == moe::F32_128_EIGHT ? "eight" : "64", q.parts);
    }
    printf("\n");
  }
}
'''


def test_fp32_products(tmp_path):
    """FC1, FC2, dgrad2, dgrad1, d_w2, d_w1: the fp32 instruction (-) or the split on 64 x 64 tiles, on 128 x 128 of four waves, of eight
    waves, cut along K into so many parts, at the sizes of the fp32 GEMM tests (which rely on each being taken in each layout) and at small ones."""
    (tmp_path / "m.cpp").write_text(F32)
    subprocess.run([build.CXX, "-std=c++17", "-I", build.CSRC, str(tmp_path / "m.cpp"), "-o", str(tmp_path / "m")], check=True)
    sizes = {(2000, 8, 1024, 2816): "128 128/3 128 128/3 128 128", (2060, 4, 1024, 1408): "128 128/3 64 64/2 64 128",
             (894, 5, 272, 1040): "64 - 64 - 64 64", (1200, 30, 48, 528): "64 - 64 - 64 64", (1027, 1, 1552, 784): "64 64 64 64 64 64",
             (512, 8, 1024, 2832): "64 64/5 64 64/5 128 128", (2077, 8, 1024, 2832): "128 64/2 128 64/2 128 128",
             (2063, 4, 1024, 1408): "128 128/3 64 64/2 64 128", (1205, 4, 496, 1008): "64 - 64 - 64 eight",
             (1500, 3, 1008, 1040): "eight 64 64 64 eight 128", (1500, 1, 784, 2064): "128 64/3 eight 128/5 64 eight",
             (1161, 8, 528, 2176): "64 64/2 64 64/2 64 128", (2008, 16, 784, 1424): "64 64 64 64 64 64", (2388, 8, 800, 2320): "64 64/3 64 64/5 64 64",
             (512, 8, 128, 256): "- - - - - -", (160, 8, 256, 512): "- - - - - -", (199, 8, 512, 1408): "64 - - - - -"}
    out = subprocess.run([str(tmp_path / "m")], input="\n".join(" ".join(map(str, k)) for k in sizes), capture_output=True, text=True, check=True)
    got = [l.strip() for l in out.stdout.split("\n") if l]
    assert got == list(sizes.values()), list(zip(sizes, got))
