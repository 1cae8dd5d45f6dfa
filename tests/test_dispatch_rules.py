"""The host rules that choose a kernel form or tile by sizes
(paper_2004_11863_amd/csrc/rules.hpp), compiled for the CPU and asked on both
sides of their lines."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2004_11863_amd", "csrc")

DRIVER = r"""
#include "rules.hpp"
#include <cstdio>
#include <cstdlib>
#include <cstring>
using namespace lbm;
static Geo geo(int mx, int my, int mz, int bytes) {
  Geo g{};
  g.D = 3;
  g.has_fine = 1;
  const int m[3] = {mx, my, mz};
  for (int k = 0; k < 3; ++k) {
    g.m[k] = m[k];
    g.nf[k] = 2 * m[k] + 1;
  }
  const int xo = 16 / bytes - 1;
  g.fxo = xo;
  g.pf = (g.nf[0] + xo + 3) / 4 * 4;
  g.Nf = (int64_t)g.nf[0] * g.nf[1] * g.nf[2];
  g.Nfp = (int64_t)g.pf * g.nf[1] * g.nf[2];
  return g;
}
int main(int argc, char** argv) {
  const char* what = argv[1];
  auto arg = [&](int k) { return atoi(argv[2 + k]); };
  if (!strcmp(what, "zcap")) {
    const Geo g = geo(arg(1), arg(2), arg(3), arg(0));
    printf("%d\n", arg(0) == 4 ? fine3_zcap<float>(g) : fine3_zcap<double>(g));
  }
  if (!strcmp(what, "fine3")) {
    const Geo g = geo(arg(1), arg(2), arg(3), arg(0));
    const double bytes = 2.0 * 19 * arg(0) * (double)g.Nfp;
    printf("%d\n", arg(0) == 4 ? fine3_by_default<float>(g, bytes) : fine3_by_default<double>(g, bytes));
  }
  if (!strcmp(what, "hrr3")) {
    const Geo g = geo(arg(1), arg(2), arg(3), arg(0));
    const double bytes = 2.0 * 19 * arg(0) * (double)g.Nfp;
    printf("%d\n", arg(0) == 4 ? hrr3_fine_by_default<float>(g, bytes) : hrr3_fine_by_default<double>(g, bytes));
  }
  if (!strcmp(what, "hrr3c")) {
    const int n[3] = {arg(1), arg(2), arg(3)};
    const double bytes = 2.0 * 19 * arg(0) * n[0] * n[1] * n[2];
    printf("%d\n", arg(0) == 4 ? hrr3_coarse_by_default<float>(n, bytes) : hrr3_coarse_by_default<double>(n, bytes));
  }
  if (!strcmp(what, "wide194")) printf("%d\n", (int)wide194(arg(0)));
  if (!strcmp(what, "tall66")) printf("%d\n", (int)tall66(arg(0), arg(1) != 0));
  if (!strcmp(what, "cap")) printf("%d\n", hrr_cap(arg(0), arg(1)));
  return 0;
}
"""


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    src, exe = d / "rules.cpp", d / "rules"
    src.write_text(DRIVER)
    subprocess.check_call(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", CSRC, "-I", "/opt/rocm/include",
                           "-Wno-attributes", "-o", str(exe), str(src)])

    def call(*args):
        return int(subprocess.check_output([str(exe), *map(str, args)]))

    return call


def longest_run(cells, nbytes):
    """Planes of a run whose storage window (four planes more, and a storage block of 32 KB per population at
    either end) stays below 2^31 bytes; none where the x-band copy (five nodes of every row on two sides) does not."""
    nf = [2 * m + 1 for m in cells]
    if 2 * 19 * 5 * nf[1] * nf[2] * nbytes >= 2 ** 31:
        return 0
    row = (nf[0] + 16 // nbytes - 1 + 3) // 4 * 4
    return max(0, (2 ** 31 - 2 * 19 * 32768) // (row * nf[1] * 19 * nbytes) - 4)


@pytest.mark.parametrize("cells,nbytes,fits", [
    ((192, 192, 192), 4, True),
    ((1186, 1186, 8), 4, True),     # planes of 428.5 MB: five of them and the blocks
    ((1187, 1187, 8), 4, False),    # 429.6 MB
    ((1200, 1200, 4), 4, False),
    ((8, 839, 840), 4, True),       # x-band copies of 2.145e9 and
    ((8, 840, 840), 4, False),      # 2.148e9 bytes
    ((4, 593, 593), 8, True),
    ((4, 594, 594), 8, False),
    ((600, 1180, 4), 8, False),
])
def test_marching_fine_kernel_limits(ask, cells, nbytes, fits):
    zcap = ask("zcap", nbytes, *cells)
    assert zcap == longest_run(cells, nbytes)
    assert (zcap > 0) == fits


@pytest.mark.parametrize("cells,nbytes,march", [
    ((42, 42, 42), 4, False), ((48, 48, 48), 4, True), ((64, 64, 64), 4, True), ((192, 192, 192), 4, True),
    # thin in y or z
    ((100, 16, 100), 4, False), ((60, 30, 60), 4, True), ((60, 60, 30), 4, True),
    ((110, 110, 28), 4, False), ((110, 36, 110), 4, False), ((110, 40, 110), 4, True),
    ((150, 150, 24), 4, False), ((200, 12, 200), 4, False), ((300, 30, 60), 4, True),
    ((300, 300, 8), 4, False), ((300, 300, 16), 4, True),
    # short rows
    ((4, 200, 200), 4, False), ((16, 150, 150), 4, False), ((26, 150, 150), 4, True),
    ((33, 100, 100), 4, False), ((40, 100, 100), 4, True), ((30, 60, 60), 4, False),
    # rows that fill tiles of 192 nodes
    ((90, 90, 24), 4, True), ((90, 28, 90), 4, True), ((90, 90, 20), 4, True), ((90, 90, 17), 4, False),
    # rows of several tiles in levels that the memory-side cache holds
    ((90, 90, 14), 4, True), ((200, 20, 30), 4, True), ((200, 60, 8), 4, True), ((300, 20, 7), 4, False),
    ((60, 60, 23), 4, False), ((110, 110, 11), 4, False), ((110, 14, 110), 4, False),
    # short runs
    ((880, 880, 16), 4, False), ((765, 765, 16), 4, True),
    # double
    ((56, 56, 56), 8, False), ((64, 64, 64), 8, True), ((4, 200, 200), 8, False), ((24, 150, 150), 8, True),
    ((300, 300, 8), 8, False), ((150, 150, 12), 8, True),
])
def test_marching_fine_kernel_by_default(ask, cells, nbytes, march):
    assert ask("fine3", nbytes, *cells) == int(march)


@pytest.mark.parametrize("cells,nbytes,one_pass", [
    ((40, 40, 40), 4, False), ((44, 44, 44), 4, True), ((128, 128, 128), 4, True),
    ((4, 200, 200), 4, False), ((18, 150, 150), 4, False), ((22, 150, 150), 4, True),
    ((150, 150, 8), 4, True), ((200, 4, 200), 4, True),
    ((4, 200, 200), 8, False), ((8, 150, 150), 8, False), ((10, 150, 150), 8, True), ((64, 64, 64), 8, True),
])
def test_one_pass_hrr_fine_by_default(ask, cells, nbytes, one_pass):
    assert ask("hrr3", nbytes, *cells) == int(one_pass)


@pytest.mark.parametrize("n,nbytes,one_pass", [
    ((200, 200, 200), 4, False), ((256, 256, 256), 4, True), ((384, 384, 384), 4, True),
    ((130, 350, 350), 4, True), ((160, 350, 350), 4, True), ((192, 300, 300), 4, True),
    ((193, 300, 300), 4, False), ((204, 300, 300), 4, False), ((205, 300, 300), 4, True),
    ((257, 300, 300), 4, False), ((297, 300, 300), 4, False), ((298, 300, 300), 4, True),
    ((180, 180, 180), 8, False), ((200, 200, 200), 8, True), ((66, 320, 320), 8, True),
])
def test_one_pass_hrr_coarse_by_default(ask, n, nbytes, one_pass):
    assert ask("hrr3c", nbytes, *n) == int(one_pass)


@pytest.mark.parametrize("row,wide", [(64, 0), (128, 0), (129, 1), (160, 1), (192, 1), (193, 0), (256, 0), (300, 0),
                                      (383, 0), (384, 0), (512, 0), (513, 1), (576, 1), (577, 0), (896, 0), (897, 1), (960, 1),
                                      (961, 0)])
def test_wide_tiles_of_192_columns(ask, row, wide):
    assert ask("wide194", row) == wide


@pytest.mark.parametrize("row,rr,hrr", [(95, 1, 0), (128, 1, 0), (129, 0, 0), (192, 0, 0), (193, 1, 1), (207, 1, 1),
                                        (215, 1, 1), (216, 0, 0), (239, 0, 0), (255, 0, 0), (257, 0, 0), (383, 0, 0)])
def test_tall_tiles_by_default(ask, row, rr, hrr):
    assert (ask("tall66", row, 0), ask("tall66", row, 1)) == (rr, hrr)


def test_two_pass_hrr_collision_residency(ask):
    """D2Q9 not capped; D3Q19 two work groups a CU (LDS variant 2), three for variant 1: an index that names a
    one-pass tile does not choose a cap."""
    assert [ask("cap", 2, v) for v in range(4)] == [0, 0, 0, 0]
    assert [ask("cap", 3, v) for v in range(4)] == [2, 1, 2, 2]
