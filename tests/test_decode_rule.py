"""CPU checks of the rule by which wc_decode picks a launch's kernel
(DecodeLaunch in csrc/wc_internal.h), compiled on its own with the host
compiler, for a device of 256 compute units that holds 24 waves a unit of the
general kernel and 32 of the 16-wave one."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
DTYPES = {"bf16": (1, 2), "u8": (3, 1), "u4": (4, 1), "fp8_e4m3": (5, 1)}
CUS = 256

DRIVER = r"""
#include <stdio.h>
#include <stdlib.h>
#include "wc_internal.h"
// argv: cus, then dtype, decoded bytes, chunk bytes, lanes, tile rows (0: none; below 0:
// in column blocks) of every tensor
int main(int argc, char** argv) {
  const uint64_t cus = strtoull(argv[1], nullptr, 10);
  wc::DecodeLaunch launch;
  for (int i = 2; i + 4 < argc; i += 5) {
    wc::TensorInfo T;
    T.dtype = uint32_t(atoi(argv[i]));
    T.out_bytes = strtoull(argv[i + 1], nullptr, 10);
    T.chunk_bytes = uint32_t(atoi(argv[i + 2]));
    T.lanes = uint32_t(atoi(argv[i + 3]));
    T.tile_r = uint32_t(abs(atoi(argv[i + 4])));
    T.tile_order = atoi(argv[i + 4]) < 0 ? WC_TILE_COLUMN_BLOCKS : WC_TILE_ROWS;
    T.n_sym = wc::symbols_of(T.dtype, T.out_bytes);
    T.n_chunks = (T.out_bytes + T.chunk_bytes - 1) / T.chunk_bytes;
    launch.add(T);
  }
  const char* names[] = {"general", "wide", "small", "few"};
  puts(names[int(launch.kernel({cus, cus * 24, cus * 32}))]);
}
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    gxx = shutil.which("g++")
    if not gxx:
        pytest.skip("no host C++ compiler")
    d = tmp_path_factory.mktemp("rule")
    src, exe = d / "rule.cpp", d / "rule"
    src.write_text(DRIVER)
    subprocess.run([gxx, "-std=c++20", "-O1", "-Wall", "-Werror",
                    "-I" + os.path.join(ROOT, "paper_2606_15789_amd", "csrc"), str(src),
                    "-o", str(exe)], check=True, capture_output=True, text=True)

    def kernel(tensors, cus=CUS, chunk_bytes=65536, lanes=64, tiled=False):
        """tensors: (dtype, chunks) pairs."""
        args = [str(cus)]
        for dt, chunks in tensors:
            args += [str(DTYPES[dt][0]), str(int(chunks * chunk_bytes)), str(chunk_bytes),
                     str(lanes), str(int(tiled))]
        return subprocess.run([str(exe), *args], check=True, capture_output=True,
                              text=True).stdout.strip()

    return kernel


def test_windows_of_one_tensor(rule):
    assert rule([("bf16", 1)]) == "few"
    assert rule([("bf16", 4 * CUS)]) == "few"
    assert rule([("u4", 4 * CUS + 1)]) == "small"
    assert rule([("u4", 8 * CUS)]) == "small"
    assert rule([("u4", 8 * CUS + 1)]) == "general"
    assert rule([("bf16", 24 * CUS)]) == "general"
    assert rule([("bf16", 24 * CUS + 1)]) == "wide"
    assert rule([("bf16", 32 * CUS)]) == "wide"
    assert rule([("bf16", 32 * CUS + 1)]) == "general"
    assert rule([("bf16", 24 * CUS + 1)], tiled=True) == "general"
    assert rule([("u8", 24 * CUS + 1)]) == "general"
    assert rule([("u8", 1)], lanes=32) == "general"
    assert rule([("u8", 1)], cus=0) == "general"


def test_small_workgroups_beyond_the_compute_units_are_no_second_round(rule):
    """Short last workgroups count: 30 tensors of 65 chunks are 270 workgroups of
    eight."""
    assert rule([("u4", 65)] * 30) == "general"
    assert rule([("u4", 64)] * 32) == "small"
    assert rule([("u4", 2017)] + [("u4", 1)] * 31) == "general"
    assert rule([("u4", 1961)] + [("u4", 1)] * 10) == "small"  # 246 + 10 workgroups
    assert rule([("u4", 1961)] + [("u4", 1)] * 11) == "general"


def test_short_chunks_take_the_general_kernel(rule):
    """A launch whose longest chunk has fewer than 32 steps (2048 symbols)."""
    for dtype, nbytes in [("bf16", 4096), ("u8", 2048), ("u4", 1024)]:
        for n, chunks in [("few", 1000), ("small", 1300)]:
            assert rule([(dtype, chunks)], chunk_bytes=nbytes) == n
            assert rule([(dtype, chunks)], chunk_bytes=nbytes // 2) == "general"
    # one chunk that its tensor does not fill
    assert rule([("u8", 2048 / 65536)]) == "few"
    assert rule([("u8", 1984 / 65536)]) == "general"
    assert rule([("u8", 1 / 65536), ("bf16", 1)]) == "few"  # the longest counts


NO_ALLOCATION = r"""
#include <stdio.h>
#include <stdlib.h>
#include <new>
#include "wc_internal.h"
static bool full = false;  // memory has run out
void* operator new(size_t n) {
  void* p = full ? nullptr : malloc(n);
  if (!p) throw std::bad_alloc();
  return p;
}
void operator delete(void* p) noexcept { free(p); }
void operator delete(void* p, size_t) noexcept { free(p); }
int main() {
  static wc::PerDevice<wc::DecodeCapacity> known;
  full = true;
  int made = 0;
  for (int pass = 0; pass < 2; pass++)
    for (int dev = 0; dev < 64; dev++)
      if (known.get(dev, [&]() -> wc::DecodeCapacity {
                made++;
                return {uint64_t(dev), 1, 2};
              }).cus != uint64_t(dev))
        return 1;
  if (made != 64) return 2;
  // devices past the table, or none: worked out each time
  for (int dev : {64, 1000, -1})
    if (known.get(dev, [&]() -> wc::DecodeCapacity { return {7, 1, 2}; }).cus != 7) return 3;
  return 0;
}
"""


def test_device_figures_are_kept_without_an_allocation(tmp_path):
    """wc_decode asks for the device's figures on every launch of 64-lane chunks
    and promises its caller no allocation: none where memory has run out, and so
    no exception out of a C entry."""
    gxx = shutil.which("g++")
    if not gxx:
        pytest.skip("no host C++ compiler")
    src, exe = tmp_path / "a.cpp", tmp_path / "a"
    src.write_text(NO_ALLOCATION)
    subprocess.run([gxx, "-std=c++20", "-O1", "-Wall", "-Werror", "-pthread",
                    "-I" + os.path.join(ROOT, "paper_2606_15789_amd", "csrc"), str(src),
                    "-o", str(exe)], check=True, capture_output=True, text=True)
    assert subprocess.run([str(exe)]).returncode == 0


def test_overlapping_launches_of_many_words_a_step_take_the_general_kernel(rule):
    """From 5.5 chunks to a compute unit (int8, fp8 and short 16-bit chunks)."""
    assert rule([("u8", 1408)]) == rule([("fp8_e4m3", 1408)]) == "small"
    assert rule([("u8", 1409)]) == rule([("fp8_e4m3", 1409)]) == "general"
    assert rule([("bf16", 1408)], chunk_bytes=16384) == "small"
    assert rule([("bf16", 1409)], chunk_bytes=16384) == "general"
    assert rule([("bf16", 2048)], chunk_bytes=32768) == "small"
    assert rule([("u4", 2048)], chunk_bytes=4096) == "small"
    assert rule([("u4", 1400), ("u8", 400)]) == "small"    # 11 x 1400 + 16 x 400 <= 88 x 256
    assert rule([("u4", 1400), ("u8", 456)]) == "general"


def test_tall_column_blocks_take_the_general_kernel_above_four_chunks(rule):
    for dtype in ("bf16", "u4"):
        for rows in (-64, -128):
            assert rule([(dtype, 4 * CUS)], tiled=rows) == "few"
            assert rule([(dtype, 4 * CUS + 1)], tiled=rows) == "general"
        for rows in (64, -32, -16):
            assert rule([(dtype, 8 * CUS)], tiled=rows) == "small"
