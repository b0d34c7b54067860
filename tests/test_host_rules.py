"""Rules of the launches that the C++ headers hold, compiled for the host and called."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEAD = '#include <cstdio>\n#include <cstdlib>\n#include <vector>\n#include "common.h"\n#include "host_util.h"\nusing namespace mplpxx;\n'


@pytest.fixture
def run(tmp_path):
    def go(body):
        src, exe = tmp_path / "rules.cpp", tmp_path / "rules"
        src.write_text(HEAD + "#define CHECK(c) do { if (!(c)) { std::printf(\"%d: %s\\n\", __LINE__, #c); std::exit(1); } } while (0)\n"
                       + "int main() {\n" + body + "\n}\n")
        cmd = ["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", f"-I{ROOT}/include",
               f"-I{ROOT}/paper_2004_08227_amd/csrc", str(src), "-o", str(exe), "-L/opt/rocm/lib", "-lamdhip64",
               "-Wl,-rpath,/opt/rocm/lib"]
        subprocess.run(cmd, check=True, capture_output=True, text=True)
        r = subprocess.run([str(exe)], capture_output=True, text=True)
        assert r.returncode == 0, r.stdout
    return go


def test_strided_launches_hold_any_count(run):
    run("""
  for (size_t c : {(size_t)0, (size_t)1, (size_t)kMaxBlocks - 1, (size_t)kMaxBlocks, (size_t)kMaxBlocks + 1, (size_t)1 << 25,
                   (size_t)1 << 26, (size_t)0x3fffffff, (size_t)0x7fffffff}) {
    const size_t b = stride_blocks(c);
    CHECK(b <= c && (c == 0 || b > 0) && b * 1024 < ((size_t)1 << 32));
  }""")


def test_iterations_of_a_launch_are_counted_in_31_bits(run):
    run("""
  for (int k : {0, 1, 7, 130000, 2147483647})
    for (long long m : {1ll, 2ll, 4950ll, 4498500ll, 0x3fffffffll})
      for (int grid : {1, 2, 100, 256, 1024}) {
        const long long owned = (m + grid - 1) / grid;
        if (owned > 1000000 && k > 130000) continue;
        int sum = 0, calls = 0;
        CHECK(in_launches(k, m, grid, [&](int done, int c) {
          CHECK(done == sum && c >= 1 && owned * c <= (c == 1 ? owned : 1ll << 30));
          sum += c;
          ++calls;
          return hipSuccess;
        }) == hipSuccess);
        CHECK(sum == k && (owned * k > (1ll << 30) || calls == (k > 0)));
      }
  int calls = 0;
  CHECK(in_launches(5, 1ll << 40, 1, [&](int, int) { return ++calls == 2 ? hipErrorUnknown : hipSuccess; }) == hipErrorUnknown);
  CHECK(calls == 2);""")


def test_workgroups_on_dies(run):
    """Every logical workgroup once, positions of one matching in blocks on the dies, and the
    plain order wherever the mapped launch would not fit or the sizes do not suit it."""
    run("""
  int mapped = 0, beyond = 0;
  for (int ms = 1; ms <= 300; ++ms)
    for (int d = 1; d <= 5; ++d)
      for (int cap : {64, 256, 512}) {
        const int G = ms * d, launch = kDies * ((ms + kDies - 1) / kDies) * d;
        const WgMap w = wg_map(G, ms, true, 1 << 20, cap);
        CHECK(w.G == G);
        if (ms < kDies || launch > cap) {
          beyond += ms >= kDies;
          CHECK(w.ms == 0 && w.launch == G);
          for (int b = 0; b < G; ++b) CHECK(wg_logical(w, b) == b);
          continue;
        }
        ++mapped;
        CHECK(w.ms == ms && w.launch == launch && launch <= cap);
        std::vector<int> seen(G, 0);
        for (int b = 0; b < launch; ++b) {
          const int g = wg_logical(w, b);
          CHECK(g >= 0 && g <= G);
          if (g == G) continue;
          ++seen[g];
          const int die = b % kDies, p = g % ms;  // the die's block of neighbouring positions
          CHECK(p >= die * ms / kDies && p < (die + 1) * ms / kDies);
        }
        for (int x : seen) CHECK(x == 1);
      }
  CHECK(mapped > 300 && beyond > 300);
  CHECK(wg_map(243, 81, true, 1 << 20, 256).ms == 0);                  // 264 workgroups
  CHECK(wg_map(20, 10, false, 1 << 20, 256).ms == 0);                  // unequal matchings
  CHECK(wg_map(21, 10, true, 1 << 20, 256).ms == 0);                   // no multiple
  CHECK(wg_map(20, 10, true, kLastLevelCache, 256).ms == 10);
  CHECK(wg_map(20, 10, true, kLastLevelCache + 1, 256).ms == 0);""")
