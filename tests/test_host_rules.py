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
