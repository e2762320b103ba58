"""The host arithmetic that buffer sizes and kernel index bounds rest on
(csrc/jpi_bounds.h), over every shape class the library accepts: a small C++
program is compiled from the header and run, no GPU needed."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2607_12659_amd", "csrc")

PROGRAMS = {
    # every prefix length that a binding accepts (action-time variant: below max_prefix) fits the bound, and the first
    # block that a wave of the few-row attention reads without knowing the length lies in the rollout's blocks
    "key_bound": """
  for (int pmax = 1; pmax <= 1100; ++pmax)
    for (int prefix = pmax > 70 ? pmax - 70 : 0; prefix <= pmax; ++prefix)
      for (int at = 0; at < 2; ++at) {
        const int bound = jpi::key_bound(prefix, pmax, at), longest = at ? (prefix < pmax ? prefix : pmax - 1) + 1 : prefix;
        CHECK(bound >= longest && bound <= pmax);
        for (int own = 1; own <= 2; ++own)
          for (int jb0 = 0; jb0 < 32; ++jb0) {
            const int last = own + jpi::kv_blocks(bound) - 1, first = jb0 < last ? jb0 : last;
            CHECK(first - own < jpi::kv_blocks(pmax));
          }
      }
""",
    # the slices of every batch of tokens fit the buffer, which stays small however many tokens a module is made for
    "xkv_slices": """
  for (int n_cu : {64, 256, 304})
    for (int N = 128; N <= 512; N *= 2) {
      const size_t Mmax = 1u << 20, room = jpi::xkv_slice_elems(Mmax, N, n_cu);
      CHECK(room <= (size_t)32768 * n_cu);
      for (int M = 1; M <= (1 << 20); M += M < 20000 ? 1 : 997) {
        const int s = jpi::xkv_slices(M, N, n_cu);
        CHECK(s == 1 || s == 2 || s == 4);
        CHECK(s == 1 || (size_t)s * M * N <= room);
        CHECK(s == 1 || (size_t)s * M * N <= jpi::xkv_slice_elems(M, N, n_cu));
        CHECK(M > 64 || s == 1);
      }
    }
""",
    # z holds the GeGLU output of every row and, in the action-time variant, the action-time MLP's W columns
    "z_columns": """
  for (size_t W = 64; W <= 4096; W += 64)
    for (size_t F = 64; F <= 4096; F += 64)
      for (int at = 0; at < 2; ++at) {
        const size_t z = jpi::z_columns(W, F, at);
        CHECK(z >= F && (!at || z >= W));
        CHECK(z == F || (at && z == W));
      }
""",
}


@pytest.mark.parametrize("name", sorted(PROGRAMS))
def test_bounds(name, tmp_path):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text('#include <cstdio>\n#include <initializer_list>\n#include "jpi_bounds.h"\n'
                   '#define CHECK(x) do { if (!(x)) { std::printf("line %d: %s\\n", __LINE__, #x); return 1; } } while (0)\n'
                   "int main() {" + PROGRAMS[name] + "  return 0;\n}\n")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], stdout=subprocess.PIPE, text=True)
    assert r.returncode == 0, r.stdout
