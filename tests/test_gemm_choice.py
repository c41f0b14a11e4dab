"""The choice of a plain product's algorithm (csrc/pa_algo_cache.hpp), on the
CPU: nothing runs in a workspace smaller than it needs, neither a fresh
candidate nor a kept choice."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2502_02414_amd", "csrc")

HARNESS = r"""
#include "pa_algo_cache.hpp"
#include <cstdio>
#include <cstdlib>
#define CHECK(c) do { if (!(c)) { std::printf("line %d: %s\n", __LINE__, #c); std::exit(1); } } while (0)
int main() {
  // candidates (runs, bytes needed): one that does not run, one too large
  const bool ok[4] = {false, true, true, true};
  const size_t need[4] = {0, 65536, 4096, 0};
  auto pick = [&](int n, size_t ws) {
    return pa::first_fit(n, ws, [&](int i) { return ok[i]; }, [&](int i) { return need[i]; });
  };
  CHECK(pick(4, 65536) == 1);
  CHECK(pick(4, 65535) == 2);
  CHECK(pick(4, 0) == 3);
  CHECK(pick(3, 0) == -1);
  CHECK(pick(0, 1 << 20) == -1);

  pa::AlgoCache<int, int> c;
  int a = 0;
  CHECK(!c.find(7, 1000000, &a));
  c.keep(7, 1000000, 11, 65536);
  CHECK(c.find(7, 1000000, &a) && a == 11);
  CHECK(c.find(7, 65536, &a) && a == 11);    // the same MiB, large enough
  CHECK(!c.find(7, 65535, &a));              // the same MiB, too small
  CHECK(!c.find(7, 0, &a));                  // no workspace
  CHECK(!c.find(8, 1000000, &a));            // another problem
  c.keep(7, 0, 12, 0);                       // a choice for the small call ...
  CHECK(c.find(7, 0, &a) && a == 12);
  CHECK(c.find(7, 1000000, &a) && a == 11);  // ... that leaves the tuned one
  CHECK(!c.find(7, 4096, &a));
  c.keep(7, 1000000, 13, 4096);              // tuned again
  CHECK(c.find(7, 1000000, &a) && a == 13);
  CHECK(c.find(7, 4096, &a) && a == 13);
  c.keep(9, 1900000, 21, 1800000);           // 1.9 MB for a call with 1.1 MB
  CHECK(!c.find(9, 1100000, &a));
  return 0;
}
"""


def test_nothing_runs_in_a_workspace_too_small_for_it(tmp_path):
    src, exe = tmp_path / "choice.cpp", tmp_path / "choice"
    src.write_text(HARNESS)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Wextra", "-Werror", "-I", CSRC, str(src), "-o",
                    str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
