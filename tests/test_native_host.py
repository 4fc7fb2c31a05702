"""Plain C++ parts of the runtime and of the kernels, compiled for the host and run without a GPU."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1911_05146_amd", "csrc")


def run_cpp(tmp_path, source):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(source)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-pthread", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
    return r.stdout.split()


@pytest.mark.parametrize("chunks", [1, 2, 8])
def test_a_collection_without_partners_ends_after_one_limit(tmp_path, chunks):
    """However many chunks of members there are; one that gets its words in time looks at all of them."""
    out = run_cpp(tmp_path, '''
#include <cstdio>
#include "hpf_wait.h"
using namespace hpf;
static unsigned looks(int nmem, unsigned in_vain_per_chunk) {
  unsigned n = 0;
  SpinBudget budget;
  for (int b = 0; more_chunks(b, nmem, budget); b += 8)
    for (unsigned k = 0;; ++k) {
      ++n;
      if (k >= in_vain_per_chunk) break;
      if (!budget.again()) break;
    }
  return n;
}
int main() { std::printf("%%u %%u %%u\\n", looks(8 * %d, ~0u), looks(8 * %d, 3), RES_SPIN_LIMIT); }
''' % (chunks, chunks))
    never, late, limit = map(int, out)
    assert never == limit + 1
    assert late == 4 * chunks
