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


def test_operands_asked_for_ahead_have_the_shape_of_the_run(tmp_path):
    """What block bi of an inference run asks for ahead belongs to a block of that run, and never to the lead, whose first matrix and table are half as large."""
    run_cpp(tmp_path, '''
#include <cstdio>
#include "hpf_ahead.h"
int main() {
  for (int lead = 0; lead < 2; ++lead)
    for (int nblk = 1; nblk < 6; ++nblk)
      for (int bi = 0; bi < nblk; ++bi)
        for (int distance = 1; distance < 3; ++distance) {
          const int b = hpf::block_ahead(lead, bi, distance, nblk);
          const bool alone = lead && nblk == 1;
          if (alone ? b != -1 : b < lead || b >= nblk || (bi + distance < nblk && b != bi + distance)) { std::printf("%d %d %d %d: %d\\n", lead, nblk, bi, distance, b); return 1; }
        }
  return 0;
}
''')


def _figures(tmp_path, kind, c, mid, px, count, lead):
    out = run_cpp(tmp_path, '''
#include <cstdio>
#include "hpf_figures.h"
int main() {
  const hpf::RunFigures f = hpf::run_figures(%d, %d, %d, %d, %d, %d);
  std::printf("%%.0f %%.0f %%.0f %%.0f %%.0f %%.0f\\n", f.forward, f.inference, f.backward, f.flops, f.wgrad, f.wgrad_flops);
}
''' % (kind, c, mid, px, count, lead))
    return [int(v) for v in out]


LED_RUNS = [(0, 32, 32, 16, 18), (0, 64, 64, 8, 1), (1, 128, 32, 16, 7), (1, 128, 64, 16, 1), (2, 64, 64, 8, 3)]


@pytest.mark.parametrize("kind,c,mid,hw,blocks,lead", [(*r, lead) for lead in (0, 1) for r in LED_RUNS] + [(1, 256, 64, 8, 4, 0)])
def test_algorithmic_figures_of_a_run(tmp_path, kind, c, mid, hw, blocks, lead):
    """Every tensor of the run once, block by block, and 2*M*K*N per contraction; the block that leads a run in has twice the image edge and half the channels in front."""
    px = hw * hw
    fwd = bwd = flops = wgrad = wflops = 0
    for i in range(blocks):
        led = lead and i == 0
        x = 4 * px * c // 2 if led else px * c            # the block's input, and its gradient
        ci, y = (c // 2 if led else c), px * c
        inner = [px * mid] * 2 if kind == 1 else [y] * (2 if kind == 2 else 1)     # outputs of the convolutions but the block's last (post-activation: all)
        extra = [y, y] if kind == 2 and led else []                               # the shortcut and relu(bn1(c1))
        if i == 0:
            fwd, bwd, infer = x, y, x + y                 # the run's input; the gradient of its output
        fwd += sum(inner) + sum(extra) + y
        if kind == 2:
            bwd += sum(inner) + y + sum(inner) + x + (y if led else 0)             # c1, c2, y read; their gradients, the input's and the shortcut's written
        else:
            bwd += x + sum(inner) + sum(inner) + x
        pairs = [(ci, mid, 1), (mid, mid, 9), (mid, c, 1)] if kind == 1 else [(ci, c, 9), (c, c, 9)]
        k = sum(a * b * t for a, b, t in pairs) + (ci * c if led else 0)
        flops += 2 * px * k
        if not led:
            wgrad += 2 * (y + sum(inner))
            wflops += 2 * px * k
    assert _figures(tmp_path, kind, c, mid, px, blocks, lead) == [fwd, infer, bwd, flops, wgrad, wflops]


FAKE_GPU = '''
#include <cstdio>
#include <cstdlib>
#include <map>
#include <random>
#include <set>
#include <thread>
#include <atomic>
#include <chrono>
#include "hpf_admission.h"
static std::set<int> g_finished;
static std::vector<std::pair<int, int>> g_waits;   // stream, event
struct Fake {
  using Stream = int; using Event = int;
  static bool finished(int ev) { return g_finished.count(ev) != 0; }
  static bool wait(int s, int ev) { g_waits.push_back({s, ev}); return true; }
};
#define CHECK(x) do { if (!(x)) { std::printf("failed: %s (line %d)\\n", #x, __LINE__); return 1; } } while (0)
'''


def test_calls_that_fit_are_admitted_while_another_one_is_issuing(tmp_path):
    """A call that is still capturing its graph holds no lock: threads with other partitions go ahead, on its device as long as both
    fit and on other devices always.  One that does not fit waits for it on the host, then for its event on the stream."""
    run_cpp(tmp_path, FAKE_GPU + '''
int main() {
  hpf::Admission<Fake> a;
  CHECK(a.enter(0, 256, 1, 200));                 // device 0, stream 1: under way from here on
  std::atomic<int> done{0};
  std::thread other([&] { a.enter(1, 256, 2, 256); a.record(1, 2, 20, nullptr); a.leave(1, 2); ++done; });
  std::thread fits([&] { a.enter(0, 256, 3, 56); a.record(0, 3, 30, nullptr); a.leave(0, 3); ++done; });
  for (int i = 0; i < 2000 && done < 2; ++i) std::this_thread::sleep_for(std::chrono::milliseconds(5));
  const int at_once = done;
  std::thread too_large([&] { a.enter(0, 256, 4, 100); a.record(0, 4, 40, nullptr); a.leave(0, 4); ++done; });
  std::this_thread::sleep_for(std::chrono::milliseconds(100));
  const int blocked = done;
  a.record(0, 1, 10, nullptr);
  a.leave(0, 1);
  other.join(); fits.join(); too_large.join();
  CHECK(at_once == 2 && blocked == 2 && done == 3);
  CHECK(g_waits.size() == 1 && g_waits[0] == std::make_pair(4, 10));   // 200 + 56 + 100 > 256: the largest holder is enough
  return 0;
}
''')


def test_two_threads_on_one_stream_keep_the_later_event(tmp_path):
    run_cpp(tmp_path, FAKE_GPU + '''
int main() {
  hpf::Admission<Fake> a;
  CHECK(a.enter(0, 256, 1, 100));
  std::atomic<int> second{0};
  std::thread t([&] { a.enter(0, 256, 1, 50); a.record(0, 1, 11, nullptr); a.leave(0, 1); second = 1; });
  std::this_thread::sleep_for(std::chrono::milliseconds(100));
  CHECK(second == 0);
  a.record(0, 1, 10, nullptr);
  a.leave(0, 1);
  t.join();
  CHECK(a.enter(0, 256, 2, 200));
  CHECK(g_waits.size() == 1 && g_waits[0] == std::make_pair(2, 11));
  // a call that fails before its first launch leaves no entry behind, a wait on whose event would be an error
  a.record(0, 2, 20, nullptr); a.leave(0, 2);
  g_finished = {11, 20};
  CHECK(a.enter(0, 256, 3, 8)); a.leave(0, 3);
  CHECK(a.enter(0, 256, 4, 256));
  CHECK(g_waits.size() == 1);
  // destroyed owners: nobody waits for their events any more
  a.record(0, 4, 40, &second); a.leave(0, 4);
  a.forget(&second);
  CHECK(a.enter(0, 256, 5, 256) && g_waits.size() == 1);
  return 0;
}
''')


@pytest.mark.parametrize("seed", [1, 2, 3])
def test_calls_that_can_overlap_always_fit(tmp_path, seed):
    """Random calls on random streams; a call overlaps everything that it does not follow through its stream or through the events that its
    stream waited for (transitively)."""
    run_cpp(tmp_path, FAKE_GPU + '''
int main() {
  std::mt19937 rng(%d);
  hpf::Admission<Fake> a;
  struct Call { int stream, cus; std::set<int> after; };
  std::map<int, Call> calls;                 // by event
  std::map<int, std::set<int>> order;        // per stream: all calls its next one follows
  for (int ev = 1; ev <= 4000; ++ev) {
    const int s = (int)(rng() %% 6), need = 8 * (1 + (int)(rng() %% (rng() %% 4 ? 8 : 32)));
    g_waits.clear();
    CHECK(a.enter(0, 256, s, need));
    for (auto& w : g_waits) { CHECK(w.first == s); order[s].insert(w.second); auto& f = calls[w.second].after; order[s].insert(f.begin(), f.end()); }
    std::map<int, int> most;                 // per other stream: the largest call that this one can overlap
    for (auto& [e, c] : calls)
      if (c.stream != s && !g_finished.count(e) && !order[s].count(e)) most[c.stream] = std::max(most[c.stream], c.cus);
    int total = need;
    for (auto& m : most) total += m.second;
    CHECK(total <= 256);
    a.record(0, s, ev, nullptr);
    a.leave(0, s);
    calls[ev] = Call{s, need, order[s]};
    order[s].insert(ev);
    if (rng() %% 8 == 0)                      // some stream drains
      for (int e : order[(int)(rng() %% 6)]) g_finished.insert(e);
    if (ev %% 64 == 0) {                      // forget what has finished
      for (int e : g_finished) { calls.erase(e); for (auto& o : order) o.second.erase(e); for (auto& c : calls) c.second.after.erase(e); }
    }
  }
  return 0;
}
''' % seed)
