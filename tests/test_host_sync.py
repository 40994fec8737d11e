"""The library's host-side order between threads, as host programs of their own: the launches of a call are enqueued together,
a limit that threads raise never falls."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2502_08246_amd", "csrc")


def run_program(tmp_path, source):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(source)
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr


def test_the_launches_of_a_call_are_enqueued_together(tmp_path):
    """Four threads on one stream, calls of three launches, one of them a call within the call."""
    run_program(tmp_path, r"""
#include <chrono>
#include <cstdio>
#include <thread>
#include <vector>
#include "host_sync.h"
std::mutex m;
std::vector<int> stream;                       // who launched, in the stream's order
void launch(int who) {
  { std::lock_guard<std::mutex> g(m); stream.push_back(who); }
  std::this_thread::sleep_for(std::chrono::microseconds(200));
}
void inner(int who) { const saap::InOrder call(&stream); launch(who); }
void outer(int who) { const saap::InOrder call(&stream); launch(who); inner(who); launch(who); }
int main() {
  std::vector<std::thread> t;
  for (int w = 0; w < 4; ++w) t.emplace_back([w] { for (int i = 0; i < 40; ++i) outer(w); });
  for (auto& x : t) x.join();
  for (size_t i = 0; i < stream.size(); i += 3)
    if (stream[i] != stream[i + 1] || stream[i] != stream[i + 2]) return printf("calls mixed at launch %zu\n", i), 1;
  return stream.size() == 480 ? 0 : 2;
}
""")


def test_a_limit_that_threads_raise_never_falls(tmp_path):
    """What is remembered is what was set last, and every thread goes on under a limit that is large enough for it."""
    run_program(tmp_path, r"""
#include <chrono>
#include <cstdio>
#include <thread>
#include <vector>
#include "host_sync.h"
std::atomic<int> set_to{0}, wrong{0};
int main() {
  for (int round = 0; round < 50; ++round) {
    std::atomic<int> limit{0};
    set_to = 0;
    std::vector<std::thread> t;
    for (int w = 0; w < 8; ++w)
      t.emplace_back([&, w] {
        const int need = 1000 * (w * 5 % 8 + 1);
        const bool ok = saap::raise_limit(limit, need, [](int bytes) {
          std::this_thread::sleep_for(std::chrono::microseconds(bytes / 100));
          set_to = bytes;
          return true;
        });
        if (!ok || set_to < need) ++wrong;
      });
    for (auto& x : t) x.join();
    if (set_to != 8000 || limit != 8000) ++wrong;
  }
  std::atomic<int> limit{5};
  if (saap::raise_limit(limit, 6, [](int) { return false; }) || limit != 5) ++wrong;
  if (wrong) printf("%d wrong\n", wrong.load());
  return wrong ? 1 : 0;
}
""")
