"""Host check of the rules by which device blocks are kept between calls
(csrc/kdt_blocks.h): the class is host code over a backend, here a model of streams
whose work finishes late, which are destroyed at any time and whose handles go to new
streams.  Whoever takes a block must be ordered after all work that still uses it, the idle
bytes stay within their limits, no block is lost or given out twice, and nothing
throws when host memory or events run out.  The same harness with every handle
trusted to name one stream for good (as if streams were never destroyed) must find a fault."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2609_18316_amd", "csrc")

HARNESS = r"""
#include <cstdio>
#include <cstdlib>
#include <map>
#include <new>
#include <random>
#include <set>
#include <vector>
#include "kdt_blocks.h"

static long g_fail_new = -1;  // operator new fails when this reaches 0
void* operator new(size_t n) {
  if (g_fail_new >= 0 && g_fail_new-- == 0) throw std::bad_alloc();
  if (void* p = std::malloc(n)) return p;
  throw std::bad_alloc();
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }

using kdt::BlockCache;
// A point on a stream's queue; a stream is named by a number of its own, never reused.
struct At { int stream; int pos; bool operator<(const At& o) const { return stream != o.stream ? stream < o.stream : pos < o.pos; } };
struct World {
  std::vector<int> queued, done;      // per stream: work queued, work finished
  std::vector<std::set<At>> waits;    // what a stream's work from here on is ordered after
  int of_handle[5];                   // the stream a handle names now (0: the null stream)
  std::map<char*, std::set<At>> uses; // work that may still use an allocated block
  std::map<char*, size_t> size;
  size_t next = 4096;
  bool events_run_out = false;
  int fresh() { queued.push_back(0); done.push_back(0); waits.emplace_back(); return (int)queued.size() - 1; }
  bool ordered(int s, At a) const {
    if (done[a.stream] >= a.pos || a.stream == s) return true;
    for (const At& w : waits[s]) if (w.stream == a.stream && w.pos >= a.pos) return true;
    return false;
  }
  void die(const char* what) { std::printf("fault: %s\n", what); std::exit(1); }
  void use_ok(char* p, int s) { for (const At& a : uses[p]) if (!ordered(s, a)) die("a block is used before earlier work is done"); }
} W;
struct Model {
  using Stream = int;   // a handle
  using Event = At;
  bool permanent(int h) {
#ifdef TRUST_HANDLES
    return true;
#else
    return h == 0;
#endif
  }
  bool record(At* e, int h) { if (W.events_run_out) return false; const int s = W.of_handle[h]; *e = At{s, W.queued[s]}; return true; }
  bool passed(At e) { return W.done[e.stream] >= e.pos; }
  bool order_after(int h, At e) {
    const long f = g_fail_new;
    g_fail_new = -1;  // (the model's own memory suffices)
    W.waits[W.of_handle[h]].insert(e);
    g_fail_new = f;
    return true;
  }
  void forget(At) {}
  bool free(void* p, int h) {
    char* c = (char*)p;
    if (!W.size.count(c)) W.die("freed twice");
    W.use_ok(c, W.of_handle[h]);
    W.size.erase(c);
    W.uses.erase(c);
    return true;
  }
  bool finish(int h, const At* e) {
    if (e) W.done[e->stream] = std::max(W.done[e->stream], e->pos);
    else W.done[W.of_handle[h]] = W.queued[W.of_handle[h]];
    return true;
  }
};

int main() {
  std::mt19937 g(2609);
  for (int h = 0; h < 5; ++h) W.of_handle[h] = W.fresh();
  auto* c = new BlockCache<Model>();
  struct Held { char* p; int handle; int stream; };
  std::vector<Held> held;
  long hits = 0, lost_streams = 0;
  for (int step = 0; step < 200000; ++step) {
    const int h = g() % 5, s = W.of_handle[h];
    W.events_run_out = g() % 64 == 0;
    const bool starve = g() % 32 == 0;  // host memory runs out somewhere in the call
    switch (g() % 8) {
      case 0: case 1: case 2: {  // a call takes a block and queues work that uses it
        const size_t bytes = g() % 3 == 0 ? (g() % 9 + 100) << 20 : size_t(1) << (8 + g() % 18);
        g_fail_new = starve ? g() % 3 : -1;
        char* p = (char*)c->take(0, bytes, h);
        g_fail_new = -1;
        if (p) {
          ++hits;
          for (const Held& x : held) if (x.p == p) W.die("a block in use is given out");
          W.use_ok(p, s);
        } else {
          p = (char*)(W.next += 4096);
          W.size[p] = kdt::block_size(bytes);
          g_fail_new = starve ? g() % 2 : -1;
          c->adopt(p, 0, W.size[p]);
          g_fail_new = -1;
        }
        if (W.size[p] < bytes) W.die("a block is too small");
        W.uses[p] = {At{s, ++W.queued[s]}};  // (ordered after every earlier use)
        held.push_back({p, h, s});
        break;
      }
      case 3: case 4: {  // a call gives its blocks on a stream back
        void* out[4];
        size_t n = 0;
        for (size_t i = 0; i < held.size() && n < 4;)
          if (held[i].handle == h && held[i].stream == s) { out[n++] = held[i].p; held.erase(held.begin() + i); }
          else ++i;
        g_fail_new = starve ? g() % 4 : -1;
        c->give(out, n, h, g() % 16 != 0);
        g_fail_new = -1;
        break;
      }
      case 5: W.done[s] += (W.queued[s] - W.done[s] + 1) / 2; break;  // work finishes
      case 6:  // a stream is destroyed with work queued; its handle names a new one
        if (h != 0 && g() % 4 == 0) {
          bool busy = false;
          for (const Held& x : held) busy |= x.stream == s;
          if (!busy) { W.of_handle[h] = W.fresh(); ++lost_streams; }
        }
        break;
      default:
        if (g() % 16 == 0) { if (!c->release(0, h)) W.die("release"); if (c->idle_bytes(0, &h)) W.die("release left blocks"); }
        else if (g() % 64 == 0) { c->release_all(0, 0); if (c->idle_bytes(0, nullptr)) W.die("release_all left blocks"); }
    }
    if (c->idle_bytes(0, nullptr) > kdt::kKeepAll || c->idle_bytes(0, &h) > kdt::kKeepStream) W.die("too much is kept");
  }
  c->release_all(0, 0);
  if (W.size.size() != held.size()) W.die("a block is lost");
  std::printf("sound: %ld blocks served again, %ld streams destroyed\n", hits, lost_streams);
  return hits > 1000 && lost_streams > 100 ? 0 : 2;
}
"""


def _run(tmp_path, extra):
    if shutil.which("g++") is None:
        pytest.skip("g++ is not available")
    src = tmp_path / "blocks.cpp"
    src.write_text(HARNESS)
    exe = tmp_path / "blocks"
    subprocess.run(["g++", "-O2", "-std=c++17", *extra, "-I", CSRC, str(src), "-o", str(exe),
                    "-lpthread"], check=True, capture_output=True, text=True)
    return subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)


def test_blocks_are_never_used_before_earlier_work_is_done(tmp_path):
    r = _run(tmp_path, [])
    assert r.returncode == 0, r.stdout + r.stderr
    assert r.stdout.startswith("sound: ")


def test_the_check_fails_where_handles_are_trusted(tmp_path):
    r = _run(tmp_path, ["-DTRUST_HANDLES"])
    assert r.returncode == 1 and r.stdout.startswith("fault: a block is used before"), r.stdout
