"""The pool of pinned memory for result downloads (wd_pinned.h), on the host
with an allocator that counts and can fail."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = r"""
#include <cassert>
#include <cstdio>
#include <cstdlib>
#include <map>
#include <thread>
#include <vector>

#include "wd_pinned.h"

static std::mutex mu;
static std::map<char*, uint64_t> live;  // (addresses only: nothing is touched)
static uint64_t largest = 0;
static int allocs = 0;
static bool fails = false;
struct Host {
  static char* alloc(uint64_t n) {
    std::lock_guard<std::mutex> lk(mu);
    if (fails) return nullptr;
    ++allocs;
    largest = n > largest ? n : largest;
    char* p = (char*)malloc(1);
    live[p] = n;
    return p;
  }
  static void release(char* p) {
    std::lock_guard<std::mutex> lk(mu);
    assert(live.erase(p) == 1);
    free(p);
  }
};
typedef wd::PinnedPool<Host> Pool;
#define CHECK(x) do { if (!(x)) { printf("line %d: %s\n", __LINE__, #x); return 1; } } while (0)

int main() {
  const uint64_t MB = 1 << 20;
  {  // at most kPinnedBlocks leased; given back with the last holder; the block that holds the bytes is taken
    Pool p;
    auto a = p.lease(10 * MB), b = p.lease(2 * MB), c = p.lease(100);
    CHECK(a && b && c && a->data() != b->data() && b->data() != c->data());
    CHECK(!p.lease(1));
    CHECK(live[c->data()] == wd::kPinnedMin);
    auto a2 = a;
    char* at = a->data();
    a.reset();
    CHECK(!p.lease(1));
    a2.reset();
    b.reset();
    const int n = allocs;
    auto d = p.lease(9 * MB);
    CHECK(d && d->data() == at && allocs == n);
    CHECK(p.lease(MB) && allocs == n);
    // the block that is never leased
    std::lock_guard<std::mutex> lk(p.stage_lock());
    char* s = p.stage(3 * MB);
    CHECK(s && s == p.stage(MB) && s != d->data());
  }
  {  // no block beyond kPinnedMax, and none for more than it
    Pool p;
    largest = 0;
    CHECK(!p.lease(wd::kPinnedMax + 1) && !p.stage(wd::kPinnedMax + 1));
    CHECK(p.lease(wd::kPinnedMax) && p.lease(wd::kPinnedMax - 5) && p.stage(wd::kPinnedMax - 1));
    CHECK(largest <= wd::kPinnedMax);
  }
  {  // memory that cannot be pinned: no block, and a block again once it can
    Pool p;
    fails = true;
    CHECK(!p.lease(MB) && !p.lease(MB) && !p.lease(MB) && !p.lease(MB) && !p.stage(MB));
    fails = false;
    auto a = p.lease(MB), b = p.lease(MB), c = p.lease(MB);
    CHECK(a && b && c && p.stage(MB));
    a.reset();
    fails = true;
    CHECK(!p.lease(50 * MB));
    fails = false;
    CHECK((a = p.lease(MB)));
  }
  {  // threads: never a block to two holders at once
    Pool p;
    std::mutex m;
    std::map<char*, int> held;
    std::vector<std::thread> th;
    bool bad = false;
    for (int t = 0; t < 8; ++t)
      th.emplace_back([&, t] {
        for (int i = 0; i < 3000; ++i) {
          auto l = p.lease((1 + (i * 7 + t) % 5) * MB);
          if (!l) continue;
          { std::lock_guard<std::mutex> lk(m); if (held[l->data()]++) bad = true; }
          { std::lock_guard<std::mutex> lk(m); --held[l->data()]; }
        }
      });
    for (auto& t : th) t.join();
    CHECK(!bad);
  }
  return 0;
}
"""


def test_pinned_pool(tmp_path):
    (tmp_path / "pool.cpp").write_text(SRC)
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-pthread", "-I",
                    os.path.join(ROOT, "paper_1804_03243_amd", "csrc"), "-o", str(tmp_path / "pool"),
                    str(tmp_path / "pool.cpp")], check=True)
    r = subprocess.run([str(tmp_path / "pool")], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
