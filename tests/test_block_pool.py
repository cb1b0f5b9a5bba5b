"""The pool of idle blocks on the CPU, over malloc: blocks are lent to one owner
at a time, kept up to the bounds, all given back in the end, and a host without
memory for the pool's own records costs a block its reuse and nothing else."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>
#include <set>
#include <thread>
#include <vector>
#include "block_pool.h"

static thread_local long countdown = -1;  // operator new fails when it reaches 0
static void* host_alloc(size_t n) {
  if (countdown == 0) throw std::bad_alloc();
  if (countdown > 0) --countdown;
  return std::malloc(n ? n : 1);
}
void* operator new(size_t n) { return host_alloc(n); }
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }

static std::atomic<long> taken{0}, given{0};
static std::atomic<size_t> most{~0ull};  // larger blocks are refused
struct Malloc {
  using Error = int;
  static constexpr Error kOk = 0;
  static Error take(bool, size_t n, void** out) {
    *out = n > most ? nullptr : std::malloc(n);
    taken += *out != nullptr;
    return *out ? 0 : 2;
  }
  static void give(bool, void* p) {
    ++given;
    std::free(p);
  }
};
using Pool = rei::BlockPool<Malloc>;

#define CHECK(x)                                                \
  do {                                                          \
    if (!(x)) {                                                 \
      std::printf("line %d: %s\n", __LINE__, #x);               \
      std::exit(1);                                             \
    }                                                           \
  } while (0)

static void* take(bool host, size_t n) {
  void* p = nullptr;
  CHECK(Pool::get().take(0, host, n, &p) == 0 && p);
  std::memset(p, 1, n);
  return p;
}

int main() {
  Pool& pool = Pool::get();
  // a block comes back for the next one of its size, the other kind's does not
  void* a = take(false, 5000);
  pool.put(0, false, a);
  CHECK(take(true, 5000) != a);
  CHECK(take(false, 8000) == a && taken == 2);
  // exact size where the rounded one is refused
  most = 70000;
  void* b = take(false, 66000);
  pool.put(0, false, b);
  CHECK(given == 1);
  void* none = &a;
  CHECK(pool.take(0, false, 80000, &none) != 0 && !none);
  most = ~0ull;
  // bounds: blocks beyond them are freed
  std::vector<void*> v;
  for (int k = 0; k < 40; ++k) v.push_back(take(false, 4 << 20));
  long before = given;
  for (void* p : v) pool.put(0, false, p);
  CHECK(given - before == 40 - (long)(Pool::bound(false) / (4 << 20)));
  pool.give_back();
  CHECK(given - before == 40);
  // the host's memory fails at every point of a life
  for (long n = 0; n < 40; ++n) {
    std::vector<void*> held(8, nullptr);
    countdown = n;
    for (int round = 0; round < 3; ++round) {
      for (size_t k = 0; k < held.size(); ++k) {
        CHECK(pool.take(k % 2, k % 3 == 0, 4096u << (k % 5), &held[k]) == 0);
        for (size_t q = 0; q < k; ++q) CHECK(held[q] != held[k]);
      }
      for (size_t k = 0; k < held.size(); ++k) pool.put(k % 2, k % 3 == 0, held[k]);
    }
    pool.give_back();
    countdown = -1;
  }
  // threads: no block has two owners
  std::vector<std::thread> ts;
  for (int t = 0; t < 8; ++t)
    ts.emplace_back([t] {
      for (int k = 0; k < 5000; ++k) {
        void* p[3];
        for (int q = 0; q < 3; ++q) {
          CHECK(Pool::get().take(0, q == 2, 3000 + 997 * q, &p[q]) == 0);
          std::memset(p[q], t * 3 + q, 3000 + 997 * q);
        }
        for (int q = 0; q < 3; ++q) {
          for (int i : {0, 1500, 2999}) CHECK(((unsigned char*)p[q])[i] == t * 3 + q);
          Pool::get().put(0, q == 2, p[q]);
        }
        if (k % 500 == 0) Pool::get().give_back();
      }
    });
  for (auto& t : ts) t.join();
  pool.give_back();
  CHECK(taken - given == 2);  // the two blocks still lent at the top
  std::puts("ok");
}
"""


def test_block_pool(tmp_path):
    src, exe = tmp_path / "pool.cpp", tmp_path / "pool"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-Wall", "-Werror", "-O1", "-pthread", "-I",
                           os.path.join(ROOT, "paper_2305_18575_amd", "csrc"), str(src), "-o", str(exe)])
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert (out.returncode, out.stdout.strip()) == (0, "ok"), (out.stdout, out.stderr)
