// Blocks of memory kept for reuse.
#pragma once

#include <cstddef>
#include <map>
#include <mutex>
#include <tuple>
#include <unordered_map>
#include <utility>
#include <vector>

namespace rei {

// Idle blocks of destroyed instances, kept for new ones: a solve that is asked
// once (created, solved, destroyed) otherwise spends most of its time
// allocating.  Pinned host blocks above all (34-120 us to allocate, 60-160 us
// to free, one or more per instance; 64 KB at most each, 4 MB kept), and
// device blocks of up to 4 MB (16 us, 7 us to free; 64 MB kept per process).
// A block comes here only when no work that uses it is left (rei_destroy
// waits for the device as a free would), so any stream may take it.
// Beyond the bounds blocks are freed; rei_trim gives all idle ones back.
// Thread-safe; never destroyed (the process's end frees it).  Nothing here
// throws: where the host has no memory to remember a block by, the block is
// freed at its end instead of kept.
//
// Memory: take(host, bytes, &p) and give(host, p), an Error type, and its value
// kOk; a refused take leaves p null.
template <class Memory>
class BlockPool {
 public:
  using Error = typename Memory::Error;
  static BlockPool& get() {
    static BlockPool* p = new BlockPool();
    return *p;
  }
  Error take(int device, bool host, size_t bytes, void** out) {
    const size_t cls = size_class_of(bytes);
    const bool small = cls <= most(host);
    if (small) {
      std::lock_guard<std::mutex> lk(mu_);
      auto it = idle_.find(Key{device, host, cls});
      if (it != idle_.end() && !it->second.empty()) {
        *out = it->second.back();
        it->second.pop_back();
        kept_[host] -= cls;
        remember(*out, cls);
        return Memory::kOk;
      }
    }
    const size_t n = held(host, bytes);
    Error e = Memory::take(host, n, out);
    if (e != Memory::kOk) {  // idle blocks may be what is missing
      give_back();
      e = Memory::take(host, n, out);
    }
    if (e != Memory::kOk && n > bytes) return Memory::take(host, bytes, out);  // (freed at its end, not kept)
    if (e == Memory::kOk && small) {
      std::lock_guard<std::mutex> lk(mu_);
      remember(*out, cls);
    }
    return e;
  }
  void put(int device, bool host, void* p) {
    if (!keep(device, host, p)) Memory::give(host, p);
  }
  // Frees every idle block.
  void give_back() {
    Idle all;
    {
      std::lock_guard<std::mutex> lk(mu_);
      all.swap(idle_);
      kept_[0] = kept_[1] = 0;
    }
    for (auto& x : all)
      for (void* p : x.second) Memory::give(std::get<1>(x.first), p);
  }
  // Bytes that a block of this many takes.
  static size_t held(bool host, size_t bytes) {
    const size_t cls = size_class_of(bytes);
    return cls <= most(host) ? cls : bytes;
  }
  static size_t bound(bool host) { return host ? 4u << 20 : 64u << 20; }

 private:
  using Key = std::tuple<int, bool, size_t>;
  using Idle = std::map<Key, std::vector<void*>>;
  static size_t most(bool host) { return host ? 64u << 10 : 4u << 20; }
  static size_t size_class_of(size_t bytes) {
    size_t c = 4096;
    while (c < bytes) c <<= 1;
    return c;
  }
  // (the caller holds mu_)
  void remember(void* p, size_t cls) {
    try {
      lent_[p] = cls;
    } catch (...) {
    }
  }
  bool keep(int device, bool host, void* p) {
    std::lock_guard<std::mutex> lk(mu_);
    auto it = lent_.find(p);
    if (it == lent_.end()) return false;
    const size_t cls = it->second;
    lent_.erase(it);
    if (kept_[host] + cls > bound(host)) return false;
    try {
      idle_[Key{device, host, cls}].push_back(p);
    } catch (...) {
      return false;
    }
    kept_[host] += cls;
    return true;
  }
  std::mutex mu_;
  Idle idle_;
  std::unordered_map<void*, size_t> lent_;  // size class of each block of a class that is in use
  size_t kept_[2] = {0, 0};
};

}  // namespace rei
