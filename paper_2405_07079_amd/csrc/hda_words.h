// Result words of call-by-call heaps (host side): pinned host memory, one
// cache line a word, 64 to a page.
#pragma once
#include <stddef.h>
#include <stdint.h>

#include <mutex>
#include <vector>

namespace hda {

// A page is made when no word is free (making one takes 0.1 ms, which each
// heap would pay).  Freeing one may wait for all work on the device, a running
// service included, so no page is freed inside the pool: give() hands a page
// that nothing uses any more to its caller, who frees it if it can afford to
// wait, and otherwise the page stays for later heaps (one page per 64 heaps
// that were alive at once, 1/1,300 of their tables at the default capacity).
class WordPool {
  struct Page {
    uint8_t* host;
    uint64_t used;  // bit i: word i is a heap's
  };
  std::mutex mu_;
  std::vector<Page> pages_;

 public:
  static constexpr size_t kPageBytes = 4096;

  // A word nobody else has; make() returns a new page (or null) and runs
  // without the lock.
  template <typename Make>
  int64_t* take(Make&& make) {
    {
      std::lock_guard<std::mutex> g(mu_);
      for (Page& p : pages_)
        if (~p.used) {
          const int i = __builtin_ctzll(~p.used);
          p.used |= 1ull << i;
          return reinterpret_cast<int64_t*>(p.host + 64 * i);
        }
    }
    uint8_t* host = static_cast<uint8_t*>(make());
    if (!host) return nullptr;
    std::lock_guard<std::mutex> g(mu_);
    pages_.push_back({host, 1ull});
    return reinterpret_cast<int64_t*>(host);
  }

  // Word w is free again.  With `drop`, returns an empty page for the caller
  // to free when another one is left, else null.
  void* give(int64_t* w, bool drop) {
    std::lock_guard<std::mutex> g(mu_);
    const uint8_t* b = reinterpret_cast<const uint8_t*>(w);
    size_t empty = 0, at = 0;
    for (size_t k = 0; k < pages_.size(); ++k) {
      Page& p = pages_[k];
      if (b >= p.host && b < p.host + kPageBytes) p.used &= ~(1ull << ((b - p.host) / 64));
      if (p.used == 0) {
        ++empty;
        at = k;
      }
    }
    if (!drop || empty < 2) return nullptr;
    void* host = pages_[at].host;
    pages_.erase(pages_.begin() + (std::ptrdiff_t)at);
    return host;
  }
};

}  // namespace hda
