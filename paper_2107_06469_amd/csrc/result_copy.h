// Host side of results on their way from the device to a caller's memory.  Nothing here calls HIP: what allocates and what copies
// is handed in.
#pragma once
#include <algorithm>
#include <atomic>
#include <cstddef>
#include <cstring>
#include <mutex>
#include <thread>
#include <vector>

namespace hydra {

// One pinned buffer of the process that all contexts' readers share: made for the first context that attaches, given back with the last
// (making one takes 0.4 ms, as long as an epoch of small models).  One reader at a time has it (StageLease).  The lock is held while
// the fields are looked at and never over a copy: contexts come and go while another's results, which may take seconds, are on their way.
class Stage {
 public:
  static constexpr size_t BYTES = (size_t)4 << 20;
  Stage(void* (*make)(size_t), void (*give_back)(void*)) : make_(make), give_back_(give_back) {}
  void attach() {
    std::lock_guard<std::mutex> l(m_);
    ++users_;
    if (!p_) p_ = make_(BYTES);  // null: readers copy without it, the next to attach tries again
  }
  void detach() {
    std::unique_lock<std::mutex> l(m_);
    --users_;
    drop(l);
  }

 private:
  friend class StageLease;
  void drop(std::unique_lock<std::mutex>& l) {  // the buffer goes once neither a context nor a reader is left
    if (users_ > 0 || leased_ || !p_) return;
    void* const p = p_;
    p_ = nullptr;
    l.unlock();
    give_back_(p);
  }
  void* (*make_)(size_t);
  void (*give_back_)(void*);
  std::mutex m_;
  void* p_ = nullptr;
  int users_ = 0;
  bool leased_ = false;
};

// p: the buffer until the lease ends, or null while another reader has it and where there is none
class StageLease {
 public:
  explicit StageLease(Stage& s) : s_(s) {
    std::lock_guard<std::mutex> l(s_.m_);
    if (s_.leased_ || !s_.p_) return;
    s_.leased_ = true;
    p = static_cast<float*>(s_.p_);
  }
  ~StageLease() {
    if (!p) return;
    std::unique_lock<std::mutex> l(s_.m_);
    s_.leased_ = false;
    s_.drop(l);
  }
  StageLease(const StageLease&) = delete;
  StageLease& operator=(const StageLease&) = delete;
  float* p = nullptr;

 private:
  Stage& s_;
};

// Requests parts 0 .. n - 1 of a copy into a leased buffer and waits for them: also where one could not be requested, since those before it
// are on their way and the buffer is another reader's once the lease ends.  The first error, 0 if there was none.
template <typename R, typename W>
int request_all(int n, const R& request, const W& wait) {
  int e = 0;
  for (int i = 0; i < n && !e; ++i) e = (int)request(i);
  const int w = (int)wait();
  return e ? e : w;
}

// work(0) on this thread and work(1) ... work(T - 1) on threads of their own, which have ended when it returns.  Where the system gives
// no more threads, or no memory for one, those there are do without it: work takes its share from a common counter, not from k.
template <typename W>
void on_threads(unsigned T, const W& work) {
  std::vector<std::thread> helpers;
  try {
    helpers.reserve(T);
    for (unsigned k = 1; k < T; ++k) helpers.emplace_back([&work, k] { work(k); });
  } catch (...) {
  }
  work(0);
  for (std::thread& t : helpers) t.join();
}

// n floats at `off` of a block go to `to` of the caller's array
struct Piece { size_t off, n, to; };

// Pieces of the block at src straight to dst.  Where they rise in the block, runs that fit 1 MB travel as one copy (some 10 us each whatever
// its size) and are taken apart here; larger pieces go to their place.  copy(to, from, floats) returns when it is done, 0 if it went well.
template <typename C>
int copy_direct(const std::vector<Piece>& ps, bool rising, const float* src, float* dst, const C& copy) {
  constexpr size_t RUN = (size_t)1 << 18;  // floats
  std::vector<float> buf;
  for (size_t j = 0; j < ps.size();) {
    size_t k = j + 1;
    while (rising && k < ps.size() && ps[k].off + ps[k].n <= ps[j].off + RUN) ++k;
    const size_t n = ps[k - 1].off + ps[k - 1].n - ps[j].off;
    const bool run = k > j + 1;
    if (run) buf.resize(n);
    if (const int e = (int)copy(run ? buf.data() : dst + ps[j].to, src + ps[j].off, n)) return e;
    const size_t at = ps[j].off;
    for (; j < k; ++j)
      if (run) memcpy(dst + ps[j].to, buf.data() + (ps[j].off - at), ps[j].n * 4);
  }
  return 0;
}

// Pieces that rise in the block, as one range in parts through a buffer of `room` floats that T threads share; thread k's copies are
// copy(k, to, from, floats).
template <typename C>
int copy_staged(const std::vector<Piece>& ps, const float* src, float* dst, float* stage, size_t room, unsigned T, const C& copy) {
  const size_t first = ps.front().off, total = ps.back().off + ps.back().n - first, part = room / T;
  std::atomic<size_t> next{0};
  std::atomic<int> err{0};
  on_threads(T, [&](unsigned k) {
    float* const buf = stage + k * part;
    for (size_t b; err.load() == 0 && (b = next.fetch_add(part)) < total;) {
      const size_t lo = first + b, hi = std::min(first + total, lo + part);
      if (const int e = (int)copy(k, buf, src + lo, hi - lo)) {
        err.store(e);
        return;
      }
      auto p = std::upper_bound(ps.begin(), ps.end(), lo, [](size_t v, const Piece& q) { return v < q.off + q.n; });
      for (; p != ps.end() && p->off < hi; ++p) {
        const size_t x = std::max(lo, p->off), y = std::min(hi, p->off + p->n);
        memcpy(dst + p->to + (x - p->off), buf + (x - lo), (y - x) * 4);
      }
    }
  });
  return err.load();
}

}  // namespace hydra
