// Host side of results on their way from the device to a caller's memory.  Nothing here calls HIP: what allocates and what copies
// is handed in.
#pragma once
#include <cstddef>
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

}  // namespace hydra
