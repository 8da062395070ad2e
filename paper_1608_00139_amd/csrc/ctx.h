// ctx.h -- the library context behind the opaque dl_ctx of include/dl.h
// (internal to the library's sources).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <memory>
#include <mutex>
#include <new>
#include <string>
#include <utility>
#include <vector>

#include "common.h"
#include "eps_solve.h"

// Fixpoints a batched call keeps in flight (each with its own workspace,
// counters and read-back event).
constexpr int kFixSlots = 2;
constexpr size_t kSlotWords = (size_t)dl::kRing + 1;  // a slot's ring and its convergence step

struct EventPair {
  hipEvent_t a, b;
};

// A tile configuration chosen for (precision, padded size) by the autotuner
// or set by the caller; ms is the measured time of one product (0 if set).
struct TuneEntry {
  int prec;
  int64_t np;
  int cfg;
  double ms;
};

// Device matrices given back by a context's programs, kept for their next
// runs: allocating and freeing the ~25 matrices of a run took 5.5 ms of a 7.6
// ms run at n = 4000 (now 2.1 ms).  At most kMaxKept bytes are kept (the oldest go first);
// the context and its programs share the pool, and the last of them frees it.
// A block is given back only when nothing in flight uses it, or to be reused
// on the same stream.
class MatPool {
 public:
  static constexpr size_t kMaxKept = (size_t)1 << 30;
  ~MatPool() { drop(); }
  hipError_t get(size_t bytes, void** p) {
    {
      std::lock_guard<std::mutex> l(m_);
      for (size_t i = kept_.size(); i-- > 0;)
        if (kept_[i].first == bytes) {
          *p = kept_[i].second;
          kept_.erase(kept_.begin() + i);
          total_ -= bytes;
          return hipSuccess;
        }
    }
    hipError_t e = hipMalloc(p, bytes);
    if (e == hipSuccess) return e;
    (void)hipGetLastError();
    drop();
    e = hipMalloc(p, bytes);
    if (e != hipSuccess) (void)hipGetLastError();
    return e;
  }
  void put(void* p, size_t bytes) {
    bool is_kept = false;
    try {
      std::lock_guard<std::mutex> l(m_);
      kept_.push_back({bytes, p});
      total_ += bytes;
      is_kept = true;
    } catch (const std::bad_alloc&) {  // no host memory for the entry
    }
    if (!is_kept) (void)hipFree(p);
    for (;;) {
      void* oldest = nullptr;
      {
        std::lock_guard<std::mutex> l(m_);
        if (total_ <= kMaxKept) return;
        total_ -= kept_.front().first;
        oldest = kept_.front().second;
        kept_.erase(kept_.begin());
      }
      (void)hipFree(oldest);
    }
  }
  // Frees what is kept (before an allocation elsewhere is given up).
  void drop() {
    std::vector<std::pair<size_t, void*>> out;
    {
      std::lock_guard<std::mutex> l(m_);
      out.swap(kept_);
      total_ = 0;
    }
    for (auto& b : out) (void)hipFree(b.second);
  }

 private:
  std::mutex m_;
  std::vector<std::pair<size_t, void*>> kept_;  // oldest first
  size_t total_ = 0;
};

// hipMalloc, once more after `kept` (if any) has given up its matrices; *p is
// null on failure.
inline hipError_t device_alloc(MatPool* kept, void** p, size_t bytes) {
  hipError_t e = hipMalloc(p, bytes);
  if (e != hipSuccess && kept) {
    (void)hipGetLastError();
    kept->drop();
    e = hipMalloc(p, bytes);
  }
  if (e != hipSuccess) {
    (void)hipGetLastError();
    *p = nullptr;
  }
  return e;
}
struct dl_ctx {
  int device = 0;
  size_t budget = 0;
  void* ws = nullptr;  // main workspace
  size_t ws_size = 0;
  unsigned long long* ring = nullptr;  // per fixpoint slot: kRing model sizes, then the slot's
                                       // convergence step (an int in one more word)
  int* conv = nullptr;                 // device scratch ints (eps bounds, solver flags)
  int* dscratch = nullptr;             // small device scratch (row max, ...)
  unsigned long long* h_ring = nullptr;  // pinned (coherent) host mirror of the slots' rings and steps
  unsigned long long* h_ring_dev = nullptr;  // its device mapping, written by k_publish
  int* h_conv = nullptr;                 // pinned scratch ints
  hipEvent_t slot_ev[kFixSlots] = {nullptr, nullptr};  // read-back events of the fixpoint slots
  bool timing = false;
  int64_t launches[3] = {0, 0, 0};
  double ms[3] = {0, 0, 0};
  std::vector<EventPair> events;    // pool of timing event pairs
  size_t ev_cursor = 0;             // pairs [0, ev_cursor) hold launches not yet resolved
  std::vector<std::pair<int, int>> pending;  // (class, pair index) to add to ms / launches
  std::shared_ptr<MatPool> mats = std::make_shared<MatPool>();  // program matrices (not with a budget)
  dl::EpsWorkspace eps;  // workspace of the epsilon solve
  std::vector<TuneEntry> tuned;  // tile configurations that override the size rule
  unsigned* fs_words = nullptr;  // counters of the one-launch plain fixpoint, then of the one on bits (zero
                                 // between launches)
  unsigned fs_tag = 0;           // tags the one-launch plain fixpoint has used (fix_small_tag)
  bool fs_dirty = false;         // a launch ended abnormally: clear them before the next
  bool fb_dirty = false;         // the same for the one on bits
  bool fl_dirty = false;         // and for the one by lists
};

namespace dl {
void set_last_error(const std::string& m);
// Tile configuration of the product kernels for (prec, Np): the tuned entry
// if there is one, else the size rule of choose_nt_config.
int pick_config(const dl_ctx* c, int prec, int64_t np);
// The tuned or set entry for (prec, Np), -1 if there is none.
int tuned_config(const dl_ctx* c, int prec, int64_t np);
}  // namespace dl
