// The streams of closed handles, kept for the next ones.
//
// Creating and checking a compute and copy pair takes about 0.8 ms, as long as the
// whole of a study of 512 samples, and a stream keeps its hardware queue for life.
// So a handle takes its pair at its first streamed study without a copy stream,
// and gives it back when it is destroyed; idle pairs (and the setup's side streams)
// wait here, at most POOL_MAX a device, in fixed arrays: nothing here throws.
#pragma once

#include <hip/hip_runtime.h>

#include <mutex>

namespace gls {

struct StreamPair {
  hipStream_t st[2] = {nullptr, nullptr};   // compute, copy
  bool checked = false;                     // a wait on the copy stream was seen not to hold up the compute stream
  bool there() const { return st[0] && st[1]; }
};

class StreamPool {
 public:
  static constexpr int POOL_MAX = 4;   // idle pairs, and idle side streams, kept per device

  // An idle pair of the device, or a new one: the copy stream is created again, at most four times, until
  // isolated(compute, copy) holds.  On failure the pair stays empty.
  template <typename Isolated>
  hipError_t take_pair(int device, Isolated isolated, StreamPair* p) {
    Entry idle;
    if (take(pairs_, device, &idle)) {
      p->st[0] = idle.st[0];
      p->st[1] = idle.st[1];
      p->checked = true;
      return hipSuccess;
    }
    hipStream_t comp = nullptr, copy = nullptr;
    hipError_t e = hipStreamCreateWithFlags(&comp, hipStreamNonBlocking);
    if (e != hipSuccess) return e;
    e = hipStreamCreateWithFlags(&copy, hipStreamNonBlocking);
    if (e != hipSuccess) {
      (void)hipStreamDestroy(comp);
      return e;
    }
    hipStream_t rejected[TRIES];   // kept until the search ends, so that their queues are not handed out again
    int n = 0;
    bool ok = isolated(comp, copy);
    while (!ok && n < TRIES) {
      hipStream_t fresh = nullptr;
      if (hipStreamCreateWithFlags(&fresh, hipStreamNonBlocking) != hipSuccess) {
        (void)hipGetLastError();
        break;
      }
      rejected[n++] = copy;
      copy = fresh;
      ok = isolated(comp, copy);
    }
    for (int i = 0; i < n; ++i) (void)hipStreamDestroy(rejected[i]);
    p->st[0] = comp;
    p->st[1] = copy;
    p->checked = ok;
    return hipSuccess;
  }

  // Waits for the pair's work.  A pair that the check never passed is not kept: the next handle searches anew.
  void give_pair(int device, StreamPair* p) {
    bool idle = p->there() && p->checked;
    for (hipStream_t s : p->st)
      if (s && hipStreamSynchronize(s) != hipSuccess) idle = false;
    if (!idle || !keep(pairs_, Entry{device, {p->st[0], p->st[1]}}))
      for (hipStream_t s : p->st)
        if (s) (void)hipStreamDestroy(s);
    *p = StreamPair{};
  }

  hipError_t take_side(int device, hipStream_t* st) {
    Entry idle;
    if (take(sides_, device, &idle)) {
      *st = idle.st[0];
      return hipSuccess;
    }
    return hipStreamCreateWithFlags(st, hipStreamNonBlocking);
  }

  // The stream has nothing left to run.
  void give_side(int device, hipStream_t st) {
    if (!keep(sides_, Entry{device, {st, nullptr}})) (void)hipStreamDestroy(st);
  }

 private:
  static constexpr int TRIES = 4, CAPACITY = 64;
  struct Entry {
    int device = 0;
    hipStream_t st[2] = {nullptr, nullptr};
  };
  struct List {
    Entry at[CAPACITY];
    int count = 0;
  };

  bool take(List& l, int device, Entry* out) {
    std::lock_guard<std::mutex> lock(mu_);
    for (int i = 0; i < l.count; ++i) {
      if (l.at[i].device != device) continue;
      *out = l.at[i];
      l.at[i] = l.at[--l.count];
      return true;
    }
    return false;
  }
  bool keep(List& l, const Entry& e) {
    std::lock_guard<std::mutex> lock(mu_);
    int have = 0;
    for (int i = 0; i < l.count; ++i) have += l.at[i].device == e.device;
    if (have >= POOL_MAX || l.count >= CAPACITY) return false;
    l.at[l.count++] = e;
    return true;
  }

  std::mutex mu_;
  List pairs_, sides_;
};

}  // namespace gls
