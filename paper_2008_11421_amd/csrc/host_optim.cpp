#include "host_optim.h"
#include "karma.h"

#include <algorithm>
#include <cmath>
#include <cstring>

namespace karma {

HostPool::HostPool(unsigned threads) {
  if (threads < 1) threads = 1;
  left_.resize(threads);
  for (unsigned i = 1; i < threads; ++i) workers_.emplace_back([this, i] { worker(i); });
}

HostPool::~HostPool() {
  {
    std::lock_guard<std::mutex> lk(mu_);
    stop_ = true;
  }
  cv_.notify_all();
  for (auto& t : workers_) t.join();
}

// Takes parts of the current call, thread `id`'s own and then the last ones of whoever has most left, until none is left;
// mu_ is held on entry and on return.
void HostPool::take_parts(unsigned id, std::unique_lock<std::mutex>& lk) {
  while (untaken_) {
    unsigned at;
    if (left_[id].next < left_[id].end) {
      at = left_[id].next++;
    } else {
      auto less = [](const Run& a, const Run& b) { return a.end - a.next < b.end - b.next; };
      at = --std::max_element(left_.begin(), left_.end(), less)->end;
    }
    --untaken_;
    const size_t lo = (size_t)at * part_, hi = std::min(n_, lo + part_);
    const std::function<void(size_t, size_t)>& fn = *fn_;
    lk.unlock();
    fn(lo, hi);
    lk.lock();
    if (--pending_ == 0) done_cv_.notify_one();
  }
}

void HostPool::worker(unsigned id) {
  std::unique_lock<std::mutex> lk(mu_);
  for (;;) {
    cv_.wait(lk, [&] { return stop_ || untaken_; });
    if (stop_) return;
    take_parts(id, lk);
  }
}

// Waking the workers takes longer (40 to 60 us) than small calls do, and the caller need not wait for it: it takes parts
// itself until none is left, and is done when those that others took are.  A step of eight layers of 256 x 256, 65792
// parameters each: 570 us with every worker given its share of each call and waited for, 390 with this.
// Each thread has a run of parts of its own, the same in every call of a size, so that it finds in its cache what it updated last
// time.  Adam again and again on one tensor, 16 threads, us, parts dealt to whoever is awake -> runs: 1 Mi elements 108 -> 80,
// 4 Mi 303 -> 127, 16 Mi 1850 -> 690; on 80 tensors of 4 Mi, which no cache holds, 345 -> 340.
void HostPool::parallel_for(size_t n, const std::function<void(size_t, size_t)>& fn) {
  constexpr size_t ALONE = 128 * 1024, LEAST = 32 * 1024;   // elements: at most this many for the caller alone; a part's least
  if (workers_.empty() || n <= ALONE) {
    if (n) fn(0, n);
    return;
  }
  std::unique_lock<std::mutex> lk(mu_);
  fn_ = &fn;
  n_ = n;
  part_ = std::max(LEAST, ((n + 4 * size() - 1) / (4 * size()) + 63) / 64 * 64);
  untaken_ = pending_ = (unsigned)((n + part_ - 1) / part_);
  for (unsigned t = 0, at = 0; t < size(); ++t) {
    left_[t].next = at;
    left_[t].end = at += untaken_ / size() + (t < untaken_ % size() ? 1 : 0);
  }
  lk.unlock();
  cv_.notify_all();
  lk.lock();
  take_parts(0, lk);
  done_cv_.wait(lk, [&] { return pending_ == 0; });
}

float bf16_to_f32(uint16_t b) {
  uint32_t u = (uint32_t)b << 16;
  float f;
  std::memcpy(&f, &u, 4);
  return f;
}

uint16_t f32_to_bf16_rne(float f) {
  uint32_t u;
  std::memcpy(&u, &f, 4);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40);   // NaN stays NaN
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

}  // namespace karma

#define HOST_OPTIM_NS avx2
#include "host_optim_loops.h"
#undef HOST_OPTIM_NS

namespace karma {

// the same loops built for AVX-512 (host_optim_avx512.cpp)
namespace avx512 {
void sgd_update(float* w, const void* g, bool g_is_bf16, size_t n, float lr, void* out, bool out_is_bf16);
void sgd_momentum_update(float* w, float* buf, const void* g, bool g_is_bf16, size_t n, float lr, float mu, void* out,
                         bool out_is_bf16);
void adam_update(float* w, float* m, float* v, const void* g, bool g_is_bf16, size_t n, float lr, float beta1, float beta2,
                 float eps, float c1, float c2, void* out, bool out_is_bf16);
void to_bf16(const float* x, size_t n, uint16_t* out);
}  // namespace avx512

static bool g_force_narrow = false;
void host_optim_force_narrow(bool on) { g_force_narrow = on; }

static bool wide_vectors() {
  static const bool yes = __builtin_cpu_supports("avx512f") && __builtin_cpu_supports("avx512bw") &&
                          __builtin_cpu_supports("avx512vl") && __builtin_cpu_supports("avx512dq");
  return yes && !g_force_narrow;
}

void to_bf16(const float* x, size_t n, uint16_t* out) {
  if (wide_vectors()) avx512::to_bf16(x, n, out);
  else avx2::to_bf16_entry(x, n, out);
}

void sgd_momentum_update(float* w, float* buf, const void* g, bool g_is_bf16, size_t n, float lr, float mu, void* out,
                         bool out_is_bf16) {
  if (wide_vectors()) avx512::sgd_momentum_update(w, buf, g, g_is_bf16, n, lr, mu, out, out_is_bf16);
  else avx2::sgd_momentum_entry(w, buf, g, g_is_bf16, n, lr, mu, out, out_is_bf16);
}

void sgd_update(float* w, const void* g, bool g_is_bf16, size_t n, float lr, void* out, bool out_is_bf16) {
  if (wide_vectors()) avx512::sgd_update(w, g, g_is_bf16, n, lr, out, out_is_bf16);
  else avx2::sgd_entry(w, g, g_is_bf16, n, lr, out, out_is_bf16);
}

void adam_update(float* w, float* m, float* v, const void* g, bool g_is_bf16, size_t n, float lr, float beta1,
                 float beta2, float eps, uint64_t step, void* out, bool out_is_bf16) {
  const float c1 = (float)(1.0 / (1.0 - std::pow((double)beta1, (double)step)));
  const float c2 = (float)(1.0 / (1.0 - std::pow((double)beta2, (double)step)));
  if (wide_vectors()) avx512::adam_update(w, m, v, g, g_is_bf16, n, lr, beta1, beta2, eps, c1, c2, out, out_is_bf16);
  else avx2::adam_entry(w, m, v, g, g_is_bf16, n, lr, beta1, beta2, eps, c1, c2, out, out_is_bf16);
}

}  // namespace karma

// One update of n parameters through the same loops the executor uses per record.
extern "C" int karma_host_update(uint32_t optimizer, float* master, float* m, float* v, const void* grad,
                                 uint32_t grad_is_bf16, uint64_t n, float lr, float beta1, float beta2, float eps,
                                 uint64_t step, void* out, uint32_t out_is_bf16, uint32_t narrow_vectors) {
  using namespace karma;
  if (!master || !grad || !out) return KARMA_E_INVAL;
  if (grad == out && (grad_is_bf16 != 0) != (out_is_bf16 != 0)) return KARMA_E_INVAL;   // in place needs equal element types
  host_optim_force_narrow(narrow_vectors != 0);
  int st = KARMA_OK;
  if (optimizer == KARMA_OPT_SGD) sgd_update(master, grad, grad_is_bf16 != 0, (size_t)n, lr, out, out_is_bf16 != 0);
  else if (optimizer == KARMA_OPT_SGD_MOMENTUM && m)
    sgd_momentum_update(master, m, grad, grad_is_bf16 != 0, (size_t)n, lr, beta1, out, out_is_bf16 != 0);
  else if (optimizer == KARMA_OPT_ADAM && m && v && step >= 1)
    adam_update(master, m, v, grad, grad_is_bf16 != 0, (size_t)n, lr, beta1, beta2, eps, step, out, out_is_bf16 != 0);
  else st = KARMA_E_INVAL;
  host_optim_force_narrow(false);
  return st;
}
