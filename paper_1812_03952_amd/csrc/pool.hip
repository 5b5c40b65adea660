// pool.hip -- the library's device memory pool.
//
// Every handle rebuilds its buffers on each Newton step (a new decoupling, a
// new hierarchy, new Krylov workspace), and hipMalloc/hipFree of buffers of
// hundreds of megabytes cost milliseconds, hipFree also synchronising the
// device.  Freed blocks therefore stay cached here and later requests of a
// similar size reuse them; memory goes back to the runtime only through
// rs_pool_trim, or when a hipMalloc fails (the cache is released and the
// allocation retried).
//
// Size classes: powers of two from 256 B to 1 MiB, multiples of 2 MiB above;
// a cached block serves a request if it is at most 1/8 larger.
#include "rs_internal.h"
#include <map>
#include <mutex>
#include <unordered_map>
#include <vector>
#include <string.h>

namespace {

struct pool_state {
  std::mutex mu;
  std::multimap<size_t, std::pair<void *, int>> free_blocks;   // size -> (pointer, device)
  std::unordered_map<void *, int> device_of;                    // live and cached blocks
  size_t cached = 0, live = 0;
};

pool_state &pool() {
  static pool_state *p = new pool_state();     // never destroyed: no HIP calls at exit
  return *p;
}

size_t size_class(size_t b) {
  if (b <= ((size_t)1 << 20)) {
    size_t r = 256;
    while (r < b) r <<= 1;
    return r;
  }
  const size_t G = (size_t)2 << 20;
  return (b + G - 1) / G * G;
}

// release every cached block of device dev (-1: all devices); caller holds the lock
void trim_locked(pool_state &P, int dev) {
  for (auto it = P.free_blocks.begin(); it != P.free_blocks.end();) {
    if (dev >= 0 && it->second.second != dev) { ++it; continue; }
    (void)hipFree(it->second.first);
    P.device_of.erase(it->second.first);
    P.cached -= it->first;
    it = P.free_blocks.erase(it);
  }
}

}  // namespace

void *rs_pool_get(size_t bytes, size_t *got) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return nullptr;
  const size_t r = size_class(bytes);
  pool_state &P = pool();
  std::lock_guard<std::mutex> lk(P.mu);
  for (auto it = P.free_blocks.lower_bound(r); it != P.free_blocks.end() && it->first <= r + r / 8; ++it) {
    if (it->second.second != dev) continue;
    void *p = it->second.first;
    *got = it->first;
    P.cached -= it->first;
    P.live += it->first;
    P.free_blocks.erase(it);
    return p;
  }
  void *p = nullptr;
  if (hipMalloc(&p, r) != hipSuccess) {
    (void)hipGetLastError();
    trim_locked(P, dev);
    p = nullptr;
    if (hipMalloc(&p, r) != hipSuccess) {
      (void)hipGetLastError();
      return nullptr;
    }
  }
  P.device_of[p] = dev;
  P.live += r;
  *got = r;
  return p;
}

void rs_pool_put(void *p, size_t bytes) {
  if (!p) return;
  pool_state &P = pool();
  std::lock_guard<std::mutex> lk(P.mu);
  auto d = P.device_of.find(p);
  int dev = d == P.device_of.end() ? 0 : d->second;
  P.free_blocks.emplace(bytes, std::make_pair(p, dev));
  P.live -= bytes;
  P.cached += bytes;
}

extern "C" void rs_pool_trim(void) {
  pool_state &P = pool();
  std::lock_guard<std::mutex> lk(P.mu);
  trim_locked(P, -1);
}

extern "C" void rs_pool_usage(size_t *live_bytes, size_t *cached_bytes) {
  pool_state &P = pool();
  std::lock_guard<std::mutex> lk(P.mu);
  if (live_bytes) *live_bytes = P.live;
  if (cached_bytes) *cached_bytes = P.cached;
}

// ---- short host waits --------------------------------------------------------
// The set-up reads a few counts and flags back (a number of aggregates, an
// error word) and waits for the stream at each, and the Krylov loops read a
// status per step.  A blocking stream synchronisation leaves the device idle
// for tens of microseconds after such a read while the host thread wakes up, a
// copy and a polled event take 15; instead the device stores the words into
// pinned memory that the host polls (9 us from the launch).  Each host thread
// has one such slot; the slot of a thread that ends goes to the next new one
// (never freed: no HIP calls at exit), so there are as many as threads at one
// time.
namespace {
#include "reduce.h"
struct slot_list {
  std::mutex mu;
  std::vector<rs_post *> free;
};
slot_list &slots() {
  static slot_list *l = new slot_list();
  return *l;
}
struct host_wait {
  rs_post *post = nullptr;
  ~host_wait() {
    if (!post) return;
    std::lock_guard<std::mutex> lk(slots().mu);
    slots().free.push_back(post);
  }
};
thread_local host_wait tw;

}  // namespace

rs_status rs_post_slot(rs_post **out) {
  if (!tw.post) {
    std::lock_guard<std::mutex> lk(slots().mu);
    if (!slots().free.empty()) {
      tw.post = slots().free.back();
      slots().free.pop_back();
    }
  }
  if (!tw.post) {
    void *p = nullptr;
    RS_HIP(hipHostMalloc(&p, sizeof(rs_post), hipHostMallocPortable | hipHostMallocCoherent));
    memset(p, 0, sizeof(rs_post));
    tw.post = (rs_post *)p;
  }
  *out = tw.post;
  return RS_OK;
}

rs_status rs_wait_post(const rs_post *p, uint64_t seq, hipStream_t s) {
  for (unsigned spin = 1;; ++spin) {
    if (__atomic_load_n(&p->seq, __ATOMIC_ACQUIRE) == seq) return RS_OK;
    if (spin % 4096) continue;
    // now and then: has the stream failed, or ended without the post?
    const hipError_t e = hipStreamQuery(s);
    if (e == hipErrorNotReady) continue;
    if (e == hipSuccess && __atomic_load_n(&p->seq, __ATOMIC_ACQUIRE) == seq) return RS_OK;
    return RS_E_HIP;
  }
}

// the words and, after them, whether an error word is set, into the post's
// values; take: the words are zero afterwards
__global__ void k_post_words(uint32_t *d, int nw, int take, const int *err0, const int *err1,
                             rs_post *__restrict__ post, uint64_t seq) {
  const int t = threadIdx.x;
  uint32_t *o = (uint32_t *)post->v;
  if (t < nw) {
    __hip_atomic_store(o + t, d[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    // at agent scope: done before the post, whatever stream the next call takes
    if (take) __hip_atomic_store(d + t, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  if (t == 0)
    __hip_atomic_store(o + RS_READ_WORDS, ((err0 && *err0) || (err1 && *err1)) ? 1u : 0u, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_SYSTEM);
  stores_done();
  if (t == 0) __hip_atomic_store(&post->seq, seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

static rs_status wait_words(void *h, uint32_t *d, size_t bytes, bool take, const int *const (&errw)[2], int *err,
                            hipStream_t s) {
  if (bytes > sizeof(uint32_t) * RS_READ_WORDS || bytes % 4) return RS_E_ARG;
  rs_post *post = nullptr;
  RS_TRY(rs_post_slot(&post));
  const uint64_t seq = rs_post_next(post);
  k_post_words<<<1, 64, 0, s>>>(d, (int)(bytes / 4), take ? 1 : 0, errw[0], errw[1], post, seq);
  RS_HIP(hipGetLastError());
  RS_TRY(rs_wait_post(post, seq, s));
  memcpy(h, post->v, bytes);
  *err = (int)((const uint32_t *)post->v)[RS_READ_WORDS];
  return RS_OK;
}

rs_status rs_wait_read_err(void *h, const void *d, size_t bytes, const int *const (&errw)[2], int *err,
                           hipStream_t s) {
  return wait_words(h, (uint32_t *)d, bytes, false, errw, err, s);
}

rs_status rs_wait_read(void *h, const void *d, size_t bytes, hipStream_t s) {
  const int *const none[2] = {nullptr, nullptr};
  int e = 0;
  return rs_wait_read_err(h, d, bytes, none, &e, s);
}

rs_status rs_wait_take(int *h, int *d, hipStream_t s) {
  const int *const none[2] = {nullptr, nullptr};
  int e = 0;
  return wait_words(h, (uint32_t *)d, sizeof(int), true, none, &e, s);
}

__global__ void k_fill32(int64_t m, uint32_t v, uint32_t *__restrict__ a) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t < m) a[t] = v;
}

rs_status rs_fill32(void *a, uint32_t v, int64_t m, hipStream_t s) {
  if (m < 1) return RS_OK;
  k_fill32<<<rs_grid(m), RS_BLOCK, 0, s>>>(m, v, (uint32_t *)a);
  RS_HIP(hipGetLastError());
  return RS_OK;
}
