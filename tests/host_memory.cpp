// Host-side checks of the device memory kept between calls, run without a GPU: this program brings its own HIP runtime
// (device memory is host memory, kernels do nothing, waits and frees do what a check asks for) and links the library.
//   host_memory <check>       exit 0: holds, 1: does not (with a line that says what)
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <atomic>
#include <chrono>
#include <condition_variable>
#include <mutex>
#include <new>
#include <set>
#include <thread>

#include "common.h"

namespace {
std::mutex mu;
std::condition_variable cv;
std::set<void*> live;                      // blocks the runtime has handed out
size_t mallocs = 0, frees = 0;
int current = 0;                           // the current device
int syncs = 0, first_failing_sync = 1 << 30;
bool hold_frees = false;                   // hipFree does not return while this is set
int frees_waiting = 0;
size_t device_bytes = (size_t)64 << 26;    // 1/64 of it: 64 MiB
size_t malloc_limit = ~(size_t)0;          // bytes that can be out at once
size_t out_bytes = 0;
std::set<std::pair<void*, size_t>> sizes;

bool host_memory_out = false;              // operator new fails

hipError_t sync_result() { return ++syncs >= first_failing_sync ? hipErrorStreamCaptureUnsupported : hipSuccess; }
}  // namespace

// (the library's allocations come here too)
void* operator new(size_t n) {
  void* p = host_memory_out ? nullptr : malloc(n ? n : 1);
  if (!p) throw std::bad_alloc();
  return p;
}
void operator delete(void* p) noexcept { free(p); }
void operator delete(void* p, size_t) noexcept { free(p); }

extern "C" {
hipError_t hipMalloc(void** p, size_t n) {
  std::lock_guard<std::mutex> l(mu);
  if (out_bytes + n > malloc_limit) { *p = nullptr; return hipErrorOutOfMemory; }
  if (posix_memalign(p, 4096, n) != 0) return hipErrorOutOfMemory;
  memset(*p, 0, n < 65536 ? n : 65536);
  ++mallocs; out_bytes += n;
  const bool was = host_memory_out;
  host_memory_out = false;                 // (these notes are not the library's)
  live.insert(*p);
  sizes.insert({*p, n});
  host_memory_out = was;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  std::unique_lock<std::mutex> l(mu);
  if (hold_frees) {
    ++frees_waiting;
    cv.notify_all();
    cv.wait(l, [] { return !hold_frees; });
    --frees_waiting;
  }
  if (p) {
    ++frees;
    live.erase(p);
    auto i = sizes.lower_bound({p, 0});
    if (i != sizes.end() && i->first == p) { out_bytes -= i->second; sizes.erase(i); }
    free(p);
  }
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { *p = calloc(1, n); return hipSuccess; }
hipError_t hipHostFree(void* p) { free(p); return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = current; return hipSuccess; }
hipError_t hipSetDevice(int d) { current = d; return hipSuccess; }
hipError_t hipGetDeviceProperties(hipDeviceProp_t* p, int) {       // (the header's macro names the version)
  memset(p, 0, sizeof(*p));
  p->totalGlobalMem = device_bytes;
  p->multiProcessorCount = 256;
  return hipSuccess;
}
hipError_t hipDeviceSynchronize() { return sync_result(); }
hipError_t hipStreamSynchronize(hipStream_t) { return sync_result(); }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "stand-in error"; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) { memset(d, v, n); return hipSuccess; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* n, hipStream_t* s) { *g = *b = dim3(1); *n = 0; *s = nullptr; return hipSuccess; }
}

using namespace gcn;

#define CHECK(c)                                                                  \
  do {                                                                            \
    if (!(c)) { printf("line %d: %s\n", __LINE__, #c); fflush(stdout); _Exit(1); } \
  } while (0)

// A graph of n vertices without edges, made by hand (kernels do nothing here).
static gcn_csr* make_handle(int n) {
  gcn_csr* A = new gcn_csr();
  A->n_global = A->nr = A->nc = A->nnz = n;
  CHECK(pool_alloc((void**)&A->rowptr, sizeof(int64_t) * (n + 1)) == GCN_OK);
  CHECK(pool_alloc((void**)&A->col, sizeof(int32_t) * n + kEntrySlack) == GCN_OK);
  CHECK(pool_alloc((void**)&A->val, sizeof(float) * n + kEntrySlack) == GCN_OK);
  for (int i = 0; i <= n; ++i) A->rowptr[i] = i;
  A->sched.n_wave_rows = n;
  for (int c = 32; c < 34; ++c) A->sched.class_begin[c] = n;      // class 31: one entry
  return A;
}

// A column-sweep plan whose last wait fails may still be written: none of its arrays is kept for other calls.
static void plan() {
  gcn_csr* A = make_handle(512);
  CHECK(gcn_debug_set_tuning("GCN_SPMM_PANEL", 1) == GCN_OK);
  float *X = (float*)aligned_alloc(256, 512 * 32 * 4), *Y = (float*)aligned_alloc(256, 512 * 32 * 4);
  const size_t before = live.size();
  for (int which = 2; which <= 3; ++which) {       // (the first wait is for the row pointers: nothing is allocated yet)
    syncs = 0; first_failing_sync = which;
    CHECK(gcn_spmm(A, X, 32, 32, GCN_F32, Y, 32, GCN_EPI_NONE, nullptr, nullptr, 0, nullptr) == GCN_EHIP);
    CHECK(syncs >= which);
    CHECK(live.size() == before + 1);              // the handle's workspace
  }
  first_failing_sync = 1 << 30;
  CHECK(gcn_spmm(A, X, 32, 32, GCN_F32, Y, 32, GCN_EPI_NONE, nullptr, nullptr, 0, nullptr) == GCN_OK);
  CHECK(A->plans.size() == 1);
  CHECK(gcn_csr_free(A) == GCN_OK);
}

// A free that the runtime holds up, be it an eviction or a block whose work may still run, holds up no other thread's calls.
static void lock() {
  void *big[2], *small, *busy;
  for (void*& b : big) CHECK(pool_alloc(&b, (size_t)40 << 20) == GCN_OK);
  CHECK(pool_alloc(&small, 100000) == GCN_OK);
  CHECK(pool_alloc(&busy, 100000) == GCN_OK);
  pool_free(small);
  pool_free(big[0]);
  for (int round = 0; round < 2; ++round) {
    { std::lock_guard<std::mutex> l(mu); hold_frees = true; }
    std::thread giver([&] {
      if (round == 0) pool_free(big[1]);           // over the limit: an older block leaves
      else pool_free(busy, false);
    });
    {
      std::unique_lock<std::mutex> l(mu);
      CHECK(cv.wait_for(l, std::chrono::seconds(20), [] { return frees_waiting > 0; }));
    }
    std::atomic<bool> done{false};
    std::thread other([&] {
      void* p = nullptr;
      CHECK(pool_alloc(&p, 5000) == GCN_OK);
      pool_free(p);
      CHECK(pool_alloc(&p, (size_t)20 << 20) == GCN_OK);
      pool_free(p);
      done = true;
    });
    for (int i = 0; i < 1000 && !done; ++i) std::this_thread::sleep_for(std::chrono::milliseconds(10));
    CHECK(done);
    { std::lock_guard<std::mutex> l(mu); hold_frees = false; }
    cv.notify_all();
    giver.join();
    other.join();
  }
}

// Memory that runs out: kept blocks go back first, also those that another thread is giving back at that moment.
static void exhausted() {
  void *a, *b, *c = nullptr;
  CHECK(pool_alloc(&a, (size_t)40 << 20) == GCN_OK);
  CHECK(pool_alloc(&b, (size_t)40 << 20) == GCN_OK);
  pool_free(a);
  { std::lock_guard<std::mutex> l(mu); hold_frees = true; malloc_limit = (size_t)100 << 20; }
  std::thread giver([&] { pool_free(b); });        // evicts a
  {
    std::unique_lock<std::mutex> l(mu);
    CHECK(cv.wait_for(l, std::chrono::seconds(20), [] { return frees_waiting > 0; }));
  }
  int rc = -100;
  std::thread taker([&] { rc = pool_alloc(&c, (size_t)90 << 20); });
  std::this_thread::sleep_for(std::chrono::milliseconds(200));
  { std::lock_guard<std::mutex> l(mu); hold_frees = false; }
  cv.notify_all();
  giver.join();
  taker.join();
  CHECK(rc == GCN_OK && c);
  CHECK(pool_alloc(&a, (size_t)90 << 20) == GCN_ENOMEM);
}

// A workspace that grows while another device is current: the wait was for that device, so the old one is not kept.
static void workspace() {
  gcn_csr* A = make_handle(512);
  CHECK(ensure_workspace(A, 1 << 20) == GCN_OK);
  size_t f = frees;
  CHECK(ensure_workspace(A, 3 << 20) == GCN_OK && frees == f);      // device 0 was waited for: kept
  current = 1;
  f = frees;
  CHECK(ensure_workspace(A, 9 << 20) == GCN_OK && frees == f + 1);
  current = 0;
  f = frees;
  first_failing_sync = 0;                                           // (a capture goes on): the old one stays
  void* ws = A->ws;
  CHECK(ensure_workspace(A, 20 << 20) == GCN_EHIP && A->ws == ws && frees == f);
}

// What is kept goes back on request; what is in use does not.
static void release() {
  void *a, *b, *c, *page;
  CHECK(pool_alloc(&a, 1000) == GCN_OK && pool_alloc(&b, (size_t)30 << 20) == GCN_OK);
  current = 1;
  CHECK(pool_alloc(&c, 70000) == GCN_OK && pinned_take(&page) == GCN_OK);
  pinned_give(page);
  pool_free(b);
  pool_free(c);
  CHECK(frees == 0);
  CHECK(gcn_release_memory() == GCN_OK && frees == 2 && live.size() == 1 && live.count(a));
  CHECK(gcn_release_memory() == GCN_OK && frees == 2);
  CHECK(pool_alloc(&b, 70000) == GCN_OK && mallocs == 4);           // nothing was left to take it from
}

// Host memory that runs out before the first block or page is asked for: calls report it or do without, none throws.
static void host() {
  host_memory_out = true;
  gcn_csr_t* A = (gcn_csr_t*)1;
  int32_t e = 0;
  CHECK(gcn_release_memory() == GCN_OK);
  CHECK(gcn_csr_build(&e, &e, 1, 1, 0, 1, nullptr, 0, nullptr, &A) == GCN_ENOMEM && !A);
  void *p = nullptr, *page = nullptr;
  CHECK(pinned_take(&page) == GCN_OK);
  pinned_give(page);
  CHECK(pool_alloc(&p, 1000) == GCN_OK && live.count(p));          // a block that is on no list
  pool_free(p);
  host_memory_out = false;
  CHECK(live.empty());
}

int main(int argc, char** argv) {
  const struct { const char* name; void (*run)(); } checks[] = {{"plan", plan}, {"lock", lock}, {"exhausted", exhausted}, {"workspace", workspace}, {"release", release}, {"host", host}};
  for (auto& c : checks)
    if (argc > 1 && !strcmp(argv[1], c.name)) { c.run(); printf("%s holds\n", c.name); fflush(stdout); _Exit(0); }
  printf("no such check\n");
  return 2;
}
