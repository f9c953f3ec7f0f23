// Host-side check of where the dense products of a layer call go, run without a GPU: this program brings its own HIP runtime (device memory is
// host memory, kernels do nothing, launches are written down by name) and links the library.
//   host_routes <overlap> <call> <d_in> <d_out> <ld> [<rows>]      one line per launch: kernel, workgroups, main | side
// call: fwd | bwd; the graph has 2^17 rows and 10^8 entries, long enough for dense products beside its sparse ones.  <ld>: the pitch of A^ H.
//       dense: the dense product alone; grad: the weight gradient alone; down, masked: the gradient handed down as well, without and with the mask of
//       the layer before; on a graph of <rows> rows and entries.
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <map>
#include <string>

#include "common.h"

namespace {
std::map<const void*, std::string>& names() {       // (the library's kernels are registered before this program's statics are made)
  static std::map<const void*, std::string>* m = new std::map<const void*, std::string>();
  return *m;
}
int side_stream;
dim3 grid_, block_;
size_t shmem_;
hipStream_t stream_;
}  // namespace

extern "C" {
void** __hipRegisterFatBinary(const void*) { static void* h; return &h; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, void*, void*, void*, void*, int*) { names()[f] = name; }
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t hipMalloc(void** p, size_t n) { *p = aligned_alloc(4096, (n + 4095) / 4096 * 4096); return *p ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipFree(void* p) { free(p); return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { *p = calloc(1, n); return hipSuccess; }
hipError_t hipHostFree(void* p) { free(p); return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDeviceProperties(hipDeviceProp_t* p, int) {       // (the header's macro names the version)
  memset(p, 0, sizeof(*p));
  p->totalGlobalMem = (size_t)288 << 30;
  p->multiProcessorCount = 256;
  return hipSuccess;
}
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = (hipStream_t)&side_stream; return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = (hipEvent_t)&side_stream; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "stand-in error"; }
hipError_t hipMemcpyAsync(void*, const void*, size_t, hipMemcpyKind, hipStream_t) { return hipErrorUnknown; }
hipError_t hipMemsetAsync(void*, int, size_t, hipStream_t) { return hipSuccess; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t n, hipStream_t s) { grid_ = g; block_ = b; shmem_ = n; stream_ = s; return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* n, hipStream_t* s) { *g = grid_; *b = block_; *n = shmem_; *s = stream_; return hipSuccess; }
hipError_t hipLaunchKernel(const void* f, dim3 g, dim3, void**, size_t, hipStream_t s) {
  printf("%s %lld %s\n", names()[f].c_str(), (long long)g.x * g.y * g.z, s == (hipStream_t)&side_stream ? "side" : "main");
  return hipSuccess;
}
}

using namespace gcn;

int main(int argc, char** argv) {
  if (argc < 6) return 2;
  const int64_t n = argc > 6 ? atol(argv[6]) : 1 << 17, nnz = argc > 6 ? n : 100000000;
  const int d_in = atoi(argv[3]), d_out = atoi(argv[4]), ld = atoi(argv[5]);
  gcn_csr A;
  A.n_global = A.nr = A.nc = n;
  A.nnz = nnz;
  void* any = aligned_alloc(4096, 4096);             // (nothing is read: kernels do nothing)
  A.rowptr = A.colptr = (int64_t*)any;
  A.col = A.rowidx = A.deg = (int32_t*)any;
  A.val = A.val_t = (float*)any;
  for (Schedule* s : {&A.sched, &A.sched_t}) {
    s->wave_rows = (int32_t*)any;
    s->n_wave_rows = n;
    for (int c = 23; c < 34; ++c) s->class_begin[c] = n;            // all rows in class 22: 512 to 1023 entries
    for (int j = 0; j <= kRowChunks; ++j) {
      s->chunk_row[j] = n / kRowChunks * j;
      for (int c = 0; c < 33; ++c) s->chunk_class_begin[j][c] = c < 22 ? 0 : c == 22 ? s->chunk_row[j] : n;
    }
  }
  if (gcn_debug_set_tuning("GCN_OVERLAP", atoi(argv[1])) != GCN_OK || gcn_debug_set_tuning("GCN_SPMM_PANEL", 0) != GCN_OK) return 2;
  float* p = (float*)any;
  const int rc = !strcmp(argv[2], "dense") ? gcn_dense_fwd(p, ld, n, p, nullptr, d_in, d_out, GCN_ACT_RELU, GCN_F32, nullptr, p + 64, round_up(d_out, 4), nullptr)
                 : !strcmp(argv[2], "grad") ? gcn_layer_bwd_ld(&A, p, round_up(d_in, 4), p + 64, ld, p, d_in, d_out, GCN_F32, p + 128, round_up(d_out, 2), nullptr, 0, p + 256,
                                                             nullptr, nullptr, 0, nullptr)
                 : !strcmp(argv[2], "down") || !strcmp(argv[2], "masked")
                     ? gcn_layer_bwd_ld(&A, p, round_up(d_in, 4), p + 64, ld, p, d_in, d_out, GCN_F32, p + 128, round_up(d_out, 4), argv[2][0] == 'm' ? p + 192 : nullptr,
                                        round_up(d_in, 4), p + 256, nullptr, p + 320, round_up(d_in, 4), nullptr)
                 : !strcmp(argv[2], "fwd")
                     ? gcn_layer_fwd_ld(&A, p, round_up(d_in, 4), p, nullptr, d_in, d_out, GCN_ACT_RELU, GCN_F32, nullptr, 0, p + 64, round_up(d_out, 4), p + 128, ld, nullptr)
                     : gcn_layer_bwd_ld(&A, p, round_up(d_in, 4), p + 64, ld, p, d_in, d_out, GCN_F32, p + 128, round_up(d_out, 4), p + 192, round_up(d_in, 4), p + 256,
                                        nullptr, p + 320, round_up(d_in, 4), nullptr);
  if (rc != GCN_OK) { printf("%d %s\n", rc, gcn_last_error()); fflush(stdout); _Exit(1); }
  fflush(stdout);
  _Exit(0);
}
