// The HIP runtime calls that the library makes, on host memory, for CPU tests
// of its host code (linked in place of the HIP runtime).  A kernel launch is
// recorded by name; those that load, lay out and start LPs run as plain loops, all
// others do nothing (an LP then runs until a limit ends it).  A device allocation can
// be made to fail.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <functional>
#include <map>
#include <string>
#include <vector>

#include "halp_types.h"
#include "kernels.h"

namespace stub {

struct Launch {
  std::string name;  // without namespace and arguments
  unsigned grid = 0, block = 0;
  size_t lds = 0;
  hipStream_t stream = nullptr;
};

// host function -> demangled name (filled before other globals are constructed)
inline std::map<const void*, std::string>& kernels() {
  static std::map<const void*, std::string> k;
  return k;
}
inline std::vector<Launch> launches;
inline std::map<void*, size_t> memory;
inline std::vector<size_t> sizes;  // of the allocations made
inline size_t bytes = 0, limit = SIZE_MAX;
inline long fail_at = -1;  // >= 0: after so many device allocations all fail
inline std::function<void(const Launch&, void**)> on_launch;

inline void reset() {
  launches.clear();
  sizes.clear();
  limit = SIZE_MAX;
  fail_at = -1;
  on_launch = nullptr;
}
inline size_t count(const std::string& part, size_t from = 0) {
  size_t n = 0;
  for (size_t i = from; i < launches.size(); ++i) n += launches[i].name.find(part) != std::string::npos;
  return n;
}
template <class V>
V& arg(void** a, int i) {
  return *static_cast<V*>(a[i]);
}

template <class K>
void radix_scatter(void** a) {
  const K* kin = arg<const K*>(a, 0);
  const int32_t* vin = arg<const int32_t*>(a, 1);
  K* kout = arg<K*>(a, 2);
  int32_t* vout = arg<int32_t*>(a, 3);
  const int64_t n = arg<int64_t>(a, 4);
  const int shift = arg<int>(a, 5);
  std::vector<int64_t> first(257, 0);
  for (int64_t i = 0; i < n; ++i) ++first[((kin[i] >> shift) & 255) + 1];
  for (int d = 0; d < 256; ++d) first[d + 1] += first[d];
  for (int64_t i = 0; i < n; ++i) {
    const int64_t at = first[(kin[i] >> shift) & 255]++;
    kout[at] = kin[i];
    vout[at] = vin[i];
  }
}

// The kernels that load, lay out and start LPs.
inline void run(const std::string& name, unsigned grid, void** a) {
  using halp::Blk;
  auto is = [&](const char* k) { return name.compare(0, strlen(k), k) == 0; };
  if (is("row_ends_kernel")) {
    for (int k = 0; k < arg<int>(a, 1); ++k) {
      const halp::LpInput& p = arg<const halp::LpInput*>(a, 0)[k];
      arg<int2*>(a, 2)[k] = make_int2(p.rp[0], p.rp[p.m]);
    }
  } else if (is("load_lps_kernel")) {
    for (unsigned k = 0; k < grid / arg<int>(a, 1); ++k) {
      const halp::LpInput& p = arg<const halp::LpInput*>(a, 0)[k];
      for (int64_t r = 0; r <= p.m; ++r) arg<int32_t*>(a, 2)[p.row0 + r] = (int32_t)(p.rp[r] + p.nz0);
      for (int64_t e = 0; e < p.nnz; ++e) arg<int32_t*>(a, 3)[p.nz0 + e] = (int32_t)(p.ci[e] + p.col0);
    }
  } else if (is("write_states_kernel")) {
    for (int i = 0; i < arg<int>(a, 5); ++i) {
      const int id = arg<const int*>(a, 3)[i];
      arg<halp::InstState*>(a, 0)[id] = arg<const halp::InstState*>(a, 4)[i];
      arg<int*>(a, 1)[id] = arg<const halp::InstState*>(a, 4)[i].status;
    }
  } else if (is("set_limit_status_kernel")) {
    for (int i = 0; i < arg<int>(a, 2); ++i)
      if (arg<halp::InstState*>(a, 0)[i].status == halp::ST_RUNNING)
        arg<halp::InstState*>(a, 0)[i].status = arg<int*>(a, 1)[i] = arg<int>(a, 3);
  } else if (is("shift_copy_kernel")) {
    for (int64_t i = 0; i < arg<int64_t>(a, 2); ++i)
      arg<int32_t*>(a, 0)[i] = (int32_t)(arg<const int32_t*>(a, 1)[i] + arg<int64_t>(a, 3));
  } else if (is("iota_kernel")) {
    for (int64_t i = 0; i < arg<int64_t>(a, 1); ++i) arg<int32_t*>(a, 0)[i] = (int32_t)i;
  } else if (is("row_ids_kernel")) {
    const int32_t* rp = arg<const int32_t*>(a, 1);
    for (unsigned b = 0; b < grid; ++b)
      for (int r = arg<const Blk*>(a, 0)[b].r0; r < arg<const Blk*>(a, 0)[b].r1; ++r)
        for (int e = rp[r]; e < rp[r + 1]; ++e) arg<int32_t*>(a, 3)[e - arg<int64_t>(a, 2)] = r;
  } else if (is("radix_scatter_kernel<unsigned int>")) {
    radix_scatter<uint32_t>(a);
  } else if (is("radix_scatter_kernel<unsigned long>")) {
    radix_scatter<uint64_t>(a);
  } else if (is("transpose_gather_kernel")) {
    const int64_t z0 = arg<int64_t>(a, 3);
    for (int64_t p = 0; p < arg<int64_t>(a, 4); ++p) {
      const int32_t e = arg<const int32_t*>(a, 0)[p];
      arg<int32_t*>(a, 5)[z0 + p] = arg<const int32_t*>(a, 1)[e];
      arg<double*>(a, 6)[z0 + p] = arg<const double*>(a, 2)[z0 + e];
    }
  } else if (is("transpose_rowptr_kernel")) {
    const uint32_t* k = arg<const uint32_t*>(a, 0);
    const int64_t nnz = arg<int64_t>(a, 1), z0 = arg<int64_t>(a, 2), c0 = arg<int64_t>(a, 3), c1 = arg<int64_t>(a, 4);
    for (int64_t j = c0; j <= c1; ++j)
      arg<int32_t*>(a, 5)[j] = (int32_t)(z0 + (std::lower_bound(k, k + nnz, (uint32_t)(j - c0)) - k));
  } else if (is("group_keys_kernel")) {
    const int32_t *rp = arg<const int32_t*>(a, 1), *ci = arg<const int32_t*>(a, 2), *gs = arg<const int32_t*>(a, 3);
    const int64_t r0 = arg<int64_t>(a, 5), z0 = arg<int64_t>(a, 6), c0 = arg<int64_t>(a, 7), len = arg<int64_t>(a, 8);
    const int ng = arg<int>(a, 4), nsl = arg<int>(a, 9), rb = arg<int>(a, 10);
    for (int g = 0; g < ng; ++g)
      for (int64_t r = gs[g]; r < gs[g + 1]; ++r)
        for (int32_t e = rp[r0 + r]; e < rp[r0 + r + 1]; ++e) {
          const int64_t c = ci[e] - c0, q = c * nsl / len, first = (q * len + nsl - 1) / nsl;
          arg<uint64_t*>(a, 11)[e - z0] =
              ((uint64_t)(g * nsl + q) << 32) | ((uint32_t)(c - first) << rb) | (uint32_t)(r - gs[g]);
          arg<int32_t*>(a, 12)[e - z0] = e;
        }
  } else if (is("group_count_kernel")) {
    const int32_t *rp = arg<const int32_t*>(a, 1), *ci = arg<const int32_t*>(a, 2), *gs = arg<const int32_t*>(a, 3);
    const int64_t r0 = arg<int64_t>(a, 5), c0 = arg<int64_t>(a, 6), len = arg<int64_t>(a, 7);
    const int ng = arg<int>(a, 4), nsl = arg<int>(a, 8);
    for (int g = 0; g < ng; ++g)
      for (int32_t e = rp[r0 + gs[g]]; e < rp[r0 + gs[g + 1]]; ++e)
        ++arg<int32_t*>(a, 9)[(int64_t)g * nsl + (ci[e] - c0) * nsl / len];
  } else if (is("segment_offsets_kernel")) {
    const uint64_t* k = arg<const uint64_t*>(a, 0);
    for (int s = 0; s <= arg<int>(a, 2); ++s)
      arg<int32_t*>(a, 3)[s] = (int32_t)(std::lower_bound(k, k + arg<int64_t>(a, 1), (uint64_t)s << 32) - k);
  }
}

}  // namespace stub

extern "C" {
hipError_t hipMalloc(void** p, size_t n) {
  *p = nullptr;
  if (stub::fail_at == 0 || n > stub::limit - std::min(stub::limit, stub::bytes)) return hipErrorOutOfMemory;
  if (stub::fail_at > 0) --stub::fail_at;
  *p = calloc(std::max<size_t>(n, 1), 1);
  stub::memory[*p] = n;
  stub::bytes += n;
  stub::sizes.push_back(n);
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  if (!p) return hipSuccess;
  auto it = stub::memory.find(p);
  if (it == stub::memory.end()) {
    fprintf(stderr, "release of memory that was not allocated\n");
    abort();
  }
  stub::bytes -= it->second;
  stub::memory.erase(it);
  free(p);
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return (*p = calloc(n, 1)) ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipHostFree(void* p) { return free(p), hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
  if (n && (!d || !s)) return hipErrorInvalidValue;
  return memcpy(d, s, n), hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind k, hipStream_t) { return hipMemcpy(d, s, n, k); }
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) { return memset(d, v, n), hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "stub error"; }
hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void* s) { return *p = const_cast<void*>(s), hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { return *s = (hipStream_t)(uintptr_t)16, hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipErrorNotSupported; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t*) { return hipErrorNotSupported; }
hipError_t hipGraphInstantiate(hipGraphExec_t*, hipGraph_t, hipGraphNode_t*, char*, size_t) { return hipErrorNotSupported; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipErrorNotSupported; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { return *e = (hipEvent_t)(uintptr_t)16, hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* t, hipEvent_t, hipEvent_t) { return *t = 0.f, hipSuccess; }

static struct {
  dim3 grid, block;
  size_t lds;
  hipStream_t stream;
} g_call;
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, hipStream_t s) { return g_call = {g, b, lds, s}, hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* lds, hipStream_t* s) {
  *g = g_call.grid;
  *b = g_call.block;
  *lds = g_call.lds;
  *s = g_call.stream;
  return hipSuccess;
}
char* __cxa_demangle(const char*, char*, size_t*, int*);
void** __hipRegisterFatBinary(const void*) {
  static void* handle;
  return &handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
  int rc = 0;
  char* d = __cxa_demangle(name, nullptr, nullptr, &rc);
  std::string s = rc == 0 ? d : name;
  free(d);
  s = s.substr(0, s.find("("));
  const size_t at = s.find("halp::");
  stub::kernels()[host] = at == std::string::npos ? s : s.substr(at + 6);
}
hipError_t hipLaunchKernel(const void* f, dim3 g, dim3 b, void** args, size_t lds, hipStream_t s) {
  if (g.x == 0 || b.x == 0 || (uint64_t)g.x * b.x > UINT32_MAX) return hipErrorInvalidConfiguration;
  stub::launches.push_back({stub::kernels().at(f), g.x, b.x, lds, s});
  stub::run(stub::launches.back().name, g.x, args);
  if (stub::on_launch) stub::on_launch(stub::launches.back(), args);
  return hipSuccess;
}
}
