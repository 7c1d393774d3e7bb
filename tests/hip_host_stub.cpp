// The HIP, rocBLAS and rocSOLVER entry points that libchefsi.so uses, on the host: loaded before
// the library in a process without a GPU, they let its host code run.  "Device" memory is host
// memory, kernels are not run: a launch appends the kernel's (or library call's) name to a list,
// and a null table handed to a kernel that reads it is counted.  stub_fail(k): the k-th allocation from now on fails.
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>

namespace {
long fail_at = 0;
long null_tables = 0;
int last_error = 0;  // until it is asked for, as in HIP
std::string launches;
std::map<const void*, std::string>& kernels() {
  static std::map<const void*, std::string> m;
  return m;
}
}  // namespace

struct dim3 {
  unsigned x, y, z;
};

#define ZERO(name) \
  int name() { return 0; }

extern "C" {
void stub_fail(long k) { fail_at = k; }
long stub_null_tables() { return null_tables; }
const char* stub_launches() { return launches.c_str(); }
void stub_clear() { launches.clear(); }

int hipMalloc(void** p, size_t n) {
  if (fail_at > 0 && --fail_at == 0) return last_error = 2;  // hipErrorOutOfMemory
  *p = std::malloc(n ? n : 1);
  return *p ? 0 : 2;
}
int hipGetLastError() {
  const int e = last_error;
  last_error = 0;
  return e;
}
int hipFree(void* p) {
  std::free(p);
  return 0;
}
int hipHostMalloc(void** p, size_t n, unsigned) {
  *p = std::calloc(n ? n : 1, 1);
  return *p ? 0 : 2;
}
int hipHostFree(void* p) {
  std::free(p);
  return 0;
}
int hipMemcpy(void* d, const void* s, size_t n, int) {
  std::memcpy(d, s, n);
  return 0;
}
int hipMemcpyAsync(void* d, const void* s, size_t n, int, void*) {
  std::memmove(d, s, n);
  return 0;
}
int hipGetSymbolAddress(void** p, const void*) {
  static void* scratch = std::malloc((size_t)64 << 20);
  *p = scratch;
  return 0;
}
int hipGetDevice(int* d) {
  *d = 0;
  return 0;
}
int hipDeviceGetAttribute(int* v, int, int) {
  *v = 256;
  return 0;
}
int hipEventElapsedTime(float* ms, void*, void*) {
  *ms = 1.f;
  return 0;
}
const char* hipGetErrorString(int) { return "stub"; }
ZERO(hipSetDevice)
ZERO(hipStreamSynchronize)
ZERO(hipEventCreate)
ZERO(hipEventDestroy)
ZERO(hipEventRecord)
ZERO(hipEventSynchronize)

void** __hipRegisterFatBinary(const void*) {
  static void* h;
  return &h;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
  if (std::strstr(name, "chefsi")) kernels()[f] = name;
}
int __hipPushCallConfiguration(dim3, dim3, size_t, void*) { return 0; }
int __hipPopCallConfiguration(dim3* g, dim3* b, size_t* lds, void** s) {
  *g = *b = dim3{1, 1, 1};
  *lds = 0;
  *s = nullptr;
  return 0;
}
int hipLaunchKernel(const void* f, dim3, dim3, void** args, size_t, void*) {
  const std::string& name = kernels()[f];
  launches += name + "\n";
  // nl_band_reduce_kernel(partial, q_slot_ptr, q_slot, gdv, ...)
  if (name.find("nl_band_reduce_kernel") != std::string::npos)
    for (int i = 0; i < 4; ++i) null_tables += *static_cast<void**>(args[i]) == nullptr;
  return 0;
}
int hipLaunchCooperativeKernel(const void* f, dim3 g, dim3 b, void** args, unsigned lds, void* s) {
  return hipLaunchKernel(f, g, b, args, lds, s);
}

int rocblas_create_handle(void** h) {
  static int one;
  *h = &one;
  return 0;
}
int rocblas_stop_device_memory_size_query(void*, size_t* n) {
  *n = 0;
  return 0;
}
int rocblas_dgemm_strided_batched() {
  launches += "rocblas_dgemm_strided_batched\n";
  return 0;
}
const char* rocblas_status_to_string(int) { return "stub"; }
ZERO(rocblas_destroy_handle)
ZERO(rocblas_set_atomics_mode)
ZERO(rocblas_set_stream)
ZERO(rocblas_set_workspace)
ZERO(rocblas_start_device_memory_size_query)
ZERO(rocblas_dgemm)
ZERO(rocblas_dtrsm)
ZERO(rocblas_zgemm)
ZERO(rocblas_zgemm_strided_batched)
ZERO(rocblas_ztrsm)
ZERO(rocsolver_dpotrf)
ZERO(rocsolver_dstedc)
ZERO(rocsolver_dsyevd)
ZERO(rocsolver_zheevd)
ZERO(rocsolver_zpotrf)
}
