// A stand-in for the HIP runtime's host calls that records launches instead of
// making them, so that the library's choice of kernels and its behaviour when a
// launch fails can be tested without a GPU.  Loaded before libtcu.so with its
// symbols global, it is what the library's references resolve to.
#include <hip/hip_runtime_api.h>

#include <cstdint>
#include <cstring>
#include <map>
#include <string>
#include <vector>

namespace {
struct Launch {
  const char *name;
  uint64_t blocks;
  uint32_t threads;
  int ints[16];   // the low words of the first arguments
  int status;
};
std::map<const void *, std::string> &names() {
  static std::map<const void *, std::string> m;
  return m;
}
std::map<const void *, int> &arity() {
  static std::map<const void *, int> m;
  return m;
}
std::vector<Launch> log_;
int fail_at = -1;   // index of the launch that fails
hipError_t last = hipSuccess;
dim3 g_grid, g_block;
size_t g_shmem;
hipStream_t g_stream;
int cus = 256;
}  // namespace

extern "C" {
void **__hipRegisterFatBinary(const void *) {
  static void *handle;
  return &handle;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *,
                           void *, void *, void *, int *) {
  names()[host] = name;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shmem, hipStream_t stream) {
  g_grid = grid;
  g_block = block;
  g_shmem = shmem;
  g_stream = stream;
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *shmem, hipStream_t *stream) {
  *grid = g_grid;
  *block = g_block;
  *shmem = g_shmem;
  *stream = g_stream;
  return hipSuccess;
}
hipError_t hipGetDeviceCount(int *n) {
  *n = 1;
  return hipSuccess;
}
hipError_t hipGetDevice(int *d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int) {
  std::memset(p, 0, sizeof(*p));
  std::strcpy(p->gcnArchName, "gfx950");
  p->multiProcessorCount = cus;
  return hipSuccess;
}
hipError_t hipGetLastError() {
  const hipError_t e = last;
  last = hipSuccess;
  return e;
}
hipError_t hipPeekAtLastError() { return last; }
hipError_t hipLaunchKernel(const void *fn, dim3 grid, dim3 block, void **args, size_t, hipStream_t) {
  Launch l{};
  const std::string &name = names()[fn];
  l.name = name.c_str();
  l.blocks = (uint64_t)grid.x * grid.y * grid.z;
  l.threads = block.x * block.y * block.z;
  for (int i = 0; i < arity()[fn] && i < 16; ++i) std::memcpy(&l.ints[i], args[i], 4);
  // the limit the runtime puts on a launch: work items per dimension in 32 bits
  if ((uint64_t)grid.x * block.x > UINT32_MAX) l.status = hipErrorInvalidConfiguration;
  if ((int)log_.size() == fail_at) l.status = hipErrorLaunchFailure;
  last = (hipError_t)l.status;
  log_.push_back(l);
  return last;
}

// The test's side.
void rec_reset(int fail) {
  log_.clear();
  fail_at = fail;
  last = hipSuccess;
}
int rec_count() { return (int)log_.size(); }
const char *rec_name(int i) { return log_[i].name; }
uint64_t rec_blocks(int i) { return log_[i].blocks; }
uint32_t rec_threads(int i) { return log_[i].threads; }
int rec_status(int i) { return log_[i].status; }
int rec_int(int i, int arg) { return log_[i].ints[arg]; }
// Arguments of the kernels whose mangled name holds `part`.
void rec_arity(const char *part, int n) {
  for (const auto &f : names())
    if (f.second.find(part) != std::string::npos) arity()[f.first] = n;
}
}
