// Which kernels the library's host code launches for a call, without a GPU:
// linked against the library's host objects and the stand-in HIP runtime below,
// which records every launch and refuses dynamic LDS beyond 64 KB where the
// kernel has not been allowed it on the current device.  Device addresses are
// made up; nothing reads them.  Reads one call a line from stdin, prints one
// line a launch ("kernel grid block lds"), then "end".
#include <cxxabi.h>

#include <cstdio>
#include <cstdlib>
#include <iostream>
#include <map>
#include <sstream>
#include <string>

#include "bandeig.h"
#include "common.h"

namespace {
// (registered before this file's own statics exist)
std::map<const void *, std::string> &names() {
  static std::map<const void *, std::string> m;
  return m;
}
std::map<std::pair<int, const void *>, int> allowed;  // dynamic LDS by device and kernel
int device = 0;
hipError_t last = hipSuccess;
struct {
  dim3 grid, block;
  size_t lds;
  hipStream_t stream;
} config;
char *address(size_t i) { return reinterpret_cast<char *>((size_t)1 << 44) + (i << 40); }
}  // namespace

extern "C" {
void **__hipRegisterFatBinary(const void *) {
  static void *handle;
  return &handle;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *f, char *, const char *name, unsigned, void *,
                           void *, void *, void *, int *) {
  int status;
  char *s = abi::__cxa_demangle(name, nullptr, nullptr, &status);
  std::string t = s ? s : name;
  std::free(s);
  const size_t a = t.find("::k_");  // bbl::(anonymous namespace)::k_name<...>(...)
  t = a == std::string::npos ? t : t.substr(a + 2);
  std::string out;
  int depth = 0;
  for (const char c : t) {
    if (c == '(' && depth == 0) break;
    depth += c == '<' ? 1 : c == '>' ? -1 : 0;
    if (c != ' ') out += c;
  }
  names()[f] = out;
}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t stream) {
  config = {grid, block, lds, stream};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, hipStream_t *stream) {
  *grid = config.grid;
  *block = config.block;
  *lds = config.lds;
  *stream = config.stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3 grid, dim3 block, void **, size_t lds,
                           hipStream_t) {
  const auto it = allowed.find({device, f});
  const bool ok = lds <= 65536 || (it != allowed.end() && (size_t)it->second >= lds);
  std::printf("%s %u %u %zu%s\n", names()[f].c_str(), grid.x * grid.y, block.x, lds,
              ok ? "" : " refused");
  if (!ok) last = hipErrorInvalidValue;
  return ok ? hipSuccess : hipErrorInvalidValue;
}
hipError_t hipFuncSetAttribute(const void *f, hipFuncAttribute, int value) {
  allowed[{device, f}] = value;
  return hipSuccess;
}
hipError_t hipGetLastError(void) {
  const hipError_t e = last;
  last = hipSuccess;
  return e;
}
const char *hipGetErrorString(hipError_t) { return "refused"; }
hipError_t hipMemcpyAsync(void *, const void *, size_t, hipMemcpyKind, hipStream_t) {
  return hipErrorInvalidValue;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipErrorInvalidValue; }
}

int main() {
  std::string line;
  while (std::getline(std::cin, line)) {
    std::istringstream in(line);
    std::string what;
    in >> what;
    try {
      if (what == "device") {
        in >> device;
      } else if (what == "band") {
        int N, kd, k;
        in >> N >> kd >> k;
        bbl::band_eigensolve(reinterpret_cast<double *>(address(0)), N, kd, k, address(1),
                             bbl::band_eig_layout(N, kd, k), nullptr, kd,
                             reinterpret_cast<double *>(address(2)),
                             reinterpret_cast<double *>(address(3)), nullptr);
      } else if (what == "spmm") {
        bbl_csr H{};
        int nvec, xdtype;
        in >> H.n >> H.nnz >> H.val_dtype >> nvec >> xdtype;
        H.row_ptr = reinterpret_cast<int64_t *>(address(0));
        H.col = reinterpret_cast<int32_t *>(address(1));
        H.val = address(2);
        bbl::launch_spmm(H, address(3), xdtype, address(4), xdtype, nvec, nullptr);
      } else if (what == "gram") {
        int64_t n;
        int xdtype, b, nblk;
        in >> n >> xdtype >> b >> nblk;
        const int parts = bbl::launch_gram(n, address(0), xdtype, b, nblk, n * b, address(1),
                                           BBL_F64, b, reinterpret_cast<double *>(address(2)),
                                           1 << 20, nullptr);
        std::printf("parts %d\n", parts);
      }
    } catch (const bbl::Error &e) {
      std::printf("error %d %s\n", e.code, e.msg.c_str());
    }
    std::printf("end\n");
    std::fflush(stdout);
  }
  return 0;
}
