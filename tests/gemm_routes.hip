// Host code of gemm.hip against a recording stand-in for the HIP runtime: which kernel instance, grid and split a
// launch takes, without a GPU (and so with the compute units of a chip that cannot be asked: 256).
#include "gemm.hip"

#include <map>
#include <string>

namespace {
std::map<const void*, std::string> g_names;
std::string g_last;
dim3 g_grid, g_block;
}  // namespace

namespace rollout {
size_t q4_code_bytes(int rows, int cols) { return (size_t)rows * cols / 2; }
}  // namespace rollout

extern "C" {
void** __hipRegisterFatBinary(const void*) {
  static void* module;
  return &module;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
  g_names[host] = name;
}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t, hipStream_t) {
  g_grid = grid;
  g_block = block;
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t*, hipStream_t*) {
  *grid = g_grid;
  *block = g_block;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3, dim3, void**, size_t, hipStream_t) {
  g_last = g_names[f];
  return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipGetDevice(int*) { return hipErrorNoDevice; }
hipError_t hipDeviceGetAttribute(int*, hipDeviceAttribute_t, int) { return hipErrorNoDevice; }

const char* last_kernel() { return g_last.c_str(); }

// A projection of more than 64 rows as the runtime launches it (swiglu, or split K with the residual added where one
// split allows it, or one split for the LM head); returns the splits, 0 where the product is added, < 0 on an error.
int project(int q4, int M, int N, int K, int max_splits, int swiglu, int residual) {
  using namespace rollout;
  g_last.clear();
  char x[1], w[1], h[1];
  float out[1];
  if (swiglu)
    return (q4 ? launch_gemm_swiglu_q4_tile(nullptr, x, w, w, M, N, K, h) : launch_gemm_swiglu(nullptr, x, w, M, N, K, h)) ? -1 : 1;
  const int s = q4 ? gemm_splits_q4(M, N, K, max_splits) : gemm_splits(ROLLOUT_DTYPE_BF16, M, N, K, max_splits);
  const bool add = residual && gemm_adds(ROLLOUT_DTYPE_BF16, M, s);
  const hipError_t e = q4 ? launch_gemm_q4_tile(nullptr, x, w, w, out, M, N, K, s, add ? 0 : 1)
                          : launch_gemm(nullptr, ROLLOUT_DTYPE_BF16, x, K, w, out, M, N, K, s, add ? 0 : 1);
  return e ? -1 : (add ? 0 : s);
}

// a plan whose nt workgroups cannot hold the matrix's weight blocks: status of its launch
int launch_plan(int nt, int M, int N, int K) {
  using namespace rollout;
  g_last.clear();
  bf16x8_t* p = nullptr;
  return launch_pp<4, 4, 2, 4, 4, false, false>(nullptr, TilePlan{T_8x16, 1, nt}, p, p, nullptr, nullptr, M, N, K, nullptr, 1);
}
}
