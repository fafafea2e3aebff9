// The one-layer kernels of persistent_large_dev.h for H = 1024 and 2048, and the kernels around them: initial states into exchange
// layout, counters of a repeated launch.
#include "persistent_large_dev.h"

namespace lstm {
namespace {

// The same for its S3 variant, one piece of 8 k per thread; and in fp32 for the kernel that may have to run the launch again.
__global__ void pack_stateL3_kernel(const float* __restrict__ h0, float* __restrict__ hx, float* __restrict__ hx0, int T, int B, int H,
                                    int b0, int nsl) {
  const long cnt = (long)nsl * 32 * (H / 8);
  for (long e = (long)blockIdx.x * blockDim.x + threadIdx.x; e < cnt; e += (long)gridDim.x * blockDim.x) {
    const int k8 = (int)(e % (H / 8)), lb = (int)((e / (H / 8)) % 32), sl = (int)(e / ((long)(H / 8) * 32));
    const int bb = b0 + 32 * sl + lb;
    float v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = (h0 && bb < B) ? h0[(size_t)bb * H + 8 * k8 + j] : 0.f;
    float* const f = hx0 + (size_t)sl * H * 32 + (size_t)k8 * 256 + 4 * lb;
    *reinterpret_cast<floatx4*>(f) = floatx4{v[0], v[2], v[4], v[6]};
    *reinterpret_cast<floatx4*>(f + 128) = floatx4{v[1], v[3], v[5], v[7]};
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] *= kUp;
    bf16x8 p[3];
    split8(v, p);
    uintx4* const o = reinterpret_cast<uintx4*>(hx + (size_t)sl * (T + 1) * H * 48) + (size_t)k8 * 32 + lb;
#pragma unroll
    for (int q = 0; q < 3; ++q) o[(size_t)q * H * 4] = __builtin_bit_cast(uintx4, p[q]);
  }
}

// h0 [B][H] of one layer (zeros if null) -> exchange slot 0 of every slice in the layout of pers_fwdL_kernel, all 32 batch columns.
__global__ void pack_stateL_kernel(const float* __restrict__ h0, float* __restrict__ hx, int T, int B, int H, int b0,
                                   int nsl) {
  const long cnt = (long)nsl * 32 * H;
  for (long e = (long)blockIdx.x * blockDim.x + threadIdx.x; e < cnt; e += (long)gridDim.x * blockDim.x) {
    const int k = (int)(e % H), lb = (int)((e / H) % 32), sl = (int)(e / ((long)H * 32));
    const int bb = b0 + 32 * sl + lb;
    const int wv = k / (H / 4), kr = k % (H / 4), k8 = kr >> 3, m = (kr >> 1) & 3, kk = kr & 1;
    hx[(size_t)sl * (T + 1) * H * 32 + ((size_t)wv * (H / 32) + k8) * 256 + (kk * 32 + lb) * 4 + m] =
        (h0 && bb < B) ? h0[(size_t)bb * H + k] : 0.f;
  }
}

// Counters at zero for a launch of pers_bwdL_kernel that is repeated on request.
__global__ void redo_bwdL_kernel(const PersBwdLArgs a, int counters) {
  if (*a.redo == 0) return;
  for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < counters; e += gridDim.x * blockDim.x) a.flagsA[e] = 0;
}

}  // namespace

hipError_t launch_fwdL_any(int H, int cell, const PersFwdLArgs& k, hipStream_t s, bool s3) {
  if (H == 2048) return launch_fwdL_cell<2048>(cell, k, s, s3);
  if (H == 1024) return launch_fwdL_cell<1024>(cell, k, s, s3);
  return launch_fwdL_mid(H, cell, k, s, s3);
}

hipError_t launch_bwdL_any(int H, int cell, const PersBwdLArgs& k, hipStream_t s, bool s3) {
  if (H == 2048) return launch_bwdL_cell<2048, 1>(cell, k, s, s3);
  if (H != 1024) return launch_bwdL_mid(H, cell, k, s, s3);
  if (k.ks == 4) return launch_bwdL_cell<1024, 4>(cell, k, s, s3);
  if (k.ks == 2) return launch_bwdL_cell<1024, 2>(cell, k, s, s3);
  return launch_bwdL_cell<1024, 1>(cell, k, s, s3);
}

hipError_t launch_pack_stateL(const float* h0, float* hx, int T, int B, int H, int b0, int nsl, hipStream_t s) {
  hipLaunchKernelGGL(pack_stateL_kernel, dim3((unsigned)((32L * nsl * H + 255) / 256)), dim3(256), 0, s, h0, hx, T, B, H, b0, nsl);
  return hipGetLastError();
}

hipError_t launch_pack_stateL3(const float* h0, float* hx, float* hx0, int T, int B, int H, int b0, int nsl, hipStream_t s) {
  hipLaunchKernelGGL(pack_stateL3_kernel, dim3((unsigned)((4L * nsl * H + 255) / 256)), dim3(256), 0, s, h0, hx, hx0, T, B, H, b0, nsl);
  return hipGetLastError();
}

hipError_t launch_redo_bwdL(const PersBwdLArgs& k, int counters, hipStream_t s) {
  hipLaunchKernelGGL(redo_bwdL_kernel, dim3(256), dim3(256), 0, s, k, counters);
  return hipGetLastError();
}

}  // namespace lstm
