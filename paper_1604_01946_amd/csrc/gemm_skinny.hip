// Products of up to 64 rows with a large second operand (the recurrent product of a step, H above what fits on chip; up to 8 rows
// where B has its unit stride along n, the others row by row): gemm_skinny_kernel.
//
// Bound: the second operand, read once, and the cutting of both operands into three bf16 parts (split3.h).  The tiles of
// gemm_split3_kernel pass through LDS with two barriers per 16 k, and a round of 64 x 64 tiles leaves one workgroup per CU, which waits
// at them: 16 x 16384 x 4096, 268 MB, takes 65 us there and 43 us = 6.2 TB/s here, 32 rows 71 and 50, 64 rows 76 and 73 (the cutting
// and the matrix instructions then take longer than the reading; 64 x 4096 x 16384 along n 82 and 66).  Here a wave multiplies all rows by 64 columns and has its own run of k: operands go from memory to registers in the layout of the matrix instructions,
// no barrier before the end, where the eight waves of a workgroup add up through LDS.
//   v_mfma_f32_16x16x32_bf16, the tile's rows are columns of the product.  Lane (q, r) needs eight k of column r (of row r of A);
//   which eight is free as long as both operands agree:
//   B with unit stride along k: k = 16 (p/4) + 4 q + p%4, 16-byte loads of which four lanes cover 64 bytes of a column;
//   B with unit stride along n: k = 8 q + p, a 16-byte load brings one k of four columns, 4 r + tile, 256 bytes of a row together.
// The sums of the first and last quarter of a wave's k and those of the middle are formed with opposite signs, as in the other kernel
// (the bf16 instructions cut low bits off downwards), and a wave with a sum that is not finite works its k out again in fp32.
#include "internal.h"
#include "persistent.h"
#include "split3.h"

#include <algorithm>

namespace lstm {
namespace {

constexpr int kLdsRow = 68;  // floats of a row of sums in LDS (64 and no bank conflicts)

struct SkinnyArgs {
  GemmProblem p;
  int slices;
  float* part;  // partial tiles [block of 64 columns][slice][64][64], slices > 1
};

template <int MT, bool KN>
__global__ __launch_bounds__(512) void gemm_skinny_kernel(const SkinnyArgs g) {
  extern __shared__ __align__(16) float red[];  // [4][16 MT][kLdsRow]
  const GemmProblem& P = g.p;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), r = lane & 15, q = lane >> 4;
  const int nb = blockIdx.x / g.slices, sl = blockIdx.x % g.slices, n0 = 64 * nb, M = P.M, N = P.N;
  // units of 32 k: of the slice, of the wave
  const int all = P.K / 32, us = (int)((long)all * sl / g.slices), ue = (int)((long)all * (sl + 1) / g.slices);
  const int u0 = us + (ue - us) * wave / 8, nu = us + (ue - us) * (wave + 1) / 8 - u0;

  floatx4 acc[4][MT];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < MT; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};

  // lane offsets in floats; rows and columns past the end repeat the last one
  unsigned oa[MT], ob[4];
#pragma unroll
  for (int j = 0; j < MT; ++j) oa[j] = (unsigned)(min(16 * j + r, M - 1) * P.sAm) + (KN ? 8 : 4) * q;
#pragma unroll
  for (int i = 0; i < 4; ++i) ob[i] = KN ? 0u : (unsigned)(min(16 * i + r, N - 1 - n0) * P.sBn) + 4 * q;
  if (KN) ob[0] = (unsigned)(8 * q * P.sBk) + (unsigned)min(4 * r, N - 4 - n0);
  const long kb = KN ? P.sBk : 1;  // floats from k to k in B
  const float* pa = P.A + 32L * u0;
  const float* pb = P.B + 32L * u0 * kb + (KN ? (long)n0 : (long)n0 * P.sBn);
  floatx4 a[MT][2], b[8];
  auto load_a = [&](int j) {
    a[j][0] = *reinterpret_cast<const floatx4*>(pa + oa[j]);
    a[j][1] = *reinterpret_cast<const floatx4*>(pa + oa[j] + (KN ? 4 : 16));
  };
  auto load_b = [&]() {
#pragma unroll
    for (int i = 0; i < 8; ++i) b[i] = *reinterpret_cast<const floatx4*>(KN ? pb + i * kb + ob[0] : pb + ob[i / 2] + 16 * (i % 2));
  };
  if (nu > 0) {
    load_b();
#pragma unroll
    for (int j = 0; j < MT; ++j) load_a(j);
  }
  const int turn = nu / 4;
  for (int u = 0; u < nu; ++u) {
    const bool minus = u >= turn && u < nu - turn;
    if (u == turn || u == nu - turn) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < MT; ++j) acc[i][j] = -acc[i][j];
    }
    const float up = minus ? -kUp : kUp;
    const bool more = u + 1 < nu;  // (the last unit is asked for again, for nobody)
    bf16x8 fb[4][3];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float v[8];
#pragma unroll
      for (int p = 0; p < 8; ++p) v[p] = (KN ? b[p][i] : b[2 * i + p / 4][p % 4]) * up;
      split8(v, fb[i]);
    }
    pa += more ? 32 : 0;
    pb += more ? 32 * kb : 0;
    load_b();
#pragma unroll
    for (int j = 0; j < MT; ++j) {
      float v[8];
#pragma unroll
      for (int p = 0; p < 8; ++p) v[p] = a[j][p / 4][p % 4] * kUp;
      bf16x8 fa[3];
      split8(v, fa);
      load_a(j);
      constexpr int pr[6][2] = {{2, 0}, {0, 2}, {1, 1}, {1, 0}, {0, 1}, {0, 0}};  // parts, smallest products first
#pragma unroll
      for (int s = 0; s < 6; ++s)
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[i][pr[s][0]], fa[pr[s][1]], acc[i][j], 0, 0, 0);
    }
  }
  if (nu > 0 && nu - turn == nu) {  // (fewer than four units: all of them with the other sign)
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < MT; ++j) acc[i][j] = -acc[i][j];
  }
  float z = 0.f;
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < MT; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        acc[i][j][e] *= kDown;
        z += acc[i][j][e] * 0.f;
      }
  if (__any(z != 0.f)) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < MT; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    for (int k = 32 * u0; k < 32 * (u0 + nu); k += 4) {
      float va[MT], vb[4];
#pragma unroll
      for (int j = 0; j < MT; ++j) va[j] = P.A[(long)min(16 * j + r, M - 1) * P.sAm + k + q];
#pragma unroll
      for (int i = 0; i < 4; ++i) vb[i] = P.B[(long)(k + q) * P.sBk + (long)min(n0 + (KN ? 4 * r + i : 16 * i + r), N - 1) * P.sBn];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < MT; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(vb[i], va[j], acc[i][j], 0, 0, 0);
    }
  }

  // ---- sums of the eight waves.  Element e of lane (q, r) in tile (i, j): row 16 j + r of the product, column 16 i + 4 q + e (KN:
  // 4 (4 q + e) + i); pieces of four columns
  auto piece = [&](int c, int j) {  // of four: KN column 16 q + 4 c, else 16 c + 4 q
    return KN ? floatx4{acc[0][j][c], acc[1][j][c], acc[2][j][c], acc[3][j][c]} : acc[c][j];
  };
  auto at = [&](int w, int c, int j) { return red + ((w * 16 * MT) + 16 * j + r) * kLdsRow + (KN ? 16 * q + 4 * c : 16 * c + 4 * q); };
  if (wave >= 4) {
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int j = 0; j < MT; ++j) *reinterpret_cast<floatx4*>(at(wave - 4, c, j)) = piece(c, j);
  }
  __syncthreads();
  if (wave < 4) {
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int j = 0; j < MT; ++j) {
        floatx4* const p = reinterpret_cast<floatx4*>(at(wave, c, j));
        *p = piece(c, j) + *p;
      }
  }
  __syncthreads();
  for (int e = threadIdx.x; e < 256 * MT; e += 512) {
    const int row = e / 16, col = 4 * (e % 16);
    const float* const p = red + row * kLdsRow + col;
    constexpr int W = 16 * MT * kLdsRow;
    auto of = [&](int w) { return *reinterpret_cast<const floatx4*>(p + w * W); };
    floatx4 v = (of(0) + of(1)) + (of(2) + of(3));
    if (row >= M) continue;
    if (g.slices > 1) {
      *reinterpret_cast<floatx4*>(g.part + ((size_t)blockIdx.x * 64 + row) * 64 + col) = v;
      continue;
    }
    float* const c = P.C + (long)row * P.ldc + n0 + col;
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (n0 + col + j < N) c[j] = P.accumulate ? c[j] + v[j] : v[j];
  }
}

template <int MT, bool KN>
hipError_t launch(const SkinnyArgs& g, hipStream_t s) {
  static bool ready;
  constexpr size_t smem = (size_t)4 * 16 * MT * kLdsRow * sizeof(float);
  if (const hipError_t e = allow_dynamic_lds((const void*)gemm_skinny_kernel<MT, KN>, smem, ready); e != hipSuccess) return e;
  hipLaunchKernelGGL((gemm_skinny_kernel<MT, KN>), dim3((g.p.N + 63) / 64 * g.slices), dim3(512), smem, s, g);
  return hipGetLastError();
}

}  // namespace

// Whether the kernel can take a product.
bool skinny_takes(const GemmProblem& p) {
  auto ok16 = [](const float* q, long stride) { return (reinterpret_cast<uintptr_t>(q) & 15u) == 0 && stride % 4 == 0 && stride >= 0 && stride < (1L << 24); };
  if (p.khead || p.M < 1 || p.M > 64 || p.N < 64 || p.K % 32 != 0 || p.sAk != 1 || !ok16(p.A, p.sAm)) return false;
  if (p.sBk == 1) return ok16(p.B, p.sBn);
  return p.sBn == 1 && p.N % 4 == 0 && ok16(p.B, p.sBk);
}

hipError_t launch_skinny(const GemmProblem& p, int slices, float* part, hipStream_t s) {
  const SkinnyArgs g{p, slices, part};
  const bool kn = p.sBk != 1;
  switch ((p.M + 15) / 16) {
    case 1: return kn ? launch<1, true>(g, s) : launch<1, false>(g, s);
    case 2: return kn ? launch<2, true>(g, s) : launch<2, false>(g, s);
    case 3: return kn ? launch<3, true>(g, s) : launch<3, false>(g, s);
    case 4: return kn ? launch<4, true>(g, s) : launch<4, false>(g, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace lstm
