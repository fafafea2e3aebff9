// One step of a few rows (online decoding: T = 1, B <= 16, an inference call): one launch per layer does the whole cell,
// lstm_cell_kernel.
//
// Bound: one trip to memory per layer and the launches.  Nothing is carried from step to step, so weights on chip, exchange
// slots and counters buy nothing here; the paths for sequences take a launch for the input product, one that clears the
// exchange, the recurrence, and two event packets (L = 2, I = H = 256, B = 1: 17.3 us).  A wave owns one hidden unit: its four rows
// of W and of R, whose columns the lanes share out in runs of 4 (16 bytes per lane), against all batch rows; vector FMAs in
// fp32; the sums meet across the lanes in a fixed order, and lane m finalises row m.  Weights are read once and in order, whatever the
// hidden size: no padding, no re-layout.  Before / now, us per call (L, B, I = H): (2, 1, 256) 17.5 / 11.1, (2, 8, 256) 27.6 / 12.5,
// (2, 1, 300) 57 / 10, (4, 16, 512) 56 / 48, (2, 16, 650) 133 / 33, (2, 8, 1024) 80 / 22, (4, 1, 2048) 215 / 113, (1, 1, 4096) 262 / 99 (537 MB of
// weights at 5.4 TB/s), (1, 16, 4096) 284 / 155.  Above 16 rows the matrix cores have enough to do; a second step would cost as many
// launches again; deep stacks of few units run as before (few_enough_layers).
//
// The hidden states of a layer are handed to the next one in the workspace; hT is written by the launch that no longer
// reads the initial states (the next layer's, or a copy behind the top layer's), so that hT may be h0; every c_T element is
// written by the lane that has read that element of c_0.
#include "../../include/lstm.h"
#include "schedule.h"
#include "knobs.h"

namespace lstm {
namespace {

struct CellArgs {
  const float *x, *h0, *c0, *W, *R, *bias;  // of this layer: [B][I], [B][H], [B][H], [4H][I], [4H][H], [4H]
  float *h, *y, *cT;                        // [B][H]: for the next layer, the result (top layer) or null, the final cell state or null
  const float* below;                       // hidden states of the layer below, to be copied to
  float* hT_below;                          // its final state (null: none)
  int B, I, H;
};

template <int MR, int V>
__global__ __launch_bounds__(256) void lstm_cell_kernel(const CellArgs a) {
  typedef float vec __attribute__((ext_vector_type(V)));
  const int lane = threadIdx.x & 63, u = (int)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), H = a.H;
  if (a.hT_below)
    for (int e = (int)(blockIdx.x * 256 + threadIdx.x); e < a.B * H; e += (int)gridDim.x * 256) a.hT_below[e] = a.below[e];
  if (u >= H) return;
  const int row = min(lane, a.B - 1);
  const bool fin = lane < a.B;
  const float c = a.c0 && fin ? a.c0[(size_t)row * H + u] : 0.f;
  float bias[4];
#pragma unroll
  for (int g = 0; g < 4; ++g) bias[g] = a.bias[g * H + u];
  float acc[4][MR];
#pragma unroll
  for (int g = 0; g < 4; ++g)
#pragma unroll
    for (int m = 0; m < MR; ++m) acc[g][m] = 0.f;
  auto product = [&](const float* __restrict__ w, const float* __restrict__ in, int K) {
    const float* const wu = w + (size_t)u * K;
#pragma unroll 2
    for (int k = V * lane; k < K; k += 64 * V) {  // (V = 4: K is a multiple of 4)
      vec wv[4], iv[MR];
#pragma unroll
      for (int g = 0; g < 4; ++g) wv[g] = *reinterpret_cast<const vec*>(wu + (size_t)g * H * K + k);
#pragma unroll
      for (int m = 0; m < MR; ++m) iv[m] = *reinterpret_cast<const vec*>(in + (size_t)min(m, a.B - 1) * K + k);
#pragma unroll
      for (int g = 0; g < 4; ++g)
#pragma unroll
        for (int m = 0; m < MR; ++m)
#pragma unroll
          for (int v = 0; v < V; ++v) acc[g][m] = fmaf(wv[g][v], iv[m][v], acc[g][m]);
    }
  };
  if (a.h0) product(a.R, a.h0, H);
  product(a.W, a.x, a.I);
  float sg[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int g = 0; g < 4; ++g)
#pragma unroll
    for (int m = 0; m < MR; ++m) {
      float v = acc[g][m];
#pragma unroll
      for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d);
      sg[g] = lane == m ? v : sg[g];
    }
  if (!fin) return;
  const float gi = sigmoidf_dev(sg[0] + bias[0]), gf = sigmoidf_dev(sg[1] + bias[1]), go = sigmoidf_dev(sg[2] + bias[2]),
              gc = tanhf_dev(sg[3] + bias[3]);
  const float cn = gf * c + gi * gc, hn = go * tanhf_dev(cn);
  const size_t e = (size_t)row * H + u;
  a.h[e] = hn;
  if (a.y) a.y[e] = hn;
  if (a.cT) a.cT[e] = cn;
}

template <int MR>
void launch_cell(const CellArgs& k, bool vec4, hipStream_t s) {
  const dim3 grid((unsigned)((k.H + 3) / 4));
  if (vec4) hipLaunchKernelGGL((lstm_cell_kernel<MR, 4>), grid, dim3(256), 0, s, k);
  else hipLaunchKernelGGL((lstm_cell_kernel<MR, 1>), grid, dim3(256), 0, s, k);
}

bool overlap(const float* a, size_t na, const float* b, size_t nb) { return a && b && a < b + nb && b < a + na; }

}  // namespace

// Whether a launch per layer is the faster way.  A launch costs 3.5 us for one row, 4.7 for up to four, 6.3 for up to
// eight and 9.3 to 14 above, whatever the layers; up to H = 512 the paths for sequences run a whole stack in one launch of some 20 us and
// 1 to 6 per layer, whose rows are nearly free.  Measured with 1 to 24 layers of 33 to 3072 units, us that way / this way:
//   one row          H = 128 (a kernel of its own, up to eight layers): 16 / 14 with four layers, 22 / 29 with eight, 61 / 53 with 16; H = 256 (the
//                    same): 24 / 22 with six, 24 / 28 with eight, 49 / 57 with 16; padded to them, H = 200: 38 / 29 with eight, 65 / 57 with 16
//   up to four rows  H = 100: 61 / 56 with twelve, 75 / 78 with 16; H = 128: 37 / 37 with eight, 61 / 74 with 16; H = 256: 95 / 77 with 16
//   up to eight      H = 100: 44 / 37 with six, 49 / 50 with eight; H = 128: 28 / 25 with four, 39 / 50 with eight; H = 192: 38 / 37 with six, 46 / 51
//                    with eight; H = 256: 105 / 103 with 16
//   up to 16         H = 64: 34 / 38 with four; H = 100: 40 / 37 with four, 44 / 56 with six; H = 128: 21 / 18 with two, 28 / 37 with four; H = 200: 49 / 37 with four, 69 / 75
//                    with eight; H = 320: 33 / 28 with two, 37 / 42 with three, 41 / 56 with four; H = 448: 45 / 42 with three, 50 / 56 with four; H = 512:
//                    318 / 288 with 24
static bool few_enough_layers(int L, int B, int H) {
  if (H > 448) return true;
  if (B > 8) return L <= (H > 192 && H <= 256 ? 4 : 3);
  if (H > 256) return true;
  if (B > 4) return L <= (H == 128 ? 4 : 6) || H > 192;
  if (B > 2) return L <= (H == 128 ? 8 : 12) || H > 128;
  if (B == 2) return true;
  return L <= 6 || !(H == 256 || (H == 128 && L <= 8));
}

// An inference call of one step and few rows.  y, hT and cT must not lie over operands that another workgroup may still
// read: hT over h0 and cT over c0, element on element, are the only overlaps that it takes.
bool cell_step_takes(const FwdArgs& a) {
  const Dims& d = a.d;
  if (d.T != 1 || d.B > 16 || !knobs().cell_step) return false;
  if (!few_enough_layers(d.L, d.B, d.H)) return false;
  const size_t BH = (size_t)d.B * d.H, S = (size_t)d.L * BH, nx = (size_t)d.B * d.I, G = 4 * (size_t)d.H;
  const size_t nW = G * d.I + (size_t)(d.L - 1) * G * d.H, nR = (size_t)d.L * G * d.H, nb = (size_t)d.L * G;
  const struct { float* p; size_t n; } out[3] = {{a.y, BH}, {a.hT, S}, {a.cT, S}};
  for (int i = 0; i < 3; ++i) {
    if (overlap(out[i].p, out[i].n, a.x, nx) || overlap(out[i].p, out[i].n, a.W, nW) || overlap(out[i].p, out[i].n, a.R, nR) ||
        overlap(out[i].p, out[i].n, a.b, nb))
      return false;
    if (overlap(out[i].p, out[i].n, a.h0, S) && !(i == 1 && a.hT == a.h0)) return false;
    if (overlap(out[i].p, out[i].n, a.c0, S) && !(i == 2 && a.cT == a.c0)) return false;
  }
  return !(overlap(a.y, BH, a.hT, S) || overlap(a.y, BH, a.cT, S) || overlap(a.hT, S, a.cT, S));
}

// a.ws: L * B * H floats of it are used.
int run_cell_step(const FwdArgs& a) {
  const Dims& d = a.d;
  const size_t BH = (size_t)d.B * d.H, G = 4 * (size_t)d.H;
  float* const h = reinterpret_cast<float*>(a.ws);
  ProfScope ps(LSTM_PHASE_FWD_RECURRENCE, a.stream);
  // (hT of a layer by the next layer's launch only where it lies over h0; otherwise its own launch writes it)
  const bool late = a.hT && a.hT == a.h0;
  for (int l = 0; l < d.L; ++l) {
    CellArgs k{};
    k.I = l ? d.H : d.I;
    k.B = d.B;
    k.H = d.H;
    k.x = l ? (late ? h + (size_t)(l - 1) * BH : a.hT ? a.hT + (size_t)(l - 1) * BH : h + (size_t)(l - 1) * BH) : a.x;
    k.h0 = a.h0 ? a.h0 + l * BH : nullptr;
    k.c0 = a.c0 ? a.c0 + l * BH : nullptr;
    k.W = a.W + (l ? G * d.I + (size_t)(l - 1) * G * d.H : 0);
    k.R = a.R + (size_t)l * G * d.H;
    k.bias = a.b + (size_t)l * G;
    k.h = a.hT && !late ? a.hT + l * BH : h + l * BH;
    k.y = l == d.L - 1 ? a.y : nullptr;
    k.cT = a.cT ? a.cT + l * BH : nullptr;
    if (late && l) {
      k.below = h + (size_t)(l - 1) * BH;
      k.hT_below = a.hT + (size_t)(l - 1) * BH;
    }
    prof_flops(2.0 * d.B * G * (k.I + (k.h0 ? d.H : 0)), "lstm_cell_kernel");
    const bool vec4 = k.I % 4 == 0 && d.H % 4 == 0;
    if (d.B == 1) launch_cell<1>(k, vec4, a.stream);
    else if (d.B == 2) launch_cell<2>(k, vec4, a.stream);
    else if (d.B <= 4) launch_cell<4>(k, vec4, a.stream);
    else if (d.B <= 8) launch_cell<8>(k, vec4, a.stream);
    else launch_cell<16>(k, vec4, a.stream);
    if (record(hipGetLastError(), "cell kernel") != hipSuccess) return LSTM_HIP_ERROR;
  }
  if (late && record(launch_ew(EW_COPY, a.hT + (size_t)(d.L - 1) * BH, d.H, h + (size_t)(d.L - 1) * BH, d.H, nullptr, 0, d.B, d.H, a.stream),
                     "copy hT") != hipSuccess)
    return LSTM_HIP_ERROR;
  return LSTM_OK;
}

}  // namespace lstm
