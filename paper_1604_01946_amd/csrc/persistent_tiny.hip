// Persistent recurrence for a single sequence (B = 1), H = 128 / 256 / 512, LSTM: pers_fwd_tiny_kernel and
// pers_bwd_tiny_kernel.
//
// With one batch row a step is a matrix-vector product of a few microseconds' worth of nothing: the time goes into the
// hop from workgroup to workgroup (Section 4 of arXiv 1604.01946 names the cost of keeping the weights on chip:
// workgroups that wait on each other) and into the instructions that a step issues around it.
//   * the data is its own flag: every exchange slot is filled with a pattern that no result can have (a NaN with a
//     payload that arithmetic never produces; a result that happens to carry it is published as the default NaN)
//     before the launch, a producer stores its values once and does nothing else, a consumer re-reads the slot with
//     agent-scope loads until no lane sees the pattern.  No acknowledgement, no counter.
//   * a layer's 32 workgroups run on the 32 CUs of one XCD, whose L2 they share: a value goes no further than that (a hop
//     from store to load takes 0.21 us, with a write-through store 0.36, to another XCD 0.51).  The workgroups find out
//     where they run and write through to memory if they are not all on one XCD.
//   * a wave owns two hidden units with all their weights over the whole K (lane i holds a few k each; the wave
//     multiplies with vector FMAs and adds up across its lanes), so no wave waits for another one's arithmetic.
//   * the H / 64 waves of a workgroup poll 1 / (H / 64) of the slot each and hand their shares to each other through
//     LDS (one barrier per step): every word of a slot is asked for once per workgroup, not once per wave.
//   * everything else -- the reserve, the values that go to the layer above or below on another XCD and come from there, the
//     input product, the bias gradient -- is the business of one more wave, through LDS: requests and acknowledgements return in
//     the order of their issue, and a poll behind a store to memory waits for that store.
//   * the half of a step's products that does not need the slot (input, gradient for the layer below) is multiplied while
//     the slot is on its way.
// Measured, L = 2, T = 500, H = 256: 0.88 us per forward step and 0.99 us per backward step (1.25 and 1.40 with write-through
// stores on all XCDs and no serving wave); H = 512, L = 1, T = 200 1.3 and 1.9 (1.7 and 1.9).
// Section 2.4's wavefront over layers is the same polling: layer l reads what layer l-1 (forward) or layer l+1 (backward)
// handed over, two to three steps behind it.  Every poll is bounded (watchdog as in the other persistent kernels).
#include "../../include/lstm.h"
#include "near_dev.h"

#include <algorithm>

namespace lstm {
namespace {

struct TinyWaiter : NearWaiter {
  // Four consecutive values per lane of a slot of n floats.  Every word is its own flag: a request that is served while the
  // producer is writing is simply partly empty.
  __device__ __forceinline__ floatx4 poll4(const float* slot, int n, int at) {
    int spins = 0;
    while (true) {
      asm volatile("" ::: "memory");  // (asked for again, it is read again)
      const floatx4 v = slot_load4<true>(slot, n, at);
      if (every_lane(top4(v, 0) != kEmpty) || give_up(spins)) return v;
    }
  }
};

constexpr int kTinyGroups = 32;  // workgroups per layer
constexpr int kTinyChunk = 8;    // steps whose reserve values pass through LDS together

// Time stamps of one workgroup's first wave, eight per step (the time-stamped instance only).
template <bool TRACE>
struct TinyTracer {
  long long* buf;  // [T][8]
  __device__ __forceinline__ void mark(int step, int slot) const {
    if (TRACE && buf && threadIdx.x == 0) {
      buf[(size_t)step * 8 + slot] = wall_clock64();
      if (slot == 0) buf[(size_t)step * 8 + 7] = clock64();
    }
  }
};

// Sums of N = 2, 4 or 8 per-lane partial values over the 64 lanes, the N sums computed together: in every stage half of
// the lanes hand their part of one value to the other half and take over the other value, so that after log2(N)
// stages each lane carries one value, and the remaining stages add up the lanes that carry the same one.  The sum of
// value r ends up in every lane whose bits 5, 4 (, 3) spell r from the low bit up: lane of_value(r).  All of it stays
// in the vector ALU: the halves of the wave and the rows of 16 lanes are exchanged with v_permlane32_swap /
// v_permlane16_swap (after the swap of x and y, x + y holds x's sum in one half and y's in the other), the rest are
// DPP moves within a row.
typedef unsigned uintx2 __attribute__((ext_vector_type(2)));
template <int CTRL>
__device__ __forceinline__ float dpp_move(float v) {
  return __uint_as_float((unsigned)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(v), CTRL, 0xf, 0xf, false));
}
__device__ __forceinline__ float merge32(float x, float y) {
  const uintx2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float merge16(float x, float y) {
  const uintx2 r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
template <int N>
__device__ __forceinline__ float reduce_lanes(const float (&a)[N], int lane) {
  static_assert(N == 2 || N == 4 || N == 8, "two, four or eight values");
  float b[N / 2];
#pragma unroll
  for (int m = 0; m < N / 2; ++m) b[m] = merge32(a[2 * m], a[2 * m + 1]);
  constexpr int NC = N > 2 ? N / 4 : 1;
  float c[NC];
#pragma unroll
  for (int m = 0; m < NC; ++m) c[m] = N > 2 ? merge16(b[2 * m], b[(2 * m + 1) % (N / 2)]) : merge16(b[0], b[0]);  // (N = 2: the two rows of a half)
  float d;
  if (N == 8) {
    const bool hi = lane & 8;
    d = (hi ? c[NC - 1] : c[0]) + dpp_move<0x128>(hi ? c[0] : c[NC - 1]);  // row_ror:8
  } else {
    d = c[0] + dpp_move<0x140>(c[0]);  // row_mirror: the other half of the row (used last: see below)
  }
  // within the remaining 8 (N = 8) or 16 (N = 2, 4) lanes: quads, then the other quad of the half row; for N < 8 the
  // mirror above has already folded the two half rows (every lane pairs with one of the other half)
  d += dpp_move<0xB1>(d);   // quad_perm [1,0,3,2]
  d += dpp_move<0x4E>(d);   // quad_perm [2,3,0,1]
  d += dpp_move<0x141>(d);  // row_half_mirror
  return d;
}
template <int N>
__device__ __forceinline__ constexpr int of_value(int r) {
  return ((r & 1) << 5) | (((r >> 1) & 1) << 4) | (N == 8 ? (((r >> 2) & 1) << 3) : 0);
}
__device__ __forceinline__ float lane_value(float v, int src_lane) {
  return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(v), src_lane));
}

// ------------------------------------------------------------------ forward
// Workgroup (l, q) of H / 64 waves and a serving one: wave w owns units u0 = 2 * (q * H / 64 + w), u0 + 1 of layer l (32
// workgroups per layer); rows r = 4*j + gate of the stacked matrices (j: which of the two units).  Exchange: hx [L][T+1][H],
// slot t+1 = h_t, slot 0 = h0 (or zeros), behind it the same values for the layer above [L][T][H], then the tables of
// all_on_one_xcd; everything but slot 0 the empty pattern before the launch.  Layer 0 takes its input product from the batched
// projection P0 [T][4H] (Section 2.3).
template <int HH, bool TRACE>
__global__ __launch_bounds__(HH + 64) void pers_fwd_tiny_kernel(const PersFwdArgs a) {
  constexpr int H = HH, G = 4 * H, NI = H / 64, NW = H / 64, NU = 2 * NW, NC = kTinyChunk;
  __shared__ __align__(16) float hs[2][H];            // [step parity]: h of the step before
  __shared__ __align__(16) float xs[2][H];            // [step parity]: input of the step after (or of the step)
  __shared__ __align__(16) float outs[2][NC][6][NU];  // [chunk parity][step][i, f, o, c', c, h][unit]
  __shared__ __align__(16) float pins[2][NC][4][NU];  // [chunk parity][step][gate][unit]: input product (layer 0)
  __shared__ int one_xcd;
  int l, q;
  if (!map_block_xcd(a.L, kTinyGroups, l, q)) return;
  const int T = a.T, lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int u0 = q * NU;  // first unit of the workgroup; a wave's are u0 + 2 * wave, + 1
  auto slot = [&](int st) { return a.hx + ((size_t)l * (T + 1) + st) * H; };
  float* const hand = a.hx + (size_t)a.L * (T + 1) * H;  // the same values for the layer above, which is on another XCD
  auto xslot = [&](int layer, int t) { return hand + ((size_t)layer * T + t) * H; };
  TinyWaiter w{{a.watchdog, a.spin_limit, false}};
  const TinyTracer<TRACE> tr{(int)blockIdx.x == a.trace_block ? a.trace : nullptr};
  float* const table = hand + (size_t)a.L * T * H + l * kTinyGroups;
  // Steps by which the input is ahead of the step that multiplies it: one, unless the layers' distances are most of a pass (L = 8,
  // T = 8, H = 256: 40 us with one, 35 with none).
  const int lead = T <= 2 * a.L ? 0 : 1;

  if (wave == NW) {  // ---- the wave that serves the others
    float* const res_l = a.res + (size_t)l * T * 6 * H;
    constexpr int NP = NC * 4 * NU / 64, NX = (H + 255) / 256;
    auto fetch_pins = [&](int t0, float (&v)[NP]) {
#pragma unroll
      for (int i = 0; i < NP; ++i) {
        const int e = 64 * i + lane, st = e / (4 * NU), g = e / NU % 4, u = e % NU;
        v[i] = t0 + st < T ? a.P0[(size_t)(t0 + st) * G + g * H + u0 + u] : 0.f;
      }
    };
    auto put_pins = [&](int t0, const float (&v)[NP]) {
#pragma unroll
      for (int i = 0; i < NP; ++i) (&pins[t0 / NC & 1][0][0][0])[64 * i + lane] = v[i];
    };
    auto write_out = [&](int t0) {  // the results of steps t0 .. t0 + NC - 1, as 16-byte pieces
      constexpr int Q = NU / 4;
      for (int i = lane; i < NC * 6 * Q; i += 64) {
        const int st = i / (6 * Q), k = i / Q % 6, u = 4 * (i % Q), t = t0 + st;
        if (t >= T) continue;
        const floatx4 v = *reinterpret_cast<const floatx4*>(&outs[t0 / NC & 1][st][k][u]);
        float* const base = k < 4 ? res_l + (size_t)t * G + k * H : res_l + (size_t)T * k * H + (size_t)t * H;  // c behind the gates, h behind c
        *reinterpret_cast<floatx4*>(base + u0 + u) = v;
        if (k == 5 && l == a.L - 1) *reinterpret_cast<floatx4*>(a.y + (size_t)t * H + u0 + u) = v;
        if (t == T - 1 && k == 5 && a.hT) *reinterpret_cast<floatx4*>(a.hT + (size_t)l * H + u0 + u) = v;
        if (t == T - 1 && k == 4 && a.cT) *reinterpret_cast<floatx4*>(a.cT + (size_t)l * H + u0 + u) = v;
      }
    };
    auto hand_over = [&](int t) {
      if (l < a.L - 1 && lane < NU) publish(xslot(l, t) + u0 + lane, outs[t / NC & 1][t % NC][5][lane], false);
    };
    uintx4 vx[NX];
    float vp[NP];
    auto request_x = [&](int t) {
#pragma unroll
      for (int i = 0; i < NX; ++i) vx[i] = remote_load4(xslot(l - 1, t), H, (256 * i + 4 * lane) % H);
    };
    auto here = [&]() {
      bool ok = true;
#pragma unroll
      for (int i = 0; i < NX; ++i)
#pragma unroll
        for (int c = 0; c < 4; ++c) ok = ok && vx[i][c] != kEmpty;
      return __all(ok);
    };
    auto take_x = [&](int t, float (&x)[H]) {
      int spins = 0;
      while (!here() && !w.give_up(spins)) request_x(t);
#pragma unroll
      for (int i = 0; i < NX; ++i) *reinterpret_cast<floatx4*>(&x[(256 * i + 4 * lane) % H]) = __builtin_bit_cast(floatx4, vx[i]);
    };
    leave_xcd(table, q, lane);
    if (l == 0) {
      fetch_pins(0, vp);
      put_pins(0, vp);
    } else {
      request_x(0);
      if (lead) {
        take_x(0, xs[1]);
        if (T > 1) request_x(1);
      }
    }
    const bool one = all_on_one_xcd(w, table, kTinyGroups, lane);
    if (lane == 0) one_xcd = one;
    __syncthreads();
    for (int t = 0; t < T; ++t) {
      if (l > 0 && t + lead < T) take_x(t + lead, xs[t & 1]);
      if (l == 0 && t % NC == 1) put_pins(t - 1 + NC, vp);
      __syncthreads();
      if (t > 0) hand_over(t - 1);
      if (t > 0 && t % NC == 0) write_out(t - NC);  // (complete since this barrier; its buffer is written again from step t + NC on)
      if (l == 0 && t % NC == 0) fetch_pins(t + NC, vp);
      if (l > 0 && t + lead + 1 < T) request_x(t + lead + 1);
    }
    __syncthreads();
    hand_over(T - 1);
    write_out((T - 1) / NC * NC);
    return;
  }

  // value m of a lane: word (64 * (m / VW) + lane) * VW + m % VW of the operand (read from LDS VW words at a time)
  constexpr int VW = NI < 4 ? NI : 4;
  typedef float vec __attribute__((ext_vector_type(VW)));
  // (H = 512: nine waves have no registers for both matrices; W lies in LDS, a lane's values VW at a time)
  constexpr bool wlds = H > 256;
  extern __shared__ __align__(16) float wx[];
  vec* const wl = reinterpret_cast<vec*>(wx) + (size_t)wave * 8 * (NI / VW) * 64;
  vec wW[8][wlds ? 1 : NI / VW], wR[8][NI / VW];
  {
    const float* Rl = a.R + (size_t)l * G * H;
    const float* Wl = a.W + (size_t)G * a.I + (size_t)(l > 0 ? l - 1 : 0) * G * H;
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      const size_t row = ((size_t)(r & 3) * H + u0 + 2 * wave + (r >> 2)) * H;
#pragma unroll
      for (int i = 0; i < NI / VW; ++i) {
        const int k = (64 * i + lane) * VW;
        wR[r][i] = *reinterpret_cast<const vec*>(Rl + row + k);
        const vec v = l > 0 ? *reinterpret_cast<const vec*>(Wl + row + k) : vec{};
        if constexpr (wlds) wl[(r * (NI / VW) + i) * 64 + lane] = v;
        else wW[r][i] = v;
      }
    }
  }
  // lanes 0 and 1 publish the two units (every lane runs the arithmetic)
  const int j = lane & 1, ul = 2 * wave + j, uj = u0 + ul, mine = 64 * wave + lane;
  float bias[4];
#pragma unroll
  for (int g = 0; g < 4; ++g) bias[g] = a.bias[(size_t)l * G + g * H + uj];
  float c_state = a.c0 ? a.c0[(size_t)l * H + uj] : 0.f;
  auto operand = [&](const float (&x)[H], vec (&v)[NI / VW]) {
#pragma unroll
    for (int i = 0; i < NI / VW; ++i) v[i] = *reinterpret_cast<const vec*>(&x[(64 * i + lane) * VW]);
  };
  auto dot = [&](const vec& x, const vec& y, float s) {
#pragma unroll
    for (int c = 0; c < VW; ++c) s = fmaf(x[c], y[c], s);
    return s;
  };
  // input half of a step, multiplied ahead of it, while the layer's own h is on its way
  float in[8];
  auto input_half = [&](const float (&x)[H]) {
    vec xi[NI / VW];
    operand(x, xi);
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      float s = 0.f;
#pragma unroll
      for (int i = 0; i < NI / VW; ++i) {
        if constexpr (wlds) s = dot(wl[(r * (NI / VW) + i) * 64 + lane], xi[i], s);
        else s = dot(wW[r][i], xi[i], s);
      }
      in[r] = s;
    }
  };
#pragma unroll
  for (int r = 0; r < 8; ++r) in[r] = 0.f;
  __syncthreads();
  const bool near = one_xcd && !a.full_fences;
  if (l > 0 && lead) input_half(xs[1]);
  for (int t = 0; t < T; ++t) {
    const int par = t & 1, ch = t / NC & 1, st = t % NC;
    tr.mark(t, 0);
    hs[par][mine] = w.poll1(slot(t) + mine);
    tr.mark(t, 1);
    // (one barrier per step: the buffer written two steps on is the one every wave has read before it arrived here)
    __syncthreads();
    tr.mark(t, 2);
    if (l > 0 && !lead) input_half(xs[par]);
    vec hr[NI / VW];
    float acc[8], pg[4];
    operand(hs[par], hr);
#pragma unroll
    for (int g = 0; g < 4; ++g) pg[g] = l == 0 ? pins[ch][st][g][ul] : 0.f;
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      float s = in[r];
#pragma unroll
      for (int i = 0; i < NI / VW; ++i) s = dot(wR[r][i], hr[i], s);
      acc[r] = s;
    }
    const float d = reduce_lanes<8>(acc, lane);
    float sg[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const float s0 = lane_value(d, of_value<8>(g)), s1 = lane_value(d, of_value<8>(4 + g));
      sg[g] = (j ? s1 : s0) + pg[g] + bias[g];
    }
    const float gi = sigmoidf_dev(sg[0]), gf = sigmoidf_dev(sg[1]), go = sigmoidf_dev(sg[2]), gc = tanhf_dev(sg[3]);
    const float cn = gf * c_state + gi * gc;
    const float hn = go * tanhf_dev(cn);
    c_state = cn;
    tr.mark(t, 3);
    if (lane < 2) publish(slot(t + 1) + uj, hn, near);
    if (lane < 12) {  // lane 2 k + j leaves value k of unit j
      const int k = lane >> 1;
      outs[ch][st][k][ul] = k < 3 ? (k == 0 ? gi : (k == 1 ? gf : go)) : (k == 3 ? gc : (k == 4 ? cn : hn));
    }
    if (l > 0 && lead && t + 1 < T) input_half(xs[par]);
  }
  __syncthreads();
}

// hx [L][T+1][H]: slot 0 <- h0 (zeros if null), the rest <- the empty pattern, as the hand-over slots and the tables behind
__global__ void tiny_prepare_fwd_kernel(float* __restrict__ hx, const float* __restrict__ h0, int L, int T, int H) {
  const long nh = (long)L * (T + 1) * H, n = nh + (long)L * T * H + L * kTinyGroups;
  for (long e = (long)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (long)gridDim.x * blockDim.x) {
    const int k = (int)(e % H), st = (int)((e / H) % (T + 1)), l = (int)(e / ((long)H * (T + 1)));
    float v = __uint_as_float(kEmpty);
    if (e < nh && st == 0) {  // (an initial state that carries the empty pattern would never be seen as written)
      v = h0 ? h0[(size_t)l * H + k] : 0.f;
      if (__float_as_uint(v) == kEmpty) v = __uint_as_float(0x7FC00000u);
    }
    hx[e] = v;
  }
}

__global__ void tiny_fill_empty_kernel(float* __restrict__ p, long n) {
  for (long e = (long)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (long)gridDim.x * blockDim.x)
    p[e] = __uint_as_float(kEmpty);
}

// ------------------------------------------------------------------ backward
// Wave w of workgroup (l, q): two units as forward, four output rows over K = 4H -- dh_{t-1} of the two units (columns of R_l)
// and the gradient dx_t for the same two units of the layer below (columns of W_l; layer 0: of the network input when
// I == H and it is wanted).  Exchange: dAx [L][T][H][4] gate gradients (the four gates of a unit side by side: one
// 16-byte store publishes them) and behind it the tables of all_on_one_xcd, dxbuf [L][T][H] hand-over gradients (slice l
// written by layer l >= 1, read by layer l-1), all of it the empty pattern before the launch.  The bias gradient of a unit is
// the sum over t of its gate gradients, which a lane of the serving wave carries along: no reduction, no atomic.
template <int HH, bool TRACE>
__global__ __launch_bounds__(HH + 64) void pers_bwd_tiny_kernel(const PersBwdArgs a) {
  constexpr int H = HH, G = 4 * H, NI = G / 64, NW = H / 64, NU = 2 * NW;
  __shared__ __align__(16) float ds[2][G];        // [step parity][word of the slot]
  __shared__ __align__(16) float raw[8][7][NU];   // [step % 8][i, f, o, c', c_t, c_{t-1}, dy][unit]
  __shared__ __align__(16) float ready[2][NU][8]; // [step parity][unit]: what the point-wise stage of the step needs
  __shared__ __align__(16) float das[2][4][NU];   // [step parity][gate][unit]: gate gradients
  __shared__ __align__(16) float dxs[2][NU];      // [step parity][unit]: gradient for the layer below
  __shared__ int one_xcd;
  int l, q;
  if (!map_block_xcd(a.L, kTinyGroups, l, q)) return;
  const int T = a.T, lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int u0 = q * NU;  // first unit of the workgroup; a wave's are u0 + 2 * wave, + 1
  const bool has_up = l < a.L - 1;
  auto dslot = [&](int t) { return a.dAx + ((size_t)l * T + t) * G; };
  auto xslot = [&](int layer, int t) { return a.dxbuf + ((size_t)layer * T + t) * H; };
  TinyWaiter w{{a.watchdog, a.spin_limit, false}};
  const TinyTracer<TRACE> tr{(int)blockIdx.x == a.trace_block ? a.trace : nullptr};
  float* const table = a.dAx + (size_t)a.L * T * G + l * kTinyGroups;

  if (wave == NW) {  // ---- the wave that serves the others
    const float* const res_l = a.res + (size_t)l * T * 6 * H;
    const float* const res_c = res_l + (size_t)T * 4 * H;
    float* const dA_l = a.dA + (size_t)l * T * G;
    constexpr int NF = (7 * NU + 63) / 64;
    float vr[NF], vd = 0.f;
    // word (k, unit) of raw, for step t >= 0 (fetch of a negative step reads step 0 for nobody): no branch, so that a count of
    // the requests behind it can be waited for
    const float* src[NF];
    const float* first[NF];  // the same word of step 0
    int stride[NF];
#pragma unroll
    for (int i = 0; i < NF; ++i) {
      const int e = min(64 * i + lane, 7 * NU - 1), k = e / NU, u = u0 + e % NU;
      stride[i] = k < 4 ? G : H;
      src[i] = k < 4 ? res_l + k * H + u : (k == 4 ? res_c + u : (k == 5 ? res_c + u - H : (has_up ? res_c + u : a.dy + u)));
      first[i] = k == 5 ? (a.c0 ? a.c0 + (size_t)l * H + u : res_c + u) : src[i];
    }
    auto fetch = [&](int t) {
#pragma unroll
      for (int i = 0; i < NF; ++i) vr[i] = *(t > 0 ? src[i] + (size_t)t * stride[i] : first[i]);
    };
    auto put = [&](int t) {
#pragma unroll
      for (int i = 0; i < NF; ++i)
        if (64 * i + lane < 7 * NU) (&raw[t & 7][0][0])[64 * i + lane] = vr[i];
    };
    leave_xcd(table, q, lane);
    const int un = lane % NU;  // the unit of the lane
    // The upstream gradient of a step is asked for a step before it is due (empty: not there yet) and polled for then.
    auto request = [&](int t) {
      if (has_up && t >= 0) vd = poll_load(xslot(l + 1, t) + u0 + un);
    };
    auto work_up = [&](int t) {
      const float (&r)[7][NU] = raw[t & 7];
      const float gi = r[0][un], gf = r[1][un], go = r[2][un], gg = r[3][un], ct = r[4][un];
      const float cp = t > 0 || a.c0 ? r[5][un] : 0.f;
      float dout = r[6][un];
      if (has_up) {
        int spins = 0;
        while (!__all(__float_as_uint(vd) != kEmpty) && !w.give_up(spins)) request(t);
        dout = vd;
      }
      const float tc = tanhf_dev(ct);
      // dc += dh * k_c; d = dc * k_i, dc * k_f, dh * k_o, dc * k_g; dc *= gf
      if (lane < NU) {
        float (&o)[8] = ready[t & 1][un];
        *reinterpret_cast<floatx4*>(&o[0]) = floatx4{go * (1.f - tc * tc), gg * gi * (1.f - gi), cp * gf * (1.f - gf), tc * go * (1.f - go)};
        *reinterpret_cast<floatx4*>(&o[4]) = floatx4{gi * (1.f - gg * gg), gf, dout, 0.f};
      }
    };
    float dbsum = 0.f;
    const int dg = lane / NU, du = lane % NU;  // gate and unit of the lane, lanes below 4 * NU
    for (int t = T - 1; t > T - 4; --t) {
      fetch(t);
      if (t >= 0) put(t);
    }
    request(T - 1);
    work_up(T - 1);
    const bool one = all_on_one_xcd(w, table, kTinyGroups, lane);
    if (lane == 0) one_xcd = one;
    request(T - 2);
    fetch(T - 4);
    __syncthreads();
    for (int t = T - 1; t >= 0; --t) {
      if (t > 0) work_up(t - 1);
      __syncthreads();
      if (t >= 3) put(t - 3);
      if (lane < 4 * NU) {
        const float v = das[t & 1][dg][du];
        dA_l[(size_t)t * G + dg * H + u0 + du] = v;
        dbsum += v;
      }
      if (t + 1 < T && lane < NU) {
        const float v = dxs[(t + 1) & 1][lane];
        if (l > 0) publish(xslot(l, t + 1) + u0 + lane, v, false);
        else if (a.dx0) a.dx0[(size_t)(t + 1) * a.I + u0 + lane] = v;
      }
      request(t - 2);  // (in front of the reserve's values, which come from further away: requests return in order)
      fetch(t - 4);
    }
    __syncthreads();
    if (lane < NU) {
      const float v = dxs[0][lane];
      if (l > 0) publish(xslot(l, 0) + u0 + lane, v, false);
      else if (a.dx0) a.dx0[u0 + lane] = v;
    }
    if (a.db && lane < 4 * NU) a.db[(size_t)l * G + dg * H + u0 + du] = dbsum;
    return;
  }

  // (H = 512: nine waves have no registers for both matrices; W lies in LDS, a lane's values four at a time)
  constexpr bool wlds = H > 256;
  extern __shared__ __align__(16) float wx[];
  float* const wl = wx + (size_t)wave * 2 * NI * 64;
  float wR[2][NI], wW[2][wlds ? 1 : NI];
  {
    const float* Rl = a.R + (size_t)l * G * H + u0 + 2 * wave;
    const float* Wl = (l > 0 ? a.W + (size_t)G * a.I + (size_t)(l - 1) * G * H : a.W) + u0 + 2 * wave;  // layer 0: [G][I], I == H
    const bool live = l > 0 || a.dx0;
    // value m of a lane: gate m % 4 of unit 64 * (m / 4) + lane (read from LDS four words at a time)
#pragma unroll
    for (int jj = 0; jj < 2; ++jj)
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const size_t k = ((size_t)(i & 3) * H + 64 * (i >> 2) + lane) * H;
        wR[jj][i] = Rl[k + jj];
        const float v = live ? Wl[k + jj] : 0.f;
        if constexpr (wlds) wl[((jj * (NI / 4) + i / 4) * 64 + lane) * 4 + i % 4] = v;
        else wW[jj][i] = v;
      }
  }
  const int j = lane & 1, ul = 2 * wave + j, uj = u0 + ul;
  const bool fin = lane < 2;
  const size_t se = (size_t)l * H + uj;
  float dc = a.dcT ? a.dcT[se] : 0.f;
  float dh_rec = a.dhT ? a.dhT[se] : 0.f;
  float da[NI];
  auto product = [&](auto from_w) {  // dh or (from_w) dx of the lane's unit
    float acc[2];
#pragma unroll
    for (int jj = 0; jj < 2; ++jj) {
      float s = 0.f;
#pragma unroll
      for (int i = 0; i < NI; i += 4) {
        floatx4 v;
        if constexpr (from_w() && wlds) v = *reinterpret_cast<const floatx4*>(&wl[((jj * (NI / 4) + i / 4) * 64 + lane) * 4]);
        else if constexpr (from_w()) v = floatx4{wW[jj][i], wW[jj][i + 1], wW[jj][i + 2], wW[jj][i + 3]};
        else v = floatx4{wR[jj][i], wR[jj][i + 1], wR[jj][i + 2], wR[jj][i + 3]};
#pragma unroll
        for (int c = 0; c < 4; ++c) s = fmaf(v[c], da[i + c], s);
      }
      acc[jj] = s;
    }
    const float r = reduce_lanes<2>(acc, lane);
    const float v0 = lane_value(r, of_value<2>(0)), v1 = lane_value(r, of_value<2>(1));
    return j ? v1 : v0;
  };
  __syncthreads();
  const bool near = one_xcd && !a.full_fences;
  for (int t = T - 1; t >= 0; --t) {
    const int par = t & 1, mine = 256 * wave + 4 * lane;
    tr.mark(t, 0);
    // ---- point-wise stage of step t
    const floatx4 ka = *reinterpret_cast<const floatx4*>(&ready[par][ul][0]), kb = *reinterpret_cast<const floatx4*>(&ready[par][ul][4]);
    const float dh = kb[2] + dh_rec;
    const float dcv = dc + dh * ka[0];
    const float d[4] = {dcv * ka[1], dcv * ka[2], dh * ka[3], dcv * kb[0]};
    dc = dcv * kb[1];
    if (fin) slot_store4(dslot(t), G, 4 * uj, floatx4{d[0], d[1], d[2], d[3]}, near);
    tr.mark(t, 1);
    if (lane < 8) das[par][lane >> 1][ul] = lane < 4 ? (lane < 2 ? d[0] : d[1]) : (lane < 6 ? d[2] : d[3]);
    // ---- dx of the step after, while the gate gradients are on their way
    if (t + 1 < T) {
      const float dx = product(std::true_type{});
      if (fin) dxs[(t + 1) & 1][ul] = dx;
    }
    tr.mark(t, 2);
    // ---- dh_{t-1}: needs dA_t of every unit of the layer (wave w polls words 256 w ... of the slot)
    const floatx4 share = w.poll4(dslot(t), G, mine);
    tr.mark(t, 3);
    *reinterpret_cast<floatx4*>(&ds[par][mine]) = share;
    __syncthreads();  // (one barrier per step is enough: see the forward kernel)
    tr.mark(t, 4);
#pragma unroll
    for (int i = 0; i < NI / 4; ++i) {
      const floatx4 qd = *reinterpret_cast<const floatx4*>(&ds[par][(64 * i + lane) * 4]);
#pragma unroll
      for (int c = 0; c < 4; ++c) da[i * 4 + c] = qd[c];
    }
    dh_rec = product(std::false_type{});
    tr.mark(t, 5);
  }
  const float dx = product(std::true_type{});
  if (fin) {
    dxs[0][ul] = dx;
    if (a.dh0) a.dh0[se] = dh_rec;
    if (a.dc0) a.dc0[se] = dc;
  }
  __syncthreads();
}

// W's rows of a workgroup, where they do not fit the registers: H / 32 units with four rows (forward) or columns each
size_t tiny_lds(int H) { return H > 256 ? (size_t)(H / 32) * 4 * H * sizeof(float) : 0; }

}  // namespace

hipError_t launch_fwd_tiny(int H, const PersFwdArgs& a, hipStream_t s) {
  const long n = (long)a.L * (2 * a.T + 1) * H + a.L * kTinyGroups;
  hipLaunchKernelGGL(tiny_prepare_fwd_kernel, dim3((unsigned)std::min<long>((n + 255) / 256, 1024)), dim3(256), 0, s, a.hx, a.h0, a.L,
                     a.T, H);
  const void* fn = H == 512 ? (const void*)pers_fwd_tiny_kernel<512, false>
                            : (H == 256 ? (const void*)pers_fwd_tiny_kernel<256, false> : (const void*)pers_fwd_tiny_kernel<128, false>);
  if (a.trace)
    fn = H == 512 ? (const void*)pers_fwd_tiny_kernel<512, true>
                  : (H == 256 ? (const void*)pers_fwd_tiny_kernel<256, true> : (const void*)pers_fwd_tiny_kernel<128, true>);
  void* params[] = {const_cast<PersFwdArgs*>(&a)};
  static bool ready[2];
  const size_t smem = tiny_lds(H);
  const hipError_t e = smem ? allow_dynamic_lds(fn, smem, ready[a.trace != nullptr]) : hipSuccess;
  if (e != hipSuccess) return e;
  return launch_resident(fn, xcd_grid(a.L, kTinyGroups), params, (unsigned)smem, s, H + 64);
}

hipError_t launch_bwd_tiny(int H, const PersBwdArgs& a, hipStream_t s) {
  const long n1 = (long)a.L * a.T * 4 * H + a.L * kTinyGroups, n2 = (long)a.L * a.T * H;
  hipLaunchKernelGGL(tiny_fill_empty_kernel, dim3((unsigned)std::min<long>((n1 + 255) / 256, 1024)), dim3(256), 0, s, a.dAx, n1);
  hipLaunchKernelGGL(tiny_fill_empty_kernel, dim3((unsigned)std::min<long>((n2 + 255) / 256, 1024)), dim3(256), 0, s, a.dxbuf, n2);
  const void* fn = H == 512 ? (const void*)pers_bwd_tiny_kernel<512, false>
                            : (H == 256 ? (const void*)pers_bwd_tiny_kernel<256, false> : (const void*)pers_bwd_tiny_kernel<128, false>);
  if (a.trace)
    fn = H == 512 ? (const void*)pers_bwd_tiny_kernel<512, true>
                  : (H == 256 ? (const void*)pers_bwd_tiny_kernel<256, true> : (const void*)pers_bwd_tiny_kernel<128, true>);
  void* params[] = {const_cast<PersBwdArgs*>(&a)};
  static bool ready[2];
  const size_t smem = tiny_lds(H);
  const hipError_t e = smem ? allow_dynamic_lds(fn, smem, ready[a.trace != nullptr]) : hipSuccess;
  if (e != hipSuccess) return e;
  return launch_resident(fn, xcd_grid(a.L, kTinyGroups), params, (unsigned)smem, s, H + 64);
}

}  // namespace lstm
