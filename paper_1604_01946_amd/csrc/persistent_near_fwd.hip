// Forward recurrence in slices of 16 batch rows whose workgroups exchange h through the L2 of one XCD: pers_fwd_near_kernel, all
// cells, multiples of 64 up to 512, 640, 768, 896 and 1024.  (Backward: persistent_near_bwd.hip.)
//
// What bounds a step here is not its products but the way from workgroup to workgroup.  The kernels with step counters pay per step
// a store, its acknowledgement, a barrier, an atomic, the poll of the counter, the fetch of the data and another barrier, about 3 us.
//   * The exchanged values are their own flags (near_dev.h): the operand loads of a step's recurrent products are its polls.
//   * A (layer, slice) group of up to 32 workgroups has an XCD to itself and stores no further than its L2; several small groups
//     share one.  Larger groups lie on all XCDs and write through to memory (PersFwdArgs::spread).
//   * Four waves split K and do nothing but poll, multiply, add up through LDS (one barrier per step) and apply the gates; four more
//     multiply the input half beside them; a ninth one brings the input product of layer 0, writes the reserve and y and hands h
//     over to the layer above, through LDS, a step behind: requests and acknowledgements return in order, so a poll behind a
//     store to memory would wait for it.
// Tile: v_mfma_f32_16x16x4_f32, MT tiles of 16 rows (unit-major, gate-minor, so that a lane's four sums are the four gates of one
// cell; single-gate cells: 16 units) x 16 batch rows.  GRU rows of a unit: r, z, W_n x, R_n h.
// A slot holds element (unit k, row n) at ((k/4)*16 + n)*4 + k%4: a lane fetches the operands of four matrix instructions at once.
#include "../../include/lstm.h"
#include "near_dev.h"

#include <algorithm>

namespace lstm {
namespace {

// FAR: groups lie on all XCDs.  IN: with the waves of the input half (layers above the launch's first).
template <int H, int CELL, int MT, bool FAR, bool IN>
__global__ __launch_bounds__(IN ? 576 : 320) void pers_fwd_near_kernel(const PersFwdArgs a) {
  constexpr int NG = CELL < 2 ? 4 : 1, NGP = CELL == 0 ? 4 : (CELL == 1 ? 3 : 1), U = 16 * MT / NG, M = H / U, GP = NGP * H;
  constexpr int NA = CELL == 0 ? 6 : (CELL == 1 ? 5 : 1), NL = H / 64, SLOT = 16 * H;
  __shared__ __align__(16) floatx4 part[2][IN ? 8 : 4][MT][64];  // [step parity][wave][tile][lane]: sums over a quarter of K (waves 4..7: input half)
  constexpr int UP = U + 4;                             // (rows of units in LDS: no bank conflicts)
  __shared__ __align__(16) float pins[2][NGP][16][UP];  // [step parity][gate][row][unit]: input product (layer 0)
  __shared__ __align__(16) float outs[2][NA][16][UP];   // [step parity][i, f, o, c', c, h (GRU r, z, n, R_n h, h)][row][unit]
  __shared__ int one_xcd;
  int g, m;
  if constexpr (FAR) map_block(a.L * a.nsl, M, g, m);
  else if (!map_block_xcd(a.L * a.nsl, M, g, m)) return;
  const int l = g / a.nsl, sl = g % a.nsl, T = a.T, B = a.B, u0 = m * U;
  const int b0 = a.b0 + 16 * sl, rows = min(16, B - b0);  // the slice's batch rows; a tile's columns past them are computed and not kept
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), q = lane >> 4, n = lane & 15;
  const size_t TB = (size_t)T * B, group = (size_t)(2 * T + 1) * SLOT;  // exchange of a group: h0, h_0 .. for itself, h_0 .. for the layer above
  float* const own = a.hx + g * group;
  float* const table = a.hx + (size_t)a.L * a.nsl * group + 64 * g;
  NearWaiter w{a.watchdog, a.spin_limit, false};

  if (wave == (IN ? 8 : 4)) {  // ---- the wave that serves the others
    if constexpr (!FAR) leave_xcd(table, m, lane);
    float* const hand = own + (size_t)(T + 1) * SLOT;
    constexpr int Q = U / 4, NP = NGP * 16 * Q, NPL = (NP + 63) / 64, NO = NA * 16 * Q, NH = 16 * Q;
    auto at_lds = [](int e) { return e / Q * UP + 4 * (e % Q); };  // 16-byte piece e of (array, row, four units) in LDS
    const float* pin_at[NPL];
    floatx4 vp[NPL];
#pragma unroll
    for (int i = 0; i < NPL; ++i) {
      const int e = min(64 * i + lane, NP - 1);
      pin_at[i] = a.P0 + (size_t)(b0 + min(e / Q % 16, rows - 1)) * GP + e / Q / 16 * H + u0 + 4 * (e % Q);
    }
    auto fetch_pins = [&](int t) {
#pragma unroll
      for (int i = 0; i < NPL; ++i) vp[i] = *reinterpret_cast<const floatx4*>(pin_at[i] + (size_t)min(t, T - 1) * B * GP);
    };
    auto put_pins = [&](int t) {
#pragma unroll
      for (int i = 0; i < NPL; ++i)
        if (64 * i + lane < NP) *reinterpret_cast<floatx4*>(&pins[t & 1][0][0][0] + at_lds(64 * i + lane)) = vp[i];
    };
    float* const res_l = a.res + (size_t)l * TB * (CELL == 0 ? 6 : (CELL == 1 ? 5 : 1)) * H;
    auto write_out = [&](int t) {
      const float* const o = &outs[t & 1][0][0][0];
      if (l < a.L - 1) {
#pragma unroll
        for (int i = 0; i < (NH + 63) / 64; ++i) {
          const int e = 64 * i + lane;
          if (e < NH) slot_store4(hand + (size_t)t * SLOT, SLOT, ((u0 / 4 + e / 16) * 16 + e % 16) * 4,
                                  *reinterpret_cast<const floatx4*>(o + ((NA - 1) * 16 + e % 16) * UP + 4 * (e / 16)), false);
        }
      }
#pragma unroll
      for (int i = 0; i < (NO + 63) / 64; ++i) {
        const int e = 64 * i + lane, k = e / NH, row = e / Q % 16, u = u0 + 4 * (e % Q);
        if (e >= NO || row >= rows) continue;
        const floatx4 v = *reinterpret_cast<const floatx4*>(o + at_lds(e));
        const size_t r = (size_t)t * B + b0 + row;
        if (a.keep) {
          float* p;
          if (CELL == 0) p = k < 4 ? res_l + r * 4 * H + k * H + u : res_l + TB * k * H + r * H + u;
          else if (CELL == 1) p = k < 4 ? res_l + TB * H + r * 4 * H + k * H + u : res_l + r * H + u;
          else p = res_l + r * H + u;
          *reinterpret_cast<floatx4*>(p) = v;
        }
        if (k == NA - 1 && l == a.L - 1) *reinterpret_cast<floatx4*>(a.y + r * H + u) = v;
      }
    };
    if (l == 0) {
      fetch_pins(0);
      put_pins(0);
      fetch_pins(1);
    }
    if constexpr (!FAR) {
      const bool one = all_on_one_xcd(w, table, M, lane);
      if (lane == 0) one_xcd = one;
    }
    __syncthreads();
    for (int t = 0; t < T; ++t) {
      __syncthreads();  // the waves' sums of step t, and their results of step t - 1
      if (l == 0) {
        put_pins(t + 1);
        fetch_pins(t + 2);
      }
      if (t > 0) write_out(t - 1);
    }
    __syncthreads();
    write_out(T - 1);
    return;
  }

  // ---- weights of waves 0..3 (recurrent half) and 4..7 (input half): lane (q, n) holds row n of tile mt at k = (wave % 4) * H/4 +
  // 16 j + 4 q + r
  const bool input = IN && wave >= 4;
  const int wk = wave & 3;
  floatx4 wt[MT][NL];
  {
    const float* mat = input ? a.W + (size_t)GP * a.I + (size_t)(l > 0 ? l - 1 : 0) * GP * H : a.R + (size_t)l * GP * H;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      const int unit = NG == 4 ? u0 + 4 * mt + (n >> 2) : u0 + 16 * mt + n, gate = NG == 4 ? n & 3 : 0;
      const size_t row = (size_t)((CELL == 1 && gate == 3 ? 2 : gate) * H + unit) * H + wk * (H / 4) + 4 * q;
      const bool has = input ? l > 0 && (CELL != 1 || gate != 3) : CELL != 1 || gate != 2;
#pragma unroll
      for (int j = 0; j < NL; ++j) wt[mt][j] = has ? *reinterpret_cast<const floatx4*>(mat + row + 16 * j) : floatx4{0.f, 0.f, 0.f, 0.f};
    }
  }
  const int kbase = (wk * (H / 16) + q) * 64 + 4 * n;  // float of the lane's first operand piece in a slot; 16 k on: 256 floats
  // Operands come in chunks of CH loads, up to DEEP chunks at a time.  On one XCD the first chunk is polled for alone; once it is there the
  // others are, and are asked for under its products.  FAR a word of each run of four units is polled for (a lane each), and then all are read
  // through the L2, once for the workgroups of an XCD; what was there too early is read again past it.
  constexpr int CH = NG == 1 && H > 768 ? 2 : (NL % 4 == 0 ? 4 : (NL % 5 == 0 ? 5 : (NL % 3 == 0 ? 3 : (NL % 7 == 0 ? 7 : NL)))), NCH = NL / CH, DMAX = IN ? 2 : 4, DEEP = NCH < DMAX ? NCH : DMAX;
  floatx4 op[DEEP * CH];
  auto ask = [&](auto past, const float* slot, int c) {
#pragma unroll
    for (int j = 0; j < CH; ++j) op[c % DEEP * CH + j] = slot_load4<decltype(past)::value>(slot, SLOT, kbase + 256 * (c * CH + j));
  };
  auto written = [&](int c) {
    unsigned m = 0;
#pragma unroll
    for (int j = 0; j < CH; ++j) m = top4(op[c % DEEP * CH + j], m);
    return every_lane(m != kEmpty);
  };
  const auto past = std::true_type{};
  const auto cached = std::false_type{};
  const int sample = (wk * (H / 16) + min(lane, H / 16 - 1)) * 64 + 63;
  // asked: the first DEEP chunks have been, through the caches
  auto multiply = [&](const float* slot, bool asked, floatx4 (&to)[MT][64]) {
    floatx4 acc[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[mt] = floatx4{0.f, 0.f, 0.f, 0.f};
    int spins = 0;
    if (!asked) {
      if constexpr (FAR) {
        while (!every_lane(__float_as_uint(poll_load(slot + sample)) != kEmpty) && !w.give_up(spins)) {
        }
#pragma unroll
        for (int c = 0; c < DEEP; ++c) ask(cached, slot, c);
      } else {
        do {
          asm volatile("" ::: "memory");
          ask(past, slot, 0);
        } while (!written(0) && !w.give_up(spins));
#pragma unroll
        for (int c = 1; c < DEEP; ++c) ask(past, slot, c);
      }
    }
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      while ((c > 0 || FAR || asked) && !written(c) && !w.give_up(spins)) {
        asm volatile("" ::: "memory");
        ask(past, slot, c);
      }
#pragma unroll
      for (int j = 0; j < CH; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int mt = 0; mt < MT; ++mt)
            acc[mt] = __builtin_amdgcn_mfma_f32_16x16x4f32(wt[mt][c * CH + j][r], op[c % DEEP * CH + j][r], acc[mt], 0, 0, 0);
      if (c + DEEP < NCH) {
        if (FAR || asked) ask(cached, slot, c + DEEP);
        else ask(past, slot, c + DEEP);
      }
    }
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) to[mt][lane] = acc[mt];
  };
  const Tracer tr{(int)blockIdx.x == a.trace_block ? a.trace : nullptr};

  if constexpr (IN)
   if (input) {  // ---- the input half of a step, beside the recurrent one
    const float* const below = a.hx + (g - a.nsl) * group + (size_t)(T + 1) * SLOT;  // (layer l > 0)
    auto request = [&](int t) {  // through the caches, which the group shares: usually there when it is looked at
#pragma unroll
      for (int c = 0; c < DEEP; ++c) ask(cached, below + (size_t)t * SLOT, c);
    };
    __syncthreads();
    if (l > 0) request(0);
    for (int t = 0; t < T; ++t) {
      if (l > 0) {
        // (matrix instructions hold up the vector instructions of the waves that apply the gates on the same SIMD: those first.
        // L = 2, T = 100, B = 16, H = 256: no pause 234 us, 384 cycles 218, 576 220, 768 227)
        __builtin_amdgcn_s_sleep(7);
        multiply(below + (size_t)t * SLOT, true, part[t & 1][wave]);
        if (t + 1 < T) request(t + 1);
      }
      __syncthreads();
    }
    __syncthreads();
    return;
  }

  // ---- wave mt < MT finalises tile mt: lane (q, n) has unit 4 mt + q (single gate: units 16 mt + 4 q ...) of row n
  const bool fin = wave < MT, valid = n < rows;
  const int ul = NG == 4 ? 4 * wave + q : 16 * wave + 4 * q;
  float bias[4] = {0.f, 0.f, 0.f, 0.f}, state = 0.f;  // state: c (LSTM), h (GRU)
  const size_t se = ((size_t)l * B + b0 + n) * H + u0 + ul;
  if (fin) {
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (NG == 1 || r < NGP) bias[r] = a.bias[(size_t)l * GP + (NG == 4 ? r * H + u0 + ul : u0 + ul + r)];
    const float* const s0 = CELL == 0 ? a.c0 : a.h0;
    if (NG == 4 && valid && s0) state = s0[se];
  }
  __syncthreads();
  const bool near = !FAR && one_xcd && !a.full_fences;
  __builtin_amdgcn_s_setprio(3);  // (a step waits for these waves: the input half fills their gaps)
  for (int t = 0; t < T; ++t) {
    const int par = t & 1;
    tr.mark(t, 0);
    multiply(own + (size_t)t * SLOT, false, part[par][wave]);
    tr.mark(t, 2);
    // (one barrier per step: `part` and `outs` of a parity are written again behind the next barrier but one)
    __syncthreads();
    tr.mark(t, 3);
    if (fin) {
      const auto& p = part[par];
      floatx4 s = (p[0][wave][lane] + p[1][wave][lane]) + (p[2][wave][lane] + p[3][wave][lane]);
      if constexpr (IN) {
        if (l > 0) s += (p[4][wave][lane] + p[5][wave][lane]) + (p[6][wave][lane] + p[7][wave][lane]);
      }
      float* const o = &outs[par][0][0][0];
      if constexpr (NG == 4) {
        float sg[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) sg[r] = s[r] + bias[r];
        if (l == 0) {
#pragma unroll
          for (int r = 0; r < NGP; ++r) sg[r] += pins[par][r][n][ul];
        }
        float h;
        if constexpr (CELL == 0) {
          const float gi = sigmoidf_dev(sg[0]), gf = sigmoidf_dev(sg[1]), go = sigmoidf_dev(sg[2]), gc = tanhf_dev(sg[3]);
          state = gf * state + gi * gc;
          h = go * tanhf_dev(state);
          slot_store1(own + (size_t)(t + 1) * SLOT, SLOT, ((u0 / 4 + wave) * 16 + n) * 4 + q, h, near);
          o[n * UP + ul] = gi;
          o[(16 + n) * UP + ul] = gf;
          o[(32 + n) * UP + ul] = go;
          o[(48 + n) * UP + ul] = gc;
          o[(64 + n) * UP + ul] = state;
          o[(80 + n) * UP + ul] = h;
          if (t == T - 1 && valid && a.cT) a.cT[se] = state;
        } else {
          const float r = sigmoidf_dev(sg[0]), z = sigmoidf_dev(sg[1]), nn = tanhf_dev(sg[2] + r * sg[3]);
          h = (1.f - z) * nn + z * state;
          state = h;
          slot_store1(own + (size_t)(t + 1) * SLOT, SLOT, ((u0 / 4 + wave) * 16 + n) * 4 + q, h, near);
          o[n * UP + ul] = r;
          o[(16 + n) * UP + ul] = z;
          o[(32 + n) * UP + ul] = nn;
          o[(48 + n) * UP + ul] = sg[3];
          o[(64 + n) * UP + ul] = h;
        }
        if (t == T - 1 && valid && a.hT) a.hT[se] = h;
      } else {
        floatx4 h;
        floatx4 pin = {0.f, 0.f, 0.f, 0.f};
        if (l == 0) pin = *reinterpret_cast<const floatx4*>(&pins[par][0][n][ul]);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float v = s[r] + pin[r] + bias[r];
          h[r] = CELL == 3 ? tanhf_dev(v) : fmaxf(v, 0.f);
        }
        slot_store4(own + (size_t)(t + 1) * SLOT, SLOT, ((u0 + ul) / 4 * 16 + n) * 4, h, near);
        *reinterpret_cast<floatx4*>(&o[n * UP + ul]) = h;
        if (t == T - 1 && valid && a.hT) *reinterpret_cast<floatx4*>(a.hT + se) = h;
      }
    }
    tr.mark(t, 4);
  }
  __syncthreads();
}

// Slot 0 of every group <- h0 (zeros without), the other slots and the tables <- the empty pattern.
__global__ __launch_bounds__(256) void near_prepare_fwd_kernel(floatx4* __restrict__ hx, const float* __restrict__ h0, int groups, int nsl, int T, int B, int H, int b0) {
  const int pieces = 4 * H;  // 16-byte pieces of a slot
  const long per = (long)(2 * T + 1) * pieces, n = groups * (per + 16);
  const float empty = __uint_as_float(kEmpty);
  for (long e = (long)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (long)gridDim.x * blockDim.x) {
    floatx4 v = {empty, empty, empty, empty};
    const long g = e / per, r = e - g * per;
    if (g < groups && r < pieces) {
      const int row = (int)r & 15, k = 4 * ((int)r >> 4), l = (int)g / nsl, b = b0 + 16 * ((int)g % nsl) + row;
      v = floatx4{0.f, 0.f, 0.f, 0.f};
      if (h0 && b < B) {  // (an initial state that carries the empty pattern would never be seen as written)
        v = *reinterpret_cast<const floatx4*>(h0 + ((size_t)l * B + b) * H + k);
#pragma unroll
        for (int c = 0; c < 4; ++c) v[c] = canonical(v[c]);
      }
    }
    hx[e] = v;
  }
}

template <int H, int CELL, int MT, bool FAR, bool IN>
hipError_t launch(const PersFwdArgs& a, hipStream_t s) {
  constexpr int M = H * (CELL < 2 ? 4 : 1) / (16 * MT);
  const int groups = a.L * a.nsl;
  const long n = groups * ((long)(2 * a.T + 1) * 4 * H + 16);
  hipLaunchKernelGGL(near_prepare_fwd_kernel, dim3((unsigned)std::min<long>((n + 255) / 256, 2048)), dim3(256), 0, s,
                     reinterpret_cast<floatx4*>(a.hx), a.h0, groups, a.nsl, a.T, a.B, H, a.b0);
  void* params[] = {const_cast<PersFwdArgs*>(&a)};
  return launch_resident((const void*)pers_fwd_near_kernel<H, CELL, MT, FAR, IN>, FAR ? groups * M : xcd_grid(groups, M), params, 0, s, IN ? 576 : 320);
}

// The instances that near_plan asks for.
template <int H, int CELL, int MT>
hipError_t launch_where(const PersFwdArgs& a, hipStream_t s) {
  constexpr int M = H * (CELL < 2 ? 4 : 1) / (16 * MT);
  if constexpr (H > 896 && CELL < 2) {
    return hipErrorInvalidValue;
  } else if constexpr (H > 512 && CELL < 2) {
    return a.L == 1 && a.spread ? launch<H, CELL, MT, true, false>(a, s) : hipErrorInvalidValue;
  } else {
    if (a.spread) return launch<H, CELL, MT, true, true>(a, s);
    if constexpr (M <= 32) return launch<H, CELL, MT, false, true>(a, s);
    return hipErrorInvalidValue;
  }
}

template <int H, int CELL>
hipError_t launch_units(int units, const PersFwdArgs& a, hipStream_t s) {
  constexpr int NG = CELL < 2 ? 4 : 1;
  if (units == 32 / NG) return launch_where<H, CELL, 2>(a, s);  // 8 units with four rows, 32 with one
  if constexpr (NG == 4 && H <= 320) {
    if (units == 16) return launch_where<H, CELL, 4>(a, s);
  }
  if constexpr (NG == 1) {
    if (units == 16) return launch_where<H, CELL, 1>(a, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_fwd_near(int cell, int H, int units, const PersFwdArgs& a, hipStream_t s) {
  return with_near_size(H, [&](auto h) {
    constexpr int HH = decltype(h)::value;
    switch (cell) {
      case 0: return launch_units<HH, 0>(units, a, s);
      case 1: return launch_units<HH, 1>(units, a, s);
      case 2: return launch_units<HH, 2>(units, a, s);
      case 3: return launch_units<HH, 3>(units, a, s);
    }
    return hipErrorInvalidValue;
  });
}

}  // namespace lstm
