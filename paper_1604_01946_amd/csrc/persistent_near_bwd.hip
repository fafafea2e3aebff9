// Backward recurrence in slices of 16 batch rows whose workgroups exchange gate gradients through the L2 of one XCD:
// pers_bwd_near_kernel, all cells, multiples of 64 up to 512, 640, 768, 896 and 1024.  The forward kernel (persistent_near_fwd.hip) names what bounds a step
// and what is done about it: values that are their own flags, a group of workgroups on an XCD of its own, a wave that
// serves the others, through LDS, with everything that comes from or goes to memory.
//
// A workgroup owns UB hidden units of one layer and slice; per step (descending t) it publishes the gate gradients of its
// units and multiplies everybody's, K = 4H (single-gate cells: H), split over waves 0..3:
//   UB = 8: one tile of 16 rows, 8 of dh_{t-1} (columns of R_l) and 8 of dx_t (the same columns of W_l), which cost nothing more;
//   UB = 16, 32: tiles of dh_{t-1} on waves 0..3, tiles of dx_t on waves 4..7 beside them, a step behind.
// dx_t goes to the layer below (layer 0: to the caller's dx where I == H) through the serving wave.
// v_mfma_f32_16x16x4_f32; K index of an LSTM or GRU unit's four gate gradients: 4 * unit + gate, so that a lane publishes a cell's
// gradients as one 16-byte piece and fetches the operands of four matrix instructions as one.  GRU: gradients with respect to the
// pre-activations of r and z, to W_n x + b_n and to R_n h.
#include "../../include/lstm.h"
#include "near_dev.h"

#include <algorithm>

namespace lstm {
namespace {

// Loads of a lane's weights per wave that stay in registers; the rest is in LDS (one tile, LSTM and GRU above H = 512).
constexpr int near_reg_loads(int H, int CELL) { return CELL < 2 ? (H > 512 ? 32 : H / 16) : H / 64; }

// FAR: groups lie on all XCDs.
template <int H, int CELL, int UB, bool FAR>
__global__ __launch_bounds__(UB == 8 ? 320 : 576) void pers_bwd_near_kernel(const PersBwdArgs a) {
  constexpr int NG = CELL < 2 ? 4 : 1, NGP = CELL == 0 ? 4 : (CELL == 1 ? 3 : 1), GP = NGP * H, G = 4 * H, M = H / UB;
  constexpr bool both = UB == 8;                  // dh and dx rows in one tile
  constexpr int NT = both ? 1 : UB / 16;          // tiles of a wave
  constexpr int SERVE = both ? 4 : 8;             // the serving wave
  constexpr int NL = NG * H / 64, SLOT = 16 * NG * H;
  constexpr int NR = CELL == 0 ? 6 : (CELL == 1 ? 5 : 1);  // arrays of the reserve that a step reads
  constexpr int CPL = both ? 1 : UB / 16;                  // cells of a lane (UB = 8: of waves 0 and 1)
  constexpr int Q = UB / 4;
  __shared__ __align__(16) floatx4 part[2][4][NT][64];               // [step parity][wave][tile][lane]: sums over a quarter of K
  __shared__ __align__(16) floatx4 xpart[both ? 1 : 2][both ? 1 : 4][both ? 1 : NT][64];  // the same of dx
  constexpr int UP = UB + 4;                               // (rows of units in LDS: no bank conflicts)
  __shared__ __align__(16) float raw[2][NR][16][UP];                 // [step parity][i, f, o, c', c_t, c_{t-1} (GRU r, z, n, R_n h, h_{t-1}; h_t)][row][unit]
  __shared__ __align__(16) float dout[2][16][UP];                    // [step parity]: upstream gradient
  __shared__ __align__(16) float das[2][NG][16][UP];                 // [step parity]: gate gradients
  __shared__ int one_xcd;
  int g, m;
  if constexpr (FAR) map_block(a.L * a.nsl, M, g, m);
  else if (!map_block_xcd(a.L * a.nsl, M, g, m)) return;
  const int l = g / a.nsl, sl = g % a.nsl, T = a.T, B = a.B, u0 = m * UB;
  const int b0 = a.b0 + 16 * sl, rows = min(16, B - b0);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), q = lane >> 4, n = lane & 15;
  const size_t TB = (size_t)T * B;
  const bool has_up = l < a.L - 1, dx_live = l > 0 || a.dx0;
  float* const own = a.dAx + (size_t)g * T * SLOT;
  float* const table = a.dAx + (size_t)a.L * a.nsl * T * SLOT + 64 * g;
  NearWaiter w{a.watchdog, a.spin_limit, false};

  if (wave == SERVE) {  // ---- the wave that serves the others
    if constexpr (!FAR) leave_xcd(table, m, lane);
    const float* const res_l = a.res + (size_t)l * TB * (CELL == 0 ? 6 : (CELL == 1 ? 5 : 1)) * H;
    constexpr int NF = NR * 16 * Q, NFL = (NF + 63) / 64, ND = 16 * Q, NDL = (ND + 63) / 64, NS = NG * 16 * Q, NSL = (NS + 63) / 64;
    auto at_lds = [](int e) { return e / Q * UP + 4 * (e % Q); };  // 16-byte piece e of (array, row, four units) in LDS
    // 16-byte piece 64 i + lane of a step's reserve values (array, row, four units); rows past the batch: zeros
    const float* src[NFL];
    const float* first[NFL];  // the same of step 0
    int stride[NFL];
    bool live[NFL], live0[NFL];
    floatx4 vr[NFL], vd[NDL];
#pragma unroll
    for (int i = 0; i < NFL; ++i) {
      const int e = min(64 * i + lane, NF - 1), k = e / ND, row = e / Q % 16, u = u0 + 4 * (e % Q);
      const size_t b = b0 + min(row, rows - 1);
      const bool gate = CELL < 2 && k < 4, before = CELL < 2 && k == NR - 1;  // one of the four gate arrays; the state of the step before
      const float* const state = CELL == 0 ? res_l + TB * 4 * H : res_l;      // c (LSTM) or h
      const float* const s0 = CELL == 0 ? a.c0 : a.h0;
      stride[i] = gate ? B * G : B * H;
      if (gate) src[i] = (CELL == 1 ? res_l + TB * H : res_l) + b * G + k * H + u;
      else src[i] = state + b * H + u;
      if (before) src[i] -= (size_t)B * H;
      first[i] = before ? (s0 ? s0 + ((size_t)l * B + b) * H + u : state + b * H + u) : src[i];
      live[i] = row < rows;
      live0[i] = live[i] && (!before || s0);
    }
    auto fetch = [&](int t) {  // (no branch, so that a count of the requests behind it can be waited for)
#pragma unroll
      for (int i = 0; i < NFL; ++i) vr[i] = *reinterpret_cast<const floatx4*>(t > 0 ? src[i] + (size_t)t * stride[i] : first[i]);
    };
    auto put = [&](int t) {
#pragma unroll
      for (int i = 0; i < NFL; ++i)
        if (64 * i + lane < NF) *reinterpret_cast<floatx4*>(&raw[t & 1][0][0][0] + at_lds(64 * i + lane)) = (t > 0 ? live[i] : live0[i]) ? vr[i] : floatx4{0.f, 0.f, 0.f, 0.f};
    };
    // upstream gradient of a step: dy, or what the layer above hands over, asked for a step before it is due and polled for then
    auto at_d = [&](int i) {  // (row, four units) -> float of a step of [B][H]; rows past the batch repeat the last one
      const int e = min(64 * i + lane, ND - 1);
      return (b0 + min(e / Q, rows - 1)) * H + u0 + 4 * (e % Q);
    };
    const size_t BH = (size_t)B * H;
    const float* const up = has_up ? a.dxbuf + (size_t)(l + 1) * TB * H : a.dy;
    auto request = [&](int t) {
#pragma unroll
      for (int i = 0; i < NDL; ++i) {
        const float* const p = up + (size_t)max(t, 0) * BH;
        vd[i] = has_up ? slot_load4<true>(p, B * H, at_d(i)) : *reinterpret_cast<const floatx4*>(p + at_d(i));
      }
    };
    auto take = [&](int t) {
      int spins = 0;
      while (has_up) {
        unsigned m = 0;
#pragma unroll
        for (int i = 0; i < NDL; ++i) m = top4(vd[i], m);
        if (every_lane(m != kEmpty) || w.give_up(spins)) break;
        asm volatile("" ::: "memory");
        request(t);
      }
#pragma unroll
      for (int i = 0; i < NDL; ++i) {
        const int e = 64 * i + lane;
        if (e < ND) *reinterpret_cast<floatx4*>(&dout[t & 1][0][0] + at_lds(e)) = e / Q < rows ? vd[i] : floatx4{0.f, 0.f, 0.f, 0.f};
      }
    };
    // dx of a step: lane (q, n) of a tile has four units of row n
    auto give_dx = [&](int t, int par) {
      if (!dx_live) return;
#pragma unroll
      for (int i = 0; i < (both ? 1 : NT); ++i) {
        floatx4 v;
        if constexpr (both) v = (part[par][0][0][lane] + part[par][1][0][lane]) + (part[par][2][0][lane] + part[par][3][0][lane]);
        else v = (xpart[par][0][i][lane] + xpart[par][1][i][lane]) + (xpart[par][2][i][lane] + xpart[par][3][i][lane]);
        const int u = u0 + (both ? 4 * (q - 2) : 16 * i + 4 * q);
        if ((both && q < 2) || n >= rows) continue;
        if (l > 0) slot_store4(a.dxbuf + (size_t)l * TB * H + (size_t)t * BH, B * H, (b0 + n) * H + u, v, false);
        else *reinterpret_cast<floatx4*>(a.dx0 + ((size_t)t * B + b0 + n) * a.I + u) = v;
      }
    };
    float* const dA_l = a.dA + (size_t)l * TB * G;
    floatx4 dbsum[NSL];
#pragma unroll
    for (int i = 0; i < NSL; ++i) dbsum[i] = floatx4{0.f, 0.f, 0.f, 0.f};

    fetch(T - 1);
    put(T - 1);
    fetch(T - 2);
    if (T > 1) put(T - 2);
    request(T - 1);
    take(T - 1);
    if constexpr (!FAR) {
      const bool one = all_on_one_xcd(w, table, M, lane);
      if (lane == 0) one_xcd = one;
    }
    request(T - 2);
    fetch(T - 3);
    __syncthreads();
    __syncthreads();  // (step T - 1 worked up: its reserve values may be overwritten)
    for (int t = T - 1; t >= 0; --t) {
      if (t > 0) take(t - 1);
      if (t > 1) put(t - 2);
      __syncthreads();  // sums and gate gradients of step t
#pragma unroll
      for (int i = 0; i < NSL; ++i) {
        const int e = 64 * i + lane, k = e / ND, row = e / Q % 16, u = u0 + 4 * (e % Q);
        if (e >= NS || row >= rows) continue;
        const floatx4 v = *reinterpret_cast<const floatx4*>(&das[t & 1][0][0][0] + at_lds(e));
        *reinterpret_cast<floatx4*>(dA_l + ((size_t)t * B + b0 + row) * G + k * H + u) = v;
        dbsum[i] += v;
      }
      if (both) give_dx(t, t & 1);
      else if (t + 1 < T) give_dx(t + 1, t & 1);
      request(t - 2);  // (in front of the reserve's values, which come from further away: requests return in order)
      fetch(t - 3);
    }
    __syncthreads();
    if (!both) give_dx(0, 1);
    // bias gradient of the slice: sums over its rows, in their order
    float* const sum = &das[0][0][0][0];  // (nobody reads it any more)
#pragma unroll
    for (int i = 0; i < NSL; ++i)
      if (64 * i + lane < NS) *reinterpret_cast<floatx4*>(sum + at_lds(64 * i + lane)) = dbsum[i];
    __builtin_amdgcn_wave_barrier();
    const int S = (B + 15) / 16;
    for (int e = lane; e < NGP * UB; e += 64) {
      float v = 0.f;
      for (int row = 0; row < rows; ++row) v += sum[(e / UB * 16 + row) * UP + e % UB];
      // (one slice: the caller's array)
      if (a.db) a.db[((size_t)l * S + b0 / 16) * GP + e / UB * H + u0 + e % UB] = v;
    }
    return;
  }

  // ---- weights: lane (q, n) holds row n of tile i (a column of R_l or W_l) at k = (wave % 4) * NG * H/4 + 16 j + 4 q + r
  // (beyond 32 j, above H = 512, they lie in LDS)
  const bool second = wave >= 4;  // waves of the dx tiles
  const int wk = wave & 3;
  constexpr int NLR = near_reg_loads(H, CELL);
  extern __shared__ __align__(16) floatx4 wlds[];
  floatx4* const wl = wlds + (size_t)wk * (NL - NLR) * 64 + lane;
  floatx4 wt[NT][NLR];
  {
    const float* const Rl = a.R + (size_t)l * GP * H;
    const float* const Wl = l > 0 ? a.W + (size_t)GP * a.I + (size_t)(l - 1) * GP * H : a.W;  // layer 0: [GP][I], I == H
    const bool from_w = both ? n >= 8 : second;
    const float* const mat = (from_w ? Wl : Rl) + u0 + (both ? n & 7 : n);
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
      for (int j = 0; j < NL; ++j) {
        floatx4 v;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int unit = NG == 4 ? wk * (H / 4) + 4 * j + q : wk * (H / 4) + 16 * j + 4 * q + r, gate = NG == 4 ? r : 0;
          const bool has = from_w ? dx_live && (CELL != 1 || gate != 3) : CELL != 1 || gate != 2;
          v[r] = has ? mat[(size_t)((CELL == 1 && gate == 3 ? 2 : gate) * H + unit) * H + 16 * i] : 0.f;
        }
        if (j < NLR) wt[i][j] = v;
        else wl[(j - NLR) * 64] = v;
      }
  }
  const int kbase = (wk * (NG * H / 16) + q) * 64 + 4 * n;  // float of the lane's first operand piece in a slot; 16 k on: 256 floats
  // Operands come in chunks of CH loads, up to DEEP chunks at a time.  On one XCD the first chunk is polled for alone (a round of all of them
  // moves 64 KB per CU at H = 256, LSTM: 0.45 us whether they are there or not); once it is there the others are, and are asked for under
  // its products.  FAR: as in the forward kernel.
  constexpr int CH = NL % 4 == 0 ? 4 : (NL % 5 == 0 ? 5 : (NL % 3 == 0 ? 3 : (NL % 7 == 0 ? 7 : NL))), NCH = NL / CH;
  constexpr int DMAX = CELL < 2 ? (H > 768 ? 2 : (H > 512 ? 3 : 4)) : (UB == 32 && H > 640 ? 2 : 4), DEEP = NCH < DMAX ? NCH : DMAX;  // (as many as there are registers for)
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
  const auto through = std::bool_constant<!FAR>{};  // past the caches, unless FAR
  const int sample = (wk * (H / 16) + min(lane, H / 16 - 1)) * 64 * NG + 64 * NG - 1;
  // asked: the first DEEP chunks have been
  auto multiply = [&](const float* slot, bool asked, floatx4 (&to)[NT][64]) {
    floatx4 acc[NT];
#pragma unroll
    for (int i = 0; i < NT; ++i) acc[i] = floatx4{0.f, 0.f, 0.f, 0.f};
    int spins = 0;
    if (!asked) {
      if constexpr (FAR) {
        while (!every_lane(__float_as_uint(poll_load(slot + sample)) != kEmpty) && !w.give_up(spins)) {
        }
        ask(through, slot, 0);
      } else {
        do {
          asm volatile("" ::: "memory");
          ask(past, slot, 0);
        } while (!written(0) && !w.give_up(spins));
      }
#pragma unroll
      for (int c = 1; c < DEEP; ++c) ask(through, slot, c);
    }
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      while ((c > 0 || FAR || asked) && !written(c) && !w.give_up(spins)) {
        asm volatile("" ::: "memory");
        ask(past, slot, c);
      }
#pragma unroll
      for (int j = 0; j < CH; ++j) {
        const int jj = c * CH + j;
        floatx4 v[NT];
#pragma unroll
        for (int i = 0; i < NT; ++i) v[i] = jj < NLR ? wt[i][jj < NLR ? jj : 0] : wl[(jj - NLR) * 64];
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int i = 0; i < NT; ++i) acc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[i][r], op[c % DEEP * CH + j][r], acc[i], 0, 0, 0);
      }
      if (c + DEEP < NCH) ask(through, slot, c + DEEP);
    }
#pragma unroll
    for (int i = 0; i < NT; ++i) to[i][lane] = acc[i];
  };
  if constexpr (!both) {
    if (second) {  // ---- dx_t, a step behind (its operands are complete once waves 0..3 have passed the step's barrier)
      __syncthreads();
      __syncthreads();
      for (int t = T - 1; t >= 0; --t) {
        if (dx_live && t + 1 < T) {
          const float* const slot = own + (size_t)(t + 1) * SLOT;
#pragma unroll
          for (int c = 0; c < DEEP; ++c) ask(through, slot, c);
          // (as in the forward kernel: the point-wise stage on the same SIMD first)
          __builtin_amdgcn_s_sleep(2);
          multiply(slot, true, xpart[t & 1][wk]);
        }
        __syncthreads();
      }
      if (dx_live) multiply(own, false, xpart[1][wk]);
      __syncthreads();
      return;
    }
  }

  // ---- cells of the point-wise stage: unit 4 wave + q + 16 i of row n
  const bool fin = !both || wave < 2, valid = n < rows;
  const int ul = 4 * wave + q;
  const size_t se = ((size_t)l * B + b0 + n) * H + u0 + ul;
  float dh[CPL], dc[CPL], k[CPL][6];  // dc: carried cell gradient (LSTM), the part of dh that passes by R (GRU)
#pragma unroll
  for (int i = 0; i < CPL; ++i) {
    dh[i] = fin && valid && a.dhT ? a.dhT[se + 16 * i] : 0.f;
    dc[i] = CELL == 0 && fin && valid && a.dcT ? a.dcT[se + 16 * i] : 0.f;
  }
  // what the point-wise stage of a step needs beside the incoming gradient
  auto work_up = [&](int t) {
#pragma unroll
    for (int i = 0; i < CPL; ++i) {
      const float* const r = &raw[t & 1][0][n][ul + 16 * i];
      constexpr int A = 16 * UP;
      if constexpr (CELL == 0) {
        const float gi = r[0], gf = r[A], go = r[2 * A], gg = r[3 * A], tc = tanhf_dev(r[4 * A]);
        k[i][0] = go * (1.f - tc * tc);
        k[i][1] = gg * gi * (1.f - gi);
        k[i][2] = r[5 * A] * gf * (1.f - gf);
        k[i][3] = tc * go * (1.f - go);
        k[i][4] = gi * (1.f - gg * gg);
        k[i][5] = gf;
      } else if constexpr (CELL == 1) {
        const float gr = r[0], z = r[A], nn = r[2 * A];
        k[i][0] = (1.f - z) * (1.f - nn * nn);
        k[i][1] = (r[4 * A] - nn) * z * (1.f - z);
        k[i][2] = r[3 * A] * gr * (1.f - gr);
        k[i][3] = gr;
        k[i][4] = z;
      } else {
        k[i][0] = CELL == 3 ? 1.f - r[0] * r[0] : r[0];
      }
    }
  };
  const Tracer tr{(int)blockIdx.x == a.trace_block ? a.trace : nullptr};
  __syncthreads();
  const bool near = !FAR && one_xcd && !a.full_fences;
  if (fin) work_up(T - 1);
  __syncthreads();
  for (int t = T - 1; t >= 0; --t) {
    const int par = t & 1;
    float* const slot = own + (size_t)t * SLOT;
    tr.mark(t, 0);
    if (fin) {
#pragma unroll
      for (int i = 0; i < CPL; ++i) {
        const float d = dh[i] + dout[par][n][ul + 16 * i];
        const int unit = u0 + ul + 16 * i;
        float* const o = &das[par][0][n][ul + 16 * i];
        constexpr int A = 16 * UP;
        if constexpr (NG == 4) {
          floatx4 v;
          if constexpr (CELL == 0) {
            const float dcv = dc[i] + d * k[i][0];
            v = floatx4{dcv * k[i][1], dcv * k[i][2], d * k[i][3], dcv * k[i][4]};
            dc[i] = dcv * k[i][5];
          } else {
            const float dn = d * k[i][0];
            v = floatx4{dn * k[i][2], d * k[i][1], dn, dn * k[i][3]};
            dc[i] = d * k[i][4];
          }
          slot_store4(slot, SLOT, (unit * 16 + n) * 4, v, near);
#pragma unroll
          for (int r = 0; r < 4; ++r) o[r * A] = v[r];
        } else {
          const float v = CELL == 3 ? d * k[i][0] : (k[i][0] > 0.f ? d : 0.f);
          slot_store1(slot, SLOT, ((unit / 4) * 16 + n) * 4 + unit % 4, v, near);
          o[0] = v;
        }
      }
      tr.mark(t, 1);
      if (t > 0) work_up(t - 1);
    }
    tr.mark(t, 2);
    multiply(slot, false, part[par][wave]);
    tr.mark(t, 4);
    // (one barrier per step: what a parity holds is written again behind the next barrier but one)
    __syncthreads();
    tr.mark(t, 5);
    if (fin) {
#pragma unroll
      for (int i = 0; i < CPL; ++i) {
        const float* const p = reinterpret_cast<const float*>(&part[par][0][i][wave * 16 + n]) + q;
        constexpr int W = NT * 64 * 4;
        dh[i] = (p[0] + p[W]) + (p[2 * W] + p[3 * W]);
        if (CELL == 1) dh[i] += dc[i];
      }
    }
  }
  if (fin && valid) {
#pragma unroll
    for (int i = 0; i < CPL; ++i) {
      if (a.dh0) a.dh0[se + 16 * i] = dh[i];
      if (CELL == 0 && a.dc0) a.dc0[se + 16 * i] = dc[i];
    }
  }
  __syncthreads();
}

// The empty pattern to n pieces at p, and to the first `own` of every `row` pieces at p2, n2 in all.
__global__ __launch_bounds__(256) void near_empty_kernel(floatx4* __restrict__ p, long n, floatx4* __restrict__ p2, long n2, int own, int row) {
  const float e = __uint_as_float(kEmpty);
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n + n2; i += (long)gridDim.x * blockDim.x) {
    const long j = i - n;
    (i < n ? p[i] : p2[own == row ? j : j / own * row + j % own]) = floatx4{e, e, e, e};
  }
}

// db[l][c] = sum over slices of part[l][slice][c], c < cols
__global__ __launch_bounds__(256) void near_bias_kernel(const float* __restrict__ part, float* __restrict__ db, int slices, int cols) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x, l = blockIdx.y;
  if (c >= cols) return;
  float v = 0.f;
  for (int s = 0; s < slices; ++s) v += part[((size_t)l * slices + s) * cols + c];
  db[(size_t)l * cols + c] = v;
}

template <int H, int CELL, int UB, bool FAR>
hipError_t launch(const PersBwdArgs& a, hipStream_t s) {
  const int groups = a.L * a.nsl, M = H / UB;
  // (of the hand-over array [L][T][B][H] the launch's rows; layer 0 hands nothing over)
  const int row4 = a.B * H / 4, own4 = std::min(16 * a.nsl, a.B - a.b0) * H / 4;
  const long n = (long)groups * (4L * (CELL < 2 ? 4 : 1) * H * a.T + 16), n2 = (long)(a.L - 1) * a.T * own4;
  hipLaunchKernelGGL(near_empty_kernel, dim3((unsigned)std::min<long>((n + n2 + 255) / 256, 2048)), dim3(256), 0, s,
                     reinterpret_cast<floatx4*>(a.dAx), n, reinterpret_cast<floatx4*>(a.dxbuf + ((size_t)a.T * a.B + a.b0) * H), n2, own4, row4);
  const void* const fn = (const void*)pers_bwd_near_kernel<H, CELL, UB, FAR>;
  constexpr size_t smem = (size_t)4 * ((CELL < 2 ? H / 16 : H / 64) - near_reg_loads(H, CELL)) * 1024;
  static bool ready;
  if (smem)
    if (const hipError_t e = allow_dynamic_lds(fn, smem, ready); e != hipSuccess) return e;
  void* params[] = {const_cast<PersBwdArgs*>(&a)};
  return launch_resident(fn, FAR ? groups * M : xcd_grid(groups, M), params, (unsigned)smem, s, UB == 8 ? 320 : 576);
}

// The instances that near_plan asks for.
template <int H, int CELL, int UB>
hipError_t launch_where(const PersBwdArgs& a, hipStream_t s) {
  if (a.spread) return launch<H, CELL, UB, true>(a, s);
  if constexpr (H / UB <= 32) return launch<H, CELL, UB, false>(a, s);
  return hipErrorInvalidValue;
}

template <int H, int CELL>
hipError_t launch_units(int units, const PersBwdArgs& a, hipStream_t s) {
  if constexpr (CELL < 2 && H <= 896) {
    if (units == 8) return launch_where<H, CELL, 8>(a, s);
  }
  if constexpr (CELL >= 2 || H <= 256) {
    if (units == 16) return launch_where<H, CELL, 16>(a, s);
  }
  if constexpr (CELL >= 2 && H <= 768) {
    if (units == 32) return launch_where<H, CELL, 32>(a, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace

// db (the caller's, [L][gates H]) from the slices' parts that launch_bwd_near left in a.db [L][slices][gates H]
hipError_t launch_near_bias(const float* part, float* db, int L, int slices, int H, int gates, hipStream_t s) {
  hipLaunchKernelGGL(near_bias_kernel, dim3((gates * H + 255) / 256, L), dim3(256), 0, s, part, db, slices, gates * H);
  return hipGetLastError();
}

hipError_t launch_bwd_near(int cell, int H, int units, const PersBwdArgs& a, hipStream_t s) {
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
