// The persistent forward recurrence with two alternating half-slices (persistent_pp.hip) on the bf16 matrix cores:
// pers_fwd_pp3_kernel.  Same tile, same chains, same counters; weights, states and inputs are cut into three bf16 parts
// (split3.h), so that the matrix instructions of a block take 3072 cycles at H = 512 instead of 8192.
//
// What bounds it.  A wave runs alone on its SIMD and pays for every instruction it issues: per block 96 matrix
// instructions (3072 cycles), 48 operand requests of 1 KB (about 1500; three parts of 2 bytes where fp32 had one of 4),
// 224 vector ALU and 25 LDS instructions (counted; about 1800) and 5 stores: 7000 cycles in all.  The exchange of a chain's h_t now has
// to fit under a block of that length, so everything about it is as early as it can be: the counter is looked at and the
// recurrent operand requested from group LAG on, one group behind the consumption of the ring slots that it goes to.
//
// Parts.  h_t is cut once, by the lane that finalises it, and travels as parts; x and the initial states are cut by the
// kernels that copy them into exchange layout; the weights when they are fetched.  The registers hold the weights of
// both operand halves (192), the ring of both chains' operands (192) and 16 sums.
//
// Exchange layout of one (layer, step, chain) slot, H x 32 x 3 bf16: part p of the 8 k = 8 k8 .. of batch row n is the
// 16-byte piece ((p * H/8 + k8) * 32 + n): what a lane (kk = lane / 32, n) feeds to a matrix instruction of 16 k, k8 = 2
// group + kk.  The 8 units of slice s are piece k8 = s of every row.
//
// Sign.  The bf16 instructions cut the low bits of their sums off downwards (gemm.hip); the waves of the first half of K
// hold their weights negated and their partial sums are subtracted, so that the bias cancels.
//
// Infinite and NaN sums raise a word; the host then has the fp32 kernel run the launch again, which reads that word and
// ends at once when it is zero (see launch_fwd_pp3's caller): a sum with an operand that has no parts comes out as in fp32.
#include "../../include/lstm.h"
#include "persistent_dev.h"
#include "split3.h"

namespace lstm {
namespace {

constexpr int pp_count(int lo, int hi, int upto) { return upto < lo ? 0 : ((upto < hi ? upto : hi) - lo + 1); }

// CELL as in pers_fwd_pp_kernel.
template <int HH, int LAG_, int GA_, int PF_, bool TRACE, int CELL = 0>
__global__ __launch_bounds__(256) void pers_fwd_pp3_kernel(const PersFwdArgs a) {
  constexpr int NGT = CELL == 0 ? 4 : (CELL == 1 ? 3 : 1);  // gate blocks of W, R, b
  constexpr int H = HH, G = NGT * H, NS = H / 8, NL = H / 16;  // G: rows of W, R, b
  constexpr int NK = H / 64;         // groups of 16 k per wave and operand half (K-quarter of H)
  constexpr int NG = 2 * NK;         // groups of a block: input half, then recurrent half
  constexpr int LAG = LAG_;          // group at which the recurrent operand's fetch begins (its counter is looked at there)
  constexpr int GA = GA_;            // group at which the other chain's previous publication is completed
  constexpr int PF = PF_;            // group at which the fetch of the other chain's next input begins
  // requests certainly issued between a publication and its completion: recurrent groups and input groups up to GA
  constexpr int NYOUNG = 3 * (pp_count(LAG, LAG + NK - 1, GA) + pp_count(PF, PF + NK - 1, GA));
  static_assert(NYOUNG >= 1 && NYOUNG < 60 && LAG >= 1 && LAG <= NK && PF + NK <= NG && GA < NG, "schedule");
  constexpr int FN = 8;
  constexpr int KS = 144, GS = 2 * KS;  // partial sums: floats from unit half to unit half, from gate to gate (no bank met twice)
  constexpr size_t SLOT = (size_t)H * 48;  // floats per slot
  __shared__ __attribute__((aligned(16))) float part[2][4][4 * GS];  // [buffer][wave][gate][kk][n][4]
  __shared__ __attribute__((aligned(16))) float stage[4][6 * 64];    // per wave: i, f, o, c', c, h of its 8 rows x 8 units

  int l, s;
  map_block(a.L, NS * a.nsl, l, s);
  const int sl = s / NS;
  s -= sl * NS;
  const int T = a.T, B = a.B;
  const int lane = threadIdx.x & 63;
  const int q = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int kk = lane >> 5, n = lane & 31;
  const int u0 = 8 * s;
  const size_t TB = (size_t)T * B;
  // The waves of a layer read a slot in orders rotated against each other (all of them would otherwise ask the same
  // L2 lines at the same time).  The rotation is a multiple of four groups where they divide into fours, so that the
  // address of a request is a scalar base plus the lane's fixed offset plus an immediate: scalar arithmetic costs a wave
  // that runs matrix instructions back to back nothing, every vector instruction costs its full issue time (one wave per
  // SIMD: nothing else to issue).
  constexpr int RU = NK % 4 == 0 ? 4 : 1, NR = NK / RU;
  const int rot = RU * ((((int)blockIdx.x >> 3) + q) % NR);

  if constexpr (TRACE) {  // (slot 5 of step 0: kernel entry under chain 1, weights in place under chain 0)
    if (a.trace && (int)blockIdx.x == a.trace_block && threadIdx.x == 0) a.trace[((size_t)T + 0) * 8 + 5] = wall_clock64();
  }
  // ---- weights -> registers.  A operand of group register i (k16 = (i + rot) % NK): row lane % 32 = 8*gate + unit,
  //      k = q*H/4 + 16*k16 + 8*kk + 0..7; negated in the first two waves
  bf16x8 wR[NK][3], wW[NK][3];
  {
    const float* Rl = a.R + (size_t)l * G * H;
    const float* Wl = l > 0 ? a.W + (size_t)G * a.I + (size_t)(l - 1) * G * H : a.W;  // layer 0: [G][I] with I <= H
    const int Il = l > 0 ? H : a.I;  // columns of Wl (x comes zero-padded to H columns)
    const int grp = n >> 3;
    const int gate = CELL >= 2 ? 0 : ((CELL == 1 && grp == 3) ? 2 : grp);  // matrix row block behind tile row group grp
    const bool useR = CELL == 0 || (CELL == 1 ? grp != 2 : grp == 0), useW = CELL == 0 || (CELL == 1 ? grp != 3 : grp == 0);
    const float* const rR = Rl + ((size_t)gate * H + u0 + (n & 7)) * H;
    const float* const rW = Wl + ((size_t)gate * H + u0 + (n & 7)) * Il;
    const float sgn = q < 2 ? -kUp : kUp;
#pragma unroll
    for (int i = 0; i < NK; ++i) {
      const int k = q * (H / 4) + 16 * wrap<NK>(i + rot) + 8 * kk;
      float vr[8], vw[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        vr[j] = useR ? sgn * rR[k + j] : 0.f;
        vw[j] = (useW && k + j < Il) ? sgn * rW[k + j] : 0.f;
      }
      split8(vr, wR[i]);
      split8(vw, wW[i]);
    }
  }

  // ---- the cell this lane finalises after the transposition (the same position in both chains): batch row
  //      8*q + lane/8 of the chain, unit lane%8
  const int nr = 8 * q + (lane >> 3);
  const int uu = lane & 7, unit = u0 + uu;
  int bb[2];
  bool valid[2];
  float c_state[2];
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    bb[c] = a.b0 + 64 * sl + 32 * c + nr;
    valid[c] = bb[c] < B;
    const float* const s0 = CELL == 0 ? a.c0 : (CELL == 1 ? a.h0 : nullptr);  // the carried state: c (LSTM), h (GRU)
    c_state[c] = (valid[c] && s0) ? s0[((size_t)l * B + bb[c]) * H + unit] : 0.f;
  }
  float bias[4];
#pragma unroll
  for (int g = 0; g < 4; ++g) bias[g] = g < NGT ? a.bias[(size_t)l * G + g * H + unit] : 0.f;

  float* const res_l = a.res + (size_t)l * TB * (CELL == 0 ? 6 : (CELL == 1 ? 5 : 1)) * H;
  float* const res_gates = CELL == 0 ? res_l : res_l + TB * H;  // LSTM, GRU
  float* const res_c = res_l + TB * 4 * H;  // LSTM only
  float* const res_h = CELL == 0 ? res_l + TB * 5 * H : res_l;
  float* const hx = a.hx + (size_t)sl * a.L * (T + 1) * 2 * SLOT;
  int* const flags = a.flags + (size_t)sl * a.L * (T + 1) * 2 * NL * kFlagStride;
  auto slot = [&](int layer, int st, int c) { return hx + (((size_t)layer * (T + 1) + st) * 2 + c) * SLOT; };
  auto flag = [&](int layer, int st, int c) { return flags + (((size_t)layer * (T + 1) + st) * 2 + c) * NL * kFlagStride; };
  const int arrive_line = ((4 * s + q) % NL) * kFlagStride;
  // the layer below is, for layer 0, the input sequence itself: x in exchange layout, all of it there before the launch
  const bool in_is_x = l == 0;
  const float* const in_base = in_is_x ? a.xin + (size_t)sl * (T + 1) * 2 * SLOT : slot(l - 1, 0, 0);
  auto in_slot = [&](int st, int c) { return in_base + ((size_t)st * 2 + c) * SLOT; };
  auto in_flag = [&](int st, int c) { return in_is_x ? flag(0, 0, c) : flag(l - 1, st, c); };  // x: never waited for

  PpWaiter<NL> w{a.watchdog, a.spin_limit, false};
  // time stamps of one workgroup's phases (diagnostic hook; a kernel instance of its own, so that the normal one carries
  // neither the branches nor the registers)
  const PpTracer trc{(TRACE && a.trace && (int)blockIdx.x == a.trace_block) ? a.trace : nullptr, T};
  struct {
    const PpTracer& t;
    __device__ __forceinline__ void mark(int c, int step, int slot) const {
      if constexpr (TRACE) t.mark(c, step, slot);
    }
  } tr{trc};
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");  // once: drop whatever earlier launches left in L1/L2

  int rv = rot / RU;
  // The lane offset as a 32-bit register that the optimiser meets anew in every block (fresh_lo): next to the scalar
  // base it then becomes the offset operand of the request instead of one 64-bit vector addition per request.
  unsigned lo = lane * 16;
  auto fresh_lo = [&]() {
    lo = lane * 16;
    asm volatile("" : "+v"(lo));
  };
  auto ldx = [&](const float* src, int i, int p) {  // src: the slot (wave-uniform); group i of this wave's K quarter, part p
    const char* const sb = reinterpret_cast<const char*>(src) + (size_t)p * H * 64 +
                           ((size_t)q * NK + RU * wrap<NR>(i / RU + rv)) * 1024;
    return __builtin_bit_cast(bf16x8, *reinterpret_cast<const uintx4*>(sb + lo + (i % RU) * 1024));
  };

  // Operands of a chain, three parts per group: at the start of the chain's block its ring holds the whole
  // input half (requested during the other chain's block); slot i is refilled with recurrent group i as soon as
  // input group i has been consumed, LAG groups behind.
  bf16x8 ring[2][NK][3];
  int seen_rec = 1 << 30;              // the next block's own-layer counter, read during the block before it

  // ---- completes the publication of chain c's step t: the store is acknowledged once at most NYOUNG younger
  //      requests are outstanding (none for the very last one); then the counter
  auto complete = [&](const int c, const int t, const bool last) {
    if (last) drain_vmem();
    else asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NYOUNG) : "memory");
    if (lane == 0) __hip_atomic_fetch_add(flag(l, t + 1, c) + arrive_line, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    tr.mark(c, t, 6);
  };

  // ---- one block: the matrix instructions of chain c's step t, then its reduction, gates and the store of h_t.
  //      Memory requests of a block, in order: the counter of the other chain's next input; recurrent groups from
  //      group LAG on; from group PF on the other chain's next input (its own if the layer below has published,
  //      else this chain's recurrent slot once more: valid memory, values unused, real fetch at the end of the
  //      block); the next block's own-layer counter; the store of h_t.  Nothing with a run-time count follows the
  //      store before the next block completes it.
  floatx16 acc;
  // ---- the first LAG groups of a block: operands long in registers, no memory request; issued together with the
  //      other chain's gates (see fused below)
  auto head = [&](const int c) {
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;
#pragma unroll
    for (int g = 0; g < LAG; ++g) acc = mfma_split3(wW[g], ring[c][g], acc);
  };
  auto block = [&](const int c, const int t) {
    tr.mark(c, t, 0);
    const int tn = c == 0 ? t + 1 : t + 2;  // input slot of the other chain's next block: its step t (c == 0) or t + 1
    const bool other_next = tn <= T;        // that block exists
    int seen_in = PpWaiter<NL>::peek(in_flag(other_next ? tn : T, 1 - c));
    const float* const rsrc = slot(l, t, c);
    fresh_lo();
    const float* nsrc = rsrc;
    bool fetched = false;
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int g = LAG; g < NG; ++g) {
      if (g == LAG) {  // h_{l,t-1} of this chain must be published (slot 0 was written before the launch)
        PpWaiter<NL>::land(seen_rec);
        w.wait(flag(l, t, c), 8, t > 0 ? seen_rec : 8);
        tr.mark(c, t, 2);
        fresh_lo();  // (after every branch: the offset has to be defined in the basic block of the requests)
      }
      if (g == PF) {
        PpWaiter<NL>::land(seen_in);
        fetched = other_next && !w.dead && (in_is_x || __all(seen_in >= 8));
        if (fetched) nsrc = in_slot(tn, 1 - c);
      }
      const bf16x8 cur[3] = {ring[c][g % NK][0], ring[c][g % NK][1], ring[c][g % NK][2]};
#pragma unroll
      for (int p = 0; p < 3; ++p) {
        if (g >= LAG && g < LAG + NK) ring[c][g - LAG][p] = ldx(rsrc, g - LAG, p);
        if (g >= PF && g < PF + NK) ring[1 - c][g - PF][p] = ldx(nsrc, g - PF, p);
      }
      acc = mfma_split3(g < NK ? wW[g % NK] : wR[g % NK], cur, acc);
      if (g == GA) {
        if (c == 1 || t > 0) complete(1 - c, c == 1 ? t : t - 1, false);  // the other chain's previous step
        fresh_lo();
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    tr.mark(c, t, 1);
    if (other_next && !fetched) {  // the layer below was late: wait for it now (before this chain's store)
      w.wait(in_flag(tn, 1 - c), 8, 0);
      const float* src = in_slot(tn, 1 - c);
#pragma unroll
      for (int i = 0; i < NK; ++i)
#pragma unroll
        for (int p = 0; p < 3; ++p) ring[1 - c][i][p] = ldx(src, i, p);
    }
    float* const mine = &part[(2 * t + c) & 1][q][0];
#pragma unroll
    for (int g = 0; g < 4; ++g)
      *reinterpret_cast<floatx4*>(mine + g * GS + kk * KS + n * 4) =
          floatx4{acc[4 * g], acc[4 * g + 1], acc[4 * g + 2], acc[4 * g + 3]};
    // the own-layer counter that the next block (the other chain's) waits for: read now, looked at LAG groups into it
    {
      const int st = c == 0 ? t : t + 1;  // that block is (1, t) or (0, t + 1): it needs h of step st - 1
      seen_rec = PpWaiter<NL>::peek(flag(l, (st > 0 && st < T) ? st : 1, 1 - c));
    }
    tr.mark(c, t, 3);
    __syncthreads();
    tr.mark(c, t, 4);
  };
  // ---- after the barrier, first part (straight-line code): K-split sums, gates, the store of h_t, the six values
  //      of the cell into the wave's corner of LDS
  float odd = 0.f;
  auto post_a = [&](const int c, const int t) {
    const float* const all = &part[(2 * t + c) & 1][0][0] + (uu >> 2) * KS + nr * 4 + (uu & 3);
    float sg[4];
#pragma unroll
    for (int g = 0; g < 4; ++g)
      sg[g] = (all[8 * GS + g * GS] + all[12 * GS + g * GS]) - (all[g * GS] + all[4 * GS + g * GS]);
    // (zero unless a sum is infinite or NaN; what it adds up to is looked at when the kernel ends)
    odd += ((sg[0] * 0.f + sg[1] * 0.f) + (sg[2] * 0.f + sg[3] * 0.f));
#pragma unroll
    for (int g = 0; g < 4; ++g) sg[g] = fmaf(sg[g], kDown, bias[g]);
    float gi, gf, go, gc, cn, hn;
    if (CELL == 0) {
      gi = sigmoidf_dev(sg[0]), gf = sigmoidf_dev(sg[1]), go = sigmoidf_dev(sg[2]), gc = tanhf_dev(sg[3]);
      cn = gf * c_state[c] + gi * gc;
      hn = go * tanhf_dev(cn);
      c_state[c] = cn;
    } else if (CELL >= 2) {
      gi = gf = go = gc = cn = 0.f;
      hn = CELL == 3 ? tanhf_dev(sg[0]) : fmaxf(sg[0], 0.f);
    } else {  // sg: r and z pre-activations, W_n x + b_n, R_n h; the four saved values: r, z, n, R_n h
      gi = sigmoidf_dev(sg[0]), gf = sigmoidf_dev(sg[1]);
      go = tanhf_dev(sg[2] + gi * sg[3]);
      gc = sg[3];
      hn = (1.f - gf) * go + gf * c_state[c];
      cn = 0.f;
      c_state[c] = hn;
    }
    // publish: the wave's 8 rows x 8 units are one 128-byte line of every part.  Neighbouring lanes hold neighbouring
    // units: both cut the pair, the even one stores the first part, the odd one the second, both the third.
    {
      const float v = valid[c] ? hn * kUp : 0.f;
      const float w2 = __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0xB1, 0xF, 0xF, true));
      const bool second = lane & 1;
      const Split2 s2 = split3(second ? w2 : v, second ? v : w2);
      unsigned* const o = reinterpret_cast<unsigned*>(slot(l, t + 1, c)) + ((size_t)s * 32 + nr) * 4 + (uu >> 1);
      __hip_atomic_store(o + (second ? (size_t)H * 16 : 0), second ? s2.m : s2.h, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(o + (size_t)H * 32, s2.l, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    // The reserve and the outputs (nobody reads them before the kernel ends) go out right behind it, as 16-byte
    // pieces: the wave's 8 rows x 8 units of each of the six arrays are transposed through a corner of LDS that only
    // this wave touches.  Stores to memory retire slowly and in order with the loads: anywhere later they would sit
    // in front of operands that the next block is about to need.
    {
      float* const st = &stage[q][0];
      const int so = lane;  // (row of the wave's eight, unit of the slice)
      st[so] = gi; st[64 + so] = gf; st[128 + so] = go; st[192 + so] = gc; st[256 + so] = cn; st[320 + so] = hn;
    }
  };
  // ---- second part: the reserve and the outputs as 16-byte pieces.  Every wave issues the same three stores in
  //      every step, whatever its rows and the call want written: a piece that is not wanted goes to a scratch line.
  //      With no branch around them the compiler knows how many requests are outstanding behind the counter that the
  //      next block looks at, and waits for that counter alone instead of for these stores to reach memory.
  auto post_b = [&](const int c, const int t) {
    const float* const st = &stage[q][0];
    const bool lastt = t == T - 1, top = l == a.L - 1;
    float* const scratch_line = a.dummy + 4 * (lane & 7);
    const int row = (lane >> 1) & 7, hf = lane & 1;
    const int br = a.b0 + 64 * sl + 32 * c + 8 * q + row;
    const bool in_batch = br < B;
    const size_t e = ((size_t)t * B + br) * H + u0 + 4 * hf;
    const size_t se = ((size_t)l * B + br) * H + u0 + 4 * hf;
    {  // gates: piece (array lane/16, row, half)
      const int arr = lane >> 4;
      const floatx4 v = *reinterpret_cast<const floatx4*>(st + arr * 64 + row * 8 + 4 * hf);
      float* const dst = (in_batch && a.keep && CELL <= 1) ? res_gates + ((size_t)t * B + br) * 4 * H + (size_t)arr * H + u0 + 4 * hf : scratch_line;
      *reinterpret_cast<floatx4*>(dst) = v;
    }
    {  // lanes 0-15: c, lanes 16-31: h (upper lanes repeat them into the scratch line)
      const int arr = 4 + ((lane >> 4) & 1);
      const floatx4 v = *reinterpret_cast<const floatx4*>(st + arr * 64 + row * 8 + 4 * hf);
      const bool mine = in_batch && lane < 32;
      float* const dst = (mine && a.keep && (CELL == 0 || arr == 5)) ? (arr == 4 ? res_c : res_h) + e : scratch_line;
      *reinterpret_cast<floatx4*>(dst) = v;
      float* const dsty = (mine && top && arr == 5) ? a.y + e : scratch_line;
      *reinterpret_cast<floatx4*>(dsty) = v;
      if (lastt && mine) {
        if (CELL == 0 && arr == 4 && a.cT) *reinterpret_cast<floatx4*>(a.cT + se) = v;
        if (arr == 5 && a.hT) *reinterpret_cast<floatx4*>(a.hT + se) = v;
      }
    }
  };
  // ---- a chain's gates and stores have no matrix instruction of their own chain to hide behind, but the other
  //      chain's next block has: its first LAG groups are issued in between (one matrix instruction, then a
  //      handful of the other instructions, and so on)
  auto fused = [&](const int cp, const int tp, const int cn) {
    post_a(cp, tp);
    head(cn);
#pragma unroll
    for (int i = 0; i < 6 * LAG; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // one matrix instruction
      __builtin_amdgcn_sched_group_barrier(0x7f7, FN, 0);  // up to FN of anything else
    }
    __builtin_amdgcn_sched_barrier(0);
    post_b(cp, tp);
  };

  tr.mark(0, 0, 5);
  // ---- chain 0's first input operand (chain 1's is requested by chain 0's first block)
  {
    if (!in_is_x) w.wait(in_flag(1, 0), 8, 0);
    const float* src = in_slot(1, 0);
#pragma unroll
    for (int i = 0; i < NK; ++i)
#pragma unroll
      for (int p = 0; p < 3; ++p) ring[0][i][p] = ldx(src, i, p);
  }
  // (the loop is rotated so that every look at a counter follows the stores before it in straight-line code)
  head(0);
  hide(rv);
  block(0, 0);
  for (int t = 0; t < T; ++t) {
    fused(0, t, 1);
    block(1, t);
    if (t + 1 < T) {
      hide(rv);
      fused(1, t, 0);
      block(0, t + 1);
    }
  }
  post_a(1, T - 1);
  post_b(1, T - 1);
  complete(1, T - 1, true);  // chain 0's last publication was completed inside chain 1's last block
  if (odd != 0.f) *a.redo = 1;  // (every writer writes the same)
}

// h0 [L][B][H] (zeros if null) -> exchange slot 0 of every (slice, layer, chain) in the layout above; rows past the
// batch hold zeros.  One piece of 8 k per thread.
__global__ void pack_state_pp3_kernel(const float* __restrict__ h0, float* __restrict__ hx, int L, int T, int B, int H, int b0,
                                      int nsl) {
  const long cnt = (long)nsl * L * 64 * (H / 8);
  for (long e = (long)blockIdx.x * blockDim.x + threadIdx.x; e < cnt; e += (long)gridDim.x * blockDim.x) {
    const int k8 = (int)(e % (H / 8)), lb = (int)((e / (H / 8)) % 64), l = (int)((e / ((long)(H / 8) * 64)) % L);
    const int sl = (int)(e / ((long)(H / 8) * 64 * L));
    const int c = lb >> 5, n = lb & 31;
    const int bb = b0 + 64 * sl + lb;
    float v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = (h0 && bb < B) ? kUp * h0[((size_t)l * B + bb) * H + 8 * k8 + j] : 0.f;
    bf16x8 p[3];
    split8(v, p);
    uintx4* const o = reinterpret_cast<uintx4*>(hx + ((((size_t)sl * L + l) * (T + 1)) * 2 + c) * H * 48) + (size_t)k8 * 32 + n;
#pragma unroll
    for (int q = 0; q < 3; ++q) o[(size_t)q * H * 4] = __builtin_bit_cast(uintx4, p[q]);
  }
}

// x [T][B][I] (I <= H) -> slots 1..T of xin [nsl][T+1][2] in the layout above, rows past the batch and columns
// past I zero (layer 0 then multiplies H columns like every other layer; its weights beyond column I are zero as well).
// Block (kb, t, sl) moves the 64 batch rows x 64 inputs [64*kb, 64*kb+64) of one step through LDS: whole rows in,
// 4 KB runs of each chain's slot and part out.
__global__ __launch_bounds__(256) void pack_x_pp3_kernel(const float* __restrict__ x, float* __restrict__ xin, int T, int B,
                                                         int I, int H, int b0, int nsl) {
  __shared__ float tile[64][65];
  const int kb = blockIdx.x, t = blockIdx.y, sl = blockIdx.z;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int e = threadIdx.x + 256 * i, lb = e >> 6, kc = e & 63;
    const int bb = b0 + 64 * sl + lb;
    tile[lb][kc] = (bb < B && 64 * kb + kc < I) ? x[((size_t)t * B + bb) * I + 64 * kb + kc] : 0.f;
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int o = threadIdx.x + 256 * i;  // piece (chain, k8 local, n): 2 x 8 x 32
    const int n = o & 31, k8 = (o >> 5) & 7, c = o >> 8;
    float v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = kUp * tile[32 * c + n][8 * k8 + j];
    bf16x8 p[3];
    split8(v, p);
    uintx4* const dst = reinterpret_cast<uintx4*>(xin + (((size_t)sl * (T + 1) + t + 1) * 2 + c) * H * 48) + (size_t)(8 * kb + k8) * 32 + n;
#pragma unroll
    for (int q = 0; q < 3; ++q) dst[(size_t)q * H * 4] = __builtin_bit_cast(uintx4, p[q]);
  }
}

template <int HH, int CELL>
hipError_t launch_pp3(int grid, const PersFwdArgs& a, hipStream_t s) {
  // Schedule (groups of the 16 / 8 of a block; forward pass, L = 4, T = 100).  H = 512, B = 64, LSTM: (LAG, GA, PF) = (2, 6, 8)
  // 0.72 ms, (2, 4, 8) 0.73, (2, 8, 8) 0.78, (2, 10, 8) 0.84; (2, 6, 4) 0.79, (2, 7, 6) 0.77; (3, 6, 8) 0.73, (4, 7, 8) 0.74.
  // H = 256, B = 128, tanh: (2, 2, 4) and (1, 2, 4) 0.45, (1, 1, 1) 0.47, (1, 3, 2) 0.54, (1, 4, 4) 0.67, (1, 6, 4) 1.02: the later the
  // completion of the other chain's publication, the more the layers above wait for it.
  constexpr int LAG = 2, GA = HH / 64 - 2, PF = HH / 64;
  const void* fn = a.trace ? (const void*)pers_fwd_pp3_kernel<HH, LAG, GA, PF, true, CELL>
                           : (const void*)pers_fwd_pp3_kernel<HH, LAG, GA, PF, false, CELL>;
  void* params[] = {const_cast<PersFwdArgs*>(&a)};
  return launch_resident(fn, grid, params, 0, s);
}

template <int CELL>
hipError_t launch_pp3_h(int H, int grid, const PersFwdArgs& a, hipStream_t s) {
  return with_on_chip_size(H, [&](auto h) {
    if constexpr (decltype(h)::value >= 256) return launch_pp3<decltype(h)::value, CELL>(grid, a, s);
    else return hipErrorInvalidValue;
  });
}

}  // namespace

hipError_t launch_fwd_pp3(int cell, int H, int grid, const PersFwdArgs& a, hipStream_t s) {  // cell 0: LSTM, 1: GRU, 2: ReLU, 3: tanh
  if (cell == 0) return launch_pp3_h<0>(H, grid, a, s);
  if (cell == 1) return launch_pp3_h<1>(H, grid, a, s);
  if (cell == 2) return launch_pp3_h<2>(H, grid, a, s);
  if (cell == 3) return launch_pp3_h<3>(H, grid, a, s);
  return hipErrorInvalidValue;
}

hipError_t launch_pack_state_pp3(const float* h0, float* hx, int L, int T, int B, int H, int b0, int nsl, hipStream_t s) {
  const long n = (long)nsl * L * 64 * (H / 8);
  hipLaunchKernelGGL(pack_state_pp3_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, h0, hx, L, T, B, H, b0, nsl);
  return hipGetLastError();
}

hipError_t launch_pack_x_pp3(const float* x, float* xin, int T, int B, int I, int H, int b0, int nsl, hipStream_t s) {
  hipLaunchKernelGGL(pack_x_pp3_kernel, dim3(H / 64, T, nsl), dim3(256), 0, s, x, xin, T, B, I, H, b0, nsl);
  return hipGetLastError();
}

}  // namespace lstm
