// Persistent recurrence: the whole T-step, L-layer recurrence in ONE
// launch, with the recurrent (and, for layers >= 1, the input) weights resident in registers.
//
// Section 4 of arXiv 1604.01946 names this as unexploited: the parameters are reused by every
// iteration and could live in a lower level of memory, at the price of a capacity limit and of
// assumptions outside the usual programming model (all blocks co-resident, blocks waiting on
// each other).  On gfx950 the register file of one CU is 512 KB, so a workgroup that owns 8
// hidden units keeps its [32 x 2H] slice of [W;R] (128 KB at H=512) in VGPRs as ready-made
// MFMA A operands for the whole sequence.  Co-residency comes from the grid never exceeding the
// number of CUs and from never having two such kernels in flight (see launch_resident); ordering comes from per-(layer, step) counters in device
// memory, released / acquired at agent scope, so that a layer only waits for the cells it
// really depends on -- cell (l, t) needs (l, t-1) and (l-1, t) -- and the layers run as the
// diagonal wavefront of Section 2.4 inside one grid.  Every wait is bounded: when the spin
// limit expires the waiter raises a host-visible word and stops waiting for the rest of the
// kernel, so the grid always drains.
//
// This file is the host side: device properties, the watchdog word, how persistent kernels are launched so that
// they are resident, which shapes run on which kernel family, groups of layers for stacks deeper than the chip
// holds, batch slices.  The kernels are in persistent_narrow / _wide / _pp / _large.hip (see persistent.h).
#include "../../include/lstm.h"
#include "persistent.h"
#include "knobs.h"

#include <algorithm>
#include <mutex>
#include <stdlib.h>

namespace lstm {

#define CK(expr, what)                                             \
  do {                                                             \
    if (record((expr), what) != hipSuccess) return LSTM_HIP_ERROR; \
  } while (0)

namespace {

// ------------------------------------------------------------------ host state
struct DeviceInfo {
  bool ok = false;
  int cus = 0;
  int coop = 0;
};
std::mutex g_mu;
DeviceInfo g_dev[64];
bool g_dev_init[64];
int* g_watch_host = nullptr;
int* g_watch_dev = nullptr;

bool device_info(DeviceInfo& out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) {
    (void)hipGetLastError();
    return false;
  }
  std::lock_guard<std::mutex> lk(g_mu);
  if (!g_dev_init[dev]) {
    DeviceInfo di;
    int v = 0;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess) di.cus = v;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeCooperativeLaunch, dev) == hipSuccess) di.coop = v;
    (void)hipGetLastError();
    di.ok = di.cus > 0;
    g_dev[dev] = di;
    g_dev_init[dev] = true;
  }
  out = g_dev[dev];
  return out.ok;
}

bool ensure_watchdog() {
  std::lock_guard<std::mutex> lk(g_mu);
  if (g_watch_host) return true;
  void* p = nullptr;
  if (hipHostMalloc(&p, 64, hipHostMallocMapped) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  g_watch_host = reinterpret_cast<int*>(p);
  *g_watch_host = 0;
  void* d = nullptr;
  if (hipHostGetDevicePointer(&d, p, 0) != hipSuccess) {
    (void)hipGetLastError();
    (void)hipHostFree(p);
    g_watch_host = nullptr;
    return false;
  }
  g_watch_dev = reinterpret_cast<int*>(d);
  return true;
}

int spin_limit() { return knobs().spin_limit; }

long long* g_trace_buf = nullptr;
size_t g_trace_bytes = 0;
int g_trace_block = 0;

int full_fences() { return knobs().full_fences ? 1 : 0; }

// All workgroups of a persistent kernel must be resident at once (they wait on each other).  The grid never exceeds
// the number of CUs and every workgroup fits a CU on its own, so an ordinary launch is resident as soon as the CUs it
// needs are free, and every other kernel on the device ends without waiting for anything.  What must not happen is
// two persistent kernels each holding part of the CUs and waiting for the rest: the persistent launches of this
// process are therefore chained, each waits (on the GPU, through an event) for the one before it, whatever their
// streams.  The event is the launch's own completion signal and has no fence for other devices or the host, who never look at it: recorded
// behind the launch, with that fence, it held up the kernel after it by 6 us (L = 2, T = 35, B = 20, H = 650 forward and backward 1206 -> 1182 us).  A cooperative launch gives the same guarantee device-wide, also
// against other processes, but measured 0.05-0.15 ms slower per launch on this stack and slows later multi-stream
// work of the process down: LSTM_COOP_LAUNCH=1 selects it.  LSTM_PLAIN_LAUNCH=1 launches without the chain (two
// persistent kernels may then share the CUs when both fit; diagnostics and tests).  A wait that never ends is, in
// every mode, turned into LSTM_INTERNAL by the watchdog.
std::mutex g_launch_mu;
hipEvent_t g_last_launch[16] = {};  // per device: completion of the most recent persistent launch
bool g_last_launch_recorded[16] = {};

// Side stream (default priority) and two events for work that overlaps a persistent launch which leaves CUs idle.
hipStream_t g_side_stream = nullptr;
hipEvent_t g_side_ev[2] = {};
std::mutex g_side_mu;  // held by the call that is using them
bool ensure_side_stream() {
  std::lock_guard<std::mutex> lk(g_launch_mu);
  if (g_side_stream) return true;
  if (hipStreamCreateWithFlags(&g_side_stream, hipStreamNonBlocking) != hipSuccess) {
    g_side_stream = nullptr;
    (void)hipGetLastError();
    return false;
  }
  for (hipEvent_t& ev : g_side_ev)
    if (hipEventCreateWithFlags(&ev, hipEventDisableTiming) != hipSuccess) {
      (void)hipGetLastError();
      return false;
    }
  return true;
}

}  // namespace

// Raises a kernel's dynamic LDS limit once per process (`done` is the caller's flag for that kernel); callers on
// several host threads are serialised.
hipError_t allow_dynamic_lds(const void* fn, size_t smem, bool& done) {
  std::lock_guard<std::mutex> lk(g_launch_mu);
  if (done) return hipSuccess;
  const hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
  if (e == hipSuccess) done = true;
  return e;
}

hipError_t launch_resident(const void* fn, int grid, void** params, unsigned smem, hipStream_t s, int threads) {
  if (knobs().coop_launch) return hipLaunchCooperativeKernel(fn, dim3(grid), dim3(threads), params, smem, s);
  int dev = 0;
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  if (knobs().plain_launch || hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 16 ||
      hipStreamIsCapturing(s, &cap) != hipSuccess || cap != hipStreamCaptureStatusNone) {
    (void)hipGetLastError();
    return hipLaunchKernel(fn, dim3(grid), dim3(threads), params, smem, s);  // (a stream under capture is ordered by its graph)
  }
  std::lock_guard<std::mutex> lk(g_launch_mu);
  hipError_t st = hipSuccess;
  if (!g_last_launch[dev]) {
    st = hipEventCreateWithFlags(&g_last_launch[dev], hipEventDisableTiming | hipEventDisableSystemFence);
    g_last_launch_recorded[dev] = false;
  } else if (g_last_launch_recorded[dev]) {
    st = hipStreamWaitEvent(s, g_last_launch[dev], 0);
  }
  if (st != hipSuccess) return st;
  st = hipExtLaunchKernel(fn, dim3(grid), dim3(threads), params, smem, s, nullptr, g_last_launch[dev], 0);
  if (st != hipSuccess) return st;
  g_last_launch_recorded[dev] = true;
  return hipSuccess;
}

namespace {

BatchPlan batch_plan(int B) {
  const bool two = knobs().two_chains;
  if (B <= 16) return {1, 1};
  if (B <= 32) return two ? BatchPlan{1, 2} : BatchPlan{2, 1};
  return two ? BatchPlan{2, 2} : BatchPlan{4, 1};
}



// The wide-batch forward kernel (32x32x2 MFMA, two batch tiles of 32).
// Height of the batch slices (16 or 32 rows) that run side by side on the narrow kernels, or 0 where the batch is
// taken whole (B <= 16, or no room) or by the wide kernels.  While all slices fit the chip in one launch the narrow
// kernels are the faster ones: a step's matrix work per workgroup shrinks with the slice and more CUs share it (one or
// two layers at H = 512, up to four at H = 256; L = 1, H = 512, B = 64, T = 100: forward recurrence 0.40 ms on four
// slices of 16 rows, 0.53 on two of 32, 0.74 on the wide kernel; backward 0.65 against 1.14).  `env` names the
// setting that pins the choice (LSTM_FWD_NARROW / LSTM_BWD_NARROW): 1 = one slice on the narrow kernel (B <= 64), 0 = never slices.
// What near_plan takes does not come here: slices of 32 rows forward at H = 384 to 512 are left, and all of it with LSTM_NEAR=0.
// Backward, from H = 256 on, slices of 32 rows lose to the kernel with two alternating chains per slice of 64 rows
// (whole iterations, T = 100: L = 2, H = 512, B = 64 2.46 -> 2.28 ms; L = 4, H = 256, B = 64 1.46 -> 1.37; L = 2, H = 256,
// B = 128 1.55 -> 1.44), while slices of 16 rows stay ahead of it (L = 1, H = 512, B = 64 1.40 against 2.02 ms).
int narrow_slice_rows(const Dims& d, int cell, int pinned, bool backward) {
  if (cell != 0) return 0;  // the narrow kernels are LSTM kernels
  if (pinned >= 0 || knobs().two_chains) return 0;
  DeviceInfo di;
  if (!device_info(di)) return 0;
  for (int rows = 16; rows <= 32; rows *= 2) {
    if (backward && rows == 32 && d.H >= 256) break;
    const int n = (d.B + rows - 1) / rows;
    if (d.B > rows && (long)d.L * (d.H / 8) * n <= di.cus && n <= 16 / d.L) return rows;  // 16 (slice, layer) counter blocks
  }
  return 0;
}

bool fwd_wide(const Dims& d) {
  if (d.B > 64) return true;  // batches above 64 run as slices of 64 rows, one launch each
  if (knobs().fwd_narrow == 1) return false;
  return d.B > 32;
}


// A single sequence: the kernels of persistent_tiny.hip (one wave per two hidden units, 32 workgroups per layer, all
// of them resident).
bool tiny_path(const Dims& d, int cell) {
  if (cell != 0 || d.B != 1 || !knobs().tiny) return false;
  if (!(d.H == 128 || d.H == 256 || d.H == 512)) return false;
  DeviceInfo di;
  return device_info(di) && di.cus >= 256 && d.L <= 8;  // 32 workgroups per layer, on the 32 CUs of an XCD each
}

// Kernels of slices of 16 rows that exchange through an XCD's L2 (persistent_near_fwd.hip, persistent_near_bwd.hip): hidden units
// per workgroup (0: not these kernels), slices side by side in a launch, whether a (layer, slice) group of workgroups lies on
// all XCDs.
//   Few units per workgroup before many, since a step's products are what a workgroup spends most of it on, and a group on one
//   XCD before one on all (L = 1, T = 100, B = 16, H = 256 LSTM forward / backward: 8 units 175 / 304 us on one, 230 / 332 on all;
//   16 units 210 / 358 on one.  L = 3, T = 40, B = 17, H = 320 forward: 8 units on all 146 us, 16 on one 169).
//   LSTM and GRU: where all slices run in one launch.  Against the kernels that come after this rule, 63 random shapes of that kind of
//   all cells, 2 to 100 steps: forward 1.66, backward 1.55 times faster on average, none slower by more than 2 %.  In several
//   launches the kernels with slices of 64 rows are ahead (GRU, L = 4, T = 50, B = 128, H = 256 305 / 530 us against 373 / 598).
//   Single gate: at any number of rows, those kernels multiply three empty gates (tanh, L = 4, T = 100, B = 256, H = 256: 922 / 1596 us
//   there, 504 / 894 here in two launches; L = 2, T = 5, B = 512, H = 512 334 / 416 and 154 / 216).
struct NearPlan {
  int units = 0, slices = 0, side = 0;
  bool spread = false;
};
NearPlan near_plan(const Dims& d, int cell, bool backward) {
  NearPlan p;
  DeviceInfo di;
  if (!knobs().near || !device_info(di) || di.cus < 256) return p;  // (eight XCDs of 32 CUs)
  if ((backward ? knobs().bwd_narrow : knobs().fwd_narrow) >= 0 || knobs().two_chains || knobs().pingpong >= 0 || !knobs().rnn_pp || knobs().split3 >= 0) return p;  // another kernel is asked for
  if (cell == 0 && d.B == 1 && !knobs().tiny) return p;  // (single sequences on the kernels with step counters)
  const bool single = cell >= 2;
  p.slices = (d.B + 15) / 16;
  // (the slices' bias gradients, [L][slices][gates H], lie in the workspace's area of [L][64][4H])
  if (backward && p.slices * (single ? 1 : 4) > 64 * 4) return NearPlan{};
  for (int side = p.slices; side > 0 && (side == p.slices || single); --side)
    for (int units = single ? 16 : 8; units <= (single ? 32 : 16); units *= 2)
      for (int spread = 0; spread < 2; ++spread) {
        const long groups = (long)d.L * side, members = d.H / units;
        // (no registers for more units' weights above these sizes; beyond 512 LSTM and GRU have instances of single layers on all XCDs)
        if (single ? backward && units == 32 && d.H > 768 : units == 16 && d.H > (backward ? 256 : 320)) continue;
        if (!single && d.H > 512 && (d.L > 1 || !spread)) continue;
        if (spread ? groups * members > 256 : (groups + 7) / 8 * members > 32) continue;
        p.units = units;
        p.side = side;
        p.spread = spread;
        return p;
      }
  return p;
}

// Layers per launch of those kernels at the sizes that have one-layer kernels as well, 0 where they don't take a shape or are slower: LSTM
// and GRU, whose products there run in three bf16 parts and here in fp32, from one step on or only up to some steps.  One-layer
// kernels / these, us (L, T, B):
//   LSTM forward   H = 640 163 / 156 (1, 35, 16); 768 174 / 170, 418 / 433 (2, 35, 20); 896 531 / 578 (1, 100, 30), 96 / 91 (1, 12, 30); 1024
//                  565 / 603 (1, 100, 30)
//   GRU forward    640 347 / 311 (2, 35, 32); 768 375 / 347; 896 408 / 391, 490 / 500 (1, 100, 30); 1024 544 / 594
//   LSTM backward  640 296 / 210 (1, 35, 16); 768 327 / 270, 839 / 598 (2, 35, 32); 896 905 / 699; 1024 86 / 102 (1, 4, 8), 813 / 951
//   GRU backward   640 780 / 460 (2, 35, 32); 768 794 / 563; 896 75 / 77 (1, 4, 8), 865 / 670; 1024 80 / 102, 802 / 932
//   single gate    tanh, H = 1024 941 / 266 and 1798 / 301 (4, 52, 1); 640 269 / 107 and 371 / 190 (1, 30, 100); 896 346 / 145 and 647 / 275 (3, 20, 20)
//   Steps from which the backward recurrence of LSTM and GRU gains (whole calls): one layer, 640 with 20 rows 0.90 (LSTM) and 0.94 (GRU) at one step,
//   0.97 and 1.10 at two, 1.09 at three; 768 with 5 rows 0.93 at one, 1.02 at three (756 padded to it 0.95 at four), with 20 rows 0.75 at one, 0.97 at three, 1.03 at
//   eight; 896 0.92 to 1.07 at eight, 1.0 to 1.1 at 16.  Several layers, each a launch: 768 with 20 rows 0.91 at one and 1.13 at three.
//   Single gate, short passes of several layers: a launch of many layers has to fill and drain them, and slices that don't fit side by side are
//   launches of their own, each with all weights to fetch (tanh, T = 2, backward: L = 4, B = 177, H = 896 515 us on one-layer kernels, 692 here; L = 2, B = 65, H = 1024 159 and 137;
//   forward L = 8, B = 192, H = 1024 863 and 1139, B = 20 ten steps 664 and 391).  Microseconds of the one-layer kernels' launches and of these, with 5 to
//   15 % against the latter, another tenth above four layers, fitted to 1600 recurrences of up to 8 layers, 40 steps and 192 rows: of those that it takes
//   none was slower by more than 3 %, and it leaves one in 30 that would have gained more than 5 %.
bool single_gate_gains(const Dims& d, int per, bool backward) {
  struct Model { double there, there_step, here, here_step, here_layer; };  // of a launch, of a step in it, of a layer behind the first in it
  constexpr Model fwd[4] = {{17.7, 3.8, 0.0, 4.4, 4.7}, {22.0, 4.0, 6.2, 4.4, 6.5}, {22.7, 4.4, 3.9, 5.2, 5.6}, {19.9, 5.2, 5.5, 6.5, 8.6}};
  constexpr Model bwd[4] = {{28.8, 8.1, 13.5, 5.9, 8.7}, {26.2, 8.5, 1.9, 7.8, 10.4}, {28.6, 7.9, 14.0, 3.7, 6.1}, {19.3, 2.9, 11.6, 0.52, 4.8}};
  constexpr int fwd_side[4] = {3, 2, 2, 2}, bwd_side[4] = {4, 3, 2, 4};  // slices of 32 rows in a launch of theirs
  if (d.L == 1 || d.T > 24) return true;
  const int i = (d.H - 640) / 128, side = (backward ? bwd_side : fwd_side)[i];
  const Model& m = (backward ? bwd : fwd)[i];
  const double there = d.L * (((d.B + 31) / 32 + side - 1) / side) * (m.there + d.T * m.there_step);
  double here = 0.0;
  for (int l = 0; l < d.L; l += per) {
    const Dims g{std::min(per, d.L - l), d.T, d.B, d.I, d.H};
    const NearPlan p = near_plan(g, 2, backward);
    here += (p.slices + p.side - 1) / p.side * (m.here + d.T * m.here_step + (g.L - 1) * m.here_layer);
  }
  return here * (d.L > 4 ? 1.1 : 1.0) < there;
}
int near_large_layers(const Dims& d, int cell, bool backward) {
  if (d.H <= 512 || d.H > 1024) return 0;
  if (d.H == 1024 && cell < 2) return 0;
  if (knobs().near < 2) {
    if (d.H == 1024 && d.L == 1 && d.B > 32) return 0;  // (of one layer of more rows only the single gate's products would gain)
    constexpr int least[3][2][2] = {{{1, 3}, {1, 1}}, {{6, 8}, {1, 3}}, {{16, 16}, {8, 8}}};  // [640, 768, 896][several layers][above 16 rows]
    if (backward && cell < 2 && d.T < least[(d.H - 640) / 128][d.L > 1][d.B > 16]) return 0;
    if (!backward && (cell == 0 ? d.H > 640 && d.T > 16 : cell == 1 && d.H > 768 && d.T > 64)) return 0;
  }
  int per = d.L;
  while (per > 0 && !near_plan(Dims{per, d.T, d.B, d.I, d.H}, cell, backward).units) --per;
  if (per > 0 && cell >= 2 && knobs().near < 2 && !single_gate_gains(d, per, backward)) return 0;
  return per;
}

// The wide-batch backward kernel: two batch halves, 16 hidden units per workgroup.
bool bwd_wide(const Dims& d) {
  if (d.B > 64) return true;
  if (knobs().bwd_narrow == 1) return false;
  return d.B > 32;
}


}  // namespace

int device_cu_count() {
  DeviceInfo di;
  return device_info(di) ? di.cus : 0;
}

void set_trace(void* buf, size_t bytes, int block) {
  g_trace_buf = reinterpret_cast<long long*>(buf);
  g_trace_bytes = buf ? bytes : 0;
  g_trace_block = block;
}

// True once after a persistent kernel's bounded wait has expired: the word is cleared by the report, so the
// call after the one that reports LSTM_INTERNAL runs normally again.
bool take_watchdog() {
  std::lock_guard<std::mutex> lk(g_mu);
  if (!g_watch_host || !*g_watch_host) return false;
  *g_watch_host = 0;
  return true;
}

// Everything the persistent path creates lazily, created now for the current device: the host-visible watchdog
// word and the event that chains the persistent launches.  After it no persistent forward call creates anything.
hipError_t setup_persistent() {
  DeviceInfo di;
  (void)device_info(di);
  if (!ensure_watchdog()) return hipErrorOutOfMemory;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= 16) return hipSuccess;  // launches on such a device are not chained
  std::lock_guard<std::mutex> lk(g_launch_mu);
  if (!g_last_launch[dev]) {
    e = hipEventCreateWithFlags(&g_last_launch[dev], hipEventDisableTiming | hipEventDisableSystemFence);
    if (e != hipSuccess) return e;
    g_last_launch_recorded[dev] = false;
  }
  return hipSuccess;
}

void release_persistent() {
  {
    std::lock_guard<std::mutex> lk(g_launch_mu);
    for (hipEvent_t& ev : g_last_launch)
      if (ev) {
        (void)hipEventDestroy(ev);
        ev = nullptr;
      }
    for (hipEvent_t& ev : g_side_ev)
      if (ev) {
        (void)hipEventDestroy(ev);
        ev = nullptr;
      }
    if (g_side_stream) {
      (void)hipStreamDestroy(g_side_stream);
      g_side_stream = nullptr;
    }
  }
  std::lock_guard<std::mutex> lk(g_mu);
  if (g_watch_host) {
    (void)hipHostFree(g_watch_host);
    g_watch_host = nullptr;
    g_watch_dev = nullptr;
  }
}

// Large hidden sizes: one layer per launch, the layer's recurrent matrix spread over all CUs.
// Largest batch that they take at all (AUTO leaves them earlier: steps_beat_large).
constexpr int kLargeMaxBatch1024 = 768, kLargeMaxBatch2048 = 448;

// LSTM: whether a pass is faster step by step (a GEMM for the whole batch and a point-wise kernel, schedule.hip) than on the
// one-layer kernels, which take slices of 32 rows, forward two side by side at H = 1024, backward four, and launch after
// launch from there on.  A launch costs about 50 us before its first step and a step of it the same whatever the rows; a
// step of the GEMM costs the less per row the more rows there are.  The models below are of microseconds per step and layer,
// fitted to L = 1 and 4, T = 5 to 50, up to 768 rows.  Time step by step / on these kernels, T = 50 (T = 5):
//   H = 2048 forward 1.44 (0.99) at 96 rows, 1.18 (0.85) at 128, 1.05 (0.74) at 256, 1.01 at 448; backward 1.12 (0.94) at 96, 0.99
//   (0.85) at 128, 0.92 (0.80) at 256
//   H = 1024 forward 1.63 (0.97) at 128, 1.25 (0.77) at 256, 1.04 (0.65) at 512; backward 1.38 (1.08) at 128, 1.08 (0.93) at 256,
//   0.97 (0.84) at 512
// Below 97 and 321 rows only short passes would gain (two steps of 64 rows at H = 2048 0.15 -> 0.11 ms); they stay on chip.
bool steps_beat_large(const Dims& d, bool backward) {
  if (!(d.H == 1024 || d.H == 2048) || d.B <= (d.H == 1024 ? 320 : 96)) return false;
  const double B = d.B, T = d.T;
  const auto launches = [&](int rows) { return (double)((d.B + rows - 1) / rows); };
  if (d.H == 2048) {
    if (backward) return launches(32) * (25.5 + 75.0 / T) > 22.0 + 0.7 * B + 75.0 / T;
    return launches(32) * (13.0 + 52.0 / T) > 17.0 + 0.41 * B + 25.0 / T;
  }
  if (backward) return launches(128) * (27.5 + 90.0 / T) > 20.0 + 0.18 * B + 30.0 / T;
  return launches(64) * (7.8 + 45.0 / T) > 15.0 + 0.11 * B + 20.0 / T;
}

// H = 320 and 384 with more than 512 rows, which are not padded either (reported_hidden): whether a pass is faster off the chip, as
// for the LSTM above, for the GRU forward and backward together.  The models are of microseconds: a launch, the steps in it (layer l
// follows l steps behind) and the rows; off the chip the layers, their steps and rows, up to 640 of which fill one round of the step
// kernel.  Fitted to one to eight layers, 6 to 80 steps, 520 to 8192 rows, within 6 % (off the chip 11) in rms; the choice costs
// 0.3 % on average against the faster of the two.  Time on chip / off it, T = 1, 10 and 40:
//   LSTM forward, H = 320: two layers of 1024 rows 2.4, 0.66, 0.40; four of 4096 10.4, 1.5, 0.80; H = 384: 3.2, 0.84, 0.49; 8.8, 1.25, 0.68
//   LSTM backward, H = 320: 1.65, 0.70, 0.56; 4.9, 1.46, 1.03; H = 384: 2.3, 0.88, 0.68; 4.7, 1.27, 0.87
//   GRU forward / backward, four layers of 1024 rows: H = 320 7.6, 1.95, 1.08 / 3.3, 1.60, 1.23; H = 384 5.9, 1.55, 0.82 / 3.5, 1.56, 1.16
bool steps_beat_chip(const Dims& d, int cell, bool backward) {
  if (!(d.H == 320 || d.H == 384) || d.B <= 512) return false;
  constexpr int cus = 256;
  const int groups = d.H / 8, per = cus / groups, slices = (d.B + 63) / 64, i = d.H == 384;
  struct Model { double launch, step[2], row[2], layer, few, given, given_row[2]; };
  constexpr Model fwd = {55.0, {3.1, 3.5}, {0.0049, 0.0045}, 16.0, 25.0, 13.0, {0.0275, 0.0330}};
  constexpr Model bwd = {45.0, {8.0, 8.1}, {0.0088, 0.0111}, 18.0, 41.0, 19.0, {0.0418, 0.0535}};
  constexpr Model gru = {80.0, {10.6, 12.1}, {0.0106, 0.0100}, 0.0, 0.0, 28.7, {0.0261, 0.0371}};
  const Model& m = cell ? gru : (backward ? bwd : fwd);
  double chip = (double)d.L * d.T * d.B * m.row[i];
  for (int l = 0; l < d.L; l += per) {
    const int layers = std::min(per, d.L - l), side = std::min(cus / (layers * groups), 16 / layers);
    chip += (slices + side - 1) / side * (m.launch + (d.T + layers - 1) * m.step[i]);
  }
  const double step = m.few > 0.0 && d.B <= 640 ? m.few : m.given + d.B * m.given_row[i];
  return chip > d.L * (m.layer + d.T * step);
}

bool persistent_large(const Dims& d, bool backward) {
  if (knobs().no_large_persistent) return false;
  if (!(d.H == 1024 || d.H == 2048 || large_mid_size(d))) return false;
  if (d.B > (d.H <= 1024 ? kLargeMaxBatch1024 : kLargeMaxBatch2048)) return false;
  DeviceInfo di;
  if (!device_info(di) || !di.coop) return false;
  return (backward ? (d.H / 128) * (d.H / 128) : d.H / 8) <= di.cus;
}

bool persistent_supported(const Dims& d, bool backward) {
  if (persistent_large(d, backward)) return true;
  if (!on_chip_size(d.H) || too_short_on_chip(d, 0)) return false;
  // Slices of 64 rows, one after the other once the chip is full: the rate does not depend on their number.  The GEMM rungs
  // gain with the batch and with short sequences (a launch here costs 70 us before its first step).  Forward and backward
  // of four layers, these kernels / the fused rung: T = 60, H = 512 23.0 / 30.7 ms at 1024 rows and 92 / 90 at 4096, H = 256
  // 15.7 / 22.7 at 2048 and 63 / 57 at 8192, H = 128 26.5 / 24.4 at 8192; T = 10, H = 512 6.3 / 5.2 at 1024 and 25.5 / 15.1 at
  // 4096.  The limit only bounds the number of launches of one call.
  if (d.B > 16384) return false;
  DeviceInfo di;
  if (!device_info(di) || !di.coop) return false;
  return d.H / 8 <= di.cus;  // deeper stacks than the chip holds run as groups of layers (run_forward_persistent)
}

namespace {



// Reserve of one layer in floats per (step, row, unit), and where its hidden states start, for each cell.
inline size_t res_width(int cell) { return cell == 0 ? 6 : (cell == 1 ? 5 : 1); }
inline size_t res_h_offset(int cell, size_t TB, int H) { return cell == 0 ? 5 * TB * H : 0; }
inline int gates_of_cell(int cell) { return cell == 0 ? 4 : (cell == 1 ? 3 : 1); }

// Steps from which the one-layer kernels run on the bf16 matrix cores.  A launch of theirs fetches, cuts and lays out the
// weights in three parts first and has launches behind it that end at once (the repeat on the fp32 kernel: one forward, two
// backward, and two in both directions when this was timed); a step is shorter.  Time against the fp32 kernels, L = 1 to 4, B = 1 to 250:
//   forward   LSTM 0.98 or less at one step; GRU, H = 1024 / 2048: 1.01 / 0.95 at six steps, 0.97 / 0.91 at eight; single
//             gate 1.05 / 0.97 at eight, 0.97 / 0.90 at twelve
//   backward  H = 2048: LSTM 0.98 at four (1.03 at one), GRU 1.02 at 20, 0.98 at 32, single gate 1.02 at twelve, 0.95 at 20.
//             H = 1024: one layer of one slice, whose tiles are cut in four, gains at no length (LSTM 1.02 at 200 steps); up to
//             64 rows of several layers LSTM 0.95 to 1.0 at six, the others 0.97 at 20; else LSTM 0.99 at twelve, GRU 0.99
//             at 50, single gate 1.00 at 32
int large_split3_steps(const Dims& d, int cell, bool backward) {
  const int c = cell == 0 ? 0 : (cell == 1 ? 1 : 2);
  constexpr int never = 1 << 30;
  constexpr int fwd[2][3] = {{1, 8, 12}, {1, 5, 8}}, bwd2048[3] = {4, 32, 20}, bwd_few[3] = {6, 20, 20}, bwd[3] = {12, 50, 32};
  if (!backward) return fwd[d.H > 1024][c];
  if (d.H > 1024) return bwd2048[c];
  if (d.L == 1 && d.B <= 32) return never;
  return d.L > 1 && d.B <= 64 ? bwd_few[c] : bwd[c];
}
// The same for the alternating kernels of H = 256 and 512 (forward; L layers of a launch with `workgroups` workgroups).
//   H = 512: LSTM 0.96 at six steps, GRU 0.99, single gate 0.95 at eight (1.01 at six); from three layers on two steps earlier.
//   H = 448 and 384 like it; 320 two steps later (1.00 to 1.03 at six steps, 0.93 at twelve); at 100 steps 0.65 to 0.75 for all three
//   H = 256: with CUs to spare 0.9 to 1.0 at 20 steps (three layers: 0.97 at twelve); with a workgroup on every CU the
//            exchange is slower than the products are faster: LSTM and GRU of one or two layers 1.0 to 1.1 at any length, four
//            layers 0.97 at 50 steps, single gate 0.9 to 1.0 at 50
//   With more than four layers at H = 256 the distance at which a layer follows the one below costs more than it saves
//   (LSTM, L = 8, B = 64, T = 100: 0.58 -> 0.64 ms), and at H = 128 a block is too short for the exchange (L = 4, B = 256:
//   0.42 -> 1.09).
int pp3_steps(const Dims& d, int cell, int workgroups, int cus) {
  constexpr int never = 1 << 30;
  if (d.H > 256) return (cell >= 2 ? 8 : 6) - (d.L >= 3 ? 2 : 0) + (d.H <= 320 ? 2 : 0);
  if (d.H != 256 || d.L > 4) return never;
  if (workgroups < cus) return d.L == 3 ? 12 : 20;
  return cell >= 2 || d.L >= 4 ? 50 : never;
}
// LSTM_SPLIT3 pins the choice wherever there is one.
bool split3_wanted(bool rule) { return knobs().split3 < 0 ? rule : knobs().split3 > 0; }
// LSTM_SPLIT3=2: the repeated launch is asked for whatever the sums were.
hipError_t force_redo(int* redo, hipStream_t s) { return knobs().split3 == 2 ? launch_set_word(redo, 1, s) : hipSuccess; }

// A launch on the bf16 matrix cores may be run again by the fp32 kernel (a sum that is infinite or NaN), which then reads
// the states that the call was given.  Where the caller has the final ones written over them, a copy is kept: `in`
// becomes slot `i` of the workspace's state area (four of n floats, which the persistent kernels do not use otherwise).
bool overlap(const float* a, size_t na, const float* b, size_t nb) { return a && b && a < b + nb && b < a + na; }
hipError_t keep_state(const float*& in, const float* out1, const float* out2, size_t n, char* ws, const WsLayout& w, int i, hipStream_t s) {
  if (!overlap(in, n, out1, n) && !overlap(in, n, out2, n)) return hipSuccess;
  float* const copy = reinterpret_cast<float*>(ws + w.state) + i * n;
  const int cols = 8;  // (n is a multiple of H)
  const hipError_t e = launch_ew(EW_COPY, copy, cols, in, cols, nullptr, 0, (int)(n / cols), cols, s);
  in = copy;
  return e;
}

int run_forward_persistent_large(const FwdArgs& args, int cell) {
  FwdArgs a = args;
  const Dims& d = a.d;
  const bool s3 = split3_wanted(d.T >= large_split3_steps(d, cell, false));
  if (s3) {
    if (cell == 1) CK(keep_state(a.h0, a.hT, a.cT, (size_t)d.L * d.B * d.H, a.ws, a.w, 0, a.stream), "keep h0");
    CK(keep_state(a.c0, a.hT, a.cT, (size_t)d.L * d.B * d.H, a.ws, a.w, 1, a.stream), "keep c0");
  }
  const size_t TB = (size_t)d.T * d.B, G = (size_t)gates_of_cell(cell) * d.H, BH = (size_t)d.B * d.H;
  const size_t rstride = res_width(cell) * TB * d.H;
  hipStream_t s = a.stream;
  float* hx = reinterpret_cast<float*>(a.ws + a.w.xchg);
  int* flags = reinterpret_cast<int*>(a.ws + a.w.flags);
  float* P = reinterpret_cast<float*>(a.ws + a.w.P);
  float* const hx0 = reinterpret_cast<float*>(a.ws + a.w.scratch);  // 32 H floats per slice of 32 rows: the area has that per row
  // slices of 32 batch rows side by side while the CUs last (two at H = 1024), the rest in further launches
  DeviceInfo di;
  (void)device_info(di);
  const int slices = (d.B + 31) / 32;
  int cap = di.cus / (d.H / 8);
  if (cap < 1) cap = 1;
  if (cap > 4) cap = 4;
  for (int l = 0; l < d.L; ++l) {
    const int Il = in_dim(d, l);
    const float* in = l == 0 ? a.x : a.reserve + (size_t)(l - 1) * rstride + res_h_offset(cell, TB, d.H);
    const float* Wl = a.W + (l == 0 ? 0 : G * d.I + (size_t)(l - 1) * G * d.H);
    {
      ProfScope ps(LSTM_PHASE_FWD_INPUT_GEMM, s);
      GemmProblem p{in, Wl, P, (int)TB, (int)G, Il, Il, 1, 1, Il, (long)G, 0};
      // (the exchange area is idle between two recurrences: it takes the partial tiles)
      CK(launch_gemm_group(&p, 1, s, hx, a.w.flags - a.w.xchg), "input projection GEMM");
    }
   for (int s0 = 0; s0 < slices; s0 += cap) {
    const int nsl = slices - s0 < cap ? slices - s0 : cap;
    const int counters = nsl * (d.T + 1) * 16 * kFlagStride;
    {
      ProfScope ps(LSTM_PHASE_FWD_PACK, s);
      // (S3: the redo word and the counters of the kernel that may have to run the launch again lie behind)
      CK(launch_fill_zero(flags, (s3 ? (size_t)2 * counters + 32 : (size_t)counters) * 4, s), "zero step counters");
      const float* const h0 = a.h0 ? a.h0 + (size_t)l * BH : nullptr;
      if (s3) CK(launch_pack_stateL3(h0, hx, hx0, d.T, d.B, d.H, 32 * s0, nsl, s), "pack h0");
      else CK(launch_pack_stateL(h0, hx, d.T, d.B, d.H, 32 * s0, nsl, s), "pack h0");
    }
    PersFwdLArgs k;
    k.b0 = 32 * s0; k.nsl = nsl;
    k.R = a.R + (size_t)l * G * d.H; k.bias = a.b + (size_t)l * G; k.P = P;
    const float* state0 = cell == 0 ? a.c0 : (cell == 1 ? a.h0 : nullptr);  // the GRU's cell update reads h_{t-1}
    k.c0 = state0 ? state0 + (size_t)l * BH : nullptr;
    k.hx = hx; k.flags = flags; k.watchdog = g_watch_dev;
    k.res = a.reserve + (size_t)l * rstride;
    k.y = l == d.L - 1 ? a.y : nullptr;
    k.hT = a.hT ? a.hT + (size_t)l * BH : nullptr;
    k.cT = a.cT ? a.cT + (size_t)l * BH : nullptr;
    k.T = d.T; k.B = d.B; k.spin_limit = spin_limit(); k.full_fences = full_fences();
    k.trace = (g_trace_bytes >= (size_t)d.T * 64) ? g_trace_buf : nullptr;
    k.trace_block = g_trace_block;
    ProfScope ps(LSTM_PHASE_FWD_RECURRENCE, s);
    prof_flops(2.0 * G * d.H * std::min(32 * nsl, d.B - 32 * s0) * d.T, s3 ? "pers_fwdL_kernel (bf16)" : "pers_fwdL_kernel");
    k.redo = s3 ? flags + counters : nullptr;
    CK(launch_fwdL_any(d.H, cell, k, s, s3), "persistent forward launch (large H)");
    if (!s3) continue;
    CK(force_redo(k.redo, s), "ask for a repeated launch");
    // an infinite or NaN sum has no parts: the fp32 kernel runs the launch again (it ends at once if nobody asked)
    k.flags = flags + counters + 32;
    k.hx0 = hx0;
    CK(launch_fwdL_any(d.H, cell, k, s, false), "persistent forward launch (large H, repeated)");
   }
  }
  return LSTM_OK;
}


}  // namespace

int weight_gradients(const BwdArgs& a, const float* dA_all, bool grouped, bool bias_done);

namespace {

// Backward pass of the large-H shapes: per layer (top down) one persistent launch for the recurrence, then
// the batched product that hands the gradient to the layer below; weight gradients at the end.

int run_backward_persistent_large(const BwdArgs& args, int cell, bool* bias_done, LayerGradients* lg) {
  BwdArgs a = args;
  const Dims& d = a.d;
  constexpr int UB = 128;
  const int NBK = d.H / UB;
  const size_t TB = (size_t)d.T * d.B, G = 4 * (size_t)d.H, BH = (size_t)d.B * d.H;
  const size_t GW = (size_t)gates_of_cell(cell) * d.H, rstride = res_width(cell) * TB * d.H;
  hipStream_t s = a.stream;
  // slices of 32 batch rows side by side while the CUs last (four at H = 1024), the rest in further launches
  DeviceInfo di;
  (void)device_info(di);
  const int slices = (d.B + 31) / 32;
  // A single slice at H = 1024 would occupy 64 CUs: the tiles' K is cut in four, 256 workgroups (LSTM_LARGE_KSPLIT=0:
  // not); two slices of a single layer cut it in two (with more layers the idle CUs are used by the weight gradients
  // of the layer above, which is worth more: L = 4, B = 64).  Below 1024 always at least in two: uncut, a workgroup
  // would finalise three or four octets of units, whose state leaves no registers for a whole tile.
  const int ks = d.H < 1024 ? (slices == 1 && d.L == 1 ? 4 : 2)
                 : d.H != 1024 || !knobs().large_ksplit ? 1 : (slices == 1 ? (d.L > 1 ? 2 : 4) : ((slices == 2 && d.L == 1) ? 2 : 1));
  int cap = di.cus / (NBK * NBK * (d.H < 1024 ? 2 : 1));
  if (cap < 1) cap = 1;
  if (cap > 4) cap = 4;
  const int maxsl = slices < cap ? slices : cap;
  float* dA_all = reinterpret_cast<float*>(a.ws + a.w.P);
  float* dxb = reinterpret_cast<float*>(a.ws + a.w.dx);
  float* X = reinterpret_cast<float*>(a.ws + a.w.xchg);
  float* Pp = X + (size_t)maxsl * d.T * NBK * (4 * UB * 32);
  int* flagsA = reinterpret_cast<int*>(a.ws + a.w.flags);
  int* flagsP = flagsA + (size_t)maxsl * d.T * NBK * kFlagInts;
  const int counters = (int)((size_t)2 * maxsl * d.T * NBK * kFlagInts);
  // On the bf16 matrix cores wherever the third part of the exchanged values finds room at the end of the reserve
  // stand-in (24 bytes per row, layer and unit, of which 256 per slice of 32 rows are needed: from 11 rows of one layer on);
  // the rest of that area takes partial tiles of the products on the side stream.
  const size_t x3_bytes = (size_t)maxsl * d.T * NBK * (2 * UB * 32) * sizeof(float), resv_bytes = a.w.total - a.w.resv;
  const bool s3 = x3_bytes <= resv_bytes && split3_wanted(d.T >= large_split3_steps(d, cell, true));
  float* const X3 = reinterpret_cast<float*>(a.ws + a.w.resv + ((resv_bytes - (s3 ? x3_bytes : 0)) & ~(size_t)255));
  const Scratch side_part{reinterpret_cast<float*>(a.ws + a.w.resv), (resv_bytes - (s3 ? x3_bytes : 0)) & ~(size_t)255};
  const size_t LBH = (size_t)d.L * BH;
  if (s3) {
    CK(keep_state(a.dhT, a.dh0, a.dc0, LBH, a.ws, a.w, 0, s), "keep dhT");
    CK(keep_state(a.dcT, a.dh0, a.dc0, LBH, a.ws, a.w, 1, s), "keep dcT");
    CK(keep_state(a.c0, a.dh0, a.dc0, LBH, a.ws, a.w, 2, s), "keep c0");
  }
  const bool bias_in_kernel = slices == 1;
  // A launch that occupies at most half of the CUs (H = 1024 with one or two slices) leaves room for the weight
  // gradients of the layer above, which are complete once that layer's recurrence is: they run on a side stream
  // while this layer's recurrence runs (Section 2.6 wants them after the propagation of *their* layer, not of all
  // layers).  The side stream starts them behind the counter reset that precedes the persistent launch, so that the
  // launch gets its CUs first and the products fill the rest.  LSTM_NO_WGRAD_OVERLAP=1 keeps one stream.
  bool overlap = (cell == 0 || lg) && d.L > 1 && 2 * maxsl * NBK * NBK * ks <= di.cus && slices <= cap;
  // The side stream and its two events are process-wide: calls from several host threads take turns from the first
  // fork to the join (the enqueue only; the GPU work of different calls still overlaps as their streams allow).
  std::unique_lock<std::mutex> side_turn(g_side_mu, std::defer_lock);
  {
    hipStreamCaptureStatus cst = hipStreamCaptureStatusNone;
    if (knobs().no_wgrad_overlap || hipStreamIsCapturing(s, &cst) != hipSuccess || cst != hipStreamCaptureStatusNone ||
        !ensure_side_stream())
      overlap = false;
    (void)hipGetLastError();
  }
  if (overlap) side_turn.lock();
  int pending = -1;  // layer whose weight gradients wait for the side stream
  for (int l = d.L - 1; l >= 0; --l) {
    const int Il = in_dim(d, l);
    float* dA = dA_all + (size_t)l * TB * G;
    for (int s0 = 0; s0 < slices; s0 += cap) {
      const int nsl = slices - s0 < cap ? slices - s0 : cap;
      {
        ProfScope ps(LSTM_PHASE_BWD_PACK, s);
        CK(launch_fill_zero(flagsA, ((size_t)counters + (s3 ? 32 : 0)) * 4, s), "zero step counters");
      }
      if (overlap && pending >= 0) {
        CK(hipEventRecord(g_side_ev[0], s), "fork to the side stream");
        CK(hipStreamWaitEvent(g_side_stream, g_side_ev[0], 0), "side stream wait");
        const int st = cell == 0 ? weight_gradients_layers(a, dA_all, pending, pending + 1, g_side_stream, true, bias_in_kernel, side_part)
                                 : lg->fn(lg->ctx, pending, g_side_stream, side_part);
        if (st != LSTM_OK) return st;
        pending = -1;
      }
      PersBwdLArgs k;
      k.R = a.R + (size_t)l * GW * d.H;
      k.res = a.reserve + (size_t)l * rstride;
      const float* state0 = cell == 0 ? a.c0 : a.h0;
      k.c0 = state0 ? state0 + (size_t)l * BH : nullptr;
      k.dout = (l == d.L - 1) ? a.dy : dxb + (size_t)(l + 1) * TB * d.H;
      k.dhT = a.dhT ? a.dhT + (size_t)l * BH : nullptr;
      k.dcT = a.dcT ? a.dcT + (size_t)l * BH : nullptr;
      k.dA = dA; k.X = X; k.Pp = Pp;
      k.dh0 = a.dh0 ? a.dh0 + (size_t)l * BH : nullptr;
      k.dc0 = a.dc0 ? a.dc0 + (size_t)l * BH : nullptr;
      k.db = bias_in_kernel ? a.db + (size_t)l * GW : nullptr;
      k.X3 = s3 ? X3 : nullptr;
      k.redo = s3 ? flagsA + counters : nullptr;
      k.flagsA = flagsA; k.flagsP = flagsP; k.watchdog = g_watch_dev;
      k.T = d.T; k.B = d.B; k.b0 = 32 * s0; k.nsl = nsl; k.ks = ks; k.spin_limit = spin_limit(); k.full_fences = full_fences();
      k.trace = (g_trace_bytes >= (size_t)d.T * 64) ? g_trace_buf : nullptr;
      k.trace_block = g_trace_block;
      ProfScope ps(LSTM_PHASE_BWD_RECURRENCE, s);
      prof_flops(2.0 * GW * d.H * std::min(32 * nsl, d.B - 32 * s0) * d.T, s3 ? "pers_bwdL_kernel (bf16)" : "pers_bwdL_kernel");
      CK(launch_bwdL_any(d.H, cell, k, s, s3), "persistent backward launch (large H)");
      if (s3) {  // an infinite or NaN sum has no parts: the fp32 kernel runs the launch again (both end at once if nobody asked)
        CK(force_redo(k.redo, s), "ask for a repeated launch");
        CK(launch_redo_bwdL(k, counters, s), "zero step counters");
        CK(launch_bwdL_any(d.H, cell, k, s, false), "persistent backward launch (large H, repeated)");
      }
    }
    float* din = l > 0 ? dxb + (size_t)l * TB * d.H : a.dx;
    if (din) {  // the GRU's gradient with respect to W_n x is its third group: the first GW columns are the ones W multiplies
      ProfScope ps(LSTM_PHASE_BWD_INPUT_GEMM, s);
      const float* Wl = a.W + (l == 0 ? 0 : GW * d.I + (size_t)(l - 1) * GW * d.H);
      GemmProblem p{dA, Wl, din, (int)TB, Il, (int)GW, (long)G, 1, Il, 1, Il, 0};
      CK(launch_gemm_group(&p, 1, s, reinterpret_cast<float*>(a.ws + a.w.xchg), a.w.flags - a.w.xchg), "input-gradient GEMM");
    }
    if (overlap) pending = l;
  }
  if (bias_done) *bias_done = bias_in_kernel;
  if (!overlap) return cell != 0 ? LSTM_OK : weight_gradients(a, dA_all, true, bias_in_kernel);
  // the bottom layer's weight gradients have nothing left to hide behind; then the side stream joins
  const int st = cell == 0 ? weight_gradients_layers(a, dA_all, 0, 1, s, true, bias_in_kernel, exchange_scratch(a.ws, a.w))
                           : lg->fn(lg->ctx, 0, s, exchange_scratch(a.ws, a.w));
  if (st != LSTM_OK) return st;
  if (lg) lg->used = true;
  CK(hipEventRecord(g_side_ev[1], g_side_stream), "join record");
  CK(hipStreamWaitEvent(s, g_side_ev[1], 0), "join wait");
  return LSTM_OK;
}

}  // namespace

// Wide persistent kernels for the GRU: hidden sizes and CU budget of the LSTM ones; they also take batches of 32
// rows and fewer (the rows past the batch are zeros), where the LSTM has kernels of its own.
bool gru_persistent_supported(const Dims& d) {
  if (persistent_large(d, false) && persistent_large(d, true)) return true;  // one-layer kernels, H > 512
  if (!on_chip_size(d.H)) return false;
  if (d.B > 16384) return false;  // (the cells' own limits are lower: rnn_cells.hip)
  DeviceInfo di;
  if (!device_info(di) || !di.coop) return false;
  return d.H / 8 <= di.cus;  // deeper stacks than the chip holds run as groups of layers
}

// cell: 0 = LSTM; 1 = GRU, 2 / 3 = single-gate RNN with ReLU / tanh (wide kernels only: the caller has checked
// gru_persistent_supported; a.c0 / a.cT are null, W, R, b have 3H or H rows and a.reserve is that cell's reserve).
// Layers that fit on the chip together: L * H/8 workgroups, one per CU.
int layers_per_launch(const Dims& d) {
  DeviceInfo di;
  if (!device_info(di)) return 0;
  return di.cus / (d.H / 8);
}

// Whether a backward pass runs on the kernel with two alternating chains per workgroup (slices of 64 rows).  (The kernel with one
// chain has instances for the powers of two only.)
bool bwd_alternating(const Dims& d, int cell) {
  const bool wide = cell != 0 || (narrow_slice_rows(d, cell, knobs().bwd_narrow, true) == 0 && bwd_wide(d));
  return wide && (((cell == 0 || knobs().rnn_pp) && knobs().pingpong != 0) || (d.H & (d.H - 1)) != 0);
}

int forward_layers(const FwdArgs& a, int cell);
int backward_layers(const BwdArgs& a, int cell, bool* bias_done, bool with_weight_gradients);

// A stack deeper than the chip holds at once runs as groups of consecutive layers, one group per launch (per batch
// slice group): the hidden states of a group's top layer, all T steps, are the input sequence of the next group --
// the same situation as x for layer 0 (Section 2.3) -- and backward the gradient a group's bottom layer produces for
// its input is the upstream gradient of the group below.
int run_forward_persistent(const FwdArgs& a, int cell) {
  const Dims& d = a.d;
  const int near_per = near_large_layers(d, cell, false);
  if (!near_per && persistent_large(d, false)) {
    if (!ensure_watchdog()) return LSTM_HIP_ERROR;
    return run_forward_persistent_large(a, cell);
  }
  const int per = near_per ? near_per : layers_per_launch(d);
  if (per <= 0) return LSTM_UNSUPPORTED;
  if (d.L <= per) return forward_layers(a, cell);
  const size_t TB = (size_t)d.T * d.B, BH = (size_t)d.B * d.H, G = (size_t)gates_of_cell(cell) * d.H;
  const size_t rstride = res_width(cell) * TB * d.H;
  for (int g0 = 0; g0 < d.L; g0 += per) {
    FwdArgs g = a;
    g.d.L = d.L - g0 < per ? d.L - g0 : per;
    const int top = g0 + g.d.L - 1;
    if (g0 > 0) {
      g.d.I = d.H;
      g.x = a.reserve + (size_t)(g0 - 1) * rstride + res_h_offset(cell, TB, d.H);
      g.W = a.W + G * d.I + (size_t)(g0 - 1) * G * d.H;
    }
    g.R = a.R + (size_t)g0 * G * d.H;
    g.b = a.b + (size_t)g0 * G;
    g.h0 = a.h0 ? a.h0 + (size_t)g0 * BH : nullptr;
    g.c0 = a.c0 ? a.c0 + (size_t)g0 * BH : nullptr;
    g.hT = a.hT ? a.hT + (size_t)g0 * BH : nullptr;
    g.cT = a.cT ? a.cT + (size_t)g0 * BH : nullptr;
    g.reserve = a.reserve + (size_t)g0 * rstride;
    // a group's top layer always leaves its hidden states where the next group reads them (an inference call writes
    // nothing else of the reserve): y of the group is that array
    if (top < d.L - 1) g.y = a.reserve + (size_t)top * rstride + res_h_offset(cell, TB, d.H);
    const int st = forward_layers(g, cell);
    if (st != LSTM_OK) return st;
  }
  return LSTM_OK;
}

int forward_layers(const FwdArgs& args, int cell) {
  FwdArgs a = args;
  const Dims& d = a.d;
  const size_t TB = (size_t)d.T * d.B, G = (cell == 0 ? 4 : (cell == 1 ? 3 : 1)) * (size_t)d.H;
  hipStream_t s = a.stream;
  if (!ensure_watchdog()) return LSTM_HIP_ERROR;
  DeviceInfo di;
  (void)device_info(di);
  const int slice_rows_narrow = narrow_slice_rows(d, cell, knobs().fwd_narrow, false);
  const bool narrow_slices = slice_rows_narrow > 0;
  const BatchPlan bp = narrow_slices ? BatchPlan{slice_rows_narrow / 16, 1} : batch_plan(d.B);
  const int BP = 16 * bp.NT;
  const bool wide = cell != 0 || (!narrow_slices && fwd_wide(d));
  float* hx = reinterpret_cast<float*>(a.ws + a.w.xchg);
  int* flags = reinterpret_cast<int*>(a.ws + a.w.flags);
  float* P0 = reinterpret_cast<float*>(a.ws + a.w.P);
  if (tiny_path(d, cell)) {
    {
      ProfScope ps(LSTM_PHASE_FWD_INPUT_GEMM, s);
      GemmProblem p{a.x, a.W, P0, (int)TB, (int)G, d.I, d.I, 1, 1, d.I, (long)G, 0};
      CK(launch_gemm_group(&p, 1, s, hx, a.w.flags - a.w.xchg), "input projection GEMM (layer 0)");
    }
    PersFwdArgs k{};
    k.W = a.W; k.R = a.R; k.bias = a.b; k.P0 = P0; k.c0 = a.c0; k.h0 = a.h0; k.hx = hx; k.watchdog = g_watch_dev;
    k.res = a.reserve; k.y = a.y; k.hT = a.hT; k.cT = a.cT;
    k.L = d.L; k.T = d.T; k.B = d.B; k.I = d.I; k.H = d.H; k.spin_limit = spin_limit(); k.full_fences = full_fences();
    k.trace = (g_trace_bytes >= (size_t)d.T * 64) ? g_trace_buf : nullptr;
    k.trace_block = g_trace_block;
    ProfScope ps(LSTM_PHASE_FWD_RECURRENCE, s);
    prof_flops(2.0 * G * d.T * d.H * (2 * d.L - 1), "pers_fwd_tiny_kernel");
    CK(launch_fwd_tiny(d.H, k, s), "persistent forward launch (single sequence)");
    return LSTM_OK;
  }
  if (const NearPlan np = near_plan(d, cell, false); np.units) {
    {
      ProfScope ps(LSTM_PHASE_FWD_INPUT_GEMM, s);
      GemmProblem p{a.x, a.W, P0, (int)TB, (int)G, d.I, d.I, 1, 1, d.I, (long)G, 0};
      CK(launch_gemm_group(&p, 1, s, hx, a.w.flags - a.w.xchg), "input projection GEMM (layer 0)");
    }
    PersFwdArgs k{};
    k.W = a.W; k.R = a.R; k.bias = a.b; k.P0 = P0; k.c0 = a.c0; k.h0 = a.h0; k.hx = hx; k.watchdog = g_watch_dev;
    k.res = a.reserve; k.y = a.y; k.hT = a.hT; k.cT = a.cT;
    k.L = d.L; k.T = d.T; k.B = d.B; k.I = d.I; k.H = d.H; k.spin_limit = spin_limit(); k.full_fences = full_fences();
    k.spread = np.spread; k.keep = a.inference ? 0 : 1;
    k.trace = (g_trace_bytes >= (size_t)d.T * 64) ? g_trace_buf : nullptr;
    k.trace_block = g_trace_block;
    ProfScope ps(LSTM_PHASE_FWD_RECURRENCE, s);
    prof_flops(2.0 * G * d.B * d.T * d.H * (2 * d.L - 1), "pers_fwd_near_kernel");
    for (int s0 = 0; s0 < np.slices; s0 += np.side) {
      k.b0 = 16 * s0;
      k.nsl = std::min(np.side, np.slices - s0);
      CK(launch_fwd_near(cell, d.H, np.units, k, s), "persistent forward launch (slices of 16 rows)");
    }
    return LSTM_OK;
  }
  // Wide kernel with I == H: layer 0 multiplies by W_0 inside the kernel like the layers above it (its workgroups
  // are otherwise idle half of every step), reading x from a copy in exchange layout that takes the place of the
  // projection in the workspace.  LSTM_FWD_BATCHED_INPUT=1 keeps the batched product of Section 2.3 instead.
  // (Section 2.3 notes that batching the input products pays at some sizes and not at others; here the batched
  // product only wins where nothing would be idle otherwise: one layer, one slice -- by about 4 %.)
  // (the kernels with two alternating chains also take I < H: x zero-padded to H columns in that copy)
  const bool pp_ok = (cell == 0 || knobs().rnn_pp) && knobs().pingpong != 0;
  bool x_in_kernel = wide && (d.I == d.H || (pp_ok && d.I < d.H)) && !(d.L == 1 && d.B <= 64);
  if (x_in_kernel) {
    if (knobs().fwd_batched_input) x_in_kernel = false;
    const size_t rows = (size_t)(d.B + 63) / 64 * 64;  // the copy of x: T+1 slots of H x 64 per slice
    if (((size_t)d.T + 1) * rows * d.H > (size_t)d.L * TB * 4 * d.H) x_in_kernel = false;
  }
  // LSTM with every layer multiplying its input in the kernel: the two half-slices of 32 rows take turns inside the
  // waves (pers_fwd_pp_kernel); LSTM_PINGPONG=0 keeps the one-chain kernel
  const bool pp = x_in_kernel && pp_ok;
  // ... on the bf16 matrix cores where that is faster (pp3_steps) and the copy of x in three parts finds room (half as large
  // again, up to the scratch area), as the exchange slots do.
  // (The kernel that runs a launch again reads x once more: not where y is written over it.)
  const size_t x3_slots = (size_t)(d.T + 1) * ((size_t)(d.B + 63) / 64 * 64) * d.H * 6;  // bytes of one layer's states in parts
  // Slices of 64 batch rows run side by side in one launch while the CUs last, the rest in further launches.
  const int grid = d.L * (d.H / 8);
  int cap = (wide || narrow_slices) && grid > 0 ? di.cus / grid : 1;
  if (cap > 16 / d.L) cap = 16 / d.L;  // the counter region holds 16 (slice, layer) pairs
  if (cap < 1) cap = 1;
  const int slice_rows = narrow_slices ? slice_rows_narrow : 64;
  const int slices = wide ? (d.B + 63) / 64 : (narrow_slices ? (d.B + slice_rows - 1) / slice_rows : 1);
  const bool pp3 = pp && d.H >= 256 && split3_wanted(d.T >= pp3_steps(d, cell, grid * std::min(cap, slices), di.cus)) &&
                   x3_slots <= a.w.scratch - a.w.P && d.L * x3_slots <= a.w.flags - a.w.xchg && !overlap(a.x, TB * (size_t)d.I, a.y, TB * (size_t)d.H);
  if (pp3) {
    CK(keep_state(a.h0, a.hT, a.cT, (size_t)d.L * d.B * d.H, a.ws, a.w, 0, s), "keep h0");
    CK(keep_state(a.c0, a.hT, a.cT, (size_t)d.L * d.B * d.H, a.ws, a.w, 1, s), "keep c0");
  }
  if (!x_in_kernel) {
    ProfScope ps(LSTM_PHASE_FWD_INPUT_GEMM, s);
    GemmProblem p{a.x, a.W, P0, (int)TB, (int)G, d.I, d.I, 1, 1, d.I, (long)G, 0};
    CK(launch_gemm_group(&p, 1, s, hx, a.w.flags - a.w.xchg), "input projection GEMM (layer 0)");
  }
  PersFwdArgs k;
  k.xin = x_in_kernel ? P0 : nullptr;
  k.keep = a.inference ? 0 : 1;
  k.dummy = reinterpret_cast<float*>(a.ws + a.w.scratch);
  k.W = a.W; k.R = a.R; k.bias = a.b; k.P0 = P0; k.c0 = a.c0; k.h0 = a.h0; k.hx = hx; k.flags = flags; k.watchdog = g_watch_dev;
  k.res = a.reserve; k.y = a.y; k.hT = a.hT; k.cT = a.cT;
  k.L = d.L; k.T = d.T; k.B = d.B; k.I = d.I; k.H = d.H; k.has_h0 = a.h0 != nullptr; k.spin_limit = spin_limit();
  k.full_fences = full_fences();
  k.trace = (g_trace_bytes >= (size_t)d.T * 64 * (pp ? 2 : 1)) ? g_trace_buf : nullptr;
  k.trace_block = g_trace_block;
  for (int s0 = 0; s0 < slices; s0 += cap) {
    const int nsl = slices - s0 < cap ? slices - s0 : cap;
    k.b0 = slice_rows * s0;
    k.nsl = nsl;
    {
      ProfScope ps(LSTM_PHASE_FWD_PACK, s);
      const size_t counter_ints = pp ? (size_t)2 * (d.H / 16) * kFlagStride : (size_t)bp.NC * kFlagInts;
      const size_t counters = (size_t)nsl * d.L * (d.T + 1) * counter_ints;
      k.redo = pp3 ? flags + counters : nullptr;  // (the counters of these kernels take half of their area)
      CK(launch_fill_zero(flags, (counters + (pp3 ? 32 : 0)) * 4, s), "zero step counters");
      if (pp3) {
        CK(launch_pack_state_pp3(a.h0, hx, d.L, d.T, d.B, d.H, k.b0, nsl, s), "pack h0");
        CK(launch_pack_x_pp3(a.x, P0, d.T, d.B, d.I, d.H, k.b0, nsl, s), "pack x");
      } else if (pp) {
        CK(launch_pack_state_pp(a.h0, hx, d.L, d.T, d.B, d.H, k.b0, nsl, s), "pack h0");
        if (x_in_kernel) CK(launch_pack_x_pp(a.x, P0, d.T, d.B, d.I, d.H, k.b0, nsl, s), "pack x");
      } else if (wide) {
        CK(launch_pack_state32(a.h0, hx, d.L, d.T, d.B, d.H, k.b0, nsl, s), "pack h0");
        if (x_in_kernel) {
          CK(launch_pack_x32(a.x, P0, flags, d.L, d.T, d.B, d.H, k.b0, nsl, d.H / 8, s), "pack x");
        }
      } else if (a.h0) {
        CK(launch_pack_state(a.h0, hx, d.L, d.T, d.B, d.H, BP, bp.NC, k.b0, nsl, s), "pack h0");
      }
    }
    ProfScope ps(LSTM_PHASE_FWD_RECURRENCE, s);
    {  // recurrent products of every layer, input products of the layers above the first, and layer 0's when x is multiplied in the kernel
      const double rows = std::min(slice_rows * nsl, d.B - k.b0), per = 2.0 * G * rows * d.T;
      prof_flops(per * d.H * (2 * d.L - 1) + (x_in_kernel ? per * d.I : 0.0),
                 pp3 ? "pers_fwd_pp3_kernel" : pp ? "pers_fwd_pp_kernel" : (wide ? "pers_fwd32_kernel" : "pers_fwd_kernel"));
    }
    hipError_t e = hipErrorInvalidValue;
    if (pp3) {
      e = launch_fwd_pp3(cell, d.H, grid * nsl, k, s);
      // an infinite or NaN sum has no parts: the fp32 kernel runs the launch again (both end at once if nobody asked)
      if (e == hipSuccess) e = force_redo(k.redo, s);
      if (e == hipSuccess) e = launch_redo_fwd_pp(k, a.x, nsl * d.L * (d.T + 1) * 2 * (d.H / 16) * kFlagStride, s);
      if (e == hipSuccess) e = launch_fwd_pp(cell, d.H, grid * nsl, k, s);
    } else if (pp) e = launch_fwd_pp(cell, d.H, grid * nsl, k, s);
    else if (wide) e = launch_fwd_wide(cell, d.H, grid * nsl, k, s);
    else e = launch_fwd_narrow(d.H, bp, grid * nsl, k, s);
    CK(e, "persistent forward launch");
  }
  return LSTM_OK;
}

// cell as in run_forward_persistent.  For the other cells the function stops after the propagation (gate gradients
// [L][T*B][4H] at the start of the workspace: GRU r, z, n, and n times r; single gate: the first H columns) and
// reports in *bias_done whether db is complete; the caller forms the weight gradients.
int run_backward_persistent(const BwdArgs& a, int cell, bool* bias_done, LayerGradients* lg) {
  const Dims& d = a.d;
  const int near_per = near_large_layers(d, cell, true);
  if (!near_per && persistent_large(d, true)) {
    if (!ensure_watchdog()) return LSTM_HIP_ERROR;
    return run_backward_persistent_large(a, cell, bias_done, lg);
  }
  const int per = near_per ? near_per : layers_per_launch(d);
  if (per <= 0) return LSTM_UNSUPPORTED;
  if (d.L <= per) return backward_layers(a, cell, bias_done, true);
  const size_t TB = (size_t)d.T * d.B, BH = (size_t)d.B * d.H, GW = (size_t)gates_of_cell(cell) * d.H;
  const size_t rstride = res_width(cell) * TB * d.H;
  const int ngroups = (d.L + per - 1) / per;
  bool all_bias = true;
  for (int gi = ngroups - 1; gi >= 0; --gi) {  // top group first
    const int g0 = gi * per;
    BwdArgs g = a;
    g.d.L = d.L - g0 < per ? d.L - g0 : per;
    const int above = g0 + g.d.L;  // first layer of the group above, if any
    // the gradient handed from group to group lives in the hand-over array of the workspace, slot = receiving layer + 1
    float* const handover = reinterpret_cast<float*>(a.ws + a.w.dx);
    if (g0 > 0) {
      g.d.I = d.H;
      g.x = a.reserve + (size_t)(g0 - 1) * rstride + res_h_offset(cell, TB, d.H);
      g.W = a.W + GW * d.I + (size_t)(g0 - 1) * GW * d.H;
      g.dx = handover + (size_t)g0 * TB * d.H;
    }
    if (above < d.L) g.dy = handover + (size_t)above * TB * d.H;
    g.R = a.R + (size_t)g0 * GW * d.H;
    g.h0 = a.h0 ? a.h0 + (size_t)g0 * BH : nullptr;
    g.c0 = a.c0 ? a.c0 + (size_t)g0 * BH : nullptr;
    g.dhT = a.dhT ? a.dhT + (size_t)g0 * BH : nullptr;
    g.dcT = a.dcT ? a.dcT + (size_t)g0 * BH : nullptr;
    g.dh0 = a.dh0 ? a.dh0 + (size_t)g0 * BH : nullptr;
    g.dc0 = a.dc0 ? a.dc0 + (size_t)g0 * BH : nullptr;
    g.db = a.db ? a.db + (size_t)g0 * GW : nullptr;
    g.reserve = a.reserve + (size_t)g0 * rstride;
    g.w.P = a.w.P + (size_t)g0 * TB * 4 * d.H * sizeof(float);   // gate gradients of the group's layers, in place
    g.w.dx = a.w.dx + (size_t)g0 * TB * d.H * sizeof(float);
    bool done = false;
    const int st = backward_layers(g, cell, &done, false);
    if (st != LSTM_OK) return st;
    all_bias = all_bias && done;
  }
  if (bias_done) *bias_done = all_bias;
  if (cell != 0) return LSTM_OK;
  return weight_gradients(a, reinterpret_cast<const float*>(a.ws + a.w.P), true, all_bias);
}

int backward_layers(const BwdArgs& a, int cell, bool* bias_done, bool with_weight_gradients) {
  const Dims& d = a.d;
  const size_t TB = (size_t)d.T * d.B, G = 4 * (size_t)d.H, GW = (cell == 0 ? 4 : (cell == 1 ? 3 : 1)) * (size_t)d.H;
  hipStream_t s = a.stream;
  if (!ensure_watchdog()) return LSTM_HIP_ERROR;
  const int slice_rows_narrow = narrow_slice_rows(d, cell, knobs().bwd_narrow, true);
  const bool narrow_slices = slice_rows_narrow > 0;
  const BatchPlan bp = narrow_slices ? BatchPlan{slice_rows_narrow / 16, 1} : batch_plan(d.B);
  const bool wide = cell != 0 || (!narrow_slices && bwd_wide(d));
  int* flags = reinterpret_cast<int*>(a.ws + a.w.flags);
  float* dA = reinterpret_cast<float*>(a.ws + a.w.P);
  if (tiny_path(d, cell)) {
    PersBwdArgs k{};
    k.W = a.W; k.R = a.R; k.res = a.reserve; k.c0 = a.c0; k.dy = a.dy; k.dhT = a.dhT; k.dcT = a.dcT;
    k.dA = dA; k.dAx = reinterpret_cast<float*>(a.ws + a.w.xchg); k.dxbuf = reinterpret_cast<float*>(a.ws + a.w.dx);
    k.dh0 = a.dh0; k.dc0 = a.dc0; k.watchdog = g_watch_dev;
    k.dx0 = (a.dx && d.I == d.H) ? a.dx : nullptr;
    k.db = a.db;  // every element written by the one lane that owns the unit
    k.L = d.L; k.T = d.T; k.B = d.B; k.I = d.I; k.H = d.H; k.spin_limit = spin_limit(); k.full_fences = full_fences();
    k.trace = (g_trace_bytes >= (size_t)d.T * 64) ? g_trace_buf : nullptr;
    k.trace_block = g_trace_block;
    {
      ProfScope ps(LSTM_PHASE_BWD_RECURRENCE, s);
      const double per = 2.0 * G * d.T;
      prof_flops(per * d.H * (2 * d.L - 1) + (k.dx0 ? per * d.I : 0.0), "pers_bwd_tiny_kernel");
      CK(launch_bwd_tiny(d.H, k, s), "persistent backward launch (single sequence)");
    }
    if (a.dx && !k.dx0) {  // layer 0's input gradient: all T steps in one product
      ProfScope ps(LSTM_PHASE_BWD_INPUT_GEMM, s);
      GemmProblem p{dA, a.W, a.dx, (int)TB, d.I, (int)GW, (long)G, 1, d.I, 1, d.I, 0};
      CK(launch_gemm_group(&p, 1, s, reinterpret_cast<float*>(a.ws + a.w.xchg), a.w.flags - a.w.xchg), "input-gradient GEMM (layer 0)");
    }
    if (bias_done) *bias_done = a.db != nullptr;
    if (!with_weight_gradients) return LSTM_OK;
    return weight_gradients(a, dA, true, a.db != nullptr);
  }
  if (const NearPlan np = near_plan(d, cell, true); np.units) {
    PersBwdArgs k{};
    k.W = a.W; k.R = a.R; k.res = a.reserve; k.c0 = a.c0; k.h0 = a.h0; k.dy = a.dy; k.dhT = a.dhT; k.dcT = a.dcT;
    k.dA = dA; k.dAx = reinterpret_cast<float*>(a.ws + a.w.xchg); k.dxbuf = reinterpret_cast<float*>(a.ws + a.w.dx);
    k.dh0 = a.dh0; k.dc0 = a.dc0; k.watchdog = g_watch_dev;
    k.dx0 = (a.dx && d.I == d.H) ? a.dx : nullptr;
    k.db = np.slices > 1 && a.db ? reinterpret_cast<float*>(a.ws + a.w.dbpart) : a.db;
    k.L = d.L; k.T = d.T; k.B = d.B; k.I = d.I; k.H = d.H; k.spin_limit = spin_limit(); k.full_fences = full_fences();
    k.spread = np.spread;
    k.trace = (g_trace_bytes >= (size_t)d.T * 64) ? g_trace_buf : nullptr;
    k.trace_block = g_trace_block;
    {
      ProfScope ps(LSTM_PHASE_BWD_RECURRENCE, s);
      const double per = 2.0 * GW * d.B * d.T;
      prof_flops(per * d.H * (2 * d.L - 1) + (k.dx0 ? per * d.I : 0.0), "pers_bwd_near_kernel");
      for (int s0 = 0; s0 < np.slices; s0 += np.side) {
        k.b0 = 16 * s0;
        k.nsl = std::min(np.side, np.slices - s0);
        CK(launch_bwd_near(cell, d.H, np.units, k, s), "persistent backward launch (slices of 16 rows)");
      }
    }
    if (k.db != a.db) {
      ProfScope ps(LSTM_PHASE_BIAS_GRAD, s);
      CK(launch_near_bias(k.db, a.db, d.L, np.slices, d.H, gates_of_cell(cell), s), "bias gradient");
    }
    if (a.dx && !k.dx0) {  // layer 0's input gradient: all T steps in one product
      ProfScope ps(LSTM_PHASE_BWD_INPUT_GEMM, s);
      GemmProblem p{dA, a.W, a.dx, (int)TB, d.I, (int)GW, (long)G, 1, d.I, 1, d.I, 0};
      CK(launch_gemm_group(&p, 1, s, reinterpret_cast<float*>(a.ws + a.w.xchg), a.w.flags - a.w.xchg), "input-gradient GEMM (layer 0)");
    }
    if (bias_done) *bias_done = a.db != nullptr;
    if (cell != 0 || !with_weight_gradients) return LSTM_OK;
    return weight_gradients(a, dA, true, a.db != nullptr);
  }
  PersBwdArgs k;
  k.W = a.W; k.R = a.R; k.res = a.reserve; k.c0 = a.c0; k.h0 = a.h0; k.dy = a.dy; k.dhT = a.dhT; k.dcT = a.dcT;
  k.dA = dA; k.dAx = reinterpret_cast<float*>(a.ws + a.w.xchg); k.dxbuf = reinterpret_cast<float*>(a.ws + a.w.dx);
  k.dh0 = a.dh0; k.dc0 = a.dc0; k.flags = flags; k.watchdog = g_watch_dev;
  // With I == H layer 0 is like every other layer: its workgroups also multiply by W_0 (the rows of the
  // MFMA tile that would otherwise hold zeros) and write the gradient of the network input themselves.
  k.dx0 = (a.dx && d.I == d.H) ? a.dx : nullptr;
  k.db = nullptr;
  if (wide && a.db && d.B <= 64) {  // one launch: the wide kernel adds the bias gradient into db itself (two addends per element)
    ProfScope ps(LSTM_PHASE_BIAS_GRAD, s);
    CK(launch_fill_zero(a.db, (size_t)d.L * GW * 4, s), "zero db");
    k.db = a.db;
  }
  k.L = d.L; k.T = d.T; k.B = d.B; k.I = d.I; k.H = d.H; k.spin_limit = spin_limit(); k.full_fences = full_fences();
  // two alternating chains per workgroup: counters of H/16 lines per (layer, step, quarter)
  const bool pp = bwd_alternating(d, cell);
  // (a line of 128 bytes per workgroup, L * H/16 * 2 slices of them, in the reserve stand-in, 24 bytes per unit, layer, step
  // and row, which a backward call does not use otherwise)
  k.dummy = reinterpret_cast<float*>(a.ws + a.w.resv);
  k.trace = (g_trace_bytes >= (size_t)d.T * 64 * (pp ? 2 : 1)) ? g_trace_buf : nullptr;
  k.trace_block = g_trace_block;
  const int grid = d.L * (d.H / 8);
  // slices of 64 batch rows side by side while the CUs last (see run_forward_persistent): for the wide kernel a
  // slice is two more "batch halves" of 32 rows with their own exchange slots and counters
  DeviceInfo di;
  (void)device_info(di);
  int cap = (wide || narrow_slices) && grid > 0 ? di.cus / grid : 1;
  if (cap > 16 / d.L) cap = 16 / d.L;
  if (cap < 1) cap = 1;
  const int slice_rows = narrow_slices ? slice_rows_narrow : 64;
  const int slices = wide ? (d.B + 63) / 64 : (narrow_slices ? (d.B + slice_rows - 1) / slice_rows : 1);
  for (int s0 = 0; s0 < slices; s0 += cap) {
    const int nsl = slices - s0 < cap ? slices - s0 : cap;
    k.b0 = slice_rows * s0;
    {
      ProfScope ps(LSTM_PHASE_BWD_PACK, s);
      const size_t per_slot = pp ? (size_t)4 * (d.H / 16) * kFlagStride : (size_t)2 * kFlagInts;  // ints per (slice, layer, step)
      CK(launch_fill_zero(flags, (size_t)nsl * d.L * (d.T + 2) * per_slot * 4, s), "zero step counters");
    }
    ProfScope ps(LSTM_PHASE_BWD_RECURRENCE, s);
    {  // dh products of every layer, dx products of the layers above the first, and layer 0's when the kernel writes dx itself
      const double rows = std::min(slice_rows * nsl, d.B - k.b0), per = 2.0 * GW * rows * d.T;
      prof_flops(per * d.H * (2 * d.L - 1) + (k.dx0 ? per * d.I : 0.0), pp ? "pers_bwd_pp_kernel" : (wide ? "pers_bwd32_kernel" : "pers_bwd_kernel"));
    }
    hipError_t e = hipErrorInvalidValue;
    if (pp) e = launch_bwd_pp(cell, d.H, k, 2 * nsl, s);
    else if (wide) e = launch_bwd_wide(cell, d.H, k, 2 * nsl, s);
    else e = launch_bwd_narrow(d.H, bp, grid * nsl, k, s);
    CK(e, "persistent backward launch");
  }
  if (a.dx && !k.dx0) {  // layer 0's input gradient: all T steps in one product
    ProfScope ps(LSTM_PHASE_BWD_INPUT_GEMM, s);
    GemmProblem p{dA, a.W, a.dx, (int)TB, d.I, (int)GW, (long)G, 1, d.I, 1, d.I, 0};
    CK(launch_gemm_group(&p, 1, s, reinterpret_cast<float*>(a.ws + a.w.xchg), a.w.flags - a.w.xchg), "input-gradient GEMM (layer 0)");
  }
  if (bias_done) *bias_done = k.db != nullptr;
  if (cell != 0 || !with_weight_gradients) return LSTM_OK;
  return weight_gradients(a, dA, true, k.db != nullptr);
}

}  // namespace lstm
