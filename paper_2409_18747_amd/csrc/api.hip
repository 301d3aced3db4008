// C-ABI entry points of libcottn: argument validation (before anything is enqueued, so it
// works on a host without a GPU), the host-side choice of the sequence split, dispatch to
// the per-dtype kernel launchers, and the optional per-kernel event timing.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <cstring>
#include <mutex>
#include <string>
#include <vector>

#include "../../include/cottn.h"
#include "launch.h"
#include "workspace.h"

namespace cottn {
namespace {

// <= 0: heuristic.  Per thread: a thread that tunes does not change what other threads get.
thread_local int g_tuned_segments = 0;

// ---- profiling state -------------------------------------------------------------------
struct PendingSpan { const char* name; hipEvent_t begin, end; };
struct KernelTotal { const char* name; long launches; double ms; };
bool g_profile_on = false;
std::vector<PendingSpan> g_pending;
std::vector<KernelTotal> g_totals;

bool is_aligned(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }

bool dim_ok(int d) { return d == 32 || d == 64 || d == 128; }

bool dims_ok(int B, int H, int N, int dk, int dv) {
  if (B < 1 || H < 1 || N < 0) return false;
  if (!dim_ok(dk) || !dim_ok(dv)) return false;
  // element counts must fit comfortably in 64-bit offsets and the grid in 31 bits
  if (double(B) * H > 16777216.0) return false;
  if (double(B) * H * double(N) * (dk > dv ? dk : dv) > 9.0e15) return false;
  return true;
}

constexpr int kComputeUnits = 256;

// What a causal forward and its backward take with g segments, in microseconds, by a model of the
// kernels: the split is the one for which this is least.
//   - A chunk step of the three scans takes `step`, as the rows are wide.  A workgroup walks its steps
//     and pays over two more to start (first rows, stored states).  The compute unit with the most
//     workgroups ends last; of `at_once` at a time each further one adds `next_one` of a step.  But the
//     rows have to come through memory, 0.86 us for every MB of Q and V.
//   - More than one segment costs the totals kernel, and the totals have to be added up, by every
//     workgroup (three scans read them), or by carry launches, which walk the segments one batch of
//     states after the other and move all of them.
// Fitted to the times of 3700 shapes (1 to 1280 units of 128 to 65536 rows, all pairs of widths, the splits
// that put up to 1300 workgroups on the chip) so that neither the forward alone nor the pair is far from
// its best: the split chosen takes 0.6 % (geometric mean of the two) longer than the best one.  At 16-bit 128 x
// 128 the totals weigh more with the pair, which a fit to both alike cut too coarsely (14 units of 777 rows 5
// segments 21 / 56 us, 13 segments 26 / 45; 2 units of 8192 rows 43 segments 29 / 68, 64 29 / 60).
double causal_call_us(long units, long N, long n_chunks, long g, int dtype, int dk, int dv) {
  const bool f32 = dtype == COTTN_F32, narrowest = dk == 32 && dv == 32, widest = dk == 128 && dv == 128;
  const int big = dk > dv ? dk : dv, small = dk > dv ? dv : dk;
  const long at_once = narrowest ? 4 : (f32 ? big == 128 && small >= 64 : widest) ? 1 : 2;
  const double next_one = f32 ? (narrowest ? 0.2 : 0.38) : narrowest ? 0.05 : 0.24;
  const double step = (f32 ? 0.07 : widest ? 0.0265 : 0.041) * (dk + dv);
  const long steps = (n_chunks + g - 1) / g, on_cu = (units * g + kComputeUnits - 1) / kComputeUnits;
  const auto together = [&](long n) { return n > 0 ? 1.0 + next_one * double(n - 1) : 0.0; };
  double us = step * (double(steps) + 2.2) * (double(on_cu / at_once) * together(at_once) + together(on_cu % at_once));
  const double rows_us = 0.86e-6 * double(units) * double(N) * (dk + dv) * (f32 ? 4 : 2);
  if (us < rows_us) us = rows_us;
  if (g > 1) {
    const double state = double(dk) * dv * 4.0 / 1024.0;   // KB
    us += 5.8 + 0.135 * step * double(steps * on_cu);
    const bool wide = widest && !f32;
    us += causal_totals_in_place(units, int(g), dk, dv, f32)
              ? (wide ? 0.037 : 0.026) * (state + 7.0) * double(g - 1)
              : (wide ? 9.0 + 0.2 * double(g) : 8.0 + 0.3 * double(g)) + 0.001 * state * double(units * g);
  }
  return us;
}

// Segments per (batch, head) for the causal calls: the least time by the model among the splits of up to
// 640 workgroups (1024 for fp32, whose scans hold the longer steps, and for 32 x 32, of which a compute
// unit runs four; 768 where both hold, whose dK/dV scan it runs three of: 64 units of 2048 rows 8 segments 24 /
// 70 us, 16 25 / 77), or none.  Finer ones gain the backward little and cost the forward, which runs three
// workgroups or more at once, a round (768 units of 1024 rows at 64 x 64: 2 segments 87 / 291 us for the
// forward / with its backward, 1 segment 64 / 270).  Others of the measured, forward / with backward: 16-bit
// 128 x 128 8 units of 2048 rows 32 segments 30 / 55 us, 16 27 / 51, 8 29 / 71; 64 x 64 64 units of 2048
// rows 6 segments 24 / 66, 8 22 / 59; 176 units of 600 rows 3 segments 19.8 / 61, 2 22.0 / 58, 1 17.8 / 62;
// fp32 40 units of 1024 rows 8 segments 33 / 94, 11 29 / 80.  Where the line costs most: 128 x 128 320 units
// of 2048 rows 2 segments 180 / 652 us, 1 167 / 645, but 3, which it leaves out, 186 / 611.
// No split at all leaves the backward waiting where units are few: up to 160 16-bit units of more than four
// chunks (of 32 x 32 fewer than 384 of more than eight) take at least two segments, but at 128 x 128, where
// one unit fills a compute unit (160 units of 300 rows at 64 x 32: 3 segments 10.0 / 26 us, 1 segment 9.1
// / 32; 352 units of 2048 rows at 32 x 32: 2 segments 41 / 125, 1 segment 37 / 136).
// (Chunks of more than 64 rows, which are for experiments: one and a half workgroups per compute unit,
// two for long chains.)
long causal_segments(long units, long N, long n_chunks, int C, int dtype, int dk, int dv) {
  if (C > 64) {
    const long want = (384 + units - 1) / units;
    return n_chunks >= 16 * want ? (512 + units - 1) / units : want;
  }
  const bool f32 = dtype == COTTN_F32, narrowest = dk == 32 && dv == 32, widest = dk == 128 && dv == 128;
  const long most = f32 && narrowest ? 768 : f32 || narrowest ? 1024 : 640;
  const bool cut = !f32 && !widest && ((n_chunks > 4 && units <= 160) || (narrowest && n_chunks > 8 && units < 384));
  double best = causal_call_us(units, N, n_chunks, 1, dtype, dk, dv);
  long best_g = 1;
  for (long steps = n_chunks - 1; steps >= 1; --steps) {
    // (only the counts that give different splits: about 2 sqrt(n_chunks) of them)
    const long g = (n_chunks + steps - 1) / steps;
    steps = (n_chunks + g - 1) / g;
    if (units * g > most) break;
    const double us = causal_call_us(units, N, n_chunks, g, dtype, dk, dv);
    if (us < best || (cut && best_g == 1)) {
      best = us;
      best_g = g;
    }
  }
  return best_g;
}

// Chunks per workgroup where a causal call walks even shares (workspace.h) instead of G segments per unit,
// or 0.  A split leaves compute units idle where units do not divide by them: 96 units at 128 x 128, of which a
// compute unit runs one workgroup, are 192 workgroups of 8 steps, or 256 shares of 6.  A share that goes on into the
// next unit costs little (its rows are prefetched across the boundary, its state starts from zero), but there are
// totals to form, also where one segment had none, and more of them to add up: 3 and 4 steps' worth of
// prologue in the comparison below, which was fitted to 360 shapes of 12 to 1100 units.
//   Forward / with backward, segments -> shares: 16-bit 128 x 128 96 units of 1024 rows 36 / 117 -> 34 / 106 us, 68 of
// 5010 117 / 379 -> 103 / 324, 272 of 1024 93 / 318 -> 80 / 261, 528 of 1464 219 / 818 -> 191 / 688; fp32 64 x 64 96
// units of 1024 rows 43 / 130 -> 38 / 120, 129 of 816 53 / 147 -> 47 / 127, 282 of 571 69 / 198 -> 59 / 173; 128 x 128
// 543 of 442 325 / 1219 -> 278 / 953; 64 x 128 308 of 582 168 / 502 -> 133 / 412.
//   Not where it does not pay: 16-bit shapes of two workgroups to a compute unit, which wait for memory more than for
// the fullest compute unit (64 x 64 96 units of 1024 rows 52.8 -> 51.9 us, 226 of 4238 at 128 x 64 167 / 599 -> 191 /
// 624); one segment per unit that fits the chip at once, where a forward has no totals to form (fp32 64 x 128 220
// units of 1719 rows 194 / 781 -> 277 / 849), or nearly (fp32 64 x 64 588 of 2516 439 / 1711 -> 472 / 1541).
long causal_even_share(long units, long n_chunks, long G, int dtype, int dk, int dv) {
  const bool f32 = dtype == COTTN_F32;
  if (!even_shares_built(dk, dv, f32)) return 0;
  const long at_once = f32 && dk == 64 && dv == 64 ? 2 : 1, places = at_once * kComputeUnits;
  const long share = (units * n_chunks + places - 1) / places;
  if (share < 3 || !causal_totals_in_place(units, int((n_chunks + share - 1) / share) + 1, dk, dv, f32)) return 0;
  const long workgroups = units * G, steps = (n_chunks + G - 1) / G;
  double rounds = 1.0;   // of the segments, as long as `steps` each
  if (workgroups <= places) {
    if (G == 1 || workgroups <= kComputeUnits * (at_once - 1)) return 0;
  } else if (f32) {
    if (at_once == 2 && G == 1) return 0;
    rounds = double((workgroups + places - 1) / places);
  } else {   // two to a compute unit then (launch.h: two_to_a_cu_forward)
    if (workgroups > 640 || (workgroups <= 512 && G == 1)) return 0;
    rounds = workgroups <= 512 ? 1.5 : 2.5;
  }
  const double gain = (rounds * double(steps) + 3.0) / (double(share) + (at_once == 2 ? 3.0 : 4.0));
  return gain >= (at_once == 2 ? 1.08 : 1.05) ? share : 0;
}

// Segments per (batch, head) for the bidirectional calls.  Their kernels have no chain to
// shorten and little to set up: about three workgroups per compute unit measured best (B24 H8 N3000
// d64, forward + backward: 155 us with 4 segments, 169 with 2), in at most four segments, whose
// totals are soon added up.  Two fit a compute unit at a time, so 193 to 256 units take two
// segments (B32 H8 N2048: 137 us, 151 us with 3), and with 342 units and more three are the start of a
// third round, which long sequences feel (352 units of 8192 rows at 32 x 32: 2 segments 146 / 391 us
// for the forward / with its backward, 3 segments 164 / 422).  At 128 x 128 one workgroup fills a
// compute unit (B8 H12 N1024 2 segments 90 us, 3 segments 114), and so it does in the dQ sweep of 16-bit
// rows with 128 and 64 or 128 and 32 columns (B16 H8 N1024 64 x 128 2 segments 62 us, 4 segments
// 73; from 129 units on, where that leaves one, four are the better again); a little more than one
// for each takes two, which even the second round out (320 units of 2048 rows: 1 segment 185 / 560 us, 2
// segments 174 / 485).  Few units with long sequences are cut further, until (nearly) every compute unit
// has a workgroup and none has two: B1 H2 N65536 128 segments 74 us, 64 segments 84;
// B1 H12 N8192 16 segments 43 us, 32 segments 53; two for the longest at 16-bit 32 x 32, of which it
// runs four (24 units of 65536 rows: 10 segments 104 / 231 us, 20 segments 73 / 206).
long bidir_segments(long units, long N, bool f32, int dk, int dv) {
  const bool widest = dk == 128 && dv == 128, narrowest = dk == 32 && dv == 32;
  const bool one_per_cu = widest || (!f32 && units <= kComputeUnits / 2 && (dk == 128 || (dk == 64 && dv == 128)));
  long want = one_per_cu ? kComputeUnits / units : (3 * kComputeUnits + units - 1) / units;
  if (units > 192 && units <= 256 && want > 2) want = 2;
  if (units > 341 && N >= 2048 && want > 2) want = 2;
  if (!f32 && widest && units > 256 && units <= 320 && N > 1024) want = 2;
  if (want > 4) want = 4;
  if (units * want < kComputeUnits && N > 512 * want - 64) {
    want = kComputeUnits / units;
    if (!f32 && narrowest && N > 4096 * want) want *= 2;
    if (want > N / 128) want = N / 128;   // at least 128 rows each
  }
  return want;
}

}  // namespace

// Split of one (batch, head) sequence into segments; see workspace.h.
bool make_plan(int op, int B, int H, int N, int dk, int dv, int chunk, int dtype, SeqPlan* plan,
               long most_segments) {
  if (dtype != COTTN_F32 && dtype != COTTN_BF16 && dtype != COTTN_F16) return false;
  if (!dims_ok(B, H, N, dk, dv)) return false;
  int C;
  if (dtype != COTTN_F32) {
    C = chunk == 0 ? 64 : chunk;
    if (C != 64 && C != 128 && C != 256) return false;
    // the larger chunks are built for d_key = d_value in {32, 64}
    if ((dk == 128 || dv == 128 || dk != dv) && C != 64) return false;
  } else {
    C = chunk == 0 ? 32 : chunk;
    if (C != 32) return false;
  }
  // (the bidirectional kernels have no quadratic part inside a chunk)
  if (op == COTTN_OP_FWD_BIDIR || op == COTTN_OP_BWD_BIDIR) C = bidir_step_rows(dtype == COTTN_F32);
  const long units = long(B) * H;
  long n_chunks = (long(N) + C - 1) / C;
  const bool bidir = op == COTTN_OP_FWD_BIDIR || op == COTTN_OP_BWD_BIDIR;
  long want = g_tuned_segments;
  plan->by_unit = want <= 0 && bidir && bidir_by_unit(units, N, dtype == COTTN_F32, dk, dv);
  if (want <= 0) {
    want = bidir ? bidir_segments(units, N, dtype == COTTN_F32, dk, dv) : causal_segments(units, N, n_chunks, C, dtype, dk, dv);
    if (most_segments > 0 && want > most_segments) want = most_segments;
  }
  if (want > n_chunks) want = n_chunks;
  if (want < 1) want = 1;
  if (bidir && !threads_fit(units * want, 4 * C)) {
    C = 64;
    plan->by_unit = false;
    n_chunks = (long(N) + C - 1) / C;
  }
  const long chunks_per_seg = n_chunks > 0 ? (n_chunks + want - 1) / want : 1;
  const long G = n_chunks > 0 ? (n_chunks + chunks_per_seg - 1) / chunks_per_seg : 1;
  if (units * G > 2147483647L / 4) return false;
  plan->C = C;
  plan->G = plan->by_unit ? 1 : int(G);
  plan->seg_rows = int((plan->by_unit ? n_chunks : chunks_per_seg) * C);
  plan->even_rows = 0;
  plan->own_prefix = !bidir && C <= 64 && own_prefix(units, int(G), plan->seg_rows, dk, dv, dtype == COTTN_F32);
  plan->slots = G > 1 ? units * G : 0;
  plan->pieces = units * G;
  if (!bidir && g_tuned_segments <= 0 && most_segments <= 0 && C <= 64 && n_chunks > 0) {
    const long share = causal_even_share(units, n_chunks, G, dtype, dk, dv);
    if (share > 0 && (units * n_chunks + share) * C < (1L << 31)) {
      const long workgroups = (units * n_chunks + share - 1) / share;
      plan->even_rows = int(share * C);
      if (plan->slots < workgroups) plan->slots = workgroups;
      if (plan->pieces < workgroups + units) plan->pieces = workgroups + units;
    }
  }
  return true;
}

namespace {

// The walk of a causal call: even shares where the plan has them, also for a padded batch (96 units of 1024
// rows at most, 16-bit 128 x 128, lengths spread evenly from a quarter of that: forward + backward 107 -> 101 us against
// segments, 272 units 287 -> 250 (with the forward alone 33 -> 37 and 93 -> 81), 68 of 5010 373 -> 322; fp32 64 x 64 282 of 571 170 -> 165), but where sequences
// are one segment each: those of a padded batch end early and make room for others, which shares of rows
// that may not exist do not (528 of 1464 515 -> 661 us, fp32 128 x 128 543 of 442 911 -> 924).
void set_walk(CausalArgs* a, const SeqPlan& plan) {
  const long units = long(a->B) * a->H;
  const bool even = plan.even_rows > 0 && (a->seq_len == nullptr || plan.G > 1);
  a->marked = plan.even_rows > 0 && plan.G == 1;
  a->C = plan.C;
  a->G = plan.G;
  a->slots = plan.slots;
  a->own_prefix = !even && plan.own_prefix;
  a->unit_rows = even ? (a->N + plan.C - 1) / plan.C * plan.C : 0;
  a->seg_rows = even ? plan.even_rows : plan.seg_rows;
  a->workgroups = int(even ? (units * a->unit_rows + a->seg_rows - 1) / a->seg_rows : units * plan.G);
}

}  // namespace

bool profile_on() { return g_profile_on; }

void profile_events(const char* kernel_name, hipEvent_t* begin, hipEvent_t* end) {
  PendingSpan sp{kernel_name, nullptr, nullptr};
  if (hipEventCreate(&sp.begin) != hipSuccess) return;
  if (hipEventCreate(&sp.end) != hipSuccess) {
    (void)hipEventDestroy(sp.begin);
    return;
  }
  g_pending.push_back(sp);
  *begin = sp.begin;
  *end = sp.end;
}

namespace {

__global__ void fill_zero_f32(float* p, long n) {
  const long i = long(blockIdx.x) * 256 + threadIdx.x;
  if (i < n) p[i] = 0.f;
}

hipError_t zero_f32(float* p, long n, hipStream_t st) {
  if (p == nullptr || n <= 0) return hipSuccess;
  return launch_kernel("fill_zero_f32", fill_zero_f32, dim3(unsigned((n + 255) / 256)), dim3(256),
                       0, st, p, n);
}

int check_common(const void* const* ptrs, int n_ptrs, int B, int H, int N, int dk, int dv,
                 int dtype, float eps) {
  for (int i = 0; i < n_ptrs; ++i)
    if (ptrs[i] == nullptr) return COTTN_E_NULL;
  if (dtype != COTTN_F32 && dtype != COTTN_BF16 && dtype != COTTN_F16) return COTTN_E_DTYPE;
  if (!dims_ok(B, H, N, dk, dv)) return COTTN_E_SHAPE;
  if (!(eps > 0.f)) return COTTN_E_ARG;
  for (int i = 0; i < n_ptrs; ++i)
    if (!is_aligned(ptrs[i], 16)) return COTTN_E_ALIGN;
  return COTTN_OK;
}

int check_workspace(const void* ws, size_t have, size_t need) {
  if (need == 0) return COTTN_OK;
  if (ws == nullptr || have < need) return COTTN_E_WORKSPACE;
  if (!is_aligned(ws, 256)) return COTTN_E_ALIGN;
  return COTTN_OK;
}

int map_hip(hipError_t e) { return e == hipSuccess ? COTTN_OK : COTTN_E_HIP; }

}  // namespace
}  // namespace cottn

using namespace cottn;

extern "C" {

size_t cottn_workspace_bytes_dkdv(int op, int B, int H, int N, int dk, int dv, int chunk,
                                  int dtype) {
  if (op == COTTN_OP_STEP) {
    return (dtype == COTTN_F32 || dtype == COTTN_BF16 || dtype == COTTN_F16) &&
                   dims_ok(B, H, 1, dk, dv)
               ? 0
               : size_t(-1);
  }
  if (op < COTTN_OP_FWD_CAUSAL || op > COTTN_OP_STEP) return size_t(-1);
  SeqPlan plan;
  if (!make_plan(op, B, H, N, dk, dv, chunk, dtype, &plan)) return size_t(-1);
  return workspace_bytes_for(op, B, H, dk, dv, plan);
}

size_t cottn_workspace_bytes(int op, int B, int H, int N, int d, int chunk, int dtype) {
  return cottn_workspace_bytes_dkdv(op, B, H, N, d, d, chunk, dtype);
}

int cottn_segments_dkdv(int op, int B, int H, int N, int dk, int dv, int chunk, int dtype) {
  if (op < COTTN_OP_FWD_CAUSAL || op > COTTN_OP_BWD_BIDIR) return 0;
  SeqPlan plan;
  if (!make_plan(op, B, H, N, dk, dv, chunk, dtype, &plan)) return 0;
  return plan.G;
}

int cottn_segments(int op, int B, int H, int N, int d, int chunk, int dtype) {
  return cottn_segments_dkdv(op, B, H, N, d, d, chunk, dtype);
}

void cottn_tune_segments(int segments) { g_tuned_segments = segments; }

const char* cottn_status_string(int status) {
  switch (status) {
    case COTTN_OK: return "ok";
    case COTTN_E_NULL: return "a required pointer is NULL";
    case COTTN_E_SHAPE: return "unsupported shape: need B,H >= 1, N >= 0, d (d_key, d_value) in "
                               "{32,64,128}, chunk in {0,64,128,256} (16-bit; 64 only when a "
                               "dimension is 128 or d_key != d_value) or {0,32} (fp32)";
    case COTTN_E_DTYPE: return "dtype must be COTTN_F32 (0), COTTN_BF16 (1) or COTTN_F16 (2)";
    case COTTN_E_ALIGN: return "tensor pointers must be 16-byte aligned, the workspace 256-byte aligned";
    case COTTN_E_WORKSPACE: return "workspace is NULL or smaller than cottn_workspace_bytes()";
    case COTTN_E_HIP: return "a HIP call failed";
    case COTTN_E_ARG: return "invalid argument";
    default: return "unknown status";
  }
}

namespace {

__global__ void copy_f32(const float* __restrict__ src, float* __restrict__ dst, long n) {
  const long i = long(blockIdx.x) * 256 + threadIdx.x;
  if (i < n) dst[i] = src[i];
}

hipError_t copy_state(float* dst, const float* src, long n, hipStream_t st) {
  return launch_kernel("copy_f32", copy_f32, dim3(unsigned((n + 255) / 256)), dim3(256), 0, st, src,
                       dst, n);
}

// seq_len != null in the *_any functions: a padded batch, with s and ds per (batch, head)
int check_lengths(const int* seq_len) {
  return seq_len == nullptr || is_aligned(seq_len, 4) ? COTTN_OK : COTTN_E_ALIGN;
}

int fwd_causal_any(const void* Q, const void* K, const void* V, const float* s, const int* seq_len,
                   const float* state_in, void* O, float* state, void* workspace,
                   size_t workspace_bytes, int B, int H, int N, int dk, int dv, int chunk, int dtype,
                   float eps, void* hip_stream, long most_segments = 0) {
  const void* req[] = {Q, K, V, s, O};
  int st = check_common(req, 5, B, H, N, dk, dv, dtype, eps);
  if (st != COTTN_OK) return st;
  if (state != nullptr && !is_aligned(state, 16)) return COTTN_E_ALIGN;
  if (state_in != nullptr && !is_aligned(state_in, 16)) return COTTN_E_ALIGN;
  if (state_in != nullptr && state_in == state) return COTTN_E_ARG;
  if ((st = check_lengths(seq_len)) != COTTN_OK) return st;
  SeqPlan plan;
  if (!make_plan(COTTN_OP_FWD_CAUSAL, B, H, N, dk, dv, chunk, dtype, &plan, most_segments)) return COTTN_E_SHAPE;
  st = check_workspace(workspace, workspace_bytes,
                       workspace_bytes_for(COTTN_OP_FWD_CAUSAL, B, H, dk, dv, plan));
  if (st != COTTN_OK) return st;
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  if (N == 0) {
    const long n = long(B) * H * dk * dv;
    if (state == nullptr) return COTTN_OK;
    if (state_in == nullptr) return map_hip(zero_f32(state, n, stream));
    return map_hip(copy_state(state, state_in, n, stream));
  }
  CausalArgs a{};
  a.Q = Q; a.K = K; a.V = V; a.s = s; a.O = O; a.state = state; a.state_in = state_in;
  a.workspace = workspace; a.seq_len = seq_len; a.s_per_unit = seq_len != nullptr;
  a.B = B; a.H = H; a.N = N; a.dk = dk; a.dv = dv;
  set_walk(&a, plan);
  a.eps = eps; a.stream = stream;
  return map_hip(dtype == COTTN_BF16 ? fwd_causal_bf16(a) : dtype == COTTN_F16 ? fwd_causal_f16(a) : fwd_causal_f32(a));
}

}  // namespace

int cottn_fwd_causal(const void* Q, const void* K, const void* V, const float* s, void* O,
                     float* state, void* workspace, size_t workspace_bytes, int B, int H, int N,
                     int d, int chunk, int dtype, float eps, void* hip_stream) {
  return fwd_causal_any(Q, K, V, s, nullptr, nullptr, O, state, workspace, workspace_bytes, B, H, N,
                        d, d, chunk, dtype, eps, hip_stream);
}

// ---- the causal forward for callers that cannot allocate ------------------------------------
// Its workspace (the fp32 segment states) is this array, part of the library's code object: every
// GPU the library runs on holds its own copy, at its own address, until the process ends.  In
// host code the name below only stands for the symbol; the address kernels can use comes from
// hipGetSymbolAddress, asked once per device with that device current.
namespace {

static __device__ __align__(256) unsigned char scratch[COTTN_STATIC_WORKSPACE_BYTES];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices] = {};

int static_workspace(void** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return COTTN_E_HIP;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (g_scratch_ptr[dev] == nullptr) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || p == nullptr)
      return COTTN_E_HIP;
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return COTTN_OK;
}

}  // namespace

int cottn_fwd_causal_static(const void* Q, const void* K, const void* V, const float* s, void* O,
                            float* state, int B, int H, int N, int d, int chunk, int dtype,
                            float eps, void* hip_stream) {
  const void* req[] = {Q, K, V, s, O};
  int st = check_common(req, 5, B, H, N, d, d, dtype, eps);
  if (st != COTTN_OK) return st;
  SeqPlan plan;
  if (!make_plan(COTTN_OP_FWD_CAUSAL, B, H, N, d, d, chunk, dtype, &plan)) return COTTN_E_SHAPE;
  size_t need = workspace_bytes_for(COTTN_OP_FWD_CAUSAL, B, H, d, d, plan);
  // a split of the library's own whose states do not fit the array gives way to the finest that does
  // (d = 128: up to 640 workgroups, 1024 for fp32, have a state of 64 KB each)
  long most = 0;
  if (need > size_t(COTTN_STATIC_WORKSPACE_BYTES)) {
    const long most_that_fit = long(COTTN_STATIC_WORKSPACE_BYTES) / (long(B) * H * d * d * long(sizeof(float)));
    most = most_that_fit < 1 ? 1 : most_that_fit;
    if (!make_plan(COTTN_OP_FWD_CAUSAL, B, H, N, d, d, chunk, dtype, &plan, most)) return COTTN_E_SHAPE;
    need = workspace_bytes_for(COTTN_OP_FWD_CAUSAL, B, H, d, d, plan);
  }
  if (need > size_t(COTTN_STATIC_WORKSPACE_BYTES)) return COTTN_E_WORKSPACE;
  void* ws = nullptr;
  if (need > 0 && (st = static_workspace(&ws)) != COTTN_OK) return st;
  // every slot of the segment-state array that a kernel reads is written earlier in the same
  // call, so what the previous call left in the array needs no clearing
  return fwd_causal_any(Q, K, V, s, nullptr, nullptr, O, state, ws, need, B, H, N,
                        d, d, chunk, dtype, eps, hip_stream, most);
}

int cottn_fwd_causal_from_state(const void* Q, const void* K, const void* V, const float* s,
                                const float* state_in, void* O, float* state, void* workspace,
                                size_t workspace_bytes, int B, int H, int N, int d, int chunk,
                                int dtype, float eps, void* hip_stream) {
  if (state_in == nullptr) return COTTN_E_NULL;
  return fwd_causal_any(Q, K, V, s, nullptr, state_in, O, state, workspace, workspace_bytes, B, H, N,
                        d, d, chunk, dtype, eps, hip_stream);
}

namespace {

int bwd_causal_any(const void* Q, const void* K, const void* V, const float* s, const int* seq_len,
                   const void* dO, const float* state_in, const float* rev_state_in, void* dQ,
                   void* dK, void* dV, float* ds, float* rev_state_out,
                   const void* fwd_workspace, size_t fwd_workspace_bytes, void* workspace,
                   size_t workspace_bytes, int B, int H, int N, int dk, int dv, int chunk, int dtype,
                   float eps, void* hip_stream) {
  const void* req[] = {Q, K, V, s, dO, dQ, dK, dV, ds};
  int st = check_common(req, 9, B, H, N, dk, dv, dtype, eps);
  if (st != COTTN_OK) return st;
  if ((st = check_lengths(seq_len)) != COTTN_OK) return st;
  if (!is_aligned(state_in, 16) || !is_aligned(rev_state_in, 16) || !is_aligned(rev_state_out, 16))
    return COTTN_E_ALIGN;
  // workgroups read the one while others write the other
  if (rev_state_out != nullptr && rev_state_out == rev_state_in) return COTTN_E_ARG;
  SeqPlan plan;
  if (!make_plan(COTTN_OP_BWD_CAUSAL, B, H, N, dk, dv, chunk, dtype, &plan)) return COTTN_E_SHAPE;
  st = check_workspace(workspace, workspace_bytes,
                       workspace_bytes_for(COTTN_OP_BWD_CAUSAL, B, H, dk, dv, plan));
  if (st != COTTN_OK) return st;
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  if (N == 0) {
    const long n = long(B) * H * dk * dv;
    hipError_t e = zero_f32(ds, seq_len != nullptr ? long(B) * H : H, stream);
    if (e == hipSuccess && rev_state_out != nullptr)
      e = rev_state_in != nullptr ? copy_state(rev_state_out, rev_state_in, n, stream)
                                  : zero_f32(rev_state_out, n, stream);
    return map_hip(e);
  }
  CausalArgs a{};
  a.Q = Q; a.K = K; a.V = V; a.s = s; a.dO = dO; a.dQ = dQ; a.dK = dK; a.dV = dV; a.ds = ds;
  a.state_in = state_in; a.rev_state_in = rev_state_in; a.rev_state_out = rev_state_out;
  a.workspace = workspace; a.seq_len = seq_len; a.s_per_unit = seq_len != nullptr;
  a.B = B; a.H = H; a.N = N; a.dk = dk; a.dv = dv;
  set_walk(&a, plan);
  a.eps = eps; a.stream = stream;
  // the forward's segment states are taken over only if the forward split the sequence as
  // the backward does
  if (fwd_workspace != nullptr && (plan.G > 1 || a.unit_rows > 0)) {
    SeqPlan fwd_plan;
    if (make_plan(COTTN_OP_FWD_CAUSAL, B, H, N, dk, dv, chunk, dtype, &fwd_plan) &&
        fwd_plan.C == plan.C && fwd_plan.G == plan.G && fwd_plan.seg_rows == plan.seg_rows &&
        fwd_plan.even_rows == plan.even_rows && fwd_plan.own_prefix == plan.own_prefix) {
      st = check_workspace(fwd_workspace, fwd_workspace_bytes,
                           workspace_bytes_for(COTTN_OP_FWD_CAUSAL, B, H, dk, dv, fwd_plan));
      if (st != COTTN_OK) return st;
      a.saved_fwd_states = static_cast<const float*>(fwd_workspace);
    }
  }
  return map_hip(dtype == COTTN_BF16 ? bwd_causal_bf16(a) : dtype == COTTN_F16 ? bwd_causal_f16(a) : bwd_causal_f32(a));
}

int fwd_bidir_any(const void* Q, const void* K, const void* V, const float* s, const int* seq_len,
                  void* O, float* state, void* workspace, size_t workspace_bytes, int B, int H,
                  int N, int dk, int dv, int dtype, float eps, void* hip_stream) {
  const void* req[] = {Q, K, V, s, O};
  int st = check_common(req, 5, B, H, N, dk, dv, dtype, eps);
  if (st != COTTN_OK) return st;
  if (state != nullptr && !is_aligned(state, 16)) return COTTN_E_ALIGN;
  if ((st = check_lengths(seq_len)) != COTTN_OK) return st;
  SeqPlan plan;
  if (!make_plan(COTTN_OP_FWD_BIDIR, B, H, N, dk, dv, 0, dtype, &plan)) return COTTN_E_SHAPE;
  st = check_workspace(workspace, workspace_bytes,
                       workspace_bytes_for(COTTN_OP_FWD_BIDIR, B, H, dk, dv, plan));
  if (st != COTTN_OK) return st;
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  if (N == 0) return map_hip(zero_f32(state, long(B) * H * dk * dv, stream));
  CausalArgs a{};
  a.Q = Q; a.K = K; a.V = V; a.s = s; a.O = O; a.state = state; a.workspace = workspace;
  a.seq_len = seq_len; a.s_per_unit = seq_len != nullptr;
  a.B = B; a.H = H; a.N = N; a.dk = dk; a.dv = dv; a.C = plan.C; a.G = plan.G; a.seg_rows = plan.seg_rows;
  a.by_unit = plan.by_unit;
  a.eps = eps; a.stream = stream;
  return map_hip(dtype == COTTN_BF16 ? fwd_bidir_bf16(a) : dtype == COTTN_F16 ? fwd_bidir_f16(a) : fwd_bidir_f32(a));
}

int bwd_bidir_any(const void* Q, const void* K, const void* V, const float* s, const int* seq_len,
                  const void* dO, void* dQ, void* dK, void* dV, float* ds,
                  const void* fwd_workspace, size_t fwd_workspace_bytes, void* workspace,
                  size_t workspace_bytes, int B, int H, int N, int dk, int dv, int dtype, float eps,
                  void* hip_stream) {
  const void* req[] = {Q, K, V, s, dO, dQ, dK, dV, ds};
  int st = check_common(req, 9, B, H, N, dk, dv, dtype, eps);
  if (st != COTTN_OK) return st;
  if ((st = check_lengths(seq_len)) != COTTN_OK) return st;
  SeqPlan plan;
  if (!make_plan(COTTN_OP_BWD_BIDIR, B, H, N, dk, dv, 0, dtype, &plan)) return COTTN_E_SHAPE;
  st = check_workspace(workspace, workspace_bytes,
                       workspace_bytes_for(COTTN_OP_BWD_BIDIR, B, H, dk, dv, plan));
  if (st != COTTN_OK) return st;
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  if (N == 0) return map_hip(zero_f32(ds, seq_len != nullptr ? long(B) * H : H, stream));
  CausalArgs a{};
  a.Q = Q; a.K = K; a.V = V; a.s = s; a.dO = dO; a.dQ = dQ; a.dK = dK; a.dV = dV; a.ds = ds;
  a.workspace = workspace; a.seq_len = seq_len; a.s_per_unit = seq_len != nullptr;
  a.B = B; a.H = H; a.N = N; a.dk = dk; a.dv = dv; a.C = plan.C; a.G = plan.G; a.seg_rows = plan.seg_rows;
  a.by_unit = plan.by_unit;
  a.eps = eps; a.stream = stream;
  if (fwd_workspace != nullptr && sum_totals_in_place(plan.G, dk, dv)) {
    SeqPlan fwd_plan;
    if (make_plan(COTTN_OP_FWD_BIDIR, B, H, N, dk, dv, 0, dtype, &fwd_plan) && fwd_plan.C == plan.C &&
        fwd_plan.G == plan.G && fwd_plan.seg_rows == plan.seg_rows) {
      st = check_workspace(fwd_workspace, fwd_workspace_bytes,
                           workspace_bytes_for(COTTN_OP_FWD_BIDIR, B, H, dk, dv, fwd_plan));
      if (st != COTTN_OK) return st;
      a.saved_fwd_states = static_cast<const float*>(fwd_workspace);
    }
  }
  return map_hip(dtype == COTTN_BF16 ? bwd_bidir_bf16(a) : dtype == COTTN_F16 ? bwd_bidir_f16(a) : bwd_bidir_f32(a));
}

}  // namespace

int cottn_bwd_causal(const void* Q, const void* K, const void* V, const float* s, const void* dO,
                     void* dQ, void* dK, void* dV, float* ds, const void* fwd_workspace,
                     size_t fwd_workspace_bytes, void* workspace, size_t workspace_bytes, int B,
                     int H, int N, int d, int chunk, int dtype, float eps, void* hip_stream) {
  return bwd_causal_any(Q, K, V, s, nullptr, dO, nullptr, nullptr, dQ, dK, dV, ds, nullptr,
                        fwd_workspace, fwd_workspace_bytes,
                        workspace, workspace_bytes, B, H, N, d, d, chunk, dtype, eps, hip_stream);
}

int cottn_bwd_causal_from_state(const void* Q, const void* K, const void* V, const float* s,
                                const void* dO, const float* state_in, const float* rev_state_in,
                                void* dQ, void* dK, void* dV, float* ds, float* rev_state_out,
                                const void* fwd_workspace, size_t fwd_workspace_bytes,
                                void* workspace, size_t workspace_bytes, int B, int H, int N, int d,
                                int chunk, int dtype, float eps, void* hip_stream) {
  return bwd_causal_any(Q, K, V, s, nullptr, dO, state_in, rev_state_in, dQ, dK, dV, ds,
                        rev_state_out, fwd_workspace, fwd_workspace_bytes, workspace,
                        workspace_bytes, B, H, N, d, d, chunk, dtype, eps, hip_stream);
}

int cottn_fwd_bidir(const void* Q, const void* K, const void* V, const float* s, void* O,
                    float* state, void* workspace, size_t workspace_bytes, int B, int H, int N,
                    int d, int dtype, float eps, void* hip_stream) {
  return fwd_bidir_any(Q, K, V, s, nullptr, O, state, workspace, workspace_bytes, B, H, N, d, d, dtype,
                       eps, hip_stream);
}

int cottn_bwd_bidir(const void* Q, const void* K, const void* V, const float* s, const void* dO,
                    void* dQ, void* dK, void* dV, float* ds, const void* fwd_workspace,
                    size_t fwd_workspace_bytes, void* workspace, size_t workspace_bytes, int B,
                    int H, int N, int d, int dtype, float eps, void* hip_stream) {
  return bwd_bidir_any(Q, K, V, s, nullptr, dO, dQ, dK, dV, ds, fwd_workspace, fwd_workspace_bytes,
                       workspace, workspace_bytes, B, H, N, d, d, dtype, eps, hip_stream);
}

// ---- padded batches: seq_len[B] rows exist per sequence; s and ds are [B][H] -------------------
int cottn_fwd_causal_varlen(const void* Q, const void* K, const void* V, const float* s,
                            const int* seq_len, void* O, float* state, void* workspace,
                            size_t workspace_bytes, int B, int H, int N, int d, int chunk,
                            int dtype, float eps, void* hip_stream) {
  if (seq_len == nullptr) return COTTN_E_NULL;
  return fwd_causal_any(Q, K, V, s, seq_len, nullptr, O, state, workspace, workspace_bytes, B, H, N,
                        d, d, chunk, dtype, eps, hip_stream);
}

int cottn_bwd_causal_varlen(const void* Q, const void* K, const void* V, const float* s,
                            const int* seq_len, const void* dO, void* dQ, void* dK, void* dV,
                            float* ds, const void* fwd_workspace, size_t fwd_workspace_bytes,
                            void* workspace, size_t workspace_bytes, int B, int H, int N, int d,
                            int chunk, int dtype, float eps, void* hip_stream) {
  if (seq_len == nullptr) return COTTN_E_NULL;
  return bwd_causal_any(Q, K, V, s, seq_len, dO, nullptr, nullptr, dQ, dK, dV, ds, nullptr,
                        fwd_workspace, fwd_workspace_bytes,
                        workspace, workspace_bytes, B, H, N, d, d, chunk, dtype, eps, hip_stream);
}

int cottn_fwd_bidir_varlen(const void* Q, const void* K, const void* V, const float* s,
                           const int* seq_len, void* O, float* state, void* workspace,
                           size_t workspace_bytes, int B, int H, int N, int d, int dtype, float eps,
                           void* hip_stream) {
  if (seq_len == nullptr) return COTTN_E_NULL;
  return fwd_bidir_any(Q, K, V, s, seq_len, O, state, workspace, workspace_bytes, B, H, N, d, d, dtype,
                       eps, hip_stream);
}

int cottn_bwd_bidir_varlen(const void* Q, const void* K, const void* V, const float* s,
                           const int* seq_len, const void* dO, void* dQ, void* dK, void* dV,
                           float* ds, const void* fwd_workspace, size_t fwd_workspace_bytes,
                           void* workspace, size_t workspace_bytes, int B, int H, int N, int d,
                           int dtype, float eps, void* hip_stream) {
  if (seq_len == nullptr) return COTTN_E_NULL;
  return bwd_bidir_any(Q, K, V, s, seq_len, dO, dQ, dK, dV, ds, fwd_workspace, fwd_workspace_bytes,
                       workspace, workspace_bytes, B, H, N, d, d, dtype, eps, hip_stream);
}

int cottn_scale_from_m(const float* m, float* s, int H, float n, void* hip_stream) {
  if (m == nullptr || s == nullptr) return COTTN_E_NULL;
  if (H < 1) return COTTN_E_SHAPE;
  if (!(n >= 1.0f) || !(n <= 3.0e38f)) return COTTN_E_ARG;
  if (!is_aligned(m, 4) || !is_aligned(s, 4)) return COTTN_E_ALIGN;
  return map_hip(launch_scale_from_m(m, s, H, n, static_cast<hipStream_t>(hip_stream)));
}

int cottn_scale_backward(const float* m, const float* ds, float* dm, int H, float n,
                         void* hip_stream) {
  if (m == nullptr || ds == nullptr || dm == nullptr) return COTTN_E_NULL;
  if (H < 1) return COTTN_E_SHAPE;
  if (!(n >= 1.0f) || !(n <= 3.0e38f)) return COTTN_E_ARG;
  if (!is_aligned(m, 4) || !is_aligned(ds, 4) || !is_aligned(dm, 4)) return COTTN_E_ALIGN;
  return map_hip(launch_scale_backward(m, ds, dm, H, n, static_cast<hipStream_t>(hip_stream)));
}

int cottn_scale_from_m_varlen(const float* m, const int* seq_len, float* s, int B, int H,
                              void* hip_stream) {
  if (m == nullptr || seq_len == nullptr || s == nullptr) return COTTN_E_NULL;
  if (B < 1 || H < 1 || double(B) * H > 16777216.0) return COTTN_E_SHAPE;
  if (!is_aligned(m, 4) || !is_aligned(seq_len, 4) || !is_aligned(s, 4)) return COTTN_E_ALIGN;
  return map_hip(launch_scale_from_m_varlen(m, seq_len, s, B, H,
                                            static_cast<hipStream_t>(hip_stream)));
}

int cottn_scale_backward_varlen(const float* m, const int* seq_len, const float* ds, float* dm,
                                int B, int H, void* hip_stream) {
  if (m == nullptr || seq_len == nullptr || ds == nullptr || dm == nullptr) return COTTN_E_NULL;
  if (B < 1 || H < 1 || double(B) * H > 16777216.0) return COTTN_E_SHAPE;
  if (!is_aligned(m, 4) || !is_aligned(seq_len, 4) || !is_aligned(ds, 4) || !is_aligned(dm, 4))
    return COTTN_E_ALIGN;
  return map_hip(launch_scale_backward_varlen(m, seq_len, ds, dm, B, H,
                                              static_cast<hipStream_t>(hip_stream)));
}

int cottn_step_dkdv(const void* q, const void* k, const void* v, const float* s, float* state,
                    void* o, int B, int H, int dk, int dv, int dtype, float eps, void* hip_stream) {
  const void* req[] = {q, k, v, s, state, o};
  int st = check_common(req, 6, B, H, 1, dk, dv, dtype, eps);
  if (st != COTTN_OK) return st;
  StepArgs a{q, k, v, s, state, o, B, H, dk, dv, eps, static_cast<hipStream_t>(hip_stream)};
  return map_hip(step_any(a, dtype));
}

int cottn_step(const void* q, const void* k, const void* v, const float* s, float* state,
               void* o, int B, int H, int d, int dtype, float eps, void* hip_stream) {
  return cottn_step_dkdv(q, k, v, s, state, o, B, H, d, d, dtype, eps, hip_stream);
}

// ---- d_key != d_value (Sec. 2.1): Q, K, dQ, dK are [B][H][N][dk]; V, O, dO, dV [B][H][N][dv] ----
int cottn_fwd_causal_dkdv(const void* Q, const void* K, const void* V, const float* s, void* O,
                          float* state, void* workspace, size_t workspace_bytes, int B, int H,
                          int N, int dk, int dv, int chunk, int dtype, float eps, void* hip_stream) {
  return fwd_causal_any(Q, K, V, s, nullptr, nullptr, O, state, workspace, workspace_bytes, B, H, N,
                        dk, dv, chunk, dtype, eps, hip_stream);
}

int cottn_bwd_causal_dkdv(const void* Q, const void* K, const void* V, const float* s,
                          const void* dO, void* dQ, void* dK, void* dV, float* ds,
                          const void* fwd_workspace, size_t fwd_workspace_bytes, void* workspace,
                          size_t workspace_bytes, int B, int H, int N, int dk, int dv, int chunk,
                          int dtype, float eps, void* hip_stream) {
  return bwd_causal_any(Q, K, V, s, nullptr, dO, nullptr, nullptr, dQ, dK, dV, ds, nullptr,
                        fwd_workspace, fwd_workspace_bytes, workspace, workspace_bytes, B, H, N, dk,
                        dv, chunk, dtype, eps, hip_stream);
}

int cottn_fwd_bidir_dkdv(const void* Q, const void* K, const void* V, const float* s, void* O,
                         float* state, void* workspace, size_t workspace_bytes, int B, int H, int N,
                         int dk, int dv, int dtype, float eps, void* hip_stream) {
  return fwd_bidir_any(Q, K, V, s, nullptr, O, state, workspace, workspace_bytes, B, H, N, dk, dv,
                       dtype, eps, hip_stream);
}

int cottn_bwd_bidir_dkdv(const void* Q, const void* K, const void* V, const float* s,
                         const void* dO, void* dQ, void* dK, void* dV, float* ds,
                         const void* fwd_workspace, size_t fwd_workspace_bytes, void* workspace,
                         size_t workspace_bytes, int B, int H, int N, int dk, int dv, int dtype,
                         float eps, void* hip_stream) {
  return bwd_bidir_any(Q, K, V, s, nullptr, dO, dQ, dK, dV, ds, fwd_workspace, fwd_workspace_bytes,
                       workspace, workspace_bytes, B, H, N, dk, dv, dtype, eps, hip_stream);
}

int cottn_profile_start(void) {
  g_pending.clear();
  g_totals.clear();
  g_profile_on = true;
  return COTTN_OK;
}

int cottn_profile_stop(void) {
  g_profile_on = false;
  int status = COTTN_OK;
  for (const PendingSpan& sp : g_pending) {
    float ms = 0.f;
    if (sp.end == nullptr || hipEventSynchronize(sp.end) != hipSuccess ||
        hipEventElapsedTime(&ms, sp.begin, sp.end) != hipSuccess) {
      status = COTTN_E_HIP;
    } else {
      KernelTotal* slot = nullptr;
      for (KernelTotal& t : g_totals)
        if (std::strcmp(t.name, sp.name) == 0) slot = &t;
      if (slot == nullptr) {
        g_totals.push_back(KernelTotal{sp.name, 0, 0.0});
        slot = &g_totals.back();
      }
      slot->launches += 1;
      slot->ms += ms;
    }
    if (sp.begin) (void)hipEventDestroy(sp.begin);
    if (sp.end) (void)hipEventDestroy(sp.end);
  }
  g_pending.clear();
  return status;
}

int cottn_profile_count(void) { return int(g_totals.size()); }
const char* cottn_profile_name(int i) {
  return (i >= 0 && i < int(g_totals.size())) ? g_totals[i].name : "";
}
long cottn_profile_launches(int i) {
  return (i >= 0 && i < int(g_totals.size())) ? g_totals[i].launches : 0;
}
double cottn_profile_ms(int i) {
  return (i >= 0 && i < int(g_totals.size())) ? g_totals[i].ms : 0.0;
}

}  // extern "C"
