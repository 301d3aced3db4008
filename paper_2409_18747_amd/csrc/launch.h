// Host-side glue between the C-ABI entry points and the kernel files: argument bundles,
// the per-dtype launch functions each kernel file defines, and the launch wrapper that
// optionally attaches timing events to a kernel.
#pragma once
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>
#include <stddef.h>

namespace cottn {

// A kernel argument that workgroups divide their index or a row number by: with it comes floor((2^32 - 1) / n), and a
// quotient is a multiplication and a correction.  The compiler's division is a chain of some twenty
// instructions through the vector ALU, and up to three of them stood before the first row was asked
// for, in every launch, with the number of workgroups, which comes by a second load.  Without them, and the scale
// asked for behind the rows, 93 instructions stand there in the 64 x 64 forward scan instead of 198.  Both together, one set of
// buffers, in turn, median of nine and lowest to highest: B8 H12 N1024 forward + backward d64 50.5 (50.3 to 50.7) -> 49.7 us (49.6
// to 49.9), five launches of 15 units of 777 rows at 64 x 128 41.0 (40.9 to 41.2) -> 40.5 (40.4 to 40.6); d128 101.7
// (101.4 to 102.7) -> 100.8 (100.6 to 102.0), where the runs of one side differ by as much.  Of d64 the backward's scans take the
// gain, 0.2 and 0.35 us; the forward's time does not change.
struct Divisor {
  int n;             // 0: nothing is divided by it
  unsigned scaled;
  constexpr explicit Divisor(int by) : n(by), scaled(by > 0 ? 0xFFFFFFFFu / unsigned(by) : 0u) {}
  __host__ __device__ constexpr operator int() const { return n; }
};
// x / d for 0 <= x: the estimate is the quotient or one less, since 2^32 - n scaled <= n.
__host__ __device__ constexpr int quotient(int x, const Divisor& d) {
  const int q = int((static_cast<unsigned long long>(static_cast<unsigned>(x)) * d.scaled) >> 32);
  return x - q * d.n >= d.n ? q + 1 : q;
}

// What a forward scan is told in one word.
enum ScanFlags { SUM_TOTALS = 1, SCALE_PER_UNIT = 2, STREAM_Q = 4, STREAM_KV = 8 };

// Sequence split chosen on the host: G segments of seg_rows rows (a multiple of C) per
// (batch, head); the last segment may be shorter.
struct CausalArgs {
  const void* Q; const void* K; const void* V; const float* s;
  const void* dO;                 // backward only
  void* O; float* state;          // forward only (state may be null)
  // a sequence processed in pieces (causal only): null, or the forward-time state Kh^T V of
  // the rows before this piece (forward and backward), the reverse-time state Qh^T dO of the
  // rows after it (backward, in), and that state with this piece added (backward, out)
  const float* state_in;
  const float* rev_state_in;
  float* rev_state_out;
  // padded batches: null, or int[B] row counts (then s and ds are [B][H], see s_per_unit)
  const int* seq_len;
  int s_per_unit;                 // s (and ds) indexed by (batch, head) instead of head
  void* dQ; void* dK; void* dV; float* ds;  // backward only
  // backward only: null, or the segment states the forward call with the same split left in
  // its workspace (then the backward does not recompute them)
  const float* saved_fwd_states;
  void* workspace;
  // dk, dv: head dimensions of queries / keys and of values / outputs (Sec. 2.1: d_H_key,
  // d_H_value); Q, K, dQ, dK are [B][H][N][dk], V, O, dO, dV [B][H][N][dv], states [dk][dv]
  int B, H, N, dk, dv, C, G, seg_rows;
  // even shares (causal; workspace.h): rows of a unit in the units laid end to end, else 0 and G segments
  // of seg_rows rows per unit; workgroups of a scan either way, and state slots of a workspace array
  int unit_rows, workgroups;
  long slots;
  // Even shares of units that would otherwise be one segment each: calls with lengths keep to those segments
  // and leave no states.  A forward notes in the last slot which it did, and a backward without lengths that
  // is handed states of none forms them itself, so that either forward suits either backward.
  bool marked;
  bool own_prefix;   // segments whose workgroups form the state before them themselves (own_prefix below)
  bool by_unit;                   // bidirectional only: a (batch, head) per workgroup, G = 1
  float eps;
  hipStream_t stream;
};

// Whether the kernels that need the states of other segments add the segment totals up
// themselves (each workgroup reads up to G - 1 states of its unit out of the L2) or a carry /
// combine kernel is launched that turns the state arrays into prefixes, suffixes or sums.  A
// launch costs about 5 us with its gap; a state of 4 KB to 64 KB takes every workgroup about 0.15 us
// to 0.6 us in each scan, and the carry kernel, which moves all of them, longer the more units there
// are.  The forward and the backward must agree on it for the backward to take over the forward's
// saved states.
//
// Causal, in place minus carried, forward / backward in us, at 2, 12 and 24 units: 64 x 64 12 segments
// -1.1 / -0.6, -2.3 / -1.4, -5.1 / -2.6; 24 segments 0.0 / +0.9, -2.9 / +1.8; 64 x 128 6 segments -0.6 /
// +0.7, -1.7 / -0.2, -3.9 / -1.7; 16 segments +1.9 / +7.3, -1.3 / +6.5, -1.9 / +6.6; 128 x 128 4 segments
// -0.7 / -0.1, -2.1 / -1.7, -4.8 / -2.3; 10 segments +2.7 / +5.5, -1.4 / +5.1, -4.8 / 0.0.  The line
// follows the number of segments where the sums of the two cross, 18 / 24 / 31 or more at 64 x 64, 7 /
// 10 / 14 at 64 x 128, 4 / 7 / 13 at 128 x 128, or one above: a launch takes the host 3 us too.  At 128 x
// 128 16-bit rows keep to 4 / 6 / 9: with more in place, 14 units of 1024 rows take 23 / 54 us for the forward
// / with its backward instead of 24 / 50, though 24 units of 4738 rows take 47 / 128 instead of 51 / 136;
// fp32 gains everywhere (24 units of 300 rows 30 / 71 instead of 39 / 75).
constexpr bool causal_totals_in_place(long units, int G, int dk, int dv, bool f32) {
  const long few = units < 32 ? units : 32;
  const long kb = dk * dv <= 64 * 64 ? 264 + 10 * few : 200 + (f32 && dk * dv == 128 * 128 ? 24 : 13) * few;
  return long(G - 1) * dk * dv * 4 <= kb * 1024;
}
// Workgroups that share the 128 value columns of a (batch, head) in a causal forward of one segment (and
// so short or of many sequences).  Such a call lasts as long as one workgroup takes: launch, first rows
// and state, a few steps, state out, and with up to 128 units half of the compute units have nothing to
// do.  A part forms the masked tiles again and reads the same query and key rows, out of the L2 it shares
// with the others (unit_and_segment).  128 x 128, whole / 2 / 4 parts: 128 units of 5 rows continued from a state
// 9.5 / 7.3 / 6.3 us (with 32-row steps; 64-row ones 7.4), of 64 rows 8.5 / 7.7 / 6.8, of 128 rows 10.4 / 9.0 /
// 9.7, 160 units of 128 rows 8.2 / 8.3 / 11.2, 512 units of 5 rows 14.9 / 17.1 / 16.7.  64 x 128, of which two
// workgroups fit a compute unit either way, 256 units of 128 rows 8.0 / 7.5 us, of 400 rows 19.3 / 17.4; fp32
// 256 units of 31 rows 7.5 / 7.0, of 100 rows 20.3 / 18.7.  At 64 columns parts of 32 gain nothing.
constexpr int value_parts(long units, int N, int dk) {
  if (units > (dk == 128 ? 128 : 256)) return 1;
  return dk == 128 && N <= 64 ? 4 : 2;
}
// 16-bit causal 128 x 128: the scans with 64-row steps fill a compute unit with one workgroup of eight
// waves.  With 32-row steps two of four waves fit, whose steps hide each other's latencies, but every
// row then pays twice for the state (its copy to LDS and the reads of it).  From 257 workgroups on, where
// the former take another round, the latter are the faster ones (the forward moves 5.4 TB/s then):
// 272 units of 300 rows forward / dQ / dK,dV 29.5 / 37.4 / 51.5 -> 27.0 / 32.6 / 41.6 us; 512 units of 1024
// rows 106 / 140 / 203 -> 94 / 125 / 157; 1024 units of 500 rows 112 / 144 / 200 -> 96 / 134 / 166; up to
// 256 workgroups they are not (256 of 512 rows 24.6 / 43.3 against 28.1 / 47.1 for forward / dK,dV).
// Their own second round is the longer one: 704 units of 1328 rows 206 / 260 / 364 -> 232 / 300 / 330, 640
// of 700 rows forward 102 -> 91, 560 of 777 rows dQ 150 -> 141..151.
// The dQ scan has registers for them only where no reverse-time totals are due (G = 1).
constexpr bool two_to_a_cu_forward(long workgroups) { return workgroups > 256 && (workgroups <= 640 || workgroups > 768); }
constexpr bool two_to_a_cu_dq(long workgroups) { return workgroups > 256 && (workgroups <= 512 || workgroups > 768); }
constexpr bool two_to_a_cu_dkdv(long workgroups) { return workgroups > 256; }
// Whether the workgroups of a causal call in segments form the state of the rows before them by themselves instead
// of adding up what a totals launch left: in the forward, which leaves it in the workspace as a carry launch would,
// and in the dQ scan of a backward that was not handed that workspace (own_prefix_dq).  A launch takes 4 us and more of a small
// call, its kernel and the totals' way through the workspace about as long again; a step of the reduction 0.3 to
// 1.2 us, one after the other over the rows before the last segment.  The line is the number of those rows up to
// which the forward alone is the faster one too.  Forward / with backward / with backward that rebuilds the state,
// totals launch -> own prefix: 64 x 64 2 units of 256 rows 10.4 / 22.9 / 35.4 -> 7.9 / 20.4 / 30.0 us, of 640 10.4
// / 22.6 / 35.0 -> 8.7 / 20.6 / 30.5, 100 of 320 10.4 / 25.7 / 34.9 -> 8.5 / 24.5 / 30.1, 15 of 777 10.9 / 25.5 /
// 35.8 -> 11.4 / 25.1 / 32.3, 100 of 512 11.5 / 32.2 / 36.2 -> 11.4 / 31.6 / 35.4, of 1024 17.3 / 50.3 / 55.6 ->
// 19.2 / 50.9 / 58.3; 32 x 32 10 units of 1024 10.5 / 22.8 / 35.2 -> 9.6 / 20.3 / 30.4; 64 x 32 15 of 777 12.9 /
// 27.2 / 40.0 -> 10.0 / 23.9 / 34.7; 64 x 128 4 of 777 14.1 / 31.0 / 44.4 -> 13.5 / 31.1 / 39.1 (between 640 and 832
// rows, forward / with backward: 2 units of 650 15.7 / 33.2 -> 12.0 / 29.4, of 700 16.1 / 33.9 -> 12.5 / 29.8, of 830
// 16.0 / 34.0 -> 13.9 / 31.3, 4 of 650 16.0 / 34.2 -> 12.2 / 29.6, of 830 16.2 / 34.3 -> 14.1 / 31.7; 32 x 128 2, 4 and
// 8 units 13.0 / 28.0 -> 9.9..11.4 / 24.3..24.8), 15 of 777 15.7 /
// 37.2 / 41.8 -> 14.1 / 34.7 / 43.0; 128 x 64 15.5 / 37.7 / 42.7 -> 15.0 / 36.3 / 46.0; 128 x 32 100 of 400 13.2 /
// 37.7 / 42.7 -> 11.7 / 36.0 / 39.8, of 512 13.6 / 39.0 / 43.6 -> 14.2 / 39.6 / 46.8; 128 x 128 40 of 256 12.9 /
// 32.4 / 39.1 -> 9.9 / 28.8 / 31.9, 100 of 640 in two segments 27.6 / 79.1 / 88.3 -> 22.4 / 73.4 / 77.6; fp32 32 x
// 32 2 of 256 10.0 / 22.3 / 35.3 -> 7.9 / 20.0 / 30.3, of 512 10.8 / 23.4 / 36.4 -> 12.1 / 22.5 / 31.3; 64 x 64 100
// of 130 14.2 / 34.6 / 41.7 -> 12.2 / 32.3 / 36.4, 40 of 256 12.4 / 34.0 / 38.7 -> 13.6 / 35.6 / 41.6; 64 x 128 100
// of 200 in two segments 26.3 / 74.9 / 82.9 -> 21.3 / 68.9 / 74.0; 128 x 128 100 of 130 38.6 / 106 / 121 -> 29.1 /
// 94 / 102.
constexpr bool own_prefix_dq(long units, int G, long seg_rows, int dk, int dv, bool f32) {
  if (G < 2) return false;
  const long workgroups = units * G, rows = (G - 1) * seg_rows;
  const bool narrow = dk * dv <= 2048, widest = dk == 128 && dv == 128;
  if (f32 && G == 2) return rows <= 224;
  if (f32 && widest) return false;
  if (f32 && dk * dv == 1024) return rows <= (workgroups <= 128 ? 288 : workgroups <= 384 ? 224 : 128);
  if (f32) return rows <= (workgroups <= 80 ? 192 : 128);
  if (widest && G == 2 && workgroups <= 256) return rows <= 1024;
  if (narrow && workgroups <= 256) return rows <= 960;
  // segments of one step: as many totals to add as steps to take
  if (seg_rows == 64 && workgroups <= 256) return rows <= (dk <= 64 && dv == 128 && workgroups <= 128 ? 768 : 576);
  return rows <= (workgroups <= 256 || narrow ? 448 : 320);
}
// The forward does so a little further than the dQ scan: with up to four segments, of several steps each, the totals
// launch lasts nearly as long as reducing the rows before the last segment in its own workgroup.  A backward that
// rebuilds the state takes the totals launch there.  Forward / with backward / with backward that rebuilds the state, totals launch -> own
// prefix, device time: 100 units of 400 rows 64 x 64 11.7 / 30.9 / 35.2 -> 10.5 / 29.4 / 34.1 us, 64 x 128 15.9 /
// 45.4 / 51.5 -> 14.5 / 43.9 / 49.7, 32 x 128 13.0 / 37.8 / 42.3 -> 11.6 / 36.2 / 40.8; 150 of 400 128 x 64 22.3 / 61.5 /
// 70.0 -> 17.2 / 56.6 / 64.6; 120 of 640 64 x 64 15.5 / 41.9 / 47.5 -> 13.8 / 39.1 / 45.2; 128 x 128 80 of 640 24.0 /
// 70.1 / 77.3 -> 19.6 / 64.5 / 72.4, of 777 29.6 / 82.8 / 94.7 -> 23.7 / 76.8 / 87.7.  Not beyond: 64 x 64 100 of 1024
// 18.4 / 50.1 -> 19.9 / 50.7, five segments 70 of 640 64 x 128 17.5 / 48.4 -> 19.1 / 48.9, and not at 128 x 32, 100 of
// 450 13.2 / 38.5 -> 14.1 / 38.9.
constexpr bool own_prefix(long units, int G, long seg_rows, int dk, int dv, bool f32) {
  if (own_prefix_dq(units, G, seg_rows, dk, dv, f32)) return true;
  if (f32 || G < 2 || G > 4 || dk * dv <= 2048 || (dk == 128 && dv == 32)) return false;
  const bool widest = dk == 128 && dv == 128;
  return units * G <= (widest ? 256 : 512) && (G - 1) * seg_rows <= (widest ? 768 : 576);
}

// Steps that they take of it at a time.  A step of narrow rows is two barriers and the waits around them more than
// work, so that four at once gain where a compute unit has room for their tiles, one workgroup each: forward / backward
// that rebuilds the state, one -> four: 32 x 32 10 units of 1024 rows 8.4 -> 7.4 / dQ 8.9 -> 8.2 us, 30 of 512 with
// backward 18.3 -> 17.3, fp32 2 of 256 7.2 -> 6.5 / 7.6 -> 7.1, 10 of 250 7.7 -> 7.0 / 8.1 -> 7.6; 64 x 32 15 of 777 forward 9.3 ->
// 8.4, dQ 9.6 -> 9.7.  Wider rows do not: 64 x 64 2 of 256 5.1 -> 4.9, 40 of 512 8.7 -> 8.6, 64 x 128 4 of 777 12.9 -> 13.9,
// 128 x 64 15 of 640 12.0 -> 12.4, 32 x 64 10 of 960 8.4 -> 8.4, fp32 10 of 192 7.2 -> 7.5; nor do more workgroups: 32 x 32
// 100 of 512 8.3 -> 9.0.
constexpr int prefix_sets_built(int dk, int dv, bool f32, bool forward) {
  return (dk == 32 && dv == 32) || (forward && !f32 && dk == 64 && dv == 32) ? 4 : 1;
}
constexpr bool prefix_by_sets(long workgroups) { return workgroups <= 256; }

// Stored states that a wave with this many 16 x 16 tiles of each loads at once when it seeds its accumulators (register
// budget), and how many where more than those are left.  More at once save latencies until the 64 bytes a cycle of the
// vector L1 are the bound.  The first number throughout / these, sums in place, forward alone and with backward in us:
// five to eight tiles, 15 units of 777 rows 16-bit 64 x 128 16.2, 37.4 / 15.0, 35.0 and 128 x 64 16.2, 37.9 / 14.9, 35.9, fp32
// 23.9, 60.4 / 22.9, 59.3 and 24.4, 62.9 / 23.9, 62.0 (fp32 whose prefixes come carried, one state each, give 0.2 to 0.8 back: 15
// of 1500 32.9, 79.8 / 32.7, 80.4 and 34.1, 86.6 / 34.0, 87.1); up to two, 4 of 2000 16-bit 64 x 32 9.6, 24.5 / 9.3, 23.7, fp32 32 x 64
// 14.5, 36.3 / 13.8, 35.1.  Not taken: 5 at four tiles, 15 of 777 at 64 x 64 forward scan 5.8 / 6.5, and 4 at 128 x 128, 96 of 1024
// forward scan 24.9 / 25.2.  Nor 6 at 64 x 64 by sixteen waves (256-row chunks), whose 128 registers a wave do not hold what they
// have: twelve more are spilled in the bf16 dQ scan, 96 of 1024 with backward 129.2 / 133.8, 16 of 16384 327.5 / 332.9.
constexpr int states_at_once(int tiles) { return tiles <= 4 ? 3 : tiles <= 8 ? 2 : 1; }
constexpr int states_at_once_of_many(int tiles, int elements, int waves) {
  if (waves >= 16 && elements >= 64 * 64) return states_at_once(tiles);
  return tiles <= 2 ? 6 : tiles > 4 && tiles <= 8 && elements < 128 * 128 ? 4 : states_at_once(tiles);
}

// Shapes built for even shares (api.hip: causal_even_share, which asks for no others).
constexpr bool even_shares_built(int dk, int dv, bool f32) {
  return (dk == 128 && dv == 128) || (f32 && dk >= 64 && dv >= 64);
}
// Bidirectional: only the sums are needed, which a backward that is handed the forward's totals takes
// over where they were left as they are; the line lies where the combine launch is the better one for
// the forward alone (64 x 64 24 segments +1.3 us at 2 units, 64 x 128 12 +0.8, 128 x 128 8 +1.2).
constexpr bool sum_totals_in_place(int G, int dk, int dv) {
  return G <= 24 && long(G - 1) * dk * dv * 4 <= 600 * 1024;
}

// Rows a step of the bidirectional kernels takes (a wave per 16 of them).  16-bit: 128; with 64 a
// workgroup has four waves to cover latencies with and twice the barriers (forward + backward, 64 ->
// 128 rows: B4 H8 N4096 d64 50 -> 42 us, B16 H8 N4096 138 -> 132 us, B1 H8 N16384 d32 45 -> 38 us, B2 H8
// N1000 d128 53 -> 46 us, B16 H16 N4096 d128 634 -> 631 us).  fp32 tiles of 128 rows and 128 columns
// would not fit the LDS.
constexpr int bidir_step_rows(bool f32) { return f32 ? 64 : 128; }

// A launch takes fewer than 2^32 threads.  8 388 608 workgroups of 512 are one too many, of 256 they are
// not: for so many (short) sequences the kernels of 512 threads give way to ones of 256, the
// bidirectional ones to 64-row steps, the 128 x 128 backward scans to one wave per row group.
constexpr bool threads_fit(long workgroups, int threads) { return workgroups * threads < (1L << 32); }

// Whether a bidirectional call with 16-bit rows takes a whole (batch, head) per workgroup, forward and
// backward in one launch each (bidir_bf16.hip: fwd_bidir_unit, bwd_bidir_unit), or splits the sequence
// over workgroups and the work over two launches each.  A unit's rows are walked one step after the
// other, so either they are few or the units alone have to fill the compute units.  Forward +
// backward, split / by unit: 8 units of 120 rows 22 / 20 us, of 250 rows at 128 x 128 32 / 33; 32 units
// of 200 rows d64 26 / 22 us; 128 units of 500 rows d64 28 / 30 us, 160 units of 512 37 / 32, 384 units
// 58 / 53; 160 units of 1024 rows 52.6 / 54.1 us, 192 units 59 / 54, 384 units 98 / 93, at 32 x 32 192
// units 29 / 33; 272 units of 1500 rows 118 / 119 us, 320 units of 2048 rows 187 / 194 us.  Where two
// rounds of workgroups leave most compute units idle in the second and sequences are long enough, the
// split is the better one too: wide rows, of which one workgroup fills a compute unit (288 units of 1500
// rows at 64 x 128 219 / 246 us, 272 of 777 at 128 x 32 92 / 104), and more than 512 units (576 of 1500
// rows at 128 x 32 326 / 365).  (fp32 steps last longer, and only 224 to 256 units gain: always split.)
constexpr bool bidir_by_unit(long units, int N, bool f32, int dk, int dv) {
  if (f32) return false;
  if (N <= 128) return true;
  if (N <= 256) return dk < 128 || dv < 128 || units >= 96;
  if (N <= 512) return units >= 160;
  if (N > 1536 || units < 192 || (dk == 32 && dv == 32)) return false;
  if (N > 1024 && (units > 512 || (units > 256 && units < 448 && (dk == 128 || dv == 128)))) return false;
  return !(dk == 128 && dv == 32 && units > 256 && units < 320);
}

struct StepArgs {
  const void* q; const void* k; const void* v; const float* s; float* state; void* o;
  int B, H, dk, dv;  // q, k are [B][H][dk]; v, o [B][H][dv]; state [B][H][dk][dv]
  float eps;
  hipStream_t stream;
};

// defined in the kernel files; every function only enqueues work on args.stream
hipError_t fwd_causal_bf16(const CausalArgs& a);
hipError_t bwd_causal_bf16(const CausalArgs& a);
hipError_t fwd_bidir_bf16(const CausalArgs& a);
hipError_t bwd_bidir_bf16(const CausalArgs& a);
hipError_t fwd_causal_f16(const CausalArgs& a);
hipError_t bwd_causal_f16(const CausalArgs& a);
hipError_t fwd_bidir_f16(const CausalArgs& a);
hipError_t bwd_bidir_f16(const CausalArgs& a);
hipError_t fwd_causal_f32(const CausalArgs& a);
hipError_t bwd_causal_f32(const CausalArgs& a);
hipError_t fwd_bidir_f32(const CausalArgs& a);
hipError_t bwd_bidir_f32(const CausalArgs& a);
// what the four above call where the fp32 matrix instruction is the better one (device_common.h: SPLIT3)
hipError_t fwd_causal_f32w(const CausalArgs& a);
hipError_t bwd_causal_f32w(const CausalArgs& a);
hipError_t fwd_bidir_f32w(const CausalArgs& a);
hipError_t bwd_bidir_f32w(const CausalArgs& a);
hipError_t step_any(const StepArgs& a, int dtype);

// small fp32 state kernels shared by all element types (defined next to their kernels)
hipError_t launch_fwd_state_carry(float* seg_state, int units, int G, int elems, hipStream_t st);
// either array may be null: then only the other one is carried
hipError_t launch_bwd_state_carry(float* fwd_tot, float* rev_tot, int units, int G, int elems,
                                  hipStream_t st);
// segment totals of Kh^T V for all segments but the last, [units][G][d][d] fp32 in `dst`
// (the first kernel of the causal forward, also used by a backward without saved states)
hipError_t launch_fwd_segment_totals_bf16(const CausalArgs& a, float* dst);
hipError_t launch_fwd_segment_totals_f16(const CausalArgs& a, float* dst);
hipError_t launch_fwd_segment_totals_f32(const CausalArgs& a, float* dst);

// The same kernel in general: dst[unit][g] = sum over the rows of segment g of N(X)^T Y
// (dk x dv) for g < n_compute (G slots per unit).
struct SegmentTotalsArgs {
  const void* X; const void* Y; float* dst;
  int units, N, dk, dv, G, n_compute, seg_rows;  // X rows are dk wide, Y rows dv wide
  float eps;
  const int* seq_len; int H;  // padded batches: rows at or beyond seq_len[unit / H] do not exist
  // dst row-major [dk][dv] per slot (false), or in the tile order the causal scan kernels read
  // their stored states in (device_common.h: tiled_state_offset, tile (key tile, value tile))
  bool tiled;
  int unit_rows, workgroups;  // even shares, as in CausalArgs (0: segments)
  hipStream_t stream;
};
hipError_t launch_segment_totals_bf16(const SegmentTotalsArgs& t);
hipError_t launch_segment_totals_f16(const SegmentTotalsArgs& t);
hipError_t launch_segment_totals_f32(const SegmentTotalsArgs& t);
hipError_t launch_segment_totals_32x32_f32w(const SegmentTotalsArgs& t);   // called by the line above
hipError_t launch_bidir_combine(float* totals, int units, int G, int elems, float* state,
                                hipStream_t st);

// the stabiliser map of Sec. 3.3 and its gradient (scale.hip)
hipError_t launch_scale_from_m(const float* m, float* s, int H, float n, hipStream_t st);
hipError_t launch_scale_backward(const float* m, const float* ds, float* dm, int H, float n,
                                 hipStream_t st);

hipError_t launch_scale_from_m_varlen(const float* m, const int* seq_len, float* s, int B, int H,
                                      hipStream_t st);
hipError_t launch_scale_backward_varlen(const float* m, const int* seq_len, const float* ds,
                                        float* dm, int B, int H, hipStream_t st);

// profiling hooks (api.hip): when profiling is on, hands out a fresh pair of events that the
// launch attaches to the kernel itself, so they time the kernel's own begin and end.
bool profile_on();
void profile_events(const char* kernel_name, hipEvent_t* begin, hipEvent_t* end);

// The block of a kernel's arguments in bytes.  Every launch writes it to memory and every workgroup begins by reading it; with more
// than 128 bytes a launch of the forward scan took 0.2 to 0.3 us longer.  Calls one after the other, 136 / 120 bytes: 12 units of 59 rows
// 128 x 128 f16 4.1 / 3.9 us, 16 of 37 fp32 32 x 32 5.3 / 5.0, 432 of 202 64 x 32 8.7 / 8.3.
template <class... Args>
constexpr size_t argument_bytes() {
  size_t at = 0;
  ((at = (at + alignof(Args) - 1) / alignof(Args) * alignof(Args) + sizeof(Args)), ...);
  return at;
}
template <class... Params>
constexpr size_t argument_bytes(void (*)(Params...)) { return argument_bytes<Params...>(); }

// Enqueues one kernel on `stream` and returns the launch status.
template <class... Params, class... Args>
inline hipError_t launch_kernel(const char* kernel_name, void (*kernel)(Params...), dim3 grid,
                                dim3 block, size_t dynamic_lds, hipStream_t stream, Args... args) {
  hipEvent_t begin = nullptr, end = nullptr;
  if (profile_on()) profile_events(kernel_name, &begin, &end);
  hipExtLaunchKernelGGL(kernel, grid, block, dynamic_lds, stream, begin, end, 0,
                        static_cast<Params>(args)...);
  return hipGetLastError();
}

}  // namespace cottn
