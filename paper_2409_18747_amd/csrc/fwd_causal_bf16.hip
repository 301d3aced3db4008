// Causal cosine attention forward: MFMA products with fp32 accumulation (gfx950).
// Written against an element type: this file builds the bfloat16 kernels, the IEEE half ones
// when it is included with COTTN_ELEM_F16 defined and the fp32 ones with COTTN_ELEM_F32.
//
// Sec. 4 eq. attn_2 writes the causal output as an inclusive cumulative sum over the sequence
// of the outer products kh_j^T v_j, contracted with qh_i.  Regrouping that sum exactly:
//   * the sequence of one (batch, head) is cut into G segments, each a whole number of chunks
//     of C rows;
//   * kernel 1 (segment totals) reduces kh^T v over every segment but the last;
//   * kernel 2 (carry, only with many segments; with few the scan adds the totals up itself)
//     turns the totals into exclusive prefixes: the state at each segment start;
//   * kernel 3 (scan) walks the chunks of its segment with the d x d state in fp32
//     accumulators:  O_c = s_h [ (Qh_c Kh_c^T (.) M) V_c + Qh_c S ],  S += Kh_c^T V_c,
//     where the first term is eq. attn_1 restricted to the chunk.
// With G = 1 only the scan kernel runs; with one chunk per segment this is the fully
// chunk-parallel form.
//
// Normalisation (Sec. 3.2): with r_i = 1/max(|q_i|,eps) and kh_j = k_j / max(|k_j|,eps),
//     O_i = s_h r_i [ sum_{j<=i} (q_i . kh_j) v_j + q_i S ],   S = sum_j kh_j^T v_j,
// so the raw Q rows are an MFMA operand and r_i multiplies the finished output row, while K,
// which is contracted over the token index in S, is rescaled to kh on its way into LDS.
//
// Work split inside the scan workgroup (C/16 waves): wave w owns query rows 16w..16w+15 of
// the chunk for the output, and a fixed set of 16x16 tiles of the state for the update.
// Tiles sit row-major in LDS; operands whose contraction index is the token are read with
// the transposing LDS read, so no transposed copy is kept.  The masked similarity tile is
// produced as P^T = K Q^T, whose accumulator layout is the operand layout the following
// product needs (with the token slots permuted the same way on the V side), so P never
// touches LDS; the V fragments read for P V are reused by the state update.  Outputs are
// accumulated transposed (O^T = V^T P^T + S^T Q^T) so that a lane ends up with 4 consecutive
// columns of one output row: one row factor per lane and 8-byte staging writes.
//
// Scheduling: the kernels wait for memory and for their own latencies, not for the MFMA
// units, so every group of MFMAs is preceded by all of its LDS reads, issued back to back into
// distinct registers (a scheduling barrier keeps the compiler from sinking a read next to its
// use), the next chunk's tiles are prefetched into registers while the current one is
// computed, and finished output rows are stored one chunk late, non-temporally.  An XCD's L2
// keeps its contents between launches and workgroups are dealt to the XCDs by index, so the
// totals kernel and the scan number their workgroups alike: the scan finds its K, V rows in L2.
#include "device_common.h"
#include "launch.h"
#include "tile_io.h"

namespace cottn {
namespace COTTN_NS {
namespace {

// DK, DV: the head dimensions of the keys / queries and of the values / outputs (Sec. 2.1:
// d_H_key and d_H_value); the state Kh^T V is DK x DV.
template <int DK, int DV, int C>
struct FwdCfg {
  static constexpr int NW = C / 16;
  static constexpr int NT = NW * 64;
  static constexpr int DTK = DK / 16, DTV = DV / 16;
  static constexpr int KSK = DK / 32;   // k steps of a contraction over the key features
  static constexpr int NP = C / 32;     // pairs of 16-token tiles in a chunk
  static constexpr int TPK = tile_pitch(DK, C), TPV = tile_pitch(DV, C);   // operand tiles
  static constexpr int SP = lds_pitch(DV);   // state copy [d_key][d_value]
  static constexpr int TILEK = C * TPK, TILEV = C * TPV;   // elements of one LDS tile
  static constexpr int STATE = DK * SP;          // elements of the bf16 state copy
  // finished output rows (DV wide) are staged in the wave's own dead query rows when those are
  // wide enough, else in a tile of their own
  static constexpr bool OWN_STAGE = ELEM * stage_pitch(DV) > LDS_ELEM * TPK;
  static constexpr int OP = stage_tile_pitch(DV, C);   // of that tile, in elem_t
  static constexpr int LDS_BYTES =
      LDS_ELEM * (2 * TILEK + TILEV + STATE) + (OWN_STAGE ? ELEM * C * OP : 0) + 4 * C;
  static constexpr int WG_PER_CU = (160 * 1024) / LDS_BYTES;
  // steps that OWN_PREFIX_SETS takes at a time, and the elements of the tiles that the second and further ones need
  // (the first of them the q tile too)
  static constexpr int PREFIX_SETS = prefix_sets_built(DK, DV, ELEM_IS_F32, true);
  static constexpr int PREFIX_TILES = PREFIX_SETS < 2 ? 0 : (PREFIX_SETS - 1) * TILEV + (PREFIX_SETS - 2) * TILEK;
  // waves per SIMD the register allocation is capped for (two workgroups per compute unit
  // when LDS allows, never more than the hardware needs for one workgroup)
  static constexpr int WAVES_RAW = (WG_PER_CU >= 2 ? 2 : 1) * NW / 4;
  // never budget registers for more than two waves per SIMD unless one workgroup alone needs
  // it: spilling costs more than the second workgroup of a large chunk gains
  static constexpr int WAVES_PER_EU = NW / 4 > 2 ? NW / 4 : (WAVES_RAW > 2 ? 2 : WAVES_RAW);
  // with CS waves per row group: one workgroup alone has NW * CS / 4 waves per SIMD; two
  // workgroups per compute unit when the LDS (one more tile for staging) allows
  template <int CS>
  static constexpr int waves_per_eu() {
    if (CS == 1) return WAVES_PER_EU;
    const int own = NW * CS / 4;
    const int wg = (160 * 1024) / (LDS_BYTES + ELEM * C * OP) >= 2 ? 2 : 1;
    return own * wg > 4 ? (own > 4 ? own : 4) : own * wg;
  }
};

// Waves per 16-row group in the scan kernel (see the kernel), chosen per shape by measurement:
// two at d = 128, where one workgroup fills the LDS of a compute unit and four waves are too
// few to cover latencies (+6 % on a 2048-token prefill of 4096 heads); at d = 64 and 32 the
// two variants time the same and the smaller workgroup is kept.
template <int DK, int DV, int C> struct FwdSplit { static constexpr int CS = ELEM_IS_F32 ? 2 : 1; };
template <> struct FwdSplit<128, 128, 64> { static constexpr int CS = 2; };
// (fp32: chunks of 32 rows are two row groups, so two waves each make a workgroup of four.  B8 H12
// N1024 d64 34.5 -> 30.5 us, operands in three parts against the fp32 matrix instruction (in even shares 28.1,
// with the range of the values noted 29.5), of which 20 us is the rows' way through HBM; 64-row steps 40 us)

// ---------------------------------------------------------------------------------------
// Kernel 1: T[unit][g] = sum over the rows of segment g of kh^T v   (fp32, d_key x d_value;
// K rows are DK wide, V rows DV wide)
// grid = units * n_slots workgroups, workgroup (unit, g) as in the scan kernels: workgroups are
// dealt to the XCDs by their index, and what this kernel reads stays in that XCD's L2 for the
// scan workgroup of the same (unit, g) in the next launch.  Segment g of a unit writes slot g
// of the unit's n_slots slots; segments at or beyond n_compute have no total to form and
// leave at once (the causal forward needs all segments but the last).  With even shares (unit_rows > 0;
// n_slots is not used) a workgroup forms the total of its last piece, unless that ends its unit.  The bidirectional
// path uses it for Kh^T V (row-major slots, TILED = false; the causal scans read theirs tile
// by tile, TILED = true).
template <int DK, int DV, int C, bool TILED>
COTTN_KERNEL((C * 4), fwd_segment_state)
    const elem_t* __restrict__ K, const elem_t* __restrict__ V, float* __restrict__ seg_state,
    int N, Divisor n_slots, int n_compute, Divisor seg_rows, float inv_eps,
    const int* __restrict__ seq_len, Divisor H, int units, Divisor unit_rows) {
  using Cfg = FwdCfg<DK, DV, C>;
  using ST = AccTiles<DK, DV, Cfg::NW>;   // key rows, value columns
  using StageK = TileStage<DK, C, Cfg::NT>;
  using StageV = TileStage<DV, C, Cfg::NT>;
  COTTN_LDS_ARRAY(lds_t, Ks, Cfg::TILEK, 0)
  COTTN_LDS_ARRAY(lds_t, Vs, Cfg::TILEV, 1)

  Unparted un;
  fetch_argument_now(K, V, seg_state, N, n_slots, n_compute, seg_rows, inv_eps, seq_len, H, units, unit_rows);
  const Span span = unit_rows == 0 ? span_of_workgroup<false, false>(units, N, n_slots, seg_rows, unit_rows)
                                   : span_of_workgroup<true, true>(units, N, n_slots, seg_rows, unit_rows);
  const int unit = span.unit;
  if (unit_rows == 0 ? span.slot - span.outermost >= n_compute : !span.mid_unit) {
    if (unit_rows > 0 && span.slot == int(gridDim.x) - 1 && threadIdx.x == 0)
      seg_state[size_t(span.slot) * DK * DV] = EVEN_MARK;
    return;
  }
  const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid / 64), l = tid % 64,
            r = l % 16, q4 = l / 16;
  const elem_t* Ku = K + size_t(unit) * N * DK;
  const elem_t* Vu = V + size_t(unit) * N * DV;
  const int row_begin = span.begin;
  const int row_end = min(valid_rows(seq_len, unit, H, N), span.end);

  f32x4 acc[ST::NCT][ST::NRT];   // layout: add_rows_to_state
#pragma unroll
  for (int x = 0; x < ST::NCT; ++x)
#pragma unroll
    for (int y = 0; y < ST::NRT; ++y) acc[x][y] = f32x4{0.f, 0.f, 0.f, 0.f};

  StageK kst;
  StageV vst;
  kst.fetch(Ku, row_begin, row_end);
  vst.fetch(Vu, row_begin, row_end);
  add_rows_to_state<DK, DV, C, Cfg::NT>(acc, kst, vst, Ks, Vs, Ku, Vu, row_begin, row_end, inv_eps, w, l, un);
  if (ST::active(w)) {
    float* out = seg_state + size_t(span.slot) * DK * DV;
#pragma unroll
    for (int x = 0; x < ST::NCT; ++x) un.results<ST::NRT>(acc[x]);
#pragma unroll
    for (int x = 0; x < ST::NCT; ++x)
#pragma unroll
      for (int y = 0; y < ST::NRT; ++y)
        store_state_words(out + (TILED ? tiled_state_offset(ST::row_tile(w, y), ST::col_tile(w, x), DV / 16, l)
                                       : (16 * ST::row_tile(w, y) + r) * DV + 16 * ST::col_tile(w, x) + 4 * q4),
                          acc[x][y]);
  }
#ifdef COTTN_SPLIT3
  __syncthreads();
  if (un.in_workgroup<Cfg::NW>(Ks)) {
    using Whole = f32w::FwdCfg<DK, DV, C>;
    static_assert(2 * Whole::TILEK <= Cfg::TILEK && 2 * Whole::TILEV <= Cfg::TILEV, "whole rows fit");
    void* const room[] = {Ks, Vs};
    f32w::fwd_segment_state<DK, DV, C, TILED>(room, K, V, seg_state, N, n_slots, n_compute, seg_rows, inv_eps, seq_len,
                                              H, units, unit_rows);
  }
#endif
}

// ---------------------------------------------------------------------------------------
// Kernel 2: in place, per (unit, element): slot g <- sum of slots < g (exclusive prefix
// along the segment axis); slot n_slots-1 never held a total and only receives its prefix.
#ifndef COTTN_REDO
__global__ __launch_bounds__(256) void fwd_state_carry(float* __restrict__ seg_state, int n_slots,
                                                       int elems_per_state, long total) {
  const long idx = (long(blockIdx.x) * 256 + threadIdx.x) * 4;  // 4 elements per thread
  if (idx >= total) return;
  const long unit = idx / elems_per_state, e = idx % elems_per_state;
  exclusive_running_sum(seg_state + unit * n_slots * elems_per_state + e, n_slots,
                        size_t(elems_per_state), false);
}
#endif

// ---------------------------------------------------------------------------------------
// Kernel 3: the chunk scan of one segment.
// The running state is held TRANSPOSED in the accumulators: tile (y, x) of the wave covers
// value rows 16*row_tile(y).. and key columns 16*col_tile(x)..; element [v] of lane (r, q4)
// is S[key 16ct + r][value 16rt + 4 q4 + v].  That way a lane holds 4 consecutive values
// of one key row, which it publishes to the row-major LDS copy Sl[key][value] with one
// 8-byte write, and the update's row-side operand is the V fragment already read for P V.
//
// CS = 2 puts two waves on every 16-row group: both form the masked similarity tile of the
// group, each accumulates one half of the output columns and owns the state tiles whose
// value side is that half.  Per-wave work and registers shrink; the workgroup has twice the
// waves to cover latencies with.
//
// LDV > DV (one segment): a workgroup takes DV of the LDV value columns, which the whole computation
// leaves apart from one another but for the masked tiles; those are formed LDV / DV times.
template <int DK, int DV, int C, int CS, int WALK, int LDV = DV>
COTTN_KERNEL((C * 4 * CS, (FwdCfg<DK, DV, C>::template waves_per_eu<CS>())), fwd_causal_scan)
    const elem_t* __restrict__ Q, const elem_t* __restrict__ K, const elem_t* __restrict__ V,
    const float* __restrict__ s, elem_t* __restrict__ O, float* __restrict__ state_out,
    float* __restrict__ seg_states, const float* __restrict__ state_in, Divisor H, Divisor G,
    Divisor seg_rows, Divisor unit_rows, int N, int units, float inv_eps, int flags,
    const int* __restrict__ lengths) {
  using Cfg = FwdCfg<DK, DV, C>;
  constexpr bool EVEN = walks_even(WALK);
  constexpr int RG = C / 16;           // row groups of a chunk
  constexpr int NOT = Cfg::DTV / CS;   // output column tiles per wave
  using ST = SplitTiles<DV, DK, RG, CS>;   // value rows, key columns (the state is held transposed)
  using StageK = TileStage<DK, C, Cfg::NT * CS>;
  using StageV = TileStage<DV, C, Cfg::NT * CS, LDV>;
  constexpr int TPK = Cfg::TPK, TPV = Cfg::TPV, SP = Cfg::SP;
  constexpr bool OWN_STAGE = CS > 1 || Cfg::OWN_STAGE;
  COTTN_LDS_ARRAY(lds_t, Qs, Cfg::TILEK, 0)   // raw q rows
  COTTN_LDS_ARRAY(lds_t, Ks, Cfg::TILEK, 1)   // kh = r_j k_j
  COTTN_LDS_ARRAY(lds_t, Vs, Cfg::TILEV, 2)   // raw v rows
  COTTN_LDS_ARRAY(lds_t, Sl, Cfg::STATE, 3)   // state, [d_key][d_value]
  // with two waves on a row group the q rows stay live in the other wave, and with outputs
  // wider than the queries they do not fit the q rows: own staging tile
  COTTN_LDS_ARRAY(elem_t, Os, OWN_STAGE ? C * Cfg::OP : 8, 4)
  COTTN_LDS_ARRAY(float, rq, C, 5)
  constexpr int SETS = WALK == OWN_PREFIX_SETS ? Cfg::PREFIX_SETS : 1;
  COTTN_LDS_ARRAY(lds_t, Ps, SETS > 1 ? Cfg::PREFIX_TILES : 8, 6)   // v and kh of further steps of an own prefix
  constexpr bool HALF_VISIBLE = F32_WHOLE && CS == 2 && C == 32, SHARE_MASKED = HALF_VISIBLE && !REDO;
  __shared__ MaskedExchange<SHARE_MASKED ? 2 : 0> masked;   // P tiles of the two key halves
  constexpr bool SKIP_UNSEEN = skips_unseen(CS, C);
  Unparted un;
  fetch_argument_now(Q, K, V, s, O, state_out, seg_states, state_in, H, G, seg_rows, unit_rows, N, units, inv_eps, flags,
                     lengths);
  const bool sum_totals = flags & SUM_TOTALS, s_per_unit = flags & SCALE_PER_UNIT, stream_q = flags & STREAM_Q,
             stream_kv = flags & STREAM_KV;
  const int* seq_len = WALK == EVEN_SHARES ? nullptr : lengths;
  Span span;
  int part = 0;
  if constexpr (LDV > DV) {
    span = Span{0, 0, N, 0, 0, 0, false};
    constexpr int PARTS = LDV / DV;   // numbered as segments are: those of a unit on one XCD
    const int index = blockIdx.x, whole = units & ~7, in_group = index % (8 * PARTS), rest = index - whole * PARTS;
    span.unit = rest < 0 ? index / (8 * PARTS) * 8 + in_group % 8 : whole + rest / PARTS;
    part = rest < 0 ? in_group / 8 : rest % PARTS;
  } else {
    span = span_of_workgroup<false, EVEN>(units, N, G, seg_rows, unit_rows);
  }
  int unit = span.unit;
  const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid / 64), l = tid % 64,
            r = l % 16, q4 = l / 16;
  const int rg = row_group<RG, CS>(w), cp = w / RG;  // row group, column part
  const elem_t* Qu = Q + size_t(unit) * N * DK;   // (of the rows fetched next, from there on)
  const elem_t* Ku = K + size_t(unit) * N * DK;
  const elem_t* Vu = V + size_t(unit) * N * LDV + part * DV;
  elem_t* Ou = O + size_t(unit) * N * LDV + part * DV;
  const int row_begin = span.begin;
  int row_end = max(row_begin, min(valid_rows(seq_len, unit, H, N), span.end));   // of the piece walked
  int piece_end = span.end;   // of the same, with the rows that do not exist

  // running state in fp32 accumulators, seeded with the segment's prefix ([d_key][d_value])
  // seg_states holds either the carried prefixes (slot g = state at the start of segment g)
  // or, with sum_totals set, the raw segment totals: then the workgroup adds up the totals of
  // the segments before its own (few segments: cheaper than a separate carry launch).
  f32x4 sacc[ST::NCT][ST::NRT];
#pragma unroll
  for (int x = 0; x < ST::NCT; ++x)
#pragma unroll
    for (int y = 0; y < ST::NRT; ++y) sacc[x][y] = f32x4{0.f, 0.f, 0.f, 0.f};
  // the first chunk's rows and the stored states are all requested before anything waits
  StageK qst, kst;
  StageV vst;
  qst.fetch(Qu, row_begin, row_end, stream_q);
  kst.fetch(Ku, row_begin, row_end, stream_kv);
  vst.fetch(Vu, row_begin, row_end, stream_kv);
  float scale = unit_scale(s, unit, H, s_per_unit);
  // the state the sequence starts from (chunked prefill) belongs to every segment's start state
  f32x4 start[ST::NCT][ST::NRT];
  const auto load_start = [&] {
    const float* src = state_in + size_t(unit) * DK * LDV + part * DV;
#pragma unroll
    for (int x = 0; x < ST::NCT; ++x)
#pragma unroll
      for (int y = 0; y < ST::NRT; ++y)
        start[x][y] = *reinterpret_cast<const f32x4*>(src + (16 * ST::col_tile(rg, cp, x) + r) * LDV +
                                                      16 * ST::row_tile(rg, cp, y) + 4 * q4);
  };
  const auto add_start = [&] {
#pragma unroll
    for (int x = 0; x < ST::NCT; ++x)
#pragma unroll
      for (int y = 0; y < ST::NRT; ++y)
#pragma unroll
        for (int v = 0; v < 4; ++v) sacc[x][y][v] += start[x][y][v];
  };
  // the state after the last row of a unit
  const auto store_final = [&] {
    float* out = state_out + size_t(unit) * DK * LDV + part * DV;
#pragma unroll
    for (int x = 0; x < ST::NCT; ++x) un.results<ST::NRT>(sacc[x]);
#pragma unroll
    for (int x = 0; x < ST::NCT; ++x)
#pragma unroll
      for (int y = 0; y < ST::NRT; ++y)
        *reinterpret_cast<f32x4*>(out + (16 * ST::col_tile(rg, cp, x) + r) * LDV +
                                  16 * ST::row_tile(rg, cp, y) + 4 * q4) = sacc[x][y];
  };
  if (state_in != nullptr && ST::active(rg, cp)) load_start();
  if constexpr (even_shares_built(DK, DV, ELEM_IS_F32) && WALK == SEGMENTS && LDV == DV)
    if (G == 1 && seg_states != nullptr && blockIdx.x == 0 && tid == 0) *seg_states = NO_EVEN_MARK;
  if constexpr (walks_own_prefix(WALK)) {
    if (span.mid_unit) {
      lds_t *k_tiles[SETS], *v_tiles[SETS];
#pragma unroll
      for (int i = 0; i < SETS; ++i) {
        k_tiles[i] = i == 0 ? Ks : i == 1 ? Qs : Ps + (SETS - 1) * Cfg::TILEV + (i - 2) * Cfg::TILEK;
        v_tiles[i] = i == 0 ? Vs : Ps + (i - 1) * Cfg::TILEV;
      }
      add_rows_before<DK, DV, C, Cfg::NT * CS, ST::NCT, ST::NRT, LDV, SETS>(
          k_tiles, v_tiles, Ku, Vu, min(row_begin, valid_rows(seq_len, unit, H, N)), inv_eps, l, ST::active(rg, cp),
          [&](int x) { return ST::col_tile(rg, cp, x); }, [&](int y) { return ST::row_tile(rg, cp, y); },
          [&](int x, int y, const frag8& kf, const frag8& vf) { sacc[x][y] = mma16_add(vf, kf, sacc[x][y]); },
          un);
      // for the backward, where a carry launch would have left it
      if (ST::active(rg, cp)) {
#pragma unroll
        for (int x = 0; x < ST::NCT; ++x) un.results<ST::NRT>(sacc[x]);
#pragma unroll
        for (int x = 0; x < ST::NCT; ++x)
#pragma unroll
          for (int y = 0; y < ST::NRT; ++y)
            store_state_words(seg_states + size_t(span.slot) * DK * DV +
                                  tiled_state_offset(ST::col_tile(rg, cp, x), ST::row_tile(rg, cp, y), DV / 16, l),
                              sacc[x][y]);
      }
    }
  } else if (LDV == DV && seg_states != nullptr && span.mid_unit && ST::active(rg, cp)) {
    const float* src = seg_states + 4 * l;
    add_stored_states<ST::STATE_BATCH, ST::STATE_MANY>(
        sacc, sum_totals ? span.outermost : span.slot, sum_totals ? span.slot - 1 : span.slot,
        [&](int slot, int x, int y) {
          return *reinterpret_cast<const f32x4*>(
              src + size_t(slot) * DK * DV +
              tiled_state_offset(ST::col_tile(rg, cp, x), ST::row_tile(rg, cp, y), DV / 16, 0));
        });
  }
  if (state_in != nullptr && ST::active(rg, cp)) add_start();

  RowPieces<DV, NOT> finished;  // output rows of the previous chunk, stored one chunk late
#pragma unroll
  for (int j = 0; j < RowPieces<DV, NOT>::PER_LANE; ++j) finished.v[j] = uint4{0u, 0u, 0u, 0u};
  void* stage = OWN_STAGE ? static_cast<void*>(Os + 16 * rg * Cfg::OP) : static_cast<void*>(Qs + 16 * rg * TPK);
  const int col0 = 16 * NOT * cp;  // first output column of this wave
  elem_t* done_O = Ou;
  int done_row = 0, done_end = 0, row0 = row_begin, left = span.left;   // done_end = 0: nothing finished yet
  for (bool more = WALK == EVEN_PADDED || row0 < row_end; more;) {
    // ---- publish the state (bf16) and this chunk's tiles
    if (ST::active(rg, cp)) {
#pragma unroll
      for (int x = 0; x < ST::NCT; ++x)
#pragma unroll
        for (int y = 0; y < ST::NRT; ++y) {
          store4_lds(Sl + (16 * ST::col_tile(rg, cp, x) + r) * SP + lds_col(16 * ST::row_tile(rg, cp, y)) + 4 * q4,
                     sacc[x][y][0], sacc[x][y][1], sacc[x][y][2], sacc[x][y][3], un);
        }
    }
    {
      float rk[StageK::PASSES], rqv[StageK::PASSES];
      qst.row_rinv(inv_eps, rqv);
      kst.row_rinv(inv_eps, rk);
      qst.commit_plain(Qs, un);
      qst.store_rinv(rq, rqv);
      kst.commit_scaled(Ks, rk, un);
      vst.commit_plain(Vs, un);
    }
    // the next step's rows: of this unit, or the first ones of the next
    const bool cross = EVEN && left > 0 && row0 + C >= row_end;
    const int next_row = cross ? 0 : row0 + C;
    const int next_end = cross ? min(valid_rows(seq_len, unit + 1, H, N), left) : row_end;
    more = (WALK == EVEN_PADDED && cross) || next_row < next_end;
    if (cross) {
      Qu += size_t(N) * DK;
      Ku += size_t(N) * DK;
      Vu += size_t(N) * LDV;
    }
    if (more) {
      qst.fetch(Qu, next_row, next_end, stream_q);
      kst.fetch(Ku, next_row, next_end, stream_kv);
      vst.fetch(Vu, next_row, next_end, stream_kv);
    }
    if (done_end > 0)
      store_row_pieces<DV, NOT, LDV>(finished, done_O, done_row + 16 * rg, done_end, l, col0);
    __syncthreads();

    if constexpr (SHARE_MASKED) {
      // this wave's half of the features of the masked tiles (key half 1 is masked for rg = 0)
#pragma unroll
      for (int half = 0; half < 2; ++half)
        if (half <= rg)
          masked.put(half, w, l, row_products<Cfg::KSK>(Ks + (16 * half + r) * TPK, Qs + (16 * rg + r) * TPK,
                                                        16 * Cfg::KSK * cp, q4));
    }

    // ---- inter-chunk part: O^T += S^T Q^T (contraction over d_key = rows of Sl)
    frag8 qf[Cfg::KSK];  // q rows of this wave: column-side operand of every product
#pragma unroll
    for (int ks = 0; ks < Cfg::KSK; ++ks)
      qf[ks] = lds_row_frag(Qs + (16 * rg + r) * TPK + lds_col(32 * ks), q4);
    // oacc[nt][v] = O[query 16 rg + r][value col0 + 16 nt + 4 q4 + v] before the row factor
    f32x4 oacc[NOT];
#pragma unroll
    for (int nt = 0; nt < NOT; ++nt) oacc[nt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < Cfg::KSK; ++ks) {
      frag8 sf[NOT];
#pragma unroll
      for (int nt = 0; nt < NOT; ++nt)
        sf[nt] = lds_col_frag_ks(Sl, SP, ks, q4, col0 + 16 * nt, r);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int nt = 0; nt < NOT; ++nt) oacc[nt] = mma16(sf[nt], qf[ks], oacc[nt]);
      __builtin_amdgcn_sched_barrier(0);
    }
    // ---- intra-chunk part and state update, two key tiles (32 tokens) at a time
#pragma unroll
    for (int p = 0; p < Cfg::NP; ++p) {
      const bool diag_or_below = 2 * p <= rg;  // wave-uniform: else every key is masked
      // k slot (q4, e) of the P fragment is token 32p + 16*(e/4) + 4*q4 + e%4; V and K are
      // read down their rows in the same order
      const int t0 = 32 * p + 4 * q4, t1 = 32 * p + 16 + 4 * q4;
      frag8 vc[NOT], kcol[ST::NCT], vrow[ST::NRT], kr[2][Cfg::KSK];
#pragma unroll
      for (int nt = 0; nt < NOT; ++nt) vc[nt] = lds_col_frag(Vs, TPV, t0, t1, col0 + 16 * nt, r);
#pragma unroll
      for (int x = 0; x < ST::NCT; ++x)
        kcol[x] = lds_col_frag(Ks, TPK, t0, t1, 16 * ST::col_tile(rg, cp, x), r);
      if (!ST::ROW_OPERAND_IS_RESULT_COLUMN) {
#pragma unroll
        for (int y = 0; y < ST::NRT; ++y)
          vrow[y] = lds_col_frag(Vs, TPV, t0, t1, 16 * ST::row_tile(rg, cp, y), r);
      }
      if (diag_or_below && !SHARE_MASKED) {
#pragma unroll
        for (int half = 0; half < 2; ++half)
#pragma unroll
          for (int ks = 0; ks < Cfg::KSK; ++ks) {
            if (SKIP_UNSEEN && half > rg) break;
            kr[half][ks] = lds_row_frag(Ks + (16 * (2 * p + half) + r) * TPK + lds_col(32 * ks), q4);
          }
      }
      if (SHARE_MASKED) __syncthreads();  // the partial tiles of the other waves are there
      __builtin_amdgcn_sched_barrier(0);
      if (diag_or_below) {
        frag8 pf;
#pragma unroll
        for (int half = 0; half < 2; ++half) {
          const int jt = 2 * p + half;
          if (SKIP_UNSEEN && half > rg) {
            put_no_half(pf, half);
            break;
          }
          f32x4 pacc = {0.f, 0.f, 0.f, 0.f};
          if constexpr (SHARE_MASKED) {
            if (half <= rg) pacc = masked.get(half, w, l);
          } else {
#pragma unroll
            for (int ks = 0; ks < Cfg::KSK; ++ks) pacc = mma16(kr[half][ks], qf[ks], pacc);
          }
          // pacc[v] = q_(16 rg + r) . k_(16jt + 4*q4 + v); keep key <= query
          const bool full = jt < rg, diag = jt == rg;
          put_half(pf, half, pacc, full || (diag && 4 * q4 + 0 <= r), full || (diag && 4 * q4 + 1 <= r),
                   full || (diag && 4 * q4 + 2 <= r), full || (diag && 4 * q4 + 3 <= r), un);
        }
        if (HALF_VISIBLE && rg == 0) {
#pragma unroll
          for (int nt = 0; nt < NOT; ++nt) oacc[nt] = mma16_half_add(vc[nt], pf, oacc[nt], 0);
        } else {
#pragma unroll
          for (int nt = 0; nt < NOT; ++nt) oacc[nt] = mma16_add(vc[nt], pf, oacc[nt]);
        }
      }
      // state update S^T += v^T kh over these 32 tokens
      if (ST::active(rg, cp)) {
#pragma unroll
        for (int y = 0; y < ST::NRT; ++y)
#pragma unroll
          for (int x = 0; x < ST::NCT; ++x)
            sacc[x][y] = mma16_add(ST::ROW_OPERAND_IS_RESULT_COLUMN ? vc[y] : vrow[y], kcol[x], sacc[x][y]);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    // ---- O rows: factor s_h r_i, staged through the wave's own (now dead) rows of Qs, or
    // through its part of the staging tile
    const float row_factor = scale * rq[16 * rg + r];
    wave_lds_sync();
    gather_rows_transposed<DV, NOT>(oacc, row_factor, stage, l, finished, un, col0);
    __syncthreads();  // all reads of Ks, Vs, Sl done before the next chunk overwrites them
    done_O = Ou;
    done_row = row0;
    done_end = row_end;
    if (cross) {   // the unit ends here
      if (state_out != nullptr && ST::active(rg, cp)) store_final();
      if (seq_len != nullptr) zero_rows<DV, LDV>(Ou, row_end, N);
      piece_end = min(N, left);
      ++unit;
      left -= unit_rows;
      Ou += size_t(N) * LDV;
      scale = unit_scale(s, unit, H, s_per_unit);
#pragma unroll
      for (int x = 0; x < ST::NCT; ++x)
#pragma unroll
        for (int y = 0; y < ST::NRT; ++y) sacc[x][y] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (state_in != nullptr && ST::active(rg, cp)) {
        load_start();
        add_start();
      }
    }
    row0 = next_row;
    row_end = next_end;
  }
  if (done_end > 0) store_row_pieces<DV, NOT, LDV>(finished, done_O, done_row + 16 * rg, done_end, l, col0);

  if (seq_len != nullptr) zero_rows<DV, LDV>(Ou, row_end, piece_end);  // rows that do not exist

  if (state_out != nullptr && piece_end == N && ST::active(rg, cp)) store_final();
#ifdef COTTN_SPLIT3
  if (un.in_workgroup<RG * CS>(rq)) {
    using Whole = f32w::FwdCfg<DK, DV, C>;
    static_assert(2 * Whole::TILEK <= Cfg::TILEK && 2 * Whole::TILEV <= Cfg::TILEV && 2 * Whole::STATE <= Cfg::STATE &&
                      CS == 2 && Whole::OP == Cfg::OP,
                  "whole rows fit, and finished ones are staged alike");
    void* const room[] = {Qs, Ks, Vs, Sl, Os, rq, Ps};
    f32w::fwd_causal_scan<DK, DV, C, CS, WALK, LDV>(room, Q, K, V, s, O, state_out, seg_states, state_in, H, G, seg_rows,
                                                    unit_rows, N, units, inv_eps, flags, lengths);
  }
#endif
}

#ifndef COTTN_REDO
template <int DK, int DV, int C>
hipError_t run_fwd_causal(const CausalArgs& a) {
  const int units = a.B * a.H;
  const elem_t* Q = static_cast<const elem_t*>(a.Q);
  const elem_t* K = static_cast<const elem_t*>(a.K);
  const elem_t* V = static_cast<const elem_t*>(a.V);
  float* ws = static_cast<float*>(a.workspace);  // [units][G] states of DK x DV (tiled) when G > 1
  const float inv_eps = 1.0f / a.eps;
  hipError_t err = hipSuccess;
  // few segments: no carry launch, each scan workgroup adds up the totals before its segment
  const bool even = a.unit_rows > 0;
  const bool sum_in_scan = even || causal_totals_in_place(units, a.G, DK, DV, ELEM_IS_F32);
  if ((a.G > 1 || even) && !a.own_prefix) {
    err = COTTN_ELEM_SYM(launch_fwd_segment_totals)(a, ws);
    if (err != hipSuccess) return err;
    if (!sum_in_scan) {
      err = launch_fwd_state_carry(ws, units, a.G, DK * DV, a.stream);
      if (err != hipSuccess) return err;
    }
  }
  // Q rows are read once here.  When the call's four tensors exceed the 256 MB last-level cache
  // nothing of them survives until a backward call either, and loading them non-temporally
  // keeps the K, V rows the totals kernel left in the L2 in place (long context: scan 98 ->
  // 87 us); below that size a backward that follows finds the rows cached, and plain loads win.
  const bool stream_q = 2.0 * units * double(a.N) * (DK + DV) * ELEM > 256.0 * 1024 * 1024;
  // Nobody reads K and V before them where there is one segment: non-temporally too once they outgrow
  // that cache by themselves (256 sequences of 2048 rows, 16 heads of 128: 1660 -> 1610 us; 64 of 1000
  // rows d64, whose K, V are found cached in part: 85 -> 105).
  const bool stream_kv = a.G == 1 && !even && 2.0 * units * double(a.N) * (DK + DV) * ELEM > 1024.0 * 1024 * 1024;
  float* states = a.G > 1 || even ? ws : nullptr;
  if (a.marked && !even) states = ws + (a.slots - 1) * DK * DV;   // (only the mark)
  const int flags = (sum_in_scan ? SUM_TOTALS : 0) | (a.s_per_unit ? SCALE_PER_UNIT : 0) | (stream_q ? STREAM_Q : 0) |
                    (stream_kv ? STREAM_KV : 0);
  const auto scan = [&](auto kernel, int threads, int parts = 1) {
    static_assert(argument_bytes(decltype(kernel){}) <= 128, "argument_bytes");
    return launch_kernel(COTTN_SYM_STR(fwd_causal_scan), kernel, dim3(a.workgroups * parts), dim3(threads), 0, a.stream, Q, K,
                         V, a.s, static_cast<elem_t*>(a.O), a.state, states, a.state_in, a.H,
                         a.G, a.seg_rows, a.unit_rows, a.N, units, inv_eps, flags, a.seq_len);
  };
  constexpr int threads = 4 * C * FwdSplit<DK, DV, C>::CS;
  if constexpr (DV == 128 && !F32_WHOLE) {
    const int parts = a.G == 1 && !even ? value_parts(units, a.N, DK) : 1;
    if constexpr (ELEM_IS_F32) {
      if (parts > 1) return scan(COTTN_SYM(fwd_causal_scan)<DK, 64, 32, 2, SEGMENTS, DV>, 256, 2);
    } else {
      if constexpr (DK == 128) {
        if (parts == 4 && a.N <= 32) return scan(COTTN_SYM(fwd_causal_scan)<DK, 32, 32, 2, SEGMENTS, DV>, 256, 4);
        if (parts == 4) return scan(COTTN_SYM(fwd_causal_scan)<DK, 32, 64, 1, SEGMENTS, DV>, 256, 4);
      }
      if (parts > 1) return scan(COTTN_SYM(fwd_causal_scan)<DK, 64, 64, 1, SEGMENTS, DV>, 256, 2);
    }
  }
  if constexpr (!ELEM_IS_F32 && DK == 128 && DV == 128)
    if (!even && !a.own_prefix && two_to_a_cu_forward(a.workgroups)) return scan(COTTN_SYM(fwd_causal_scan)<DK, DV, 32, 2, SEGMENTS>, 256);
  if constexpr (even_shares_built(DK, DV, ELEM_IS_F32))
    if (even)
      return a.seq_len == nullptr
                 ? scan(COTTN_SYM(fwd_causal_scan)<DK, DV, C, FwdSplit<DK, DV, C>::CS, EVEN_SHARES>, threads)
                 : scan(COTTN_SYM(fwd_causal_scan)<DK, DV, C, FwdSplit<DK, DV, C>::CS, EVEN_PADDED>, threads);
  if constexpr (C <= 64)
    if (a.own_prefix) {
      if constexpr (FwdCfg<DK, DV, C>::PREFIX_SETS > 1)
        if (prefix_by_sets(a.workgroups))
          return scan(COTTN_SYM(fwd_causal_scan)<DK, DV, C, FwdSplit<DK, DV, C>::CS, OWN_PREFIX_SETS>, threads);
      return scan(COTTN_SYM(fwd_causal_scan)<DK, DV, C, FwdSplit<DK, DV, C>::CS, OWN_PREFIX>, threads);
    }
  return scan(COTTN_SYM(fwd_causal_scan)<DK, DV, C, FwdSplit<DK, DV, C>::CS, SEGMENTS>, threads);
}
#endif  // COTTN_REDO

}  // namespace
}  // namespace COTTN_NS

#ifndef COTTN_REDO
using namespace COTTN_NS;

template <int DK, int DV, bool TILED>
static hipError_t run_segment_totals(const SegmentTotalsArgs& t) {
  const elem_t* X = static_cast<const elem_t*>(t.X);
  const elem_t* Y = static_cast<const elem_t*>(t.Y);
  const float inv_eps = 1.0f / t.eps;
  // The totals kernel takes 128-row tiles when the segment is that long: a 512-thread
  // workgroup has all of its loads in flight at once instead of paying one memory latency per
  // 64-row chunk, and several workgroups still fit a compute unit (two 256-row tiles of the
  // operand-tile pitch would leave room for one: measured 0.6 us slower on the GPT shape;
  // fp32 rows in parts fit twice only with 64 rows, but 32 x 32 and 32 x 64).
  const dim3 grid(t.unit_rows > 0 ? t.workgroups : t.units * t.G);
  constexpr bool TALL = LDS_ELEM * 128 * (lds_pitch(DK) + lds_pitch(DV)) <= 80 * 1024;
  if constexpr (TALL)
    if (t.seg_rows >= 128)
      return launch_kernel(COTTN_SYM_STR(fwd_segment_state), COTTN_SYM(fwd_segment_state)<DK, DV, 128, TILED>, grid, dim3(512),
                         0, t.stream, X, Y, t.dst, t.N, t.G, t.n_compute, t.seg_rows, inv_eps,
                         t.seq_len, t.H, t.units, t.unit_rows);
  return launch_kernel(COTTN_SYM_STR(fwd_segment_state), COTTN_SYM(fwd_segment_state)<DK, DV, 64, TILED>, grid, dim3(256), 0,
                       t.stream, X, Y, t.dst, t.N, t.G, t.n_compute, t.seg_rows, inv_eps, t.seq_len, t.H,
                       t.units, t.unit_rows);
}

#ifdef COTTN_F32_WHOLE
hipError_t launch_segment_totals_32x32_f32w(const SegmentTotalsArgs& t) {
  return t.tiled ? run_segment_totals<32, 32, true>(t) : run_segment_totals<32, 32, false>(t);
}
#else
hipError_t COTTN_SYM(launch_segment_totals)(const SegmentTotalsArgs& t) {
  switch (t.dk * 1000 + t.dv) {
#ifdef COTTN_ELEM_F32   // device_common.h: SPLIT3
    case 32032: return launch_segment_totals_32x32_f32w(t);
#else
    case 32032: return t.tiled ? run_segment_totals<32, 32, true>(t) : run_segment_totals<32, 32, false>(t);
#endif
    case 32064: return t.tiled ? run_segment_totals<32, 64, true>(t) : run_segment_totals<32, 64, false>(t);
    case 32128: return t.tiled ? run_segment_totals<32, 128, true>(t) : run_segment_totals<32, 128, false>(t);
    case 64032: return t.tiled ? run_segment_totals<64, 32, true>(t) : run_segment_totals<64, 32, false>(t);
    case 64064: return t.tiled ? run_segment_totals<64, 64, true>(t) : run_segment_totals<64, 64, false>(t);
    case 64128: return t.tiled ? run_segment_totals<64, 128, true>(t) : run_segment_totals<64, 128, false>(t);
    case 128032: return t.tiled ? run_segment_totals<128, 32, true>(t) : run_segment_totals<128, 32, false>(t);
    case 128064: return t.tiled ? run_segment_totals<128, 64, true>(t) : run_segment_totals<128, 64, false>(t);
    case 128128: return t.tiled ? run_segment_totals<128, 128, true>(t) : run_segment_totals<128, 128, false>(t);
    default: return hipErrorInvalidValue;
  }
}

hipError_t COTTN_SYM(launch_fwd_segment_totals)(const CausalArgs& a, float* dst) {
  SegmentTotalsArgs t{};
  t.X = a.K; t.Y = a.V; t.dst = dst;
  t.units = a.B * a.H; t.N = a.N; t.dk = a.dk; t.dv = a.dv; t.G = a.G; t.n_compute = a.G - 1;
  t.seg_rows = a.seg_rows; t.eps = a.eps; t.stream = a.stream;
  t.seq_len = a.seq_len; t.H = a.H; t.unit_rows = a.unit_rows; t.workgroups = a.workgroups;
  t.tiled = true;  // read by the scan kernels only
  return COTTN_SYM(launch_segment_totals)(t);
}
#endif

#if !defined(COTTN_ELEM_F16) && !defined(COTTN_ELEM_F32)  // not specific to the element type
hipError_t launch_fwd_state_carry(float* seg_state, int units, int G, int elems, hipStream_t st) {
  const long total = long(units) * elems;
  return launch_kernel("fwd_state_carry", fwd_state_carry, dim3(unsigned((total / 4 + 255) / 256)),
                       dim3(256), 0, st, seg_state, G, elems, total);
}
#endif

hipError_t COTTN_SYM(fwd_causal)(const CausalArgs& a) {
#if defined(COTTN_F32_WHOLE)
  switch ((a.dk * 1000 + a.dv) * 1000 + a.C) {
    case 32128032: return run_fwd_causal<32, 128, 32>(a);
    case 128032032: return run_fwd_causal<128, 32, 32>(a);
    case 128128032: return run_fwd_causal<128, 128, 32>(a);
    default: return hipErrorInvalidValue;
  }
#elif defined(COTTN_ELEM_F32)
  switch ((a.dk * 1000 + a.dv) * 1000 + a.C) {
    case 32032032: return run_fwd_causal<32, 32, 32>(a);
    case 32064032: return run_fwd_causal<32, 64, 32>(a);
    case 32128032: case 128032032: case 128128032: return fwd_causal_f32w(a);   // device_common.h: SPLIT3
    case 64032032: return run_fwd_causal<64, 32, 32>(a);
    case 64064032: return run_fwd_causal<64, 64, 32>(a);
    case 64128032: return run_fwd_causal<64, 128, 32>(a);
    case 128064032: return run_fwd_causal<128, 64, 32>(a);
    default: return hipErrorInvalidValue;
  }
#else
  // d_key != d_value: chunks of 64 rows
  switch ((a.dk * 1000 + a.dv) * 1000 + a.C) {
    case 32032064: return run_fwd_causal<32, 32, 64>(a);
    case 32032128: return run_fwd_causal<32, 32, 128>(a);
    case 32032256: return run_fwd_causal<32, 32, 256>(a);
    case 64064064: return run_fwd_causal<64, 64, 64>(a);
    case 64064128: return run_fwd_causal<64, 64, 128>(a);
    case 64064256: return run_fwd_causal<64, 64, 256>(a);
    case 128128064: return run_fwd_causal<128, 128, 64>(a);
    case 32064064: return run_fwd_causal<32, 64, 64>(a);
    case 32128064: return run_fwd_causal<32, 128, 64>(a);
    case 64032064: return run_fwd_causal<64, 32, 64>(a);
    case 64128064: return run_fwd_causal<64, 128, 64>(a);
    case 128032064: return run_fwd_causal<128, 32, 64>(a);
    case 128064064: return run_fwd_causal<128, 64, 64>(a);
    default: return hipErrorInvalidValue;
  }
#endif
}

#endif  // COTTN_REDO

}  // namespace cottn
