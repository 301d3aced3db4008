// Bidirectional cosine attention, forward and backward: MFMA products with fp32 accumulation
// (gfx950).  Written against an element type: this file builds the bfloat16 kernels, the IEEE
// half ones when it is included with COTTN_ELEM_F16 defined and the fp32 ones with
// COTTN_ELEM_F32.
//
// Sec. 4 eq. subQuadCos: without a mask the product reassociates to O = s_h Qh (Kh^T V), so
// the d x d matrix S = Kh^T V is reduced once over the whole sequence and then applied to
// every query row.  The gradient formulas of Sec. 4 with M removed collapse the same way:
// with G = Qh^T dO (also d x d),
//     dQh = s dO S^T,   dKh = s V G^T,   dV = s Kh G,   ds = <S, G> (Frobenius product),
// followed by the chain rule through the row normalisation.
//
// Launches per call:
//   forward   totals: the segment-totals kernel of the causal forward reduces Kh^T V over one
//             segment of rows per workgroup (split over the sequence because B*H alone may not
//             fill the chip); apply: streams the Q rows and multiplies them with S;
//   backward  first sweep (Q, dO -> dQ): dQ needs only S, which the forward left behind, so
//             the sweep that has to read Q and dO for G = Qh^T dO forms dQ on the way and
//             leaves G's segment totals and the shares of ds (= sum_i qh_i . dqh_i, the same
//             number as <S, G>); second sweep (K, V -> dK, dV) applies G.  Every row of the
//             seven tensors is moved once.  A backward that was not handed the forward's
//             totals reduces Kh^T V first;
//   by unit   16-bit rows, short sequences or many of them: the two launches of a call are one.
//   combine   only with many segments: sums the segment totals per (batch, head) into slot 0;
//             with few, the kernels add the totals up themselves while staging them.
//
// The apply kernels follow the scheme of the causal kernels: raw rows as MFMA operands,
// normalisation factors on result rows, results accumulated transposed and staged through
// the wave's own (dead) tile rows, stores one chunk late.
#include "device_common.h"
#include "launch.h"
#include "tile_io.h"
#include "workspace.h"

namespace cottn {
namespace COTTN_NS {
namespace {

// DK, DV: head dimensions of queries / keys and of values / outputs (Sec. 2.1); the matrices
// S = Kh^T V and G = Qh^T dO are DK x DV.
template <int DK, int DV, int C>
struct BiCfg {
  static constexpr int NW = C / 16;
  static constexpr int NT = NW * 64;
  static constexpr int DTK = DK / 16, DTV = DV / 16;
  static constexpr int KSK = DK / 32, KSV = DV / 32;
  static constexpr int TPK = tile_pitch(DK, C), TPV = tile_pitch(DV, C);   // operand tiles
  // the DK x DV matrices are written once per workgroup and then only read, as row fragments
  // too: they take the operand tiles' pitch
  static constexpr int SP = tile_pitch(DV, C);
  static constexpr int TILEK = C * TPK, TILEV = C * TPV;
  static constexpr int STATE = DK * SP;
  // Whether a backward sweep over segments asks for the scale before its first rows, as the forwards do.  Behind them
  // that is one request less to wait for (most backwards take 0.2 to 0.7 us less), but the
  // compiler waits for it where it is first used, in the loop, and with it in every step for the rows of the next one.  The
  // forwards lose by that (scale behind / before: 20 sequences of 18749 rows of 32 f16 23.0 / 21.2 us, 48 of
  // 7621 bf16 21.5 / 20.1, 24 of 7380 at 64 x 64 21.8 / 21.3, 384 of 512 by workgroup 18.0 / 17.8), and of the backwards those
  // of narrow 16-bit values, whose steps are short (34.2 / 33.1, 43.6 / 42.5; short sequences there give 0.3 back, 8 of 437 at
  // 64 x 32 7.4 / 7.7; 64 x 64 45.9 / 45.9, fp32 36 of 197 13.9 / 14.2).
  static constexpr bool BWD_SCALE_FIRST = !ELEM_IS_F32 && DV == 32;
  // the forward stages finished output rows (DV wide) in the wave's own dead query rows when
  // those are wide enough, else in a tile of their own
  static constexpr bool FWD_OWN_STAGE = ELEM * stage_pitch(DV) > LDS_ELEM * TPK;
  // the dQ sweep stages finished rows in a tile of their own when the LDS has room for it,
  // otherwise behind a barrier in the dead dO tile (fp32 with wide heads); SPLIT3: when that does
  // not cost a workgroup, otherwise in the dead Q tile, whose rows are always wide enough
  static constexpr int DQ_BYTES = LDS_ELEM * (TILEK + TILEV + STATE) + 8 * C;
  static constexpr int DQ_STAGE_BYTES = ELEM * C * stage_tile_pitch(DK, C);
  static constexpr bool DQ_STAGE_IN_Q = SPLIT3 || REDO;
  static constexpr bool DQ_OWN_STAGE =
      REDO ? false :
      SPLIT3 ? 160 * 1024 / (DQ_BYTES + DQ_STAGE_BYTES) == 160 * 1024 / DQ_BYTES
             : ELEM * stage_pitch(DK) > LDS_ELEM * TPV || DQ_BYTES + DQ_STAGE_BYTES <= 160 * 1024;
};

// Slot 0 <- sum over g of the slots, one matrix element per thread (grid: elems/256 workgroups
// per (batch, head)); `state` (may be null) receives it too.
#ifndef COTTN_REDO
__global__ __launch_bounds__(256) void bidir_combine(float* __restrict__ totals, int G, int elems,
                                                     float* __restrict__ state) {
  // one grid dimension: (unit, 256-element block of the matrix), so that B*H is not limited to
  // the 65535 of the other grid dimensions
  const int blocks_per_unit = elems / 256;
  const int unit = blockIdx.x / blocks_per_unit, blk = blockIdx.x % blocks_per_unit;
  const int e = blk * 256 + threadIdx.x;
  float* p = totals + size_t(unit) * G * elems;
  float a = 0.f;
  constexpr int BATCH = 16;   // loads in flight per thread
  for (int g0 = 0; g0 < G; g0 += BATCH) {
    float t[BATCH];
#pragma unroll
    for (int i = 0; i < BATCH; ++i) t[i] = g0 + i < G ? p[size_t(g0 + i) * elems + e] : 0.f;
#pragma unroll
    for (int i = 0; i < BATCH; ++i) a += t[i];
  }
  p[e] = a;
  if (state != nullptr) state[size_t(unit) * elems + e] = a;
}
#endif

// dst (LDS, elements, row-major [DK][DV] with row pitch SP) <- sum of the first n_sum of the
// [DK][DV] fp32 matrices at src; the fp32 sum also goes to `copy` when that is not null.
template <int DK, int DV, int NT, int SP>
__device__ __forceinline__ void stage_summed_matrix(lds_t* dst, const float* __restrict__ src,
                                                    int n_sum, float* __restrict__ copy, Unparted& un) {
  // up to 16 of a thread's loads are in flight before the first is waited for: PIECES pieces of
  // BATCH matrices (a batch that reaches beyond the last matrix re-reads it and drops it)
  constexpr int PASSES = DK * DV / (4 * NT), PIECES = PASSES < 1 ? 1 : PASSES < 4 ? PASSES : 4;
  constexpr int BATCH = 16 / PIECES < 4 ? 16 / PIECES : 4;
  static_assert(PASSES % PIECES == 0, "whole passes of the workgroup (or less than one)");
  for (int e0 = 4 * threadIdx.x; e0 < DK * DV; e0 += 4 * NT * PIECES) {
    f32x4 sum[PIECES];
#pragma unroll
    for (int i = 0; i < PIECES; ++i) sum[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int j0 = 0; j0 < n_sum; j0 += BATCH) {
      f32x4 t[BATCH][PIECES];
#pragma unroll
      for (int b = 0; b < BATCH; ++b)
#pragma unroll
        for (int i = 0; i < PIECES; ++i)
          t[b][i] = *reinterpret_cast<const f32x4*>(src + size_t(min(j0 + b, n_sum - 1)) * DK * DV + e0 +
                                                    4 * NT * i);
#pragma unroll
      for (int b = 0; b < BATCH; ++b) {
        const bool keep = j0 + b < n_sum;
#pragma unroll
        for (int i = 0; i < PIECES; ++i)
#pragma unroll
          for (int v = 0; v < 4; ++v) sum[i][v] += keep ? t[b][i][v] : 0.f;
      }
    }
#pragma unroll
    for (int i = 0; i < PIECES; ++i) {
      const int e = e0 + 4 * NT * i;
      if (copy != nullptr) *reinterpret_cast<f32x4*>(copy + e) = sum[i];
      store4_lds(dst + (e / DV) * SP + lds_col(e % DV), sum[i][0], sum[i][1], sum[i][2], sum[i][3], un);
    }
  }
}

// O_i = s r_i (q_i S) for the rows row_begin .. row_end - 1 of one unit, with S in Sl (not yet
// behind a barrier); the first C rows have been fetched.  Own: staging tile, or null.
template <int DK, int DV, int C>
__device__ __forceinline__ void apply_rows(TileStage<DK, C, BiCfg<DK, DV, C>::NT>& qst, lds_t* Qs, const lds_t* Sl,
                                           elem_t* Os, float* rq, const elem_t* __restrict__ Qu,
                                           elem_t* __restrict__ Ou, float scale, int row_begin, int row_end,
                                           float inv_eps, int w, int l, Unparted& un) {
  using Cfg = BiCfg<DK, DV, C>;
  using Stage = TileStage<DK, C, Cfg::NT>;
  constexpr int TP = Cfg::TPK, SP = Cfg::SP;
  const int r = l % 16, q4 = l / 16;
  RowPieces<DV> finished;  // output rows of the previous chunk, stored one chunk late
#pragma unroll
  for (int j = 0; j < RowPieces<DV>::PER_LANE; ++j) finished.v[j] = uint4{0u, 0u, 0u, 0u};
  void* stage = Cfg::FWD_OWN_STAGE ? static_cast<void*>(Os + 16 * w * stage_tile_pitch(DV, C))
                                   : static_cast<void*>(Qs + 16 * w * TP);
  for (int row0 = row_begin; row0 < row_end; row0 += C) {
    {
      float rqv[Stage::PASSES];
      qst.row_rinv(inv_eps, rqv);
      qst.commit_plain(Qs, un);
      qst.store_rinv(rq, rqv);
    }
    if (row0 + C < row_end) qst.fetch(Qu, row0 + C, row_end);
    if (row0 > row_begin) store_row_pieces<DV>(finished, Ou, row0 - C + 16 * w, row_end, l);
    __syncthreads();
    // oacc[nt][v] = (q S)[query 16w + r][value 16 nt + 4 q4 + v]
    f32x4 oacc[Cfg::DTV];
#pragma unroll
    for (int nt = 0; nt < Cfg::DTV; ++nt) oacc[nt] = f32x4{0.f, 0.f, 0.f, 0.f};
    frag8 qf[Cfg::KSK], sf[Cfg::KSK][Cfg::DTV];
#pragma unroll
    for (int ks = 0; ks < Cfg::KSK; ++ks) {
      qf[ks] = lds_row_frag(Qs + (16 * w + r) * TP + lds_col(32 * ks), q4);
#pragma unroll
      for (int nt = 0; nt < Cfg::DTV; ++nt)
        sf[ks][nt] = lds_col_frag_ks(Sl, SP, ks, q4, 16 * nt, r);
    }
    __builtin_amdgcn_sched_barrier(0);  // all LDS reads are issued before the first MFMA
#pragma unroll
    for (int ks = 0; ks < Cfg::KSK; ++ks)
#pragma unroll
      for (int nt = 0; nt < Cfg::DTV; ++nt) oacc[nt] = mma16(sf[ks][nt], qf[ks], oacc[nt]);
    __builtin_amdgcn_sched_barrier(0);
    const float row_factor = scale * rq[16 * w + r];
    wave_lds_sync();  // this wave's reads of its Qs rows precede the staging writes
    gather_rows_transposed<DV>(oacc, row_factor, stage, l, finished, un);
    __syncthreads();
  }
  if (row_begin < row_end) {
    const int last = row_begin + (row_end - row_begin - 1) / C * C;
    store_row_pieces<DV>(finished, Ou, last + 16 * w, row_end, l);
  }
}

// O rows of one segment: O_i = s r_i (q_i S), accumulated as O^T = S^T Q^T.  `totals` holds
// n_sum stored matrices per unit at a stride of `slots` matrices; the workgroup of segment 0
// writes their sum to `state` when that is asked for.
template <int DK, int DV, int C>
COTTN_KERNEL((C * 4), fwd_bidir_apply)
    const elem_t* __restrict__ Q, const float* __restrict__ s, elem_t* __restrict__ O,
    const float* __restrict__ totals, int slots, int n_sum, float* __restrict__ state, Divisor H, int N,
    Divisor G, int seg_rows, float inv_eps, const int* __restrict__ seq_len, int s_per_unit, int units) {
  using Cfg = BiCfg<DK, DV, C>;
  using Stage = TileStage<DK, C, Cfg::NT>;
  COTTN_LDS_ARRAY(lds_t, Qs, Cfg::TILEK, 0)  // raw q
  COTTN_LDS_ARRAY(lds_t, Sl, Cfg::STATE, 1)  // [d_key][d_value]
  COTTN_LDS_ARRAY(elem_t, Os, Cfg::FWD_OWN_STAGE ? C * stage_tile_pitch(DV, C) : 8, 2)
  COTTN_LDS_ARRAY(float, rq, C, 3)

  Unparted un;
  fetch_argument_now(Q, s, O, totals, slots, n_sum, state, H, N, G, seg_rows, inv_eps, seq_len,
                     s_per_unit, units);
  int unit, g;
  unit_and_segment(blockIdx.x, units, G, unit, g);
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), l = threadIdx.x % 64;
  const elem_t* Qu = Q + size_t(unit) * N * DK;
  elem_t* Ou = O + size_t(unit) * N * DV;
  const float scale = unit_scale(s, unit, H, s_per_unit);
  const int row_begin = g * seg_rows;
  const int seg_end = min(N, row_begin + seg_rows);
  const int row_end = max(row_begin, min(valid_rows(seq_len, unit, H, N), seg_end));

  Stage qst;
  qst.fetch(Qu, row_begin, row_end);
  stage_summed_matrix<DK, DV, Cfg::NT, Cfg::SP>(Sl, totals + size_t(unit) * slots * DK * DV, n_sum,
                                  (state != nullptr && g == 0) ? state + size_t(unit) * DK * DV
                                                               : nullptr, un);

  apply_rows<DK, DV, C>(qst, Qs, Sl, Cfg::FWD_OWN_STAGE ? Os : nullptr, rq, Qu, Ou, scale, row_begin, row_end,
                        inv_eps, w, l, un);
  if (seq_len != nullptr) zero_rows<DV>(Ou, row_end, seg_end);  // rows that do not exist
#ifdef COTTN_SPLIT3
  if (un.in_workgroup<Cfg::NW>(rq)) {
    using Whole = f32w::BiCfg<DK, DV, C>;
    static_assert(2 * Whole::TILEK <= Cfg::TILEK && 2 * Whole::STATE <= Cfg::STATE &&
                  Whole::FWD_OWN_STAGE == Cfg::FWD_OWN_STAGE, "whole rows fit, and finished ones are staged alike");
    void* const room[] = {Qs, Sl, Os, rq};
    f32w::fwd_bidir_apply<DK, DV, C>(room, Q, s, O, totals, slots, n_sum, state, H, N, G, seg_rows, inv_eps, seq_len, s_per_unit, units);
  }
#endif
}

// dQ rows row_begin .. row_end - 1 of one unit, with S in Sl (not yet behind a barrier); the first C
// rows have been fetched.  Adds the rows' Qh^T dO to racc (element [v] of lane (r, q4) is
// G[key 16 ct + r][value 16 rt + 4 q4 + v]) and their qh . dqh to ds_lane of the first lane row.
template <int DK, int DV, int C, class RT = AccTiles<DV, DK, C / 16>>
__device__ __forceinline__ void dq_rows(TileStage<DK, C, BiCfg<DK, DV, C>::NT>& qst,
                                        TileStage<DV, C, BiCfg<DK, DV, C>::NT>& gst,
                                        f32x4 (&racc)[RT::NCT][RT::NRT], float& ds_lane, lds_t* Qs, lds_t* Gs,
                                        elem_t* Os, const lds_t* Sl, float* rq, const elem_t* __restrict__ Qu,
                                        const elem_t* __restrict__ Gu, elem_t* __restrict__ dQu, float scale,
                                        int row_begin, int row_end, float inv_eps, int w, int l, Unparted& un) {
  using Cfg = BiCfg<DK, DV, C>;
  using StageK = TileStage<DK, C, Cfg::NT>;
  constexpr int TPK = Cfg::TPK, TPV = Cfg::TPV, SP = Cfg::SP;
  const int r = l % 16, q4 = l / 16;
  RowPieces<DK> finished;  // dQ rows of the previous chunk, stored one chunk late
#pragma unroll
  for (int j = 0; j < RowPieces<DK>::PER_LANE; ++j) finished.v[j] = uint4{0u, 0u, 0u, 0u};
  for (int row0 = row_begin; row0 < row_end; row0 += C) {
    {
      float rqv[StageK::PASSES];
      qst.row_rinv(inv_eps, rqv);
      qst.commit_scaled(Qs, rqv, un);
      qst.store_rinv(rq, rqv);
      gst.commit_plain(Gs, un);
    }
    if (row0 + C < row_end) {
      qst.fetch(Qu, row0 + C, row_end);
      gst.fetch(Gu, row0 + C, row_end);
    }
    if (row0 > row_begin) store_row_pieces<DK>(finished, dQu, row0 - C + 16 * w, row_end, l);
    __syncthreads();

    // dq[nt][v] = dqh[row 16w + r][key feature 16 nt + 4 q4 + v]
    f32x4 dq[Cfg::DTK];
#pragma unroll
    for (int nt = 0; nt < Cfg::DTK; ++nt) dq[nt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < Cfg::KSV; ++ks) {
      const frag8 gf = lds_row_frag(Gs + (16 * w + r) * TPV + lds_col(32 * ks), q4);
      frag8 srow[Cfg::DTK];
#pragma unroll
      for (int nt = 0; nt < Cfg::DTK; ++nt)
        srow[nt] = lds_row_frag(Sl + (16 * nt + r) * SP + lds_col(32 * ks), q4);
      __builtin_amdgcn_sched_barrier(0);  // all LDS reads are issued before the first MFMA
#pragma unroll
      for (int nt = 0; nt < Cfg::DTK; ++nt) dq[nt] = mma16(srow[nt], gf, dq[nt]);
      __builtin_amdgcn_sched_barrier(0);
    }
    // G^T += dO^T qh over the chunk's tokens, 32 at a time (rows beyond the sequence are zero)
    if (RT::active(w)) {
#pragma unroll
      for (int p = 0; p < C / 32; ++p) {
        const int t0 = 32 * p + 4 * q4, t1 = 32 * p + 16 + 4 * q4;
        frag8 qcol[RT::NCT], grow[RT::NRT];
#pragma unroll
        for (int x = 0; x < RT::NCT; ++x)
          qcol[x] = lds_col_frag(Qs, TPK, t0, t1, 16 * RT::col_tile(w, x), r);
#pragma unroll
        for (int y = 0; y < RT::NRT; ++y)
          grow[y] = lds_col_frag(Gs, TPV, t0, t1, 16 * RT::row_tile(w, y), r);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int y = 0; y < RT::NRT; ++y)
#pragma unroll
          for (int x = 0; x < RT::NCT; ++x) racc[x][y] = mma16_add(grow[y], qcol[x], racc[x][y]);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    const float ri = rq[16 * w + r];
    float xv[Cfg::DTK][4];
    const float t = dot_with_row<Cfg::DTK, TPK>(dq, Qs + 16 * w * TPK, 0, xv, r, q4);
    const float rho = project_out_row<Cfg::DTK, true>(dq, xv, t, ri, inv_eps);
    if (q4 == 0) ds_lane += rho;
    if (!Cfg::DQ_OWN_STAGE) __syncthreads();  // every wave is done with the dO tile
    gather_rows_transposed<DK>(dq, scale * ri,
                               Cfg::DQ_OWN_STAGE ? static_cast<void*>(Os + 16 * w * stage_tile_pitch(DK, C))
                               : Cfg::DQ_STAGE_IN_Q ? static_cast<void*>(Qs + 16 * w * TPK)
                                                 : static_cast<void*>(Gs + 16 * w * TPV),
                               l, finished, un);
    __syncthreads();
  }
  if (row_begin < row_end) {
    const int last = row_begin + (row_end - row_begin - 1) / C * C;
    store_row_pieces<DK>(finished, dQu, last + 16 * w, row_end, l);
  }
}

// Backward, first sweep: dQ rows of one segment and the segment's total of Qh^T dO.  It needs
// only S = Kh^T V, which the forward already reduced, so the rows of Q and dO are read once,
// here, for both dQ and the matrix G that the second sweep applies:
//   dqh^T = S dO^T (over d_value),  dq_i = s r_i (dqh_i - qh_i (qh_i . dqh_i)),
//   G_segment = sum over the rows of qh_i^T dO_i,  ds share = sum of qh_i . dqh_i.
// Q is stored in LDS as qh = r_i q_i: it is contracted over the tokens in G, and the chain
// rule wants the normalised row anyway.  Every wave reads all rows of both tiles (the total
// contracts them over the tokens), so finished dQ rows are staged in a tile of their own where
// that fits.
template <int DK, int DV, int C>
COTTN_KERNEL((C * 4), bwd_bidir_dq)
    const elem_t* __restrict__ Q, const elem_t* __restrict__ dO, const float* __restrict__ s,
    elem_t* __restrict__ dQ, const float* __restrict__ s_totals, int slots, int n_sum,
    float* __restrict__ g_totals, float* __restrict__ ds_partial, Divisor H, int N, Divisor G,
    int seg_rows, float inv_eps, const int* __restrict__ seq_len, int s_per_unit, int units) {
  using Cfg = BiCfg<DK, DV, C>;
  using RT = AccTiles<DV, DK, Cfg::NW>;   // total of Qh^T dO: value rows, key columns
  using StageK = TileStage<DK, C, Cfg::NT>;
  using StageV = TileStage<DV, C, Cfg::NT>;
  COTTN_LDS_ARRAY(lds_t, Qs, Cfg::TILEK, 0)   // qh = r_i q_i
  COTTN_LDS_ARRAY(lds_t, Gs, Cfg::TILEV, 1)   // dO
  COTTN_LDS_ARRAY(elem_t, Os, Cfg::DQ_OWN_STAGE ? C * stage_tile_pitch(DK, C) : 8, 2)   // finished dQ rows
  COTTN_LDS_ARRAY(lds_t, Sl, Cfg::STATE, 3)   // Kh^T V, [d_key][d_value]
  COTTN_LDS_ARRAY(float, rq, C, 4)
  COTTN_LDS_ARRAY(float, ds_wave, Cfg::NW, 5)

  Unparted un;
  fetch_argument_now(Q, dO, s, dQ, s_totals, slots, n_sum, g_totals, ds_partial, H, N, G, seg_rows,
                     inv_eps, seq_len, s_per_unit, units);
  int unit, g;
  unit_and_segment(blockIdx.x, units, G, unit, g);
  const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid / 64), l = tid % 64,
            r = l % 16, q4 = l / 16;
  const elem_t* Qu = Q + size_t(unit) * N * DK;
  const elem_t* Gu = dO + size_t(unit) * N * DV;
  elem_t* dQu = dQ + size_t(unit) * N * DK;
  float scale = 0.f;
  if (Cfg::BWD_SCALE_FIRST) scale = unit_scale(s, unit, H, s_per_unit);
  const int row_begin = g * seg_rows;
  const int seg_end = min(N, row_begin + seg_rows);
  const int row_end = max(row_begin, min(valid_rows(seq_len, unit, H, N), seg_end));

  StageK qst;
  StageV gst;
  qst.fetch(Qu, row_begin, row_end);
  gst.fetch(Gu, row_begin, row_end);
  if (!Cfg::BWD_SCALE_FIRST) scale = unit_scale(s, unit, H, s_per_unit);
  stage_summed_matrix<DK, DV, Cfg::NT, Cfg::SP>(Sl, s_totals + size_t(unit) * slots * DK * DV, n_sum, nullptr, un);

  // racc[x][y]: element [v] of lane (r, q4) is G[key 16 ct + r][value 16 rt + 4 q4 + v]
  f32x4 racc[RT::NCT][RT::NRT];
#pragma unroll
  for (int x = 0; x < RT::NCT; ++x)
#pragma unroll
    for (int y = 0; y < RT::NRT; ++y) racc[x][y] = f32x4{0.f, 0.f, 0.f, 0.f};
  float ds_lane = 0.f;
  dq_rows<DK, DV, C>(qst, gst, racc, ds_lane, Qs, Gs, Cfg::DQ_OWN_STAGE ? Os : nullptr, Sl, rq, Qu, Gu, dQu, scale,
                     row_begin, row_end, inv_eps, w, l, un);
  if (seq_len != nullptr) zero_rows<DK>(dQu, row_end, seg_end);  // rows that do not exist

  if (RT::active(w)) {
    float* out = g_totals + (size_t(unit) * slots + g) * DK * DV;
#pragma unroll
    for (int x = 0; x < RT::NCT; ++x) un.results<RT::NRT>(racc[x]);
#pragma unroll
    for (int x = 0; x < RT::NCT; ++x)
#pragma unroll
      for (int y = 0; y < RT::NRT; ++y)
        store_state_words(out + (16 * RT::col_tile(w, x) + r) * DV + 16 * RT::row_tile(w, y) + 4 * q4,
                          racc[x][y]);
  }
  // the segment's share of ds: lanes of the first lane row hold the row sums
  ds_lane = group_sum<64>(ds_lane);
  if (l == 0) ds_wave[w] = ds_lane;
  __syncthreads();
  if (tid == 0) {
    float t = 0.f;
#pragma unroll
    for (int i = 0; i < Cfg::NW; ++i) t += ds_wave[i];
    ds_partial[size_t(unit) * G + g] = t;
  }
#ifdef COTTN_SPLIT3
  if (un.in_workgroup<Cfg::NW>(rq)) {
    using Whole = f32w::BiCfg<DK, DV, C>;
    static_assert(2 * Whole::TILEK <= Cfg::TILEK && 2 * Whole::TILEV <= Cfg::TILEV && 2 * Whole::STATE <= Cfg::STATE, "whole rows fit");
    void* const room[] = {Qs, Gs, Os, Sl, rq, ds_wave};
    f32w::bwd_bidir_dq<DK, DV, C>(room, Q, dO, s, dQ, s_totals, slots, n_sum, g_totals, ds_partial, H, N, G, seg_rows, inv_eps,
                                  seq_len, s_per_unit, units);
  }
#endif
}

// dK and dV rows row_begin .. row_end - 1 of one unit, with G in Gl (not yet behind a barrier);
// the first C rows have been fetched.
template <int DK, int DV, int C>
__device__ __forceinline__ void dkdv_rows(TileStage<DK, C, BiCfg<DK, DV, C>::NT>& kst,
                                          TileStage<DV, C, BiCfg<DK, DV, C>::NT>& vst, lds_t* Ks, lds_t* Vs,
                                          const lds_t* Gl, float* rk, const elem_t* __restrict__ Ku,
                                          const elem_t* __restrict__ Vu, elem_t* __restrict__ dKu,
                                          elem_t* __restrict__ dVu, float scale, int row_begin, int row_end,
                                          float inv_eps, int w, int l, Unparted& un) {
  using Cfg = BiCfg<DK, DV, C>;
  using StageK = TileStage<DK, C, Cfg::NT>;
  constexpr int TPK = Cfg::TPK, TPV = Cfg::TPV, SP = Cfg::SP;
  const int r = l % 16, q4 = l / 16;
  RowPieces<DK> done_k;  // rows of the previous chunk, stored one chunk late
  RowPieces<DV> done_v;
#pragma unroll
  for (int j = 0; j < RowPieces<DK>::PER_LANE; ++j) done_k.v[j] = uint4{0u, 0u, 0u, 0u};
#pragma unroll
  for (int j = 0; j < RowPieces<DV>::PER_LANE; ++j) done_v.v[j] = uint4{0u, 0u, 0u, 0u};
  for (int row0 = row_begin; row0 < row_end; row0 += C) {
    {
      float rkv[StageK::PASSES];
      kst.row_rinv(inv_eps, rkv);
      kst.commit_plain(Ks, un);
      kst.store_rinv(rk, rkv);
      vst.commit_plain(Vs, un);
    }
    if (row0 + C < row_end) {
      kst.fetch(Ku, row0 + C, row_end);
      vst.fetch(Vu, row0 + C, row_end);
    }
    if (row0 > row_begin) {
      store_row_pieces<DK>(done_k, dKu, row0 - C + 16 * w, row_end, l);
      store_row_pieces<DV>(done_v, dVu, row0 - C + 16 * w, row_end, l);
    }
    __syncthreads();

    // d*[nt][v] = result[row 16w + r][feature 16 nt + 4 q4 + v]
    f32x4 dk[Cfg::DTK], dv[Cfg::DTV];
#pragma unroll
    for (int nt = 0; nt < Cfg::DTK; ++nt) dk[nt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int nt = 0; nt < Cfg::DTV; ++nt) dv[nt] = f32x4{0.f, 0.f, 0.f, 0.f};
    // G V^T contracts over d_value (row fragments of Gl along its rows)
#pragma unroll
    for (int ks = 0; ks < Cfg::KSV; ++ks) {
      const frag8 vf = lds_row_frag(Vs + (16 * w + r) * TPV + lds_col(32 * ks), q4);
      frag8 grow[Cfg::DTK];
#pragma unroll
      for (int nt = 0; nt < Cfg::DTK; ++nt)
        grow[nt] = lds_row_frag(Gl + (16 * nt + r) * SP + lds_col(32 * ks), q4);
      __builtin_amdgcn_sched_barrier(0);  // all LDS reads are issued before the first MFMA
#pragma unroll
      for (int nt = 0; nt < Cfg::DTK; ++nt) dk[nt] = mma16(grow[nt], vf, dk[nt]);
      __builtin_amdgcn_sched_barrier(0);
    }
    // G^T k^T contracts over d_key (fragments down the rows of Gl)
#pragma unroll
    for (int ks = 0; ks < Cfg::KSK; ++ks) {
      const frag8 kf = lds_row_frag(Ks + (16 * w + r) * TPK + lds_col(32 * ks), q4);
      frag8 gcol[Cfg::DTV];
#pragma unroll
      for (int nt = 0; nt < Cfg::DTV; ++nt)
        gcol[nt] = lds_col_frag_ks(Gl, SP, ks, q4, 16 * nt, r);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int nt = 0; nt < Cfg::DTV; ++nt) dv[nt] = mma16(gcol[nt], kf, dv[nt]);
      __builtin_amdgcn_sched_barrier(0);
    }
    // every tile row is private to its wave here: chain rule on the raw rows, then the
    // results are staged in place (K rows for dK, V rows for dV)
    const float rj = rk[16 * w + r];
    float xv[Cfg::DTK][4];
    const float t = dot_with_row<Cfg::DTK, TPK>(dk, Ks + 16 * w * TPK, 0, xv, r, q4);
    project_out_row<Cfg::DTK, false>(dk, xv, t, rj, inv_eps);
    wave_lds_sync();  // own rows of Ks, Vs were read before the staging writes
    gather_rows_transposed<DK>(dk, scale * rj, Ks + 16 * w * TPK, l, done_k, un);
    gather_rows_transposed<DV>(dv, scale * rj, Vs + 16 * w * TPV, l, done_v, un);
    __syncthreads();
  }
  if (row_begin < row_end) {
    const int last = row_begin + (row_end - row_begin - 1) / C * C;
    store_row_pieces<DK>(done_k, dKu, last + 16 * w, row_end, l);
    store_row_pieces<DV>(done_v, dVu, last + 16 * w, row_end, l);
  }
}

// Backward, second sweep: dK and dV rows of one segment from G = Qh^T dO (the sum of the n_sum
// stored matrices at g_totals); the first H workgroups also finish ds from the n_ds partial
// sums per (batch, head) that the first sweep left.  Accumulated transposed:
//   dkh^T = G V^T (over d_value),  (k G)^T = G^T k^T (over d_key),
//   dk_j = s r_j (dkh_j - kh_j (kh_j . dkh_j)),  dv_j = s r_j (k_j G).
template <int DK, int DV, int C>
COTTN_KERNEL((C * 4), bwd_bidir_dkdv)
    const elem_t* __restrict__ K, const elem_t* __restrict__ V, const float* __restrict__ s,
    elem_t* __restrict__ dK, elem_t* __restrict__ dV, const float* __restrict__ g_totals, int slots,
    int n_sum, const float* __restrict__ ds_partial, int n_ds, float* __restrict__ ds, int B, Divisor H,
    int N, Divisor G, int seg_rows, float inv_eps, const int* __restrict__ seq_len, int s_per_unit) {
  using Cfg = BiCfg<DK, DV, C>;
  using StageK = TileStage<DK, C, Cfg::NT>;
  using StageV = TileStage<DV, C, Cfg::NT>;
  COTTN_LDS_ARRAY(lds_t, Ks, Cfg::TILEK, 0)   // raw k
  COTTN_LDS_ARRAY(lds_t, Vs, Cfg::TILEV, 1)
  COTTN_LDS_ARRAY(lds_t, Gl, Cfg::STATE, 2)   // Qh^T dO, [d_key][d_value]
  COTTN_LDS_ARRAY(float, rk, C, 3)

  Unparted un;
  fetch_argument_now(K, V, s, dK, dV, g_totals, slots, n_sum, ds_partial, n_ds, ds, B, H, N, G,
                     seg_rows, inv_eps, seq_len, s_per_unit);
  int unit, g;
  unit_and_segment(blockIdx.x, B * H, G, unit, g);
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), l = threadIdx.x % 64;
  const elem_t* Ku = K + size_t(unit) * N * DK;
  const elem_t* Vu = V + size_t(unit) * N * DV;
  elem_t* dKu = dK + size_t(unit) * N * DK;
  elem_t* dVu = dV + size_t(unit) * N * DV;
  float scale = 0.f;
  if (Cfg::BWD_SCALE_FIRST) scale = unit_scale(s, unit, H, s_per_unit);
  const int row_begin = g * seg_rows;
  const int seg_end = min(N, row_begin + seg_rows);
  const int row_end = max(row_begin, min(valid_rows(seq_len, unit, H, N), seg_end));

  StageK kst;
  StageV vst;
  kst.fetch(Ku, row_begin, row_end);
  vst.fetch(Vu, row_begin, row_end);
  if (!Cfg::BWD_SCALE_FIRST) scale = unit_scale(s, unit, H, s_per_unit);

  // ds[h] = sum of the shares of all batches (ds[b][h], one batch, with a scale per unit)
  if (int(blockIdx.x) < (s_per_unit ? B * H.n : H.n) && w == 0) {
    float t = 0.f;
    const int n = s_per_unit ? n_ds : B * n_ds;
    for (int i = l; i < n; i += 64)
      t += s_per_unit ? ds_partial[size_t(blockIdx.x) * n_ds + i]
                      : ds_partial[(size_t(i / n_ds) * H + blockIdx.x) * n_ds + (i % n_ds)];
    t = group_sum<64>(t);
    if (l == 0) ds[blockIdx.x] = t;
  }
  stage_summed_matrix<DK, DV, Cfg::NT, Cfg::SP>(Gl, g_totals + size_t(unit) * slots * DK * DV, n_sum, nullptr, un);

  dkdv_rows<DK, DV, C>(kst, vst, Ks, Vs, Gl, rk, Ku, Vu, dKu, dVu, scale, row_begin, row_end, inv_eps, w, l, un);
  if (seq_len != nullptr) {  // rows that do not exist
    zero_rows<DK>(dKu, row_end, seg_end);
    zero_rows<DV>(dVu, row_end, seg_end);
  }
#ifdef COTTN_SPLIT3
  if (un.in_workgroup<Cfg::NW>(rk)) {
    using Whole = f32w::BiCfg<DK, DV, C>;
    static_assert(2 * Whole::TILEK <= Cfg::TILEK && 2 * Whole::TILEV <= Cfg::TILEV && 2 * Whole::STATE <= Cfg::STATE, "whole rows fit");
    void* const room[] = {Ks, Vs, Gl, rk};
    f32w::bwd_bidir_dkdv<DK, DV, C>(room, K, V, s, dK, dV, g_totals, slots, n_sum, ds_partial, n_ds, ds, B, H, N, G, seg_rows,
                                    inv_eps, seq_len, s_per_unit);
  }
#endif
}

// ---------------------------------------------------------------------------------------
// 16-bit rows, short sequences or many of them (launch.h: bidir_by_unit): a whole (batch, head) per
// workgroup, forward and backward in one launch each.  Split over launches such a call is in large
// part launches, first loads and the matrix on its way through the workspace into every workgroup
// (16 KB of fp32 for each segment's 64 x 64 total, 32 KB of rows behind it).  128-row steps and eight
// waves keep the walk short; B16 H12 N389 f16 with lengths from a quarter of N up: forward 14.7 -> 10.6
// us, backward 21.4 -> 17.9; B32 H12 N512 bf16 22 -> 18.5 and 36 -> 32 us, 5.4 TB/s of its rows.
#ifndef COTTN_ELEM_F32
// Forward: S = Kh^T V over the sequence in the accumulators, published to LDS (and to the workspace,
// for the backward), then applied to the Q rows.
template <int DK, int DV, int C>
__global__ __launch_bounds__(C * 4) void COTTN_SYM(fwd_bidir_unit)(
    const elem_t* __restrict__ Q, const elem_t* __restrict__ K, const elem_t* __restrict__ V,
    const float* __restrict__ s, elem_t* __restrict__ O, float* __restrict__ totals,
    float* __restrict__ state, Divisor H, int N, float inv_eps, const int* __restrict__ seq_len,
    int s_per_unit) {
  using Cfg = BiCfg<DK, DV, C>;
  using ST = AccTiles<DK, DV, Cfg::NW>;   // key rows, value columns
  constexpr int SP = Cfg::SP;
  __shared__ __attribute__((aligned(16))) lds_t Ks[Cfg::TILEK];   // kh, then raw q
  __shared__ __attribute__((aligned(16))) lds_t Vs[Cfg::TILEV];   // v, then finished rows
  __shared__ __attribute__((aligned(16))) lds_t Sl[Cfg::STATE];   // [d_key][d_value]
  __shared__ float rq[C];

  Unparted un;
  fetch_argument_now(Q, K, V, s, O, totals, state, H, N, inv_eps, seq_len, s_per_unit);
  const int unit = blockIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), l = threadIdx.x % 64, r = l % 16, q4 = l / 16;
  const elem_t* Qu = Q + size_t(unit) * N * DK;
  const elem_t* Ku = K + size_t(unit) * N * DK;
  const elem_t* Vu = V + size_t(unit) * N * DV;
  elem_t* Ou = O + size_t(unit) * N * DV;
  const float scale = unit_scale(s, unit, H, s_per_unit);
  const int row_end = valid_rows(seq_len, unit, H, N);

  f32x4 acc[ST::NCT][ST::NRT];   // layout: add_rows_to_state
#pragma unroll
  for (int x = 0; x < ST::NCT; ++x)
#pragma unroll
    for (int y = 0; y < ST::NRT; ++y) acc[x][y] = f32x4{0.f, 0.f, 0.f, 0.f};
  TileStage<DK, C, Cfg::NT> kst, qst;
  TileStage<DV, C, Cfg::NT> vst;
  kst.fetch(Ku, 0, row_end);
  vst.fetch(Vu, 0, row_end);
  qst.fetch(Qu, 0, row_end);
  add_rows_to_state<DK, DV, C, Cfg::NT>(acc, kst, vst, Ks, Vs, Ku, Vu, 0, row_end, inv_eps, w, l, un);
  if (ST::active(w)) {
#pragma unroll
    for (int x = 0; x < ST::NCT; ++x)
#pragma unroll
      for (int y = 0; y < ST::NRT; ++y) {
        const int key = 16 * ST::row_tile(w, y) + r, value = 16 * ST::col_tile(w, x) + 4 * q4;
        store4(Sl + key * SP + value, acc[x][y][0], acc[x][y][1], acc[x][y][2], acc[x][y][3]);
        const size_t at = size_t(unit) * DK * DV + key * DV + value;
        store_state_words(totals + at, acc[x][y]);
        if (state != nullptr) *reinterpret_cast<f32x4*>(state + at) = acc[x][y];
      }
  }
  __syncthreads();  // every wave is done with the K and V tiles
  apply_rows<DK, DV, C>(qst, Ks, Sl, Cfg::FWD_OWN_STAGE ? Vs : nullptr, rq, Qu, Ou, scale, 0, row_end, inv_eps, w, l, un);
  if (seq_len != nullptr) zero_rows<DV>(Ou, row_end, N);  // rows that do not exist
}

// Backward: the dQ sweep with G = Qh^T dO in the accumulators, G published to LDS in the place of S,
// then the dK/dV sweep.  The unit's share of ds goes to ds_out[unit]: ds itself where a scale belongs
// to one unit, else a partial sum for bidir_sum_ds.
template <int DK, int DV, int C>
__global__ __launch_bounds__(C * 4) void COTTN_SYM(bwd_bidir_unit)(
    const elem_t* __restrict__ Q, const elem_t* __restrict__ K, const elem_t* __restrict__ V,
    const elem_t* __restrict__ dO, const float* __restrict__ s, elem_t* __restrict__ dQ,
    elem_t* __restrict__ dK, elem_t* __restrict__ dV, const float* __restrict__ s_totals,
    float* __restrict__ ds_out, Divisor H, int N, float inv_eps, const int* __restrict__ seq_len,
    int s_per_unit) {
  using Cfg = BiCfg<DK, DV, C>;
  using RT = AccTiles<DV, DK, Cfg::NW>;   // total of Qh^T dO: value rows, key columns
  constexpr int SP = Cfg::SP;
  __shared__ __attribute__((aligned(16))) lds_t Qs[Cfg::TILEK];   // qh, then raw k
  __shared__ __attribute__((aligned(16))) lds_t Gs[Cfg::TILEV];   // dO, then v
  __shared__ __attribute__((aligned(16))) elem_t Os[Cfg::DQ_OWN_STAGE ? C * stage_tile_pitch(DK, C) : 8];   // finished dQ rows
  __shared__ __attribute__((aligned(16))) lds_t Sl[Cfg::STATE];   // Kh^T V, then Qh^T dO, [d_key][d_value]
  __shared__ float rq[C];
  __shared__ float ds_wave[Cfg::NW];

  Unparted un;
  fetch_argument_now(Q, K, V, dO, s, dQ, dK, dV, s_totals, ds_out, H, N, inv_eps, seq_len, s_per_unit);
  const int unit = blockIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), l = threadIdx.x % 64, r = l % 16, q4 = l / 16;
  const size_t k_rows = size_t(unit) * N * DK, v_rows = size_t(unit) * N * DV;
  const int row_end = valid_rows(seq_len, unit, H, N);

  TileStage<DK, C, Cfg::NT> qst, kst;
  TileStage<DV, C, Cfg::NT> gst, vst;
  qst.fetch(Q + k_rows, 0, row_end);
  gst.fetch(dO + v_rows, 0, row_end);
  const float scale = unit_scale(s, unit, H, s_per_unit);
  stage_summed_matrix<DK, DV, Cfg::NT, SP>(Sl, s_totals + size_t(unit) * DK * DV, 1, nullptr, un);
  f32x4 racc[RT::NCT][RT::NRT];
#pragma unroll
  for (int x = 0; x < RT::NCT; ++x)
#pragma unroll
    for (int y = 0; y < RT::NRT; ++y) racc[x][y] = f32x4{0.f, 0.f, 0.f, 0.f};
  float ds_lane = 0.f;
  dq_rows<DK, DV, C>(qst, gst, racc, ds_lane, Qs, Gs, Cfg::DQ_OWN_STAGE ? Os : nullptr, Sl, rq, Q + k_rows,
                     dO + v_rows, dQ + k_rows, scale, 0, row_end, inv_eps, w, l, un);
  kst.fetch(K + k_rows, 0, row_end);
  vst.fetch(V + v_rows, 0, row_end);
  if (seq_len != nullptr) zero_rows<DK>(dQ + k_rows, row_end, N);  // rows that do not exist

  ds_lane = group_sum<64>(ds_lane);   // lanes of the first lane row hold the row sums
  if (l == 0) ds_wave[w] = ds_lane;
  __syncthreads();  // (also where the sequence is empty and Sl has only just been staged)
  if (threadIdx.x == 0) {
    float t = 0.f;
#pragma unroll
    for (int i = 0; i < Cfg::NW; ++i) t += ds_wave[i];
    ds_out[unit] = t;
  }
  if (RT::active(w)) {
#pragma unroll
    for (int x = 0; x < RT::NCT; ++x)
#pragma unroll
      for (int y = 0; y < RT::NRT; ++y)
        store4(Sl + (16 * RT::col_tile(w, x) + r) * SP + 16 * RT::row_tile(w, y) + 4 * q4, racc[x][y][0],
               racc[x][y][1], racc[x][y][2], racc[x][y][3]);
  }
  dkdv_rows<DK, DV, C>(kst, vst, Qs, Gs, Sl, rq, K + k_rows, V + v_rows, dK + k_rows, dV + v_rows, scale, 0, row_end,
                       inv_eps, w, l, un);
  if (seq_len != nullptr) {  // rows that do not exist
    zero_rows<DK>(dK + k_rows, row_end, N);
    zero_rows<DV>(dV + v_rows, row_end, N);
  }
}

// ds[h] = sum over the batch of the units' shares (one wave per head)
__global__ __launch_bounds__(64) void bidir_sum_ds(const float* __restrict__ ds_partial, float* __restrict__ ds,
                                                   int B, int H) {
  float t = 0.f;
  for (int b = threadIdx.x; b < B; b += 64) t += ds_partial[size_t(b) * H + blockIdx.x];
  t = group_sum<64>(t);
  if (threadIdx.x == 0) ds[blockIdx.x] = t;
}
#endif  // COTTN_ELEM_F32

#ifndef COTTN_REDO
SegmentTotalsArgs totals_args(const CausalArgs& a, const void* X, const void* Y, float* dst) {
  SegmentTotalsArgs t{};
  t.X = X; t.Y = Y; t.dst = dst;
  t.units = a.B * a.H; t.N = a.N; t.dk = a.dk; t.dv = a.dv; t.G = a.G; t.n_compute = a.G;
  t.seg_rows = a.seg_rows; t.eps = a.eps; t.stream = a.stream;
  t.seq_len = a.seq_len; t.H = a.H;
  return t;
}

template <int DK, int DV, int C>
hipError_t run_fwd_bidir_rows(const CausalArgs& a) {
  const int units = a.B * a.H;
  float* totals = static_cast<float*>(a.workspace);
  // 16-bit 128 x 128 beyond one workgroup per compute unit: one by unit fills a compute unit, and so the
  // second round finds most of them idle; the totals and the apply kernel fit twice, the latter in
  // 64-row steps (by unit or 128-row steps / so: 288 units of 777 rows 79.7 / 73.8 us, 320 of 2048 200 /
  // 185, 896 of 513 151 / 142; up to 256 workgroups the other way round, 256 of 1024 rows 47.7 / 59.4).
  const bool in_rounds = !ELEM_IS_F32 && DK == 128 && DV == 128 && long(units) * a.G > 256;
#ifndef COTTN_ELEM_F32
  if constexpr (C == bidir_step_rows(false))
    if (a.by_unit && !in_rounds)
      return launch_kernel(COTTN_SYM_STR(fwd_bidir_unit), COTTN_SYM(fwd_bidir_unit)<DK, DV, C>, dim3(units),
                           dim3(C * 4), 0, a.stream, static_cast<const elem_t*>(a.Q),
                           static_cast<const elem_t*>(a.K), static_cast<const elem_t*>(a.V), a.s,
                           static_cast<elem_t*>(a.O), totals, a.state, a.H, a.N, 1.0f / a.eps, a.seq_len, a.s_per_unit);
#endif
  hipError_t err = COTTN_ELEM_SYM(launch_segment_totals)(totals_args(a, a.K, a.V, totals));
  if (err != hipSuccess) return err;
  // few segments: the apply workgroups add the totals up themselves (and write `state`)
  const bool sum_in_apply = sum_totals_in_place(a.G, DK, DV);
  if (!sum_in_apply) {
    err = launch_bidir_combine(totals, units, a.G, DK * DV, a.state, a.stream);
    if (err != hipSuccess) return err;
  }
  const auto apply = [&](auto kernel, int rows) {
    return launch_kernel(COTTN_SYM_STR(fwd_bidir_apply), kernel, dim3(units * a.G), dim3(rows * 4), 0, a.stream,
                         static_cast<const elem_t*>(a.Q), a.s, static_cast<elem_t*>(a.O), totals, a.G,
                         sum_in_apply ? a.G : 1, sum_in_apply ? a.state : nullptr, a.H, a.N, a.G, a.seg_rows,
                         1.0f / a.eps, a.seq_len, a.s_per_unit, units);
  };
  if constexpr (!ELEM_IS_F32 && DK == 128 && DV == 128)
    if (in_rounds) return apply(COTTN_SYM(fwd_bidir_apply)<DK, DV, 64>, 64);
  return apply(COTTN_SYM(fwd_bidir_apply)<DK, DV, C>, C);
}

template <int DK, int DV, int C>
hipError_t run_bwd_bidir_rows(const CausalArgs& a) {
  using Cfg = BiCfg<DK, DV, C>;
  const int units = a.B * a.H;
  char* ws = static_cast<char*>(a.workspace);
  float* s_totals = reinterpret_cast<float*>(ws);
  const size_t pair_stride = state_array_bytes(a.B, a.H, DK, DV, a.G) / sizeof(float);
  float* g_totals = s_totals + pair_stride;
  float* ds_partial = reinterpret_cast<float*>(ws + 2 * state_array_bytes(a.B, a.H, DK, DV, a.G));
  // few segments: the sweeps add the segment totals up themselves while staging them; many:
  // the combine kernel leaves the sum in slot 0
  const bool few = sum_totals_in_place(a.G, DK, DV);
  hipError_t err;
  // S = Kh^T V: the totals the forward left behind (slot 0 is their sum already when the
  // forward ran the combine kernel), or reduced here
  const float* s_src = a.saved_fwd_states;
  if (s_src == nullptr) {
    err = COTTN_ELEM_SYM(launch_segment_totals)(totals_args(a, a.K, a.V, s_totals));
    if (err != hipSuccess) return err;
    if (!few) {
      err = launch_bidir_combine(s_totals, units, a.G, DK * DV, nullptr, a.stream);
      if (err != hipSuccess) return err;
    }
    s_src = s_totals;
  }
#ifndef COTTN_ELEM_F32
  if constexpr (C == bidir_step_rows(false))
    if (a.by_unit) {
      // with a scale per unit, or one batch, a unit's share of ds is ds
      const bool whole = a.s_per_unit || a.B == 1;
      err = launch_kernel(COTTN_SYM_STR(bwd_bidir_unit), COTTN_SYM(bwd_bidir_unit)<DK, DV, C>, dim3(units),
                          dim3(C * 4), 0, a.stream, static_cast<const elem_t*>(a.Q),
                          static_cast<const elem_t*>(a.K), static_cast<const elem_t*>(a.V),
                          static_cast<const elem_t*>(a.dO), a.s, static_cast<elem_t*>(a.dQ),
                          static_cast<elem_t*>(a.dK), static_cast<elem_t*>(a.dV), s_src, whole ? a.ds : ds_partial,
                          a.H, a.N, 1.0f / a.eps, a.seq_len, a.s_per_unit);
      if (err != hipSuccess || whole) return err;
      return launch_kernel("bidir_sum_ds", bidir_sum_ds, dim3(a.H), dim3(64), 0, a.stream, ds_partial, a.ds, a.B, a.H);
    }
#endif
  err = launch_kernel(COTTN_SYM_STR(bwd_bidir_dq), COTTN_SYM(bwd_bidir_dq)<DK, DV, C>, dim3(units * a.G),
                      dim3(Cfg::NT), 0, a.stream, static_cast<const elem_t*>(a.Q),
                      static_cast<const elem_t*>(a.dO), a.s, static_cast<elem_t*>(a.dQ), s_src, a.G,
                      few ? a.G : 1, g_totals, ds_partial, a.H, a.N, a.G, a.seg_rows, 1.0f / a.eps,
                      a.seq_len, a.s_per_unit, units);
  if (err != hipSuccess) return err;
  if (!few) {
    err = launch_bidir_combine(g_totals, units, a.G, DK * DV, nullptr, a.stream);
    if (err != hipSuccess) return err;
  }
  return launch_kernel(COTTN_SYM_STR(bwd_bidir_dkdv), COTTN_SYM(bwd_bidir_dkdv)<DK, DV, C>, dim3(units * a.G),
                       dim3(Cfg::NT), 0, a.stream, static_cast<const elem_t*>(a.K),
                       static_cast<const elem_t*>(a.V), a.s, static_cast<elem_t*>(a.dK),
                       static_cast<elem_t*>(a.dV), g_totals, a.G, few ? a.G : 1, ds_partial, a.G, a.ds,
                       a.B, a.H, a.N, a.G, a.seg_rows, 1.0f / a.eps, a.seq_len, a.s_per_unit);
}

// The plan's rows per step: the usual ones, or 64 for very many sequences (launch.h: threads_fit), whose
// states of more than 64 x 64 no card holds.
template <int DK, int DV>
hipError_t run_fwd_bidir(const CausalArgs& a) {
  constexpr int C = bidir_step_rows(ELEM_IS_F32);
  if (a.C == C) return run_fwd_bidir_rows<DK, DV, C>(a);
  if constexpr (DK * DV <= 64 * 64)
    if (a.C == 64) return run_fwd_bidir_rows<DK, DV, 64>(a);
  return hipErrorInvalidValue;
}
template <int DK, int DV>
hipError_t run_bwd_bidir(const CausalArgs& a) {
  constexpr int C = bidir_step_rows(ELEM_IS_F32);
  if (a.C == C) return run_bwd_bidir_rows<DK, DV, C>(a);
  if constexpr (DK * DV <= 64 * 64)
    if (a.C == 64) return run_bwd_bidir_rows<DK, DV, 64>(a);
  return hipErrorInvalidValue;
}
#endif  // COTTN_REDO

}  // namespace
}  // namespace COTTN_NS

#ifndef COTTN_REDO
using namespace COTTN_NS;

#if !defined(COTTN_ELEM_F16) && !defined(COTTN_ELEM_F32)  // not specific to the element type
hipError_t launch_bidir_combine(float* totals, int units, int G, int elems, float* state,
                                hipStream_t st) {
  return launch_kernel("bidir_combine", bidir_combine, dim3(unsigned(elems / 256) * units), dim3(256), 0, st,
                       totals, G, elems, state);
}
#endif

#if defined(COTTN_F32_WHOLE)
hipError_t fwd_bidir_f32w(const CausalArgs& a) {
  return a.dk == 32 ? run_fwd_bidir<32, 32>(a) : run_fwd_bidir<128, 128>(a);
}
hipError_t bwd_bidir_f32w(const CausalArgs& a) {
  return a.dk == 32 ? run_bwd_bidir<32, 32>(a) : run_bwd_bidir<128, 128>(a);
}
#else
#ifdef COTTN_ELEM_F32   // device_common.h: SPLIT3
#define COTTN_SQUARE(D, CALL, WHOLE) WHOLE(a)
#else
#define COTTN_SQUARE(D, CALL, WHOLE) CALL<D, D>(a)
#endif
#define COTTN_FOR_EACH_DK_DV(CALL, WHOLE)                                                       \
  switch (a.dk * 1000 + a.dv) {                                                                 \
    case 32032: return COTTN_SQUARE(32, CALL, WHOLE);                                           \
    case 32064: return CALL<32, 64>(a);                                                         \
    case 32128: return CALL<32, 128>(a);                                                        \
    case 64032: return CALL<64, 32>(a);                                                         \
    case 64064: return CALL<64, 64>(a);                                                         \
    case 64128: return CALL<64, 128>(a);                                                        \
    case 128032: return CALL<128, 32>(a);                                                       \
    case 128064: return CALL<128, 64>(a);                                                       \
    case 128128: return COTTN_SQUARE(128, CALL, WHOLE);                                         \
    default: return hipErrorInvalidValue;                                                       \
  }

hipError_t COTTN_SYM(fwd_bidir)(const CausalArgs& a) { COTTN_FOR_EACH_DK_DV(run_fwd_bidir, fwd_bidir_f32w) }

hipError_t COTTN_SYM(bwd_bidir)(const CausalArgs& a) { COTTN_FOR_EACH_DK_DV(run_bwd_bidir, bwd_bidir_f32w) }
#endif

#endif  // COTTN_REDO

}  // namespace cottn
