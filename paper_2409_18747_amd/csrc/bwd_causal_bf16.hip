// Causal cosine attention backward: MFMA products with fp32 accumulation (gfx950).
// Written against an element type: this file builds the bfloat16 kernels, the IEEE half ones
// when it is included with COTTN_ELEM_F16 defined and the fp32 ones with COTTN_ELEM_F32.
//
// Sec. 4 gives, for the normalised operands Qh, Kh (A = dO V^T, P = Qh Kh^T, M the
// lower-triangular mask),
//     dQh = (A (.) M) Kh,    dKh = (A (.) M)^T Qh,    dV = (P (.) M)^T dO,
// and notes that dQh is a cumulative sum running forward in time while dKh and dV use one
// running backward.  With S_t = sum_{j<=t} kh_j^T v_j and R_t = sum_{i>=t} qh_i^T dO_i:
//     dqh_t = s dO_t S_t^T,    dkh_t = s v_t R_t^T,    dv_t = s kh_t R_t.
// Both sums are regrouped exactly into chunks of C rows inside G segments per (batch, head):
//   forward-time states   per-segment totals of Kh^T V (d_key x d_value, stored tile by tile
//             like all states that only these kernels exchange): taken over from the
//             forward call when it hands its workspace on, else rebuilt by the forward's
//             totals kernel; with many segments a carry kernel turns totals into prefixes
//             (and the reverse-time totals into suffixes), with few the scans add them up;
//   dQ scan   forward-time: dQ of a segment, chunk by chunk, first to last; it has Q and dO
//             in LDS anyway and leaves the segment's reverse-time total Qh^T dO behind;
//   dK/dV scan  reverse-time: dK and dV of a segment, chunk by chunk, last to first (so it
//             starts on the rows the dQ scan read last, which are still in the XCD's L2);
//             its first workgroups also add up ds from the dQ scan's partial sums.
//
// Normalisation factors r_i = 1/max(|q_i|, eps), r_j = 1/max(|k_j|, eps) are not applied to
// Q and K element-wise where a row factor does the same:
//   dQ pass    K is contracted over the token index everywhere and is stored as kh = r_j k_j;
//              V stays raw; Q is only needed normalised (for the chain rule below and for
//              the reverse-time total) and is stored as qh;
//              dqh_i = sum_j A_ij kh_j + dO_i S^T,  S = sum kh_j^T v_j;
//   dK/dV pass Q is rescaled to r_i q_i (it is contracted over the token index in the
//              reverse state R = sum (r_i q_i)^T dO_i); K and V stay raw;
//              dv_j = s r_j [ sum_i ((r_i q_i).k_j) dO_i + k_j R ],
//              dkh_j = sum_i A_ij (r_i q_i) + v_j R^T.
// The chain rule through x/max(||x||, eps), with t = x . dxh on the raw row:
//     dx = s r (dxh - x r^2 t) = s r (dxh - xh (xh . dxh))   (rows at or below eps: dx = s r dxh),
// and ds_h = sum over rows of qh_i . dqh_i before scaling by s.
//
// Inside a chunk the masked A and P tiles are produced directly in the register layout the
// next product needs as an operand, so they never pass through LDS; operands contracted
// over the token index are read from the row-major LDS tiles with the transposing LDS read,
// and the fragments read for the intra-chunk products are reused by the state updates.
// Results are accumulated transposed (a lane holds 4 consecutive columns of one result row),
// which makes every row factor a per-lane scalar and the staging writes 8 bytes wide.
// Scheduling follows the forward file: all LDS reads of a group of MFMAs are issued first,
// and the next chunk's tiles are prefetched into registers.
#include "device_common.h"
#include "launch.h"
#include "tile_io.h"
#include "workspace.h"

namespace cottn {
namespace COTTN_NS {
namespace {

// DK, DV: the head dimensions of the keys / queries and of the values / outputs (Sec. 2.1:
// d_H_key and d_H_value); Q, K, dQ, dK rows are DK wide, V, dO, dV rows DV wide, and both
// running states (Kh^T V forward in time, Qh^T dO backward in time) are DK x DV.
// CS waves share a 16-row group of a chunk: each forms the masked tiles of the group and
// accumulates its part of the result columns.
template <int DK, int DV, int C, int CS>
struct BwdCfg {
  static constexpr int RG = C / 16;        // row groups of a chunk
  static constexpr int NW = RG * CS;
  static constexpr int NT = NW * 64;
  static constexpr int DTK = DK / 16, DTV = DV / 16;
  static constexpr int NKT = DTK / CS, NVT = DTV / CS;   // result column tiles of a wave
  static constexpr int KSK = DK / 32, KSV = DV / 32;
  static constexpr int NP = C / 32;
  static constexpr int TPK = tile_pitch(DK, C), TPV = tile_pitch(DV, C);   // operand tiles
  static constexpr int SPV = lds_pitch(DV);   // state copies
  static constexpr int TILEK = C * TPK, TILEV = C * TPV;
  // the copy of the running state in elements, [d_key][d_value] in both scans
  static constexpr int STATE = DK * SPV;
  static constexpr int LDS_BYTES = LDS_ELEM * (2 * TILEK + 2 * TILEV + STATE) + 4 * C * CS + 4 * C + 64;
  static constexpr int WG_PER_CU = (160 * 1024) / LDS_BYTES;
  // the dQ kernel adds a staging tile when that does not lower the workgroups per compute
  // unit, and must when the finished rows (DK wide) do not fit the rows of the dO tile (the parts of
  // SPLIT3 rows leave room for them in the Q tile)
  static constexpr int OP = stage_tile_pitch(DK, C);   // of that tile, in elem_t
  static constexpr bool DQ_STAGE_IN_Q = SPLIT3 || REDO;
  static constexpr bool DQ_OWN_STAGE =
      (!DQ_STAGE_IN_Q && ELEM * stage_pitch(DK) > LDS_ELEM * TPV) ||
      (CS == 1 && LDS_BYTES + ELEM * C * OP <= 160 * 1024 &&
       (160 * 1024) / (LDS_BYTES + ELEM * C * OP) == WG_PER_CU);
  // The operands of a 32-token step are read in several groups (masked tiles first), each used
  // up before the next is read, instead of all at once: fewer registers in use at a time.  For
  // 128 x 128, where everything at once does not fit, and for fp32, whose products take so long
  // that one group's reads hide behind the other wave's.
  static constexpr bool PHASED = CS == 2 && (ELEM_IS_F32 || (DK == 128 && DV == 128));
  // So does the 16-bit dK/dV scan at 32 x 128, whose eight tiles of dV leave 17 to 20 registers spilled
  // otherwise: 512 units of 512 rows 53.3 -> 39.4 us, 96 of 1024 26.0 -> 18.5.
  static constexpr bool DKDV_PHASED = PHASED || (!ELEM_IS_F32 && CS == 1 && DK == 32 && DV == 128);
  // masked tiles formed by the two waves of a row group together (MaskedExchange); 32-row chunks
  static constexpr bool HALF_VISIBLE = F32_WHOLE && CS == 2 && C == 32, SHARE_MASKED = HALF_VISIBLE && !REDO;
  // steps that OWN_PREFIX_SETS takes at a time: the second through the tiles of Q and dO, two more through their own
  static constexpr int PREFIX_SETS = prefix_sets_built(DK, DV, ELEM_IS_F32, false);
  static constexpr bool SKIP_UNSEEN = skips_unseen(CS, C), DQ_SKIP_UNSEEN = SKIP_UNSEEN && DV == 128;
  static constexpr int WAVES_RAW = (WG_PER_CU >= 2 ? 2 : 1) * NW / 4;
  // never budget registers for more than two waves per SIMD unless one workgroup alone needs
  // it: spilling costs more than the second workgroup of a large chunk gains
  static constexpr int WAVES_PER_EU =
      NW / 4 > 2 ? NW / 4 : (WAVES_RAW > 2 ? 2 : WAVES_RAW);
};

// Rows a kernel takes at a time (CR, a divisor of the chunk: the regrouping is exact for any)
// and waves per row group (CS).
//
// 16-bit: 64-row steps with one wave per row group, except where the two states and the result of
// a wave do not fit its registers next to the operand fragments (64 x 128 and 128 x 64: up to 300
// spilled registers, or one wave per SIMD without spills).  Two waves per row group halve states
// and results per wave, 32-row steps keep the workgroup at four waves and two to a compute
// unit: dQ / dK/dV scan at B4 H12 N2048 64 x 128 59 / 55 -> 24 / 26 us, 128 x 64 36 / 38 -> 27 /
// 27 us.  Square and 32-wide shapes are slower that way (64 x 64 by 3 %, 32 x 32 by 30 %:
// shorter steps, the masked tiles formed twice).  At 128 x 128 one workgroup fills the LDS of a
// compute unit, and four waves on it wait for LDS reads with nothing to switch to: 64-row steps
// with two waves per row group, eight waves in all (B8 H12 N1024 40 / 48 -> 37 / 41 us, B4 H12
// N2048 38 / 45 -> 33 / 38 us).  That takes smaller groups of LDS reads (PHASED): with everything
// read at once 9 and 18 registers spill, a spilled register comes back behind the rows
// prefetched for the next step, and the scans take 43 / 52 us.
//
// fp32: 32-row chunks are two row groups, and two waves on each make a workgroup of four, of which the
// tiles and the state in parts (device_common.h: SPLIT3) leave room for two at 64 x 64.  B8 H12 N1024 d64:
// dQ 46 -> 38 us, dK/dV 52 -> 44 against the fp32 matrix instruction, both in segments and before a value's
// range was noted (in even shares 36.8 / 41.1 without that note, 38.2 / 43.5 with it); the scans' rows take 25 and 30 us
// through HBM.  The vector ALU bounds them: 6.5 instructions part an element and note its range, of the rows
// once and of the state once a step.  64-row steps with eight waves, one workgroup to a compute unit, take 51 and 63
// us; products of results straight into their sums (no instruction for the addition) 38 and 45, at
// 1.2 times the error.
// Where the whole fp32 kernels stand, an MFMA has a sixteenth of the bf16 rate: 32 rows instead of 64
// save a fifth of the masked products, and the two waves of a row group form them together and only
// where something is visible (MaskedExchange).  A third workgroup on the compute unit (168 registers)
// spills and is slower.
template <int DK, int DV, int C> struct BwdSplit {
  static constexpr bool WIDE = DK != DV && DK >= 64 && DV >= 64;
  static constexpr int CR = WIDE ? 32 : C, CS = ELEM_IS_F32 || WIDE || (DK == 128 && DV == 128) ? 2 : 1;
};

// ---------------------------------------------------------------------------------------
// Kernel 2: blockIdx.y == 0: slot g <- sum of fwd totals of segments < g;
//           blockIdx.y == 1: slot g <- sum of rev totals of segments > g.
// Totals that were never computed (fwd slot G-1, rev slot 0) are not read; a null array is
// skipped.
#ifndef COTTN_REDO
__global__ __launch_bounds__(256) void bwd_state_carry(float* __restrict__ fwd_tot,
                                                       float* __restrict__ rev_tot, int G,
                                                       int elems_per_state, long total) {
  const long idx = (long(blockIdx.x) * 256 + threadIdx.x) * 4;  // 4 elements per thread
  float* tot = blockIdx.y == 0 ? fwd_tot : rev_tot;
  if (idx >= total || tot == nullptr) return;
  const long unit = idx / elems_per_state, e = idx % elems_per_state;
  exclusive_running_sum(tot + unit * G * elems_per_state + e, G, size_t(elems_per_state),
                        blockIdx.y == 1);
}
#endif

// ---------------------------------------------------------------------------------------
// Kernel 3: dQ of one segment, chunks in forward order.  Wave w owns query rows 16w..16w+15.
// The running state S ([d_key][d_value]) sits in accumulators with the keys along the lanes:
// element [v] of lane (r, q4) of tile (key tile y, value tile x) is
// S[16 rt + r][16 ct + 4 q4 + v], the orientation the forward scan and the totals kernel use
// (so the stored states are read tile by tile, one 1 KB instruction per tile).  A lane holds 4
// consecutive values of one key row and publishes them with one 8-byte write to the row-major
// LDS copy St[d_key][d_value]; the update's key-side operand is the K fragment already read
// for the intra-chunk product.
//
// REV: whether the launch has segments to leave reverse-time totals for.
template <int DK, int DV, int C, int CS, bool REV, int WALK>
COTTN_KERNEL((C * 4 * CS, (BwdCfg<DK, DV, C, CS>::WAVES_PER_EU)), bwd_dq_scan)
    const elem_t* __restrict__ Q, const elem_t* __restrict__ K, const elem_t* __restrict__ V,
    const elem_t* __restrict__ dO, const float* __restrict__ s, elem_t* __restrict__ dQ,
    const float* __restrict__ fwd_states, float* __restrict__ rev_totals,
    float* __restrict__ ds_partial, Divisor H, int N, Divisor G, Divisor seg_rows, float inv_eps,
    int sum_totals, const int* __restrict__ lengths, int s_per_unit,
    const float* __restrict__ state_in, int units, Divisor unit_rows) {
  using Cfg = BwdCfg<DK, DV, C, CS>;
  constexpr bool EVEN = walks_even(WALK);
  using AT = SplitTiles<DK, DV, Cfg::RG, CS>;   // forward-time state: key rows, value columns
  using RT = SplitTiles<DV, DK, Cfg::RG, CS>;   // reverse-time total: value rows, key columns
  using StageK = TileStage<DK, C, Cfg::NT>;
  using StageV = TileStage<DV, C, Cfg::NT>;
  constexpr int TPK = Cfg::TPK, TPV = Cfg::TPV, SP = Cfg::SPV;
  COTTN_LDS_ARRAY(lds_t, Qs, Cfg::TILEK, 0)   // qh = r_i q_i
  COTTN_LDS_ARRAY(lds_t, Ks, Cfg::TILEK, 1)   // kh = r_j k_j
  COTTN_LDS_ARRAY(lds_t, Vs, Cfg::TILEV, 2)   // raw v
  COTTN_LDS_ARRAY(lds_t, Gs, Cfg::TILEV, 3)   // dO
  COTTN_LDS_ARRAY(lds_t, St, Cfg::STATE, 4)   // state, [d_key][d_value]
  // Every wave reads all rows of all four tiles until the end of a chunk (the reverse total
  // contracts Qs and Gs over the tokens), so finished dQ rows are staged in a tile of their
  // own when LDS has room for one; otherwise behind a barrier in the dead dO (SPLIT3: Q) tile.
  COTTN_LDS_ARRAY(elem_t, Os, Cfg::DQ_OWN_STAGE ? C * Cfg::OP : 8, 5)
  COTTN_LDS_ARRAY(float, rq, C, 6)
  COTTN_LDS_ARRAY(float, xdot, CS > 1 ? CS * C : 1, 7)   // row dot products of the column parts
  COTTN_LDS_ARRAY(float, ds_wave, Cfg::NW, 8)
  constexpr int SETS = WALK == OWN_PREFIX_SETS ? Cfg::PREFIX_SETS : 1;
  COTTN_LDS_ARRAY(lds_t, Ps, SETS > 2 ? (SETS - 2) * (Cfg::TILEK + Cfg::TILEV) : 8, 9)   // kh and v of further steps
  // A tiles of the two key halves: in the staging tile where there is one (it is written a
  // barrier after the last of them is read), so that 128 x 32 keeps two workgroups
  constexpr bool IN_STAGE = Cfg::SHARE_MASKED && Cfg::DQ_OWN_STAGE;
  using Masked = MaskedExchange<Cfg::SHARE_MASKED ? 2 : 0>;
  static_assert(!IN_STAGE || int(sizeof(Masked)) <= ELEM * C * Cfg::OP, "the tiles fit the staging tile");
  __shared__ __attribute__((aligned(16))) char masked_lds[Cfg::SHARE_MASKED && !IN_STAGE ? sizeof(Masked) : 16];
  Masked& masked = *reinterpret_cast<Masked*>(IN_STAGE ? reinterpret_cast<char*>(Os) : masked_lds);

  Unparted un;
  fetch_argument_now(Q, K, V, dO, s, dQ, fwd_states, rev_totals, ds_partial, H, N, G, seg_rows,
                     inv_eps, sum_totals, lengths, s_per_unit, state_in, units, unit_rows);
  const int* seq_len = WALK == EVEN_SHARES ? nullptr : lengths;
  const Span span = span_of_workgroup<false, EVEN>(units, N, G, seg_rows, unit_rows);
  int unit = span.unit;
  const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid / 64), l = tid % 64,
            r = l % 16, q4 = l / 16;
  const int rg = row_group<Cfg::RG, CS>(w), cp = w / Cfg::RG;   // row group, column part
  const elem_t* Qu = Q + size_t(unit) * N * DK;   // (of the rows fetched next, from there on)
  const elem_t* Ku = K + size_t(unit) * N * DK;
  const elem_t* Vu = V + size_t(unit) * N * DV;
  const elem_t* Gu = dO + size_t(unit) * N * DV;
  elem_t* dQu = dQ + size_t(unit) * N * DK;
  const int row_begin = span.begin;
  int row_end = max(row_begin, min(valid_rows(seq_len, unit, H, N), span.end));   // of the piece walked
  int piece_end = span.end;   // of the same, with the rows that do not exist

  // fwd_states holds the carried prefixes (slot g = state at the start of segment g) or, with
  // sum_totals set, the raw segment totals, which this workgroup then adds up itself
  f32x4 sacc[AT::NCT][AT::NRT];
  // By-product for the dK/dV kernel: the first piece's total of qh^T dO (unless it begins its
  // unit; the workgroups before this one need it), accumulated in that kernel's layout: element [v] of
  // lane (r, q4) of tile (y, x) is R[key 16 ct + r][value 16 rt + 4 q4 + v].
  f32x4 racc[RT::NCT][RT::NRT];
  bool with_rev = REV && rev_totals != nullptr && span.mid_unit;
#pragma unroll
  for (int x = 0; x < AT::NCT; ++x)
#pragma unroll
    for (int y = 0; y < AT::NRT; ++y) sacc[x][y] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int x = 0; x < RT::NCT; ++x)
#pragma unroll
    for (int y = 0; y < RT::NRT; ++y) racc[x][y] = f32x4{0.f, 0.f, 0.f, 0.f};
  // the first chunk's rows and the stored states are all requested before anything waits
  float ds_lane = 0.f;
  StageK qst, kst;
  StageV vst, gst;
  qst.fetch(Qu, row_begin, row_end);
  kst.fetch(Ku, row_begin, row_end);
  vst.fetch(Vu, row_begin, row_end);
  gst.fetch(Gu, row_begin, row_end);
  float scale = unit_scale(s, unit, H, s_per_unit);
  const auto form_prefix = [&] {
    lds_t *k_tiles[SETS], *v_tiles[SETS];
#pragma unroll
    for (int i = 0; i < SETS; ++i) {
      k_tiles[i] = i == 0 ? Ks : i == 1 ? Qs : Ps + (i - 2) * Cfg::TILEK;
      v_tiles[i] = i == 0 ? Vs : i == 1 ? Gs : Ps + (SETS - 2) * Cfg::TILEK + (i - 2) * Cfg::TILEV;
    }
    add_rows_before<DK, DV, C, Cfg::NT, AT::NRT, AT::NCT, DV, SETS>(
        k_tiles, v_tiles, Ku, Vu, min(row_begin, valid_rows(seq_len, unit, H, N)), inv_eps, l, AT::active(rg, cp),
        [&](int y) { return AT::row_tile(rg, cp, y); }, [&](int x) { return AT::col_tile(rg, cp, x); },
        [&](int y, int x, const frag8& kf, const frag8& vf) { sacc[x][y] = mma16_add(vf, kf, sacc[x][y]); },
        un);
  };
  bool no_states = walks_own_prefix(WALK);
  if constexpr (WALK == EVEN_SHARES)   // (sum_totals 2: the states are a forward's that may have left none)
    no_states = sum_totals == 2 && fwd_states[size_t(gridDim.x - 1) * DK * DV] != EVEN_MARK;
  if ((walks_own_prefix(WALK) || WALK == EVEN_SHARES) && no_states) {
    if (span.mid_unit) form_prefix();
  } else if (fwd_states != nullptr && span.mid_unit && AT::active(rg, cp)) {
    add_stored_states<AT::STATE_BATCH, AT::STATE_MANY>(
        sacc, sum_totals ? span.outermost : span.slot, sum_totals ? span.slot - 1 : span.slot,
        [&](int slot, int x, int y) {
          return *reinterpret_cast<const f32x4*>(
              fwd_states + size_t(slot) * DK * DV +
              tiled_state_offset(AT::row_tile(rg, cp, y), AT::col_tile(rg, cp, x), DV / 16, l));
        });
  }
  // the state of the rows before this piece of the sequence belongs to every segment's start
  const auto add_state_in = [&] {
    const float* src = state_in + size_t(unit) * DK * DV;
#pragma unroll
    for (int x = 0; x < AT::NCT; ++x)
#pragma unroll
      for (int y = 0; y < AT::NRT; ++y)
        sacc[x][y] += *reinterpret_cast<const f32x4*>(src + (16 * AT::row_tile(rg, cp, y) + r) * DV +
                                                      16 * AT::col_tile(rg, cp, x) + 4 * q4);
  };
  if (state_in != nullptr && AT::active(rg, cp)) add_state_in();
  const auto store_rev_total = [&] {
    float* out = rev_totals + size_t(span.slot) * DK * DV;
#pragma unroll
    for (int x = 0; x < RT::NCT; ++x) un.results<RT::NRT>(racc[x]);
#pragma unroll
    for (int x = 0; x < RT::NCT; ++x)
#pragma unroll
      for (int y = 0; y < RT::NRT; ++y)
        store_state_words(out + tiled_state_offset(RT::col_tile(rg, cp, x), RT::row_tile(rg, cp, y), DV / 16, l),
                          racc[x][y]);
  };
  // the piece's share of ds: lanes of the first lane row hold the row sums.  Pieces are numbered in the
  // order of their rows: slot + unit with even shares (one more piece for every unit begun)
  const auto store_ds = [&] {
    ds_lane = group_sum<64>(ds_lane);
    if (l == 0) ds_wave[w] = ds_lane;
    __syncthreads();
    if (tid == 0) {
      float t = 0.f;
#pragma unroll
      for (int i = 0; i < Cfg::NW; ++i) t += ds_wave[i];
      ds_partial[span.slot + (EVEN ? unit : 0)] = t;
    }
    ds_lane = 0.f;
  };

  constexpr int NKT = Cfg::NKT;
  const int colk = 16 * NKT * cp;  // first result column of this wave
  RowPieces<DK, NKT> finished;  // dQ rows of the previous chunk, stored one chunk late
#pragma unroll
  for (int j = 0; j < RowPieces<DK, NKT>::PER_LANE; ++j) finished.v[j] = uint4{0u, 0u, 0u, 0u};
  elem_t* done_dQ = dQu;
  int done_row = 0, done_end = 0, row0 = row_begin, left = span.left;   // done_end = 0: nothing finished yet
  for (bool more = WALK == EVEN_PADDED || row0 < row_end; more;) {
    if (AT::active(rg, cp)) {
#pragma unroll
      for (int x = 0; x < AT::NCT; ++x)
#pragma unroll
        for (int y = 0; y < AT::NRT; ++y) {
          store4_lds(St + (16 * AT::row_tile(rg, cp, y) + r) * SP + lds_col(16 * AT::col_tile(rg, cp, x)) + 4 * q4,
                     sacc[x][y][0], sacc[x][y][1], sacc[x][y][2], sacc[x][y][3], un);
        }
    }
    {
      float rqv[StageK::PASSES], rkv[StageK::PASSES];
      qst.row_rinv(inv_eps, rqv);
      kst.row_rinv(inv_eps, rkv);
      qst.commit_scaled(Qs, rqv, un);
      qst.store_rinv(rq, rqv);
      kst.commit_scaled(Ks, rkv, un);
      vst.commit_plain(Vs, un);
      gst.commit_plain(Gs, un);
    }
    // the next step's rows: of this unit, or the first ones of the next
    const bool cross = EVEN && left > 0 && row0 + C >= row_end;
    const int next_row = cross ? 0 : row0 + C;
    const int next_end = cross ? min(valid_rows(seq_len, unit + 1, H, N), left) : row_end;
    more = (WALK == EVEN_PADDED && cross) || next_row < next_end;
    if (cross) {
      Qu += size_t(N) * DK;
      Ku += size_t(N) * DK;
      Vu += size_t(N) * DV;
      Gu += size_t(N) * DV;
    }
    if (more) {
      qst.fetch(Qu, next_row, next_end);
      kst.fetch(Ku, next_row, next_end);
      vst.fetch(Vu, next_row, next_end);
      gst.fetch(Gu, next_row, next_end);
    }
    if (done_end > 0) store_row_pieces<DK, NKT>(finished, done_dQ, done_row + 16 * rg, done_end, l, colk);
    __syncthreads();

    if constexpr (Cfg::SHARE_MASKED) {
      // this wave's half of the features of the masked tiles (key half 1 is masked for rg = 0)
#pragma unroll
      for (int half = 0; half < 2; ++half)
        if (half <= rg)
          masked.put(half, w, l, row_products<Cfg::KSV>(Vs + (16 * half + r) * TPV, Gs + (16 * rg + r) * TPV,
                                                        16 * Cfg::KSV * cp, q4));
    }

    // earlier chunks: dqh^T += S dO^T (contraction over d_value = along the rows of St)
    frag8 gf[Cfg::KSV];  // dO rows of this wave: column-side operand of every product
#pragma unroll
    for (int ks = 0; ks < Cfg::KSV; ++ks)
      gf[ks] = lds_row_frag(Gs + (16 * rg + r) * TPV + lds_col(32 * ks), q4);
    // dq[nt][v] = dqh[query 16 rg + r][key feature colk + 16 nt + 4 q4 + v]
    f32x4 dq[NKT];
#pragma unroll
    for (int nt = 0; nt < NKT; ++nt) dq[nt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < Cfg::KSV; ++ks) {
      frag8 sf[NKT];
#pragma unroll
      for (int nt = 0; nt < NKT; ++nt)
        sf[nt] = lds_row_frag(St + (colk + 16 * nt + r) * SP + lds_col(32 * ks), q4);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int nt = 0; nt < NKT; ++nt) dq[nt] = mma16(sf[nt], gf[ks], dq[nt]);
      __builtin_amdgcn_sched_barrier(0);
    }

    // this chunk: dqh^T += Kh^T (A (.) M)^T with A^T = V dO^T, and the state update,
    // 32 tokens at a time
#pragma unroll
    for (int p = 0; p < Cfg::NP; ++p) {
      const bool diag_or_below = 2 * p <= rg;
      const int t0 = 32 * p + 4 * q4, t1 = 32 * p + 16 + 4 * q4;  // token order of the A slots
      frag8 af;
      frag8 vr[2][Cfg::KSV];
      const auto read_values = [&] {
#pragma unroll
        for (int half = 0; half < 2; ++half)
#pragma unroll
          for (int ks = 0; ks < Cfg::KSV; ++ks) {
            if (Cfg::DQ_SKIP_UNSEEN && half > rg) break;
            vr[half][ks] = lds_row_frag(Vs + (16 * (2 * p + half) + r) * TPV + lds_col(32 * ks), q4);
          }
      };
      const auto form_masked = [&] {
#pragma unroll
        for (int half = 0; half < 2; ++half) {
          const int jt = 2 * p + half;
          if (Cfg::DQ_SKIP_UNSEEN && half > rg) {
            put_no_half(af, half);
            break;
          }
          f32x4 t = {0.f, 0.f, 0.f, 0.f};
          if constexpr (Cfg::SHARE_MASKED) {
            if (half <= rg) t = masked.get(half, w, l);
          } else {
#pragma unroll
            for (int ks = 0; ks < Cfg::KSV; ++ks) t = mma16(vr[half][ks], gf[ks], t);
          }
          // t[v] = dO_(16 rg + r) . v_(16jt + 4 q4 + v); keep key <= query
          const bool full = jt < rg, diag = jt == rg;
          put_half(af, half, t, full || (diag && 4 * q4 + 0 <= r), full || (diag && 4 * q4 + 1 <= r),
                   full || (diag && 4 * q4 + 2 <= r), full || (diag && 4 * q4 + 3 <= r), un);
        }
      };
      frag8 qcol[RT::NCT], grow[RT::NRT];
      const bool rev_here = with_rev && RT::active(rg, cp);
      const auto read_reverse = [&] {
#pragma unroll
        for (int x = 0; x < RT::NCT; ++x)
          qcol[x] = lds_col_frag(Qs, TPK, t0, t1, 16 * RT::col_tile(rg, cp, x), r);
#pragma unroll
        for (int y = 0; y < RT::NRT; ++y)
          grow[y] = lds_col_frag(Gs, TPV, t0, t1, 16 * RT::row_tile(rg, cp, y), r);
      };
      if (Cfg::SHARE_MASKED) __syncthreads();  // the partial tiles of the other waves are there
      if (Cfg::PHASED && diag_or_below) {
        if (!Cfg::SHARE_MASKED) read_values();
        __builtin_amdgcn_sched_barrier(0);
        form_masked();
        __builtin_amdgcn_sched_barrier(0);
      }
      frag8 kc[NKT], vcol[AT::NCT], krow[AT::NRT];
#pragma unroll
      for (int nt = 0; nt < NKT; ++nt) kc[nt] = lds_col_frag(Ks, TPK, t0, t1, colk + 16 * nt, r);
#pragma unroll
      for (int x = 0; x < AT::NCT; ++x)
        vcol[x] = lds_col_frag(Vs, TPV, t0, t1, 16 * AT::col_tile(rg, cp, x), r);
      if (!AT::ROW_OPERAND_IS_RESULT_COLUMN) {
#pragma unroll
        for (int y = 0; y < AT::NRT; ++y)
          krow[y] = lds_col_frag(Ks, TPK, t0, t1, 16 * AT::row_tile(rg, cp, y), r);
      }
      if (!Cfg::PHASED) {
        if (rev_here) read_reverse();
        if (diag_or_below) read_values();
      }
      __builtin_amdgcn_sched_barrier(0);
      if (diag_or_below) {
        if (!Cfg::PHASED) form_masked();
        if (Cfg::HALF_VISIBLE && rg == 0) {
#pragma unroll
          for (int nt = 0; nt < NKT; ++nt) dq[nt] = mma16_half_add(kc[nt], af, dq[nt], 0);
        } else {
#pragma unroll
          for (int nt = 0; nt < NKT; ++nt) dq[nt] = mma16_add(kc[nt], af, dq[nt]);
        }
      }
      // state update: S += kh^T v over these 32 tokens
      if (AT::active(rg, cp)) {
#pragma unroll
        for (int y = 0; y < AT::NRT; ++y)
#pragma unroll
          for (int x = 0; x < AT::NCT; ++x)
            sacc[x][y] = mma16_add(vcol[x], AT::ROW_OPERAND_IS_RESULT_COLUMN ? kc[y] : krow[y], sacc[x][y]);
      }
      if (Cfg::PHASED) {
        __builtin_amdgcn_sched_barrier(0);
        if (rev_here) read_reverse();
        __builtin_amdgcn_sched_barrier(0);
      }
      // reverse total: R^T += dO^T qh over the same tokens
      if (rev_here) {
#pragma unroll
        for (int y = 0; y < RT::NRT; ++y)
#pragma unroll
          for (int x = 0; x < RT::NCT; ++x) racc[x][y] = mma16_add(grow[y], qcol[x], racc[x][y]);
      }
      __builtin_amdgcn_sched_barrier(0);
    }

    // epilogue: normalisation chain rule on the rows (Qs holds qh), then s r_i and the store
    const float ri = rq[16 * rg + r];
    float xv[NKT][4];
    float t = dot_with_row<NKT, TPK>(dq, Qs + 16 * rg * TPK, colk, xv, r, q4);
    if (CS > 1) {  // the row's dot product over the columns of all its waves
      if (q4 == 0) xdot[cp * C + 16 * rg + r] = t;
      __syncthreads();
      t = 0.f;
#pragma unroll
      for (int c = 0; c < CS; ++c) t += xdot[c * C + 16 * rg + r];
    }
    const float rho = project_out_row<NKT, true>(dq, xv, t, ri, inv_eps);
    if (q4 == 0 && cp == 0) ds_lane += rho;
    if (CS == 1 && !Cfg::DQ_OWN_STAGE) __syncthreads();  // every wave is done with the dO tile
    gather_rows_transposed<DK, NKT>(dq, scale * ri,
                                    Cfg::DQ_OWN_STAGE ? static_cast<void*>(Os + 16 * rg * Cfg::OP)
                                    : Cfg::DQ_STAGE_IN_Q ? static_cast<void*>(Qs + 16 * rg * TPK)
                                                    : static_cast<void*>(Gs + 16 * rg * TPV),
                                    l, finished, un, colk);
    __syncthreads();
    done_dQ = dQu;
    done_row = row0;
    done_end = row_end;
    if (cross) {   // the unit ends here
      if (with_rev && RT::active(rg, cp)) store_rev_total();
      with_rev = false;
      store_ds();
      if (seq_len != nullptr) zero_rows<DK>(dQu, row_end, N);
      piece_end = min(N, left);
      ++unit;
      left -= unit_rows;
      dQu += size_t(N) * DK;
      scale = unit_scale(s, unit, H, s_per_unit);
#pragma unroll
      for (int x = 0; x < AT::NCT; ++x)
#pragma unroll
        for (int y = 0; y < AT::NRT; ++y) sacc[x][y] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (state_in != nullptr && AT::active(rg, cp)) add_state_in();
    }
    row0 = next_row;
    row_end = next_end;
  }
  if (done_end > 0) store_row_pieces<DK, NKT>(finished, done_dQ, done_row + 16 * rg, done_end, l, colk);

  if (seq_len != nullptr) zero_rows<DK>(dQu, row_end, piece_end);  // rows that do not exist

  if (with_rev && RT::active(rg, cp)) store_rev_total();
  store_ds();
#ifdef COTTN_SPLIT3
  if (un.in_workgroup<Cfg::NW>(rq)) {
    using Whole = f32w::BwdCfg<DK, DV, C, CS>;
    static_assert(2 * Whole::TILEK <= Cfg::TILEK && 2 * Whole::TILEV <= Cfg::TILEV && 2 * Whole::STATE <= Cfg::STATE, "whole rows fit");
    void* const room[] = {Qs, Ks, Vs, Gs, St, Os, rq, xdot, ds_wave, Ps};
    f32w::bwd_dq_scan<DK, DV, C, CS, REV, WALK>(room, Q, K, V, dO, s, dQ, fwd_states, rev_totals, ds_partial, H, N, G,
                                                seg_rows, inv_eps, sum_totals, lengths, s_per_unit, state_in, units,
                                                unit_rows);
  }
#endif
}

// ---------------------------------------------------------------------------------------
// Kernel 4: dK and dV of one segment, chunks in reverse order.  Wave w owns key rows
// 16w..16w+15 of the chunk.  The running reverse state R ([d_key][d_value]) sits transposed
// in the accumulators (value rows, key columns): element [v] of lane (r, q4) of tile (y, x)
// is R[16 ct + r][16 rt + 4 q4 + v], published with one 8-byte write to the row-major LDS
// copy Rl[d_key][d_value]; the update's row-side operand is the dO fragment already read
// for the intra-chunk dV product.
template <int DK, int DV, int C, int CS, int WALK>
COTTN_KERNEL((C * 4 * CS, (BwdCfg<DK, DV, C, CS>::WAVES_PER_EU)), bwd_dkdv_scan)
    const elem_t* __restrict__ Q, const elem_t* __restrict__ K, const elem_t* __restrict__ V,
    const elem_t* __restrict__ dO, const float* __restrict__ s, elem_t* __restrict__ dK,
    elem_t* __restrict__ dV, const float* __restrict__ rev_states,
    const float* __restrict__ ds_partial, float* __restrict__ ds, int B, Divisor H, int N, Divisor G,
    Divisor seg_rows, float inv_eps, int sum_totals, const int* __restrict__ lengths, int s_per_unit,
    const float* __restrict__ rev_in, float* __restrict__ rev_out, Divisor unit_rows) {
  using Cfg = BwdCfg<DK, DV, C, CS>;
  constexpr bool EVEN = walks_even(WALK);
  using AT = SplitTiles<DV, DK, Cfg::RG, CS>;   // value rows, key columns (the state is held transposed)
  using StageK = TileStage<DK, C, Cfg::NT>;
  using StageV = TileStage<DV, C, Cfg::NT>;
  constexpr int TPK = Cfg::TPK, TPV = Cfg::TPV, SP = Cfg::SPV;
  COTTN_LDS_ARRAY(lds_t, Qs, Cfg::TILEK, 0)   // r_i q_i
  COTTN_LDS_ARRAY(lds_t, Ks, Cfg::TILEK, 1)   // raw k
  COTTN_LDS_ARRAY(lds_t, Vs, Cfg::TILEV, 2)   // raw v
  COTTN_LDS_ARRAY(lds_t, Gs, Cfg::TILEV, 3)   // dO
  COTTN_LDS_ARRAY(lds_t, Rl, Cfg::STATE, 4)   // reverse state, [d_key][d_value]
  COTTN_LDS_ARRAY(float, rk, C, 5)
  COTTN_LDS_ARRAY(float, xdot, CS > 1 ? CS * C : 1, 6)   // row dot products of the column parts
  // P tiles of the two query halves, then the A tiles
  __shared__ MaskedExchange<Cfg::SHARE_MASKED ? 4 : 0> masked;

  Unparted un;
  fetch_argument_now(Q, K, V, dO, s, dK, dV, rev_states, ds_partial, ds, B, H, N, G, seg_rows,
                     inv_eps, sum_totals, lengths, s_per_unit, rev_in, rev_out, unit_rows);
  const int* seq_len = WALK == EVEN_SHARES ? nullptr : lengths;
  const Span span = span_of_workgroup<true, EVEN>(B * H, N, G, seg_rows, unit_rows);
  int unit = span.unit;
  const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid / 64), l = tid % 64,
            r = l % 16, q4 = l / 16;
  const int rg = row_group<Cfg::RG, CS>(w), cp = w / Cfg::RG;   // row group, column part
  const elem_t* Qu = Q + size_t(unit) * N * DK;   // (of the rows fetched next, from there on)
  const elem_t* Ku = K + size_t(unit) * N * DK;
  const elem_t* Vu = V + size_t(unit) * N * DV;
  const elem_t* Gu = dO + size_t(unit) * N * DV;
  elem_t* dKu = dK + size_t(unit) * N * DK;
  elem_t* dVu = dV + size_t(unit) * N * DV;
  int row_begin = span.begin;   // of the piece walked, and its end
  int row_end = max(row_begin, min(valid_rows(seq_len, unit, H, N), span.end));
  int piece_end = span.end;   // with the rows that do not exist

  // rev_states holds the carried suffixes (slot g = reverse state at the end of segment g)
  // or, with sum_totals set, the raw segment totals of the later segments to be added up here
  f32x4 racc[AT::NCT][AT::NRT];
#pragma unroll
  for (int x = 0; x < AT::NCT; ++x)
#pragma unroll
    for (int y = 0; y < AT::NRT; ++y) racc[x][y] = f32x4{0.f, 0.f, 0.f, 0.f};
  // the last chunk's rows and the stored states are all requested before anything waits
  StageK qst, kst;
  StageV vst, gst;
  bool more = WALK == EVEN_PADDED || row_begin < row_end;   // (a segment of a padded batch can be empty)
  int row0 = row_begin + (row_end - row_begin - 1) / C * C;
  if (more) {
    qst.fetch(Qu, row0, row_end);
    kst.fetch(Ku, row0, row_end);
    vst.fetch(Vu, row0, row_end);
    gst.fetch(Gu, row0, row_end);
  }
  float scale = unit_scale(s, unit, H, s_per_unit);
  // the first H workgroups also finish ds: ds[h] = sum over batches and segments of the
  // partial sums the dQ kernel left behind (with a scale per (batch, head): the first B*H
  // workgroups, ds[b][h] = sum over the segments; with even shares there can be fewer workgroups)
  if constexpr (EVEN) {
    if (w == 0)
      for (int h = blockIdx.x; h < (seq_len != nullptr ? B * H.n : H.n); h += gridDim.x) {
        float t = 0.f;
        for (int b = l; b < (seq_len != nullptr ? 1 : B); b += 64) {
          const int u = b * H + h, last = quotient((u + 1) * unit_rows - 1, seg_rows);
          for (int slot = quotient(u * unit_rows, seg_rows); slot <= last; ++slot) t += ds_partial[slot + u];
        }
        t = group_sum<64>(t);
        if (l == 0) ds[h] = t;
      }
  } else if (int(blockIdx.x) < (s_per_unit ? B * H.n : H.n) && w == 0) {
    float t = 0.f;
    const int n = s_per_unit ? G.n : B * G.n;
    for (int i = l; i < n; i += 64)
      t += s_per_unit ? ds_partial[size_t(blockIdx.x) * G + i]
                      : ds_partial[(size_t(quotient(i, G)) * H + blockIdx.x) * G + (i - quotient(i, G) * G)];
    t = group_sum<64>(t);
    if (l == 0) ds[blockIdx.x] = t;
  }
  if (rev_states != nullptr && span.mid_unit && AT::active(rg, cp)) {
    add_stored_states<AT::STATE_BATCH, AT::STATE_MANY>(
        racc, sum_totals ? span.slot + 1 : span.slot, sum_totals ? span.outermost : span.slot,
        [&](int slot, int x, int y) {
          return *reinterpret_cast<const f32x4*>(
              rev_states + size_t(slot) * DK * DV +
              tiled_state_offset(AT::col_tile(rg, cp, x), AT::row_tile(rg, cp, y), DV / 16, l));
        });
  }
  // the reverse state of the rows after this piece of the sequence belongs to every segment
  const auto add_rev_in = [&] {
    const float* src = rev_in + size_t(unit) * DK * DV;
#pragma unroll
    for (int x = 0; x < AT::NCT; ++x)
#pragma unroll
      for (int y = 0; y < AT::NRT; ++y)
        racc[x][y] += *reinterpret_cast<const f32x4*>(src + (16 * AT::col_tile(rg, cp, x) + r) * DV +
                                                      16 * AT::row_tile(rg, cp, y) + 4 * q4);
  };
  if (rev_in != nullptr && AT::active(rg, cp)) add_rev_in();
  // at the first row of a unit: the reverse state of the whole piece and what followed it
  const auto store_rev_out = [&] {
    float* out = rev_out + size_t(unit) * DK * DV;
#pragma unroll
    for (int x = 0; x < AT::NCT; ++x) un.results<AT::NRT>(racc[x]);
#pragma unroll
    for (int x = 0; x < AT::NCT; ++x)
#pragma unroll
      for (int y = 0; y < AT::NRT; ++y)
        *reinterpret_cast<f32x4*>(out + (16 * AT::col_tile(rg, cp, x) + r) * DV +
                                  16 * AT::row_tile(rg, cp, y) + 4 * q4) = racc[x][y];
  };

  constexpr int NKT = Cfg::NKT, NVT = Cfg::NVT;
  const int colk = 16 * NKT * cp, colv = 16 * NVT * cp;  // first result columns of this wave
  RowPieces<DK, NKT> done_k;  // dK and dV rows of the previous chunk, stored one chunk late
  RowPieces<DV, NVT> done_v;
#pragma unroll
  for (int j = 0; j < RowPieces<DK, NKT>::PER_LANE; ++j) done_k.v[j] = uint4{0u, 0u, 0u, 0u};
#pragma unroll
  for (int j = 0; j < RowPieces<DV, NVT>::PER_LANE; ++j) done_v.v[j] = uint4{0u, 0u, 0u, 0u};
  elem_t *done_dK = dKu, *done_dV = dVu;
  int done_row = 0, done_end = 0, left = span.left;   // done_end = 0: nothing finished yet
  while (more) {
    if (AT::active(rg, cp)) {
#pragma unroll
      for (int x = 0; x < AT::NCT; ++x)
#pragma unroll
        for (int y = 0; y < AT::NRT; ++y) {
          store4_lds(Rl + (16 * AT::col_tile(rg, cp, x) + r) * SP + lds_col(16 * AT::row_tile(rg, cp, y)) + 4 * q4,
                     racc[x][y][0], racc[x][y][1], racc[x][y][2], racc[x][y][3], un);
        }
    }
    {
      float rqv[StageK::PASSES], rkv[StageK::PASSES];
      qst.row_rinv(inv_eps, rqv);
      kst.row_rinv(inv_eps, rkv);
      qst.commit_scaled(Qs, rqv, un);
      kst.commit_plain(Ks, un);
      kst.store_rinv(rk, rkv);
      vst.commit_plain(Vs, un);
      gst.commit_plain(Gs, un);
    }
    // the next step's rows: of this unit, or the last ones of the unit before
    const bool cross = EVEN && left > 0 && row0 == row_begin;
    const int next_begin = cross ? max(0, unit_rows - left) : row_begin;
    const int next_end = cross ? max(next_begin, valid_rows(seq_len, unit - 1, H, N)) : row_end;
    const int next_row = cross ? next_begin + (next_end - next_begin - 1) / C * C : row0 - C;
    more = cross || row0 > row_begin;
    if (cross) {
      Qu -= size_t(N) * DK;
      Ku -= size_t(N) * DK;
      Vu -= size_t(N) * DV;
      Gu -= size_t(N) * DV;
    }
    if (more) {
      qst.fetch(Qu, next_row, next_end);
      kst.fetch(Ku, next_row, next_end);
      vst.fetch(Vu, next_row, next_end);
      gst.fetch(Gu, next_row, next_end);
    }
    if (EVEN ? done_end > 0 : row0 + C < row_end) {
      store_row_pieces<DK, NKT>(done_k, EVEN ? done_dK : dKu, (EVEN ? done_row : row0 + C) + 16 * rg,
                                EVEN ? done_end : row_end, l, colk);
      store_row_pieces<DV, NVT>(done_v, EVEN ? done_dV : dVu, (EVEN ? done_row : row0 + C) + 16 * rg,
                                EVEN ? done_end : row_end, l, colv);
    }
    __syncthreads();

    if constexpr (Cfg::SHARE_MASKED) {
      // this wave's half of the features of the masked tiles (query half 0 is masked for rg = 1)
#pragma unroll
      for (int half = 0; half < 2; ++half)
        if (half >= rg) {
          masked.put(half, w, l, row_products<Cfg::KSK>(Qs + (16 * half + r) * TPK, Ks + (16 * rg + r) * TPK,
                                                        16 * Cfg::KSK * cp, q4));
          masked.put(2 + half, w, l, row_products<Cfg::KSV>(Gs + (16 * half + r) * TPV, Vs + (16 * rg + r) * TPV,
                                                            16 * Cfg::KSV * cp, q4));
        }
    }

    frag8 kf[Cfg::KSK], vf[Cfg::KSV];  // this wave's key rows and value rows (column side)
#pragma unroll
    for (int ks = 0; ks < Cfg::KSK; ++ks)
      kf[ks] = lds_row_frag(Ks + (16 * rg + r) * TPK + lds_col(32 * ks), q4);
#pragma unroll
    for (int ks = 0; ks < Cfg::KSV; ++ks)
      vf[ks] = lds_row_frag(Vs + (16 * rg + r) * TPV + lds_col(32 * ks), q4);
    // dk[nt][v] = dkh[key 16 rg + r][feature colk + 16 nt + 4 q4 + v]; dv likewise before s r_j
    f32x4 dk[NKT], dv[NVT];
#pragma unroll
    for (int nt = 0; nt < NKT; ++nt) dk[nt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int nt = 0; nt < NVT; ++nt) dv[nt] = f32x4{0.f, 0.f, 0.f, 0.f};

    // later chunks: dv^T += R^T k^T (over d_key), dkh^T += R v^T (over d_value)
    constexpr int KS_BOTH = Cfg::KSK < Cfg::KSV ? Cfg::KSK : Cfg::KSV;
#pragma unroll
    for (int ks = 0; ks < (Cfg::KSK > Cfg::KSV ? Cfg::KSK : Cfg::KSV); ++ks) {
      frag8 rcol[NVT], rrow[NKT];
      if (ks < Cfg::KSK) {
#pragma unroll
        for (int nt = 0; nt < NVT; ++nt)
          rcol[nt] = lds_col_frag_ks(Rl, SP, ks, q4, colv + 16 * nt, r);
      }
      if (ks < Cfg::KSV) {
#pragma unroll
        for (int nt = 0; nt < NKT; ++nt)
          rrow[nt] = lds_row_frag(Rl + (colk + 16 * nt + r) * SP + lds_col(32 * ks), q4);
      }
      __builtin_amdgcn_sched_barrier(0);
      if (ks < KS_BOTH && NKT == NVT) {
#pragma unroll
        for (int nt = 0; nt < NKT; ++nt) {
          dv[nt] = mma16(rcol[nt], kf[ks], dv[nt]);
          dk[nt] = mma16(rrow[nt], vf[ks], dk[nt]);
        }
      } else {
        if (ks < Cfg::KSK) {
#pragma unroll
          for (int nt = 0; nt < NVT; ++nt) dv[nt] = mma16(rcol[nt], kf[ks], dv[nt]);
        }
        if (ks < Cfg::KSV) {
#pragma unroll
          for (int nt = 0; nt < NKT; ++nt) dk[nt] = mma16(rrow[nt], vf[ks], dk[nt]);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }

    // this chunk: query tiles it >= rg two at a time, and the reverse state update
#pragma unroll
    for (int p = 0; p < Cfg::NP; ++p) {
      const bool diag_or_above = 2 * p + 1 >= rg;
      const int t0 = 32 * p + 4 * q4, t1 = 32 * p + 16 + 4 * q4;  // token order of the slots
      frag8 qr[2][Cfg::KSK], gr[2][Cfg::KSV], qc[NKT];
      frag8 pf, af;
      const auto read_queries = [&](int half) {
#pragma unroll
        for (int ks = 0; ks < Cfg::KSK; ++ks)
          qr[half][ks] = lds_row_frag(Qs + (16 * (2 * p + half) + r) * TPK + lds_col(32 * ks), q4);
      };
      const auto read_out_grads = [&](int half) {
#pragma unroll
        for (int ks = 0; ks < Cfg::KSV; ++ks)
          gr[half][ks] = lds_row_frag(Gs + (16 * (2 * p + half) + r) * TPV + lds_col(32 * ks), q4);
      };
      const auto read_query_columns = [&] {
#pragma unroll
        for (int nt = 0; nt < NKT; ++nt) qc[nt] = lds_col_frag(Qs, TPK, t0, t1, colk + 16 * nt, r);
      };
      // tile of query tile 2p + half and this wave's keys; t[v]: query 16 it + 4 q4 + v, key
      // 16 rg + r; keep key <= query
      const auto put_masked = [&](frag8& f, int half, f32x4 t) {
        const int it = 2 * p + half;
        const bool full = it > rg, diag = it == rg;
        put_half(f, half, t, full || (diag && r <= 4 * q4 + 0), full || (diag && r <= 4 * q4 + 1),
                 full || (diag && r <= 4 * q4 + 2), full || (diag && r <= 4 * q4 + 3), un);
      };
      const auto form_p = [&](int half) {
        f32x4 t = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < Cfg::KSK; ++ks) t = mma16(qr[half][ks], kf[ks], t);
        return t;
      };
      const auto form_a = [&](int half) {
        f32x4 t = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < Cfg::KSV; ++ks) t = mma16(gr[half][ks], vf[ks], t);
        return t;
      };
      if constexpr (Cfg::SHARE_MASKED) {
        __syncthreads();  // the partial tiles of the other waves are there
#pragma unroll
        for (int half = 0; half < 2; ++half) {
          f32x4 tp = {0.f, 0.f, 0.f, 0.f}, ta = {0.f, 0.f, 0.f, 0.f};
          if (half >= rg) {
            tp = masked.get(half, w, l);
            ta = masked.get(2 + half, w, l);
          }
          put_masked(pf, half, tp);
          put_masked(af, half, ta);
        }
        __builtin_amdgcn_sched_barrier(0);
      } else if (Cfg::DKDV_PHASED && diag_or_above) {
#pragma unroll
        for (int half = 0; half < 2; ++half) {
          if (Cfg::SKIP_UNSEEN && half < rg) {
            put_no_half(pf, half);
            put_no_half(af, half);
            continue;
          }
          read_queries(half);
          __builtin_amdgcn_sched_barrier(0);
          put_masked(pf, half, form_p(half));
          __builtin_amdgcn_sched_barrier(0);
          read_out_grads(half);
          __builtin_amdgcn_sched_barrier(0);
          put_masked(af, half, form_a(half));
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      frag8 gc[NVT], qcol[AT::NCT], grow[AT::NRT];
#pragma unroll
      for (int nt = 0; nt < NVT; ++nt) gc[nt] = lds_col_frag(Gs, TPV, t0, t1, colv + 16 * nt, r);
#pragma unroll
      for (int x = 0; x < AT::NCT; ++x)
        qcol[x] = lds_col_frag(Qs, TPK, t0, t1, 16 * AT::col_tile(rg, cp, x), r);
      if (!AT::ROW_OPERAND_IS_RESULT_COLUMN) {
#pragma unroll
        for (int y = 0; y < AT::NRT; ++y)
          grow[y] = lds_col_frag(Gs, TPV, t0, t1, 16 * AT::row_tile(rg, cp, y), r);
      }
      __builtin_amdgcn_sched_barrier(0);
      // reverse state update: R^T += dO^T (r q) over these 32 tokens
      if (AT::active(rg, cp)) {
#pragma unroll
        for (int y = 0; y < AT::NRT; ++y)
#pragma unroll
          for (int x = 0; x < AT::NCT; ++x)
            racc[x][y] = mma16_add(AT::ROW_OPERAND_IS_RESULT_COLUMN ? gc[y] : grow[y], qcol[x], racc[x][y]);
      }
      if (diag_or_above) {
        if (Cfg::DKDV_PHASED) {
          if (Cfg::HALF_VISIBLE && rg == 1) {
#pragma unroll
            for (int nt = 0; nt < NVT; ++nt) dv[nt] = mma16_half_add(gc[nt], pf, dv[nt], 1);
          } else {
#pragma unroll
            for (int nt = 0; nt < NVT; ++nt) dv[nt] = mma16_add(gc[nt], pf, dv[nt]);
          }
          __builtin_amdgcn_sched_barrier(0);
          read_query_columns();
          __builtin_amdgcn_sched_barrier(0);
        } else {
#pragma unroll
          for (int half = 0; half < 2; ++half) {
            read_queries(half);
            read_out_grads(half);
          }
          read_query_columns();
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int half = 0; half < 2; ++half) {
            const f32x4 tp = form_p(half), ta = form_a(half);
            put_masked(pf, half, tp);
            put_masked(af, half, ta);
          }
#pragma unroll
          for (int nt = 0; nt < NVT; ++nt) dv[nt] = mma16_add(gc[nt], pf, dv[nt]);
        }
        if (Cfg::HALF_VISIBLE && rg == 1) {
#pragma unroll
          for (int nt = 0; nt < NKT; ++nt) dk[nt] = mma16_half_add(qc[nt], af, dk[nt], 1);
        } else {
#pragma unroll
          for (int nt = 0; nt < NKT; ++nt) dk[nt] = mma16_add(qc[nt], af, dk[nt]);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }

    // epilogue: dv_j = s r_j dv; dk_j through the normalisation chain rule; both staged in
    // the row group's own (dead) rows of Vs and Ks
    const float rj = rk[16 * rg + r];
    float xv[NKT][4];
    float t = dot_with_row<NKT, TPK>(dk, Ks + 16 * rg * TPK, colk, xv, r, q4);
    if (CS > 1) {  // the row's dot product over the columns of all its waves
      if (q4 == 0) xdot[cp * C + 16 * rg + r] = t;
      __syncthreads();  // and the rows of Ks / Vs were read by all of them
      t = 0.f;
#pragma unroll
      for (int i = 0; i < CS; ++i) t += xdot[i * C + 16 * rg + r];
    }
    project_out_row<NKT, false>(dk, xv, t, rj, inv_eps);
    if (CS == 1) wave_lds_sync();  // own Ks / Vs rows (kf, vf, raw k) were read before the staging writes
    gather_rows_transposed<DK, NKT>(dk, scale * rj, Ks + 16 * rg * TPK, l, done_k, un, colk);
    gather_rows_transposed<DV, NVT>(dv, scale * rj, Vs + 16 * rg * TPV, l, done_v, un, colv);
    __syncthreads();
    done_dK = dKu;
    done_dV = dVu;
    done_row = row0;
    done_end = row_end;
    if (cross) {   // the unit begins here
      if (rev_out != nullptr && AT::active(rg, cp)) store_rev_out();
      if (seq_len != nullptr) {
        zero_rows<DK>(dKu, row_end, piece_end);
        zero_rows<DV>(dVu, row_end, piece_end);
      }
      piece_end = N;
      --unit;
      left -= unit_rows;
      dKu -= size_t(N) * DK;
      dVu -= size_t(N) * DV;
      scale = unit_scale(s, unit, H, s_per_unit);
#pragma unroll
      for (int x = 0; x < AT::NCT; ++x)
#pragma unroll
        for (int y = 0; y < AT::NRT; ++y) racc[x][y] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (rev_in != nullptr && AT::active(rg, cp)) add_rev_in();
    }
    row_begin = next_begin;
    row0 = next_row;
    row_end = next_end;
  }
  if (EVEN ? done_end > 0 : row_begin < row_end) {
    store_row_pieces<DK, NKT>(done_k, EVEN ? done_dK : dKu, (EVEN ? done_row : row_begin) + 16 * rg,
                              EVEN ? done_end : row_end, l, colk);
    store_row_pieces<DV, NVT>(done_v, EVEN ? done_dV : dVu, (EVEN ? done_row : row_begin) + 16 * rg,
                              EVEN ? done_end : row_end, l, colv);
  }
  if (seq_len != nullptr) {  // rows that do not exist
    zero_rows<DK>(dKu, row_end, piece_end);
    zero_rows<DV>(dVu, row_end, piece_end);
  }
  if (rev_out != nullptr && row_begin == 0 && AT::active(rg, cp)) store_rev_out();
#ifdef COTTN_SPLIT3
  if (un.in_workgroup<Cfg::NW>(rk)) {
    using Whole = f32w::BwdCfg<DK, DV, C, CS>;
    static_assert(2 * Whole::TILEK <= Cfg::TILEK && 2 * Whole::TILEV <= Cfg::TILEV && 2 * Whole::STATE <= Cfg::STATE, "whole rows fit");
    void* const room[] = {Qs, Ks, Vs, Gs, Rl, rk, xdot};
    f32w::bwd_dkdv_scan<DK, DV, C, CS, WALK>(room, Q, K, V, dO, s, dK, dV, rev_states, ds_partial, ds, B, H, N, G, seg_rows,
                                             inv_eps, sum_totals, lengths, s_per_unit, rev_in, rev_out, unit_rows);
  }
#endif
}

#ifndef COTTN_REDO
template <int DK, int DV, int C, int CR = BwdSplit<DK, DV, C>::CR, int CS = BwdSplit<DK, DV, C>::CS>
hipError_t run_bwd_causal(const CausalArgs& a) {
  using Cfg = BwdCfg<DK, DV, CR, CS>;
  const int units = a.B * a.H;
  const elem_t* Q = static_cast<const elem_t*>(a.Q);
  const elem_t* K = static_cast<const elem_t*>(a.K);
  const elem_t* V = static_cast<const elem_t*>(a.V);
  const elem_t* dO = static_cast<const elem_t*>(a.dO);
  char* ws = static_cast<char*>(a.workspace);
  const float* fwd_states = nullptr;
  float* rev_states = nullptr;
  const dim3 grid(a.workgroups);
  const bool even = a.unit_rows > 0;
  const float inv_eps = 1.0f / a.eps;
  // few segments: no carry launches, the scan workgroups add up the totals they need
  const bool sum_in_scan = even || causal_totals_in_place(units, a.G, DK, DV, ELEM_IS_F32);
  // an own-prefix forward leaves carried prefixes
  const bool carried = a.own_prefix && a.saved_fwd_states != nullptr;
  const bool rebuild = a.own_prefix && !carried && own_prefix_dq(units, a.G, a.seg_rows, DK, DV, ELEM_IS_F32);
  hipError_t err;
  if (a.G > 1 || even) {
    // Forward-time states: taken over from the forward call when it left them behind (raw
    // totals or carried prefixes, by the same rule as here), else recomputed from K and V.
    float* own_fwd = reinterpret_cast<float*>(ws);
    rev_states = reinterpret_cast<float*>(ws + state_slots_bytes(a.slots, DK, DV));
    ws += 2 * state_slots_bytes(a.slots, DK, DV);
    if (a.saved_fwd_states != nullptr) {
      fwd_states = a.saved_fwd_states;
    } else if (!rebuild) {
      err = COTTN_ELEM_SYM(launch_fwd_segment_totals)(a, own_fwd);
      if (err != hipSuccess) return err;
      if (!sum_in_scan) {
        err = launch_bwd_state_carry(own_fwd, nullptr, units, a.G, DK * DV, a.stream);
        if (err != hipSuccess) return err;
      }
      fwd_states = own_fwd;
    }
  }
  float* ds_partial = reinterpret_cast<float*>(ws);
  // the dQ scan leaves the reverse-time segment totals (of qh^T dO) behind for the dK/dV scan
  const auto dq_scan = [&](auto kernel, int threads) {
    return launch_kernel(COTTN_SYM_STR(bwd_dq_scan), kernel, grid, dim3(threads), 0, a.stream, Q, K, V, dO, a.s,
                         static_cast<elem_t*>(a.dQ), fwd_states, rev_states, ds_partial, a.H, a.N, a.G, a.seg_rows,
                         inv_eps, sum_in_scan && !carried ? (a.marked && a.saved_fwd_states != nullptr ? 2 : 1) : 0, a.seq_len, a.s_per_unit, a.state_in,
                         units, a.unit_rows);
  };
  // (one wave per row group at 128 x 128 is for more workgroups than a split or shares ever make: threads_fit)
  constexpr bool VERY_MANY = !ELEM_IS_F32 && DK == 128 && DV == 128 && CS == 1;
  constexpr bool EVEN_BUILT = even_shares_built(DK, DV, ELEM_IS_F32) && !VERY_MANY;
  constexpr bool HALVED = !ELEM_IS_F32 && DK == 128 && DV == 128 && CR == 64 && CS == 2;
  if (HALVED && a.G == 1 && !even && two_to_a_cu_dq(a.workgroups)) {
    if constexpr (HALVED) err = dq_scan(COTTN_SYM(bwd_dq_scan)<DK, DV, 32, CS, false, SEGMENTS>, 256);
  } else if (even) {
    if constexpr (EVEN_BUILT)
      err = a.seq_len == nullptr ? dq_scan(COTTN_SYM(bwd_dq_scan)<DK, DV, CR, CS, true, EVEN_SHARES>, Cfg::NT)
                                 : dq_scan(COTTN_SYM(bwd_dq_scan)<DK, DV, CR, CS, true, EVEN_PADDED>, Cfg::NT);
  } else if (rebuild) {
    const bool by_sets = Cfg::PREFIX_SETS > 1 && prefix_by_sets(a.workgroups);
    if constexpr (Cfg::PREFIX_SETS > 1 && C <= 64)
      if (by_sets) err = dq_scan(COTTN_SYM(bwd_dq_scan)<DK, DV, CR, CS, true, OWN_PREFIX_SETS>, Cfg::NT);
    if constexpr (C <= 64 && !VERY_MANY)
      if (!by_sets) err = dq_scan(COTTN_SYM(bwd_dq_scan)<DK, DV, CR, CS, true, OWN_PREFIX>, Cfg::NT);
  } else {
    err = dq_scan(COTTN_SYM(bwd_dq_scan)<DK, DV, CR, CS, true, SEGMENTS>, Cfg::NT);
  }
  if (err != hipSuccess) return err;
  if (!sum_in_scan) {
    err = launch_bwd_state_carry(nullptr, rev_states, units, a.G, DK * DV, a.stream);
    if (err != hipSuccess) return err;
  }
  // the dK/dV kernel also reduces the ds partial sums written by the dQ kernel
  const auto dkdv_scan = [&](auto kernel, int threads) {
    return launch_kernel(COTTN_SYM_STR(bwd_dkdv_scan), kernel, grid, dim3(threads), 0, a.stream, Q, K, V, dO, a.s,
                         static_cast<elem_t*>(a.dK), static_cast<elem_t*>(a.dV), rev_states, ds_partial, a.ds, a.B,
                         a.H, a.N, a.G, a.seg_rows, inv_eps, sum_in_scan ? 1 : 0, a.seq_len, a.s_per_unit,
                         a.rev_state_in, a.rev_state_out, a.unit_rows);
  };
  if constexpr (HALVED)
    if (!even && two_to_a_cu_dkdv(a.workgroups))
      return dkdv_scan(COTTN_SYM(bwd_dkdv_scan)<DK, DV, 32, CS, SEGMENTS>, 256);
  if constexpr (EVEN_BUILT)
    if (even)
      return a.seq_len == nullptr ? dkdv_scan(COTTN_SYM(bwd_dkdv_scan)<DK, DV, CR, CS, EVEN_SHARES>, Cfg::NT)
                                  : dkdv_scan(COTTN_SYM(bwd_dkdv_scan)<DK, DV, CR, CS, EVEN_PADDED>, Cfg::NT);
  return dkdv_scan(COTTN_SYM(bwd_dkdv_scan)<DK, DV, CR, CS, SEGMENTS>, Cfg::NT);
}
#endif  // COTTN_REDO

}  // namespace
}  // namespace COTTN_NS

#ifndef COTTN_REDO
using namespace COTTN_NS;

#if !defined(COTTN_ELEM_F16) && !defined(COTTN_ELEM_F32)  // not specific to the element type
hipError_t launch_bwd_state_carry(float* fwd_tot, float* rev_tot, int units, int G, int elems,
                                  hipStream_t st) {
  const long total = long(units) * elems;
  return launch_kernel("bwd_state_carry", bwd_state_carry, dim3(unsigned((total / 4 + 255) / 256), 2),
                       dim3(256), 0, st, fwd_tot, rev_tot, G, elems, total);
}
#endif

hipError_t COTTN_SYM(bwd_causal)(const CausalArgs& a) {
#if defined(COTTN_F32_WHOLE)
  switch ((a.dk * 1000 + a.dv) * 1000 + a.C) {
    case 32128032: return run_bwd_causal<32, 128, 32>(a);
    case 128032032: return run_bwd_causal<128, 32, 32>(a);
    case 128128032: return run_bwd_causal<128, 128, 32>(a);
    default: return hipErrorInvalidValue;
  }
#elif defined(COTTN_ELEM_F32)
  switch ((a.dk * 1000 + a.dv) * 1000 + a.C) {
    case 32032032: return run_bwd_causal<32, 32, 32>(a);
    case 32064032: return run_bwd_causal<32, 64, 32>(a);
    case 32128032: case 128032032: case 128128032: return bwd_causal_f32w(a);   // device_common.h: SPLIT3
    case 64032032: return run_bwd_causal<64, 32, 32>(a);
    case 64064032: return run_bwd_causal<64, 64, 32>(a);
    case 64128032: return run_bwd_causal<64, 128, 32>(a);
    case 128064032: return run_bwd_causal<128, 64, 32>(a);
    default: return hipErrorInvalidValue;
  }
#else
  // d_key != d_value: chunks of 64 rows
  switch ((a.dk * 1000 + a.dv) * 1000 + a.C) {
    case 32032064: return run_bwd_causal<32, 32, 64>(a);
    case 32032128: return run_bwd_causal<32, 32, 128>(a);
    case 32032256: return run_bwd_causal<32, 32, 256>(a);
    case 64064064: return run_bwd_causal<64, 64, 64>(a);
    case 64064128: return run_bwd_causal<64, 64, 128>(a);
    case 64064256: return run_bwd_causal<64, 64, 256>(a);
    case 128128064:
      return threads_fit(long(a.B) * a.H * a.G, 512) ? run_bwd_causal<128, 128, 64>(a)
                                                     : run_bwd_causal<128, 128, 64, 64, 1>(a);
    case 32064064: return run_bwd_causal<32, 64, 64>(a);
    case 32128064: return run_bwd_causal<32, 128, 64>(a);
    case 64032064: return run_bwd_causal<64, 32, 64>(a);
    case 64128064: return run_bwd_causal<64, 128, 64>(a);
    case 128032064: return run_bwd_causal<128, 32, 64>(a);
    case 128064064: return run_bwd_causal<128, 64, 64>(a);
    default: return hipErrorInvalidValue;
  }
#endif
}

#endif  // COTTN_REDO

}  // namespace cottn
