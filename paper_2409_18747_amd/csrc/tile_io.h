// Global -> register -> LDS staging of [rows][D] tiles of elements, with the row L2 norm of
// Sec. 3.2 computed on the way (16-bit: sum of squares with the packed dot instruction; reduced
// over the lanes that share a row with DPP moves).
//
// The normalisation x / max(||x||, eps) is applied element by element only where it must be.
// With r_i = 1 / max(||q_i||, eps) and r_j likewise for k_j, every product of the method is
// linear in qh_i = r_i q_i and kh_j = r_j k_j.  Where the rows of a result belong to the
// normalised operand's rows, the raw rows are the MFMA operand and the factor multiplies the
// finished fp32 result row; only an operand that is contracted over the token index is
// rescaled on its way into LDS (K in the forward and dQ passes, Q in the dK/dV pass).  A
// rescaled row has norm at most 1, so this is safe in IEEE half precision too: no row is
// ever multiplied by the factor of another row, which is 1/eps when that row is zero.
// Included behind device_common.h, and as often.

namespace cottn {
namespace COTTN_NS {

// A workgroup of NT threads moves a tile of C rows x D columns.  Each lane owns 16
// consecutive bytes (EPP columns) of a row; D/EPP neighbouring lanes share a row, so a
// wavefront reads whole rows: fully coalesced.
__device__ __forceinline__ uint4 load_rows(const elem_t* p, bool stream) {
  if (stream) {
    const u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
    return uint4{v.x, v.y, v.z, v.w};
  }
  return *reinterpret_cast<const uint4*>(p);
}

// (LD: elements from a row of the tensor to the next, more than D where D columns of it are taken.)
template <int D, int C, int NT, int LD = D>
struct TileStage {
  static constexpr int LPR = D / EPP;     // lanes per row
  static constexpr int RPP = NT / LPR;    // rows per pass
  static constexpr int PASSES = (C + RPP - 1) / RPP;
  static_assert(NT % LPR == 0, "thread count must cover whole rows");
  static_assert(C % RPP == 0 || C < RPP, "tile rows must be a multiple of rows per pass");

  uint4 regs[PASSES];

  // rows >= n_rows (end of the sequence or of the segment) read as zero; `stream` (uniform
  // over the workgroup) marks the loads non-temporal: rows nothing will find in a cache again
  __device__ __forceinline__ void fetch(const elem_t* __restrict__ base, int row0, int n_rows,
                                        bool stream = false) {
    const int tid = threadIdx.x;
    // a base that is the same for all lanes plus a 32-bit lane offset that is the same for all
    // tiles: the addresses then take scalar registers and one vector register
    const elem_t* rows = base + size_t(row0) * LD;
    const unsigned lane = unsigned((tid / LPR) * LD + (tid % LPR) * EPP);
    if (C % RPP == 0 && row0 + C <= n_rows) {
      // whole tile in range (workgroup-uniform): plain loads at constant strides
#pragma unroll
      for (int p = 0; p < PASSES; ++p)
        regs[p] = load_rows(rows + p * RPP * LD + lane, stream);
      return;
    }
#pragma unroll
    for (int p = 0; p < PASSES; ++p) {
      const int lr = p * RPP + tid / LPR;
      uint4 v = {0u, 0u, 0u, 0u};
      if (lr < C && row0 + lr < n_rows) v = load_rows(rows + p * RPP * LD + lane, stream);
      regs[p] = v;
    }
  }

  // rinv[p] = min(1/||row||, inv_eps) = 1 / max(||row||, eps) for the row this lane holds in
  // pass p (every lane of the row gets the same value).
  __device__ __forceinline__ void row_rinv(float inv_eps, float* rinv) const {
    float sum_sq[PASSES];
#pragma unroll
    for (int p = 0; p < PASSES; ++p) sum_sq[p] = group_sum<LPR>(piece_sum_sq(regs[p]));
    row_inv_norms<PASSES>(sum_sq, inv_eps, rinv);
  }

  // out[local row] = rinv of that row (one lane per row writes)
  __device__ __forceinline__ void store_rinv(float* out, const float* rinv) const {
    const int tid = threadIdx.x;
#pragma unroll
    for (int p = 0; p < PASSES; ++p) {
      const int lr = p * RPP + tid / LPR;
      if ((C % RPP == 0 || lr < C) && (tid % LPR) == 0) out[lr] = rinv[p];
    }
  }

  __device__ __forceinline__ void commit_plain(lds_t* tile, Unparted& un) const {
    const int tid = threadIdx.x;
    const int col = lds_col((tid % LPR) * EPP);
#pragma unroll
    for (int p = 0; p < PASSES; ++p) {
      const int lr = p * RPP + tid / LPR;
      if (C % RPP == 0 || lr < C) store_piece_lds<false>(tile + lr * tile_pitch(D, C) + col, regs[p], 1.f, un);
    }
  }

  // tile[lr][:] = scale[p] * row, rounded to the element type
  __device__ __forceinline__ void commit_scaled(lds_t* tile, const float* scale, Unparted& un) const {
    const int tid = threadIdx.x;
    const int col = lds_col((tid % LPR) * EPP);
#pragma unroll
    for (int p = 0; p < PASSES; ++p) {
      const int lr = p * RPP + tid / LPR;
      if (C % RPP == 0 || lr < C)
        store_piece_lds<true>(tile + lr * tile_pitch(D, C) + col, regs[p], scale[p], un);
    }
  }
};

// Which 16x16 tiles of a DR x DC fp32 accumulator matrix a wave owns, for a workgroup of NW
// waves.  The matrix is cut into (DR/16) x (DC/16) tiles indexed (row tile, column tile).  A
// wave keeps one or more whole tile columns when there are fewer waves than columns (so the
// column-side operand is loaded once per wave); otherwise the waves that share a tile column
// split its row tiles.  (The state K^T V is d_key x d_value; which of the two is the row side
// depends on the kernel's accumulator orientation.)
template <int DR, int DC, int NW>
struct AccTiles {
  static constexpr int RT = DR / 16, CT = DC / 16;
  static constexpr int NCT = (NW >= CT) ? 1 : CT / NW;      // column tiles per wave
  static constexpr int WPC = (NW >= CT) ? NW / CT : 1;      // waves per tile column
  static constexpr int NRT = (WPC >= RT) ? 1 : RT / WPC;    // row tiles per wave
  __device__ static __forceinline__ bool active(int w) { return (w / CT) * NRT < RT; }
  __device__ static __forceinline__ int col_tile(int w, int x) { return (w % CT) + x * NW; }
  __device__ static __forceinline__ int row_tile(int w, int y) {
    return (NW >= CT) ? (w / CT) * NRT + y : y;
  }
};

// The same ownership when the RG row groups of a chunk are each served by CS waves that split
// the result columns between them (wave = (row group rg, column part cp)).  CS = 1 is AccTiles
// over the row groups.  CS > 1: a wave owns the row tiles of its own column part, which are the
// tiles whose fragments it reads for its result columns anyway, and the column tiles rg, rg +
// RG, ...
template <int DR, int DC, int RG, int CS>
struct SplitTiles {
  using One = AccTiles<DR, DC, RG>;
  static constexpr int RT = DR / 16, CT = DC / 16;
  static constexpr int NCT = CS == 1 ? One::NCT : (RG >= CT ? 1 : CT / RG);
  static constexpr int NRT = CS == 1 ? One::NRT : RT / CS;
  // whether the row-side operand of the state update is among the fragments of the wave's
  // result columns (else it is read separately)
  static constexpr bool ROW_OPERAND_IS_RESULT_COLUMN = CS == 1 ? One::WPC == 1 : true;
  // stored states a wave loads at once when it seeds its accumulators, up to BATCH of them and beyond
  static constexpr int TILES = NCT * NRT, STATE_BATCH = states_at_once(TILES),
                       STATE_MANY = states_at_once_of_many(TILES, DR * DC, RG * CS);
  static_assert(CS == 1 || RT % CS == 0, "column parts must be whole tiles");
  __device__ static __forceinline__ bool active(int rg, int cp) {
    return CS == 1 ? One::active(rg) : rg < CT;
  }
  __device__ static __forceinline__ int col_tile(int rg, int cp, int x) {
    return CS == 1 ? One::col_tile(rg, x) : rg % CT + x * RG;
  }
  __device__ static __forceinline__ int row_tile(int rg, int cp, int y) {
    return CS == 1 ? One::row_tile(rg, y) : cp * NRT + y;
  }
};

// Whole fp32, two waves on each of the two row groups of a 32-row chunk: both need the group's masked
// tiles, and an fp32 MFMA is slow enough that forming them twice shows (8 of the 24 products a
// wave has in a chunk of the dK/dV scan at d = 64).  Each wave contracts half of the features and
// passes its partial tile on through LDS: slot = one per tile of the group.
template <int TILES>
struct MaskedExchange {
  f32x4 part[TILES][4][64];   // [tile][wave][lane]
  __device__ __forceinline__ void put(int tile, int w, int l, f32x4 t) { part[tile][w][l] = t; }
  // both halves of the features (waves w and w ^ 2 serve the same row group)
  __device__ __forceinline__ f32x4 get(int tile, int w, int l) const {
    return part[tile][w & 1][l] + part[tile][w | 2][l];
  }
};

// Row group and column part of a wave.  With the masked tiles of a chunk skipped where nothing is
// visible, one of the two row groups of the fp32 scans has less to do; wave w runs on SIMD w % 4,
// so every second round of workgroups (256 compute units) swaps the groups.
template <int RG, int CS>
__device__ __forceinline__ int row_group(int w) {
  return ELEM_IS_F32 && RG == 2 ? (w + (blockIdx.x >> 8)) % RG : w % RG;
}

// fp32 in parts, two waves on each of the two row groups of a 32-row chunk: one row group sees only half of the keys (or
// queries), and the masked tile of the other half, which costs twelve to 24 matrix instructions and the parting of its
// values, is left out (the two workgroups of a compute unit have opposite groups on a SIMD, see above).  Causal kernels,
// formed / left out: B8 H12 N1024 d64 forward 28.6 -> 28.0 us, dK/dV 40.3 -> 39.2; 300 units of 1000 rows 64 x 128 173.5 -> 169.6, dQ
// 228 -> 204, dK/dV 260 -> 255; 40 of 1024 at 128 x 64 forward 34.1 -> 31.1.  (At d64 that is what the runs of the whole pair differ
// by: 117.3, 116.0 to 120.1 -> 116.8, 113.0 to 119.0.)  The dQ scan takes it at 128 value columns only: at
// 64 x 64 the branch costs 16 spilled registers (35.7 -> 37.4), at 32 columns it makes no difference.
constexpr bool skips_unseen(int waves_per_group, int rows) { return SPLIT3 && waves_per_group == 2 && rows == 32; }

// acc += the wave's tiles of the stored states first..last, `load(state, x, y)` returning
// tile (x, y) of one of them.  States are taken BATCH at a time with every load of a batch
// issued before the first addition, so a batch costs one memory latency, not one per state; MANY at a time
// while there are more than BATCH of them.
// Slots of the last batch beyond `last` re-read `last` (an address already in flight) and
// are discarded.
template <int BATCH, int NCT, int NRT, class LoadTile>
__device__ __forceinline__ void add_stored_batch(f32x4 (&acc)[NCT][NRT], int base, int last, LoadTile load) {
  f32x4 t[BATCH][NCT][NRT];
#pragma unroll
  for (int i = 0; i < BATCH; ++i)
#pragma unroll
    for (int x = 0; x < NCT; ++x)
#pragma unroll
      for (int y = 0; y < NRT; ++y) t[i][x][y] = load(min(base + i, last), x, y);
#pragma unroll
  for (int i = 0; i < BATCH; ++i) {
    const bool keep = base + i <= last;
#pragma unroll
    for (int x = 0; x < NCT; ++x)
#pragma unroll
      for (int y = 0; y < NRT; ++y)
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[x][y][v] += keep ? t[i][x][y][v] : 0.f;
  }
}
template <int BATCH, int MANY, int NCT, int NRT, class LoadTile>
__device__ __forceinline__ void add_stored_states(f32x4 (&acc)[NCT][NRT], int first, int last,
                                                  LoadTile load) {
  int base = first;
  if constexpr (MANY > BATCH)
    for (; base + BATCH <= last; base += MANY) add_stored_batch<MANY>(acc, base, last, load);
  for (; base <= last; base += BATCH) add_stored_batch<BATCH>(acc, base, last, load);
}

// acc += kh^T v over rows row_begin .. row_end - 1 of one unit, C rows at a time; the first C rows
// of K and V have been fetched.  acc[x][y] = S tile (key tile row_tile(y), value tile col_tile(x)),
// held with the keys along the lanes: element [v] of lane (r, q4) is S[16 kt + r][16 vt + 4 q4 + v],
// the orientation the forward and the dQ scan keep their running state in.  Ends with the tiles
// still being read: a barrier has to follow before they are written again.
template <int DK, int DV, int C, int NT, class ST = AccTiles<DK, DV, NT / 64>>
__device__ __forceinline__ void add_rows_to_state(f32x4 (&acc)[ST::NCT][ST::NRT], TileStage<DK, C, NT>& kst,
                                                  TileStage<DV, C, NT>& vst, lds_t* Ks, lds_t* Vs,
                                                  const elem_t* __restrict__ Ku, const elem_t* __restrict__ Vu,
                                                  int row_begin, int row_end, float inv_eps, int w, int l, Unparted& un) {
  constexpr int TPK = tile_pitch(DK, C), TPV = tile_pitch(DV, C);
  const int r = l % 16, q4 = l / 16;
  for (int row0 = row_begin; row0 < row_end; row0 += C) {
    float rk[TileStage<DK, C, NT>::PASSES];
    kst.row_rinv(inv_eps, rk);
    __syncthreads();  // previous chunk's reads of Ks/Vs are done
    kst.commit_scaled(Ks, rk, un);
    vst.commit_plain(Vs, un);
    if (row0 + C < row_end) {
      kst.fetch(Ku, row0 + C, row_end);
      vst.fetch(Vu, row0 + C, row_end);
    }
    __syncthreads();
    if (ST::active(w)) {
#pragma unroll
      for (int p = 0; p < C / 32; ++p) {
        frag8 bv[ST::NCT], ak[ST::NRT];
#pragma unroll
        for (int x = 0; x < ST::NCT; ++x)
          bv[x] = lds_col_frag_ks(Vs, TPV, p, q4, 16 * ST::col_tile(w, x), r);
#pragma unroll
        for (int y = 0; y < ST::NRT; ++y)
          ak[y] = lds_col_frag_ks(Ks, TPK, p, q4, 16 * ST::row_tile(w, y), r);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int y = 0; y < ST::NRT; ++y)
#pragma unroll
          for (int x = 0; x < ST::NCT; ++x) acc[x][y] = mma16_add(bv[x], ak[y], acc[x][y]);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
}

// acc += kh^T v over rows 0 .. n_rows - 1 of one unit, SETS x C rows at a time (each C rows through tiles of their
// own, Ks[i] and Vs[i]), the tiles of the state dealt to the waves as in the scan that goes on from them: key
// tiles key_tile(i), value tiles value_tile(j), and add(i, j, k fragment, v fragment).  Ends behind a barrier.
template <int DK, int DV, int C, int NT, int NK, int NV, int LDV, int SETS, class KeyTile, class ValueTile, class Add>
__device__ __forceinline__ void add_rows_before(lds_t* (&Ks)[SETS], lds_t* (&Vs)[SETS],
                                                const elem_t* __restrict__ Ku, const elem_t* __restrict__ Vu, int n_rows,
                                                float inv_eps, int l, bool active, KeyTile key_tile, ValueTile value_tile,
                                                Add add, Unparted& un) {
  constexpr int TPK = tile_pitch(DK, C), TPV = tile_pitch(DV, C);
  const int r = l % 16, q4 = l / 16;
  TileStage<DK, C, NT> kst[SETS];
  TileStage<DV, C, NT, LDV> vst[SETS];
  const auto fetch = [&](int row0) {
#pragma unroll
    for (int i = 0; i < SETS; ++i) {
      if (i > 0 && row0 + i * C >= n_rows) break;
      kst[i].fetch(Ku, row0 + i * C, n_rows);
      vst[i].fetch(Vu, row0 + i * C, n_rows);
    }
  };
  fetch(0);
  for (int row0 = 0; row0 < n_rows; row0 += SETS * C) {
#pragma unroll
    for (int i = 0; i < SETS; ++i) {
      if (i > 0 && row0 + i * C >= n_rows) break;
      float rk[TileStage<DK, C, NT>::PASSES];
      kst[i].row_rinv(inv_eps, rk);
      kst[i].commit_scaled(Ks[i], rk, un);
      vst[i].commit_plain(Vs[i], un);
    }
    if (row0 + SETS * C < n_rows) fetch(row0 + SETS * C);
    __syncthreads();
    if (active) {
#pragma unroll
      for (int i = 0; i < SETS; ++i) {
        if (i > 0 && row0 + i * C >= n_rows) break;
#pragma unroll
        for (int p = 0; p < C / 32; ++p) {
          frag8 kf[NK], vf[NV];
#pragma unroll
          for (int x = 0; x < NK; ++x) kf[x] = lds_col_frag_ks(Ks[i], TPK, p, q4, 16 * key_tile(x), r);
#pragma unroll
          for (int y = 0; y < NV; ++y) vf[y] = lds_col_frag_ks(Vs[i], TPV, p, q4, 16 * value_tile(y), r);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int x = 0; x < NK; ++x)
#pragma unroll
            for (int y = 0; y < NV; ++y) add(x, y, kf[x], vf[y]);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
    __syncthreads();
  }
}

// A wave's finished result block (16 rows x NTILES*16 columns, by default all D columns) as
// whole 16-byte pieces of rows, one or more per lane, ready for coalesced global stores.
template <int D, int NTILES = D / 16>
struct RowPieces {
  static constexpr int PPR = 16 * NTILES / EPP;  // 16-byte pieces per row
  static constexpr int PIECES = 16 * PPR;    // in the wave's 16 rows
  static constexpr int PER_LANE = (PIECES + 63) / 64;
  uint4 v[PER_LANE];
};

// Turns a wave's result block whose accumulators are laid out TRANSPOSED (acc[nt][v] =
// result[row r][column col0 + 16 nt + 4 q4 + v], i.e. each lane holds 4 consecutive columns
// of one row) into row pieces: scales by the per-lane row factor, rounds to the element type, passes the
// block through a staging area private to the wave (16 rows of stage_pitch(D) elements from
// stage_rows on, columns col0..; it fits the wave's 16 rows of an operand tile, whose pitch is
// larger) with 8-byte writes (fp32: 16) and reads it back as 16-byte pieces.
template <int D, int NTILES = D / 16>
__device__ __forceinline__ void gather_rows_transposed(const f32x4* acc, float row_factor,
                                                       void* stage, int l,
                                                       RowPieces<D, NTILES>& out, Unparted& un, int col0 = 0) {
  using RP = RowPieces<D, NTILES>;
  constexpr int PITCH = stage_pitch(D);
  elem_t* stage_rows = static_cast<elem_t*>(stage);
  const int r = l % 16, q4 = l / 16;
  un.results<NTILES>(acc, row_factor);
#pragma unroll
  for (int nt = 0; nt < NTILES; ++nt) {
    store4(stage_rows + r * PITCH + col0 + 16 * nt + 4 * q4, row_factor * acc[nt][0],
           row_factor * acc[nt][1], row_factor * acc[nt][2], row_factor * acc[nt][3]);
  }
  wave_lds_sync();
#pragma unroll
  for (int j = 0; j < RP::PER_LANE; ++j) {
    const int i = l + 64 * j;
    const int lr = i / RP::PPR, col = col0 + (i % RP::PPR) * EPP;
    if (RP::PIECES % 64 == 0 || i < RP::PIECES)
      out.v[j] = *reinterpret_cast<const uint4*>(stage_rows + lr * PITCH + col);
  }
}

// Writes the pieces to rows first_row.. (columns col0..) of dst; rows at or beyond row_end are
// not written.  The scan kernels call this one chunk late (after the next chunk's loads have
// been issued): the wait for those loads at the top of a chunk step is a wait for every
// outstanding memory operation, and must not find stores that were issued a moment ago.
template <int D, int NTILES = D / 16, int LD = D>
__device__ __forceinline__ void store_row_pieces(const RowPieces<D, NTILES>& p,
                                                 elem_t* __restrict__ dst, int first_row,
                                                 int row_end, int l, int col0 = 0) {
  using RP = RowPieces<D, NTILES>;
  elem_t* rows = dst + size_t(first_row) * LD + col0;   // uniform over the wave
#pragma unroll
  for (int j = 0; j < RP::PER_LANE; ++j) {
    const int i = l + 64 * j;
    const int lr = i / RP::PPR;
    if ((RP::PIECES % 64 == 0 || i < RP::PIECES) && first_row + lr < row_end)
      store_streaming(rows + unsigned(lr * LD + (i % RP::PPR) * EPP), p.v[j]);
  }
}

// Sum of x over the four 16-lane rows of the wave (lanes r, r+16, r+32, r+48); every lane
// gets the total of its column.
__device__ __forceinline__ float sum_over_lane_rows(float x) {
  x += __shfl_xor(x, 16, 64);
  x += __shfl_xor(x, 32, 64);
  return x;
}

// Chain rule through the row normalisation on a wave's transposed 16-row block of NTILES * 16
// columns: acc[nt][v] = dxh[row r][column col0 + 16 nt + 4 q4 + v].  In two halves, because the
// waves of a row group may share its columns:
// dot_with_row reads the columns of the row into xv from `x_rows` (the 16 rows of the group in
// an LDS tile, row pitch PITCH, holding either the raw row x or xh = r x) and returns their dot
// product with dxh;
template <int NTILES, int PITCH>
__device__ __forceinline__ float dot_with_row(const f32x4* acc, const lds_t* x_rows, int col0,
                                              float (&xv)[NTILES][4], int r, int q4) {
  float t = 0.f;
#pragma unroll
  for (int nt = 0; nt < NTILES; ++nt) {
    load4_lds(x_rows + r * PITCH + lds_col(col0 + 16 * nt) + 4 * q4, xv[nt]);
#pragma unroll
    for (int v = 0; v < 4; ++v) t += xv[nt][v] * acc[nt][v];
  }
  return sum_over_lane_rows(t);
}
// project_out_row takes that product over the whole row and replaces acc by dxh - xh (xh . dxh)
// (no projection for rows at or below eps).  Returns xh . dxh.
template <int NTILES, bool NORMALISED>
__device__ __forceinline__ float project_out_row(f32x4* acc, const float (&xv)[NTILES][4], float t,
                                                 float rinv, float inv_eps) {
  const float c = (rinv == inv_eps) ? 0.f : (NORMALISED ? t : rinv * (rinv * t));
#pragma unroll
  for (int nt = 0; nt < NTILES; ++nt)
#pragma unroll
    for (int v = 0; v < 4; ++v) acc[nt][v] -= xv[nt][v] * c;
  return NORMALISED ? t : rinv * t;
}

}  // namespace COTTN_NS
}  // namespace cottn
