// Device-side primitives shared by the gfx950 kernels: vector types, the MFMA wrapper, LDS
// fragment reads (plain and transposing), packing, lane reductions.
// Nothing in here knows about attention.
//
// The MFMA kernels are written once for a floating-point element and compiled for three:
// bfloat16 by default, IEEE half when the translation unit defines COTTN_ELEM_F16 before
// including anything, fp32 with COTTN_ELEM_F32 (the *_f16.hip and *_f32.hip files do exactly
// that and then include the kernel source).  fp32 comes in two ways, see SPLIT3 below.
// COTTN_SYM(name) appends the element's suffix to kernel and launcher names.
//
// No include guard: a translation unit includes this once for each way it computes in, each time in a
// namespace of its own (COTTN_NS).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "launch.h"

#undef COTTN_NS
#undef COTTN_SYM
#undef COTTN_SYM_STR
#undef COTTN_ELEM_SYM
#undef COTTN_SPLIT3
#if defined(COTTN_ELEM_F32) && defined(COTTN_F32_WHOLE)
#define COTTN_NS f32w
#elif defined(COTTN_ELEM_F32)
#define COTTN_NS f32
#elif defined(COTTN_ELEM_F16)
#define COTTN_NS f16
#else
#define COTTN_NS bf16
#endif

namespace cottn {
namespace COTTN_NS {

// fp32 elements: how their products are formed.
//   SPLIT3  every operand in three bfloat16 parts x = x0 + x1 + x2 (each the rest rounded to
//           nearest: from 2^-110 up to 3.38e38 the sum is x exactly), six of the nine products of
//           parts on the bf16 matrix instruction.  Left out are x1 y2, x2 y1 and x2 y2: together just
//           under 2^-24 of a product at most, 2^-27.4 in the root mean square of normal values, where
//           an fp32 addition rounds to 2^-24 at most.  The bf16 rate is sixteen times the fp32 one, so
//           this takes 6/16 of the time, and the operands that are contracted over the tokens can take
//           the transposing LDS read.
//           Beyond that range, and where something is infinite or not a number, the workgroup that
//           meets it does its work again with whole products (Unparted).
//   else    the fp32 matrix instruction (COTTN_F32_WHOLE: the *_f32w.hip files), where the parts do
//           not fit the LDS (128 x 128) or fit it for one causal workgroup instead of two (128 x 32
//           and 32 x 128: B4 H8 N2048 forward + backward 121 / 140 and 108 / 123 us, whole / parts), and
//           where a row's few products are soon formed either way (32 x 32 without a mask, 32 / 33 us,
//           and the segment totals of that shape, 4.8 / 5.6).
// Elsewhere the parts are the faster way: forward + backward, whole / parts, B4 H8 N2048 causal 32 x
// 32 50 / 47 us, 64 x 64 106 / 88, 64 x 128 181 / 152, bidirectional 64 x 64 66 / 63, 128 x 64 122 /
// 105; B32 H16 N512 causal 64 x 64 271 / 227.  Then the vector ALU is what they wait for (it issues in
// 46 to 50 % of the cycles of the 64 x 64 scans, the matrix units are busy in 26 to 30 %): 6.5 instructions to part
// an element and note its range, about half of a step's.
#if defined(COTTN_ELEM_F32) && defined(COTTN_F32_WHOLE)
typedef float elem_native;  // the compiler's type for one element of an MFMA operand
typedef float elem_t;       // storage type of an element in global memory
typedef float lds_t;        // what the operand tiles and state copies in LDS are made of
#define COTTN_SYM(name) name##_f32w
#define COTTN_SYM_STR(name) #name "_f32w"
#elif defined(COTTN_ELEM_F32)
typedef __bf16 elem_native;
typedef float elem_t;
typedef uint16_t lds_t;
#define COTTN_SYM(name) name##_f32
#define COTTN_SYM_STR(name) #name "_f32"
#elif defined(COTTN_ELEM_F16)
typedef _Float16 elem_native;
typedef uint16_t elem_t;
typedef uint16_t lds_t;
#define COTTN_SYM(name) name##_f16
#define COTTN_SYM_STR(name) #name "_f16"
#else
typedef __bf16 elem_native;
typedef uint16_t elem_t;
typedef uint16_t lds_t;
#define COTTN_SYM(name) name##_bf16
#define COTTN_SYM_STR(name) #name "_bf16"
#endif
// launchers that both fp32 builds call and one defines
#if defined(COTTN_ELEM_F32)
#define COTTN_ELEM_SYM(name) name##_f32
#else
#define COTTN_ELEM_SYM(name) COTTN_SYM(name)
#endif
#ifdef COTTN_ELEM_F32
constexpr bool ELEM_IS_F32 = true;
#else
constexpr bool ELEM_IS_F32 = false;
#endif
#if defined(COTTN_ELEM_F32) && !defined(COTTN_F32_WHOLE)
#define COTTN_SPLIT3
constexpr bool SPLIT3 = true;
#else
constexpr bool SPLIT3 = false;
#endif
constexpr bool F32_WHOLE = ELEM_IS_F32 && !SPLIT3;
constexpr int ELEM = int(sizeof(elem_t));
constexpr int LDS_ELEM = int(sizeof(lds_t));
constexpr int EPP = 16 / ELEM;  // elements in a 16-byte piece of a row
typedef __attribute__((ext_vector_type(8))) elem_native native8;
#ifdef COTTN_SPLIT3
struct frag8 { native8 part[3]; };   // one MFMA operand fragment
#else
typedef native8 frag8;
#endif
typedef __attribute__((ext_vector_type(2))) elem_native elem2;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(8))) short s16x8;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;

#undef COTTN_LDS
#define COTTN_LDS __attribute__((address_space(3)))

// Where column c of a row lies in an LDS tile or state copy.  SPLIT3: every 32 columns are 32
// first, 32 second and 32 third parts, so that parts of an element are always 32 apart.
constexpr int PART = 32;
__host__ __device__ constexpr int lds_col(int c) { return SPLIT3 ? (c >> 5) * (3 * PART) + (c & (PART - 1)) : c; }

// Row pitches (in lds_t) of 16-bit LDS arrays.  The LDS moves 64 lanes x 16 bytes in 4
// cycles and 64 x 8 bytes in 2.4 at best (4 for a transposing read of rows that are 8 apart);
// how the 64 addresses of an instruction fall into banks decides whether it gets there.
// Measured on gfx950 with every access pattern of these kernels (cycles per wave instruction,
// 16 waves issuing; the same at d = 32, 64, 128):
//                                         pitch = cols + 8        pitch = cols + 16
//   16-byte row fragments (16 rows)            8.0                     4.1
//   transposing reads over the tokens          4.1                     2.4
//   8-byte writes / reads of 4 cols of a row   8.0 / 2.4              16.0 / 4.1
//   16-byte pieces read back row by row        8.0                    12.0
//   (16-byte writes cost 13 and transposing reads of a state 4.1 with either.)
// So the [rows][cols] operand tiles (read as row fragments and token-column fragments) use
// cols + 16 (unless four such tiles and a state copy would not fit the 160 KB of a compute
// unit: 256-row chunks at d = 64), the state copies and the staging of finished rows
// (8-byte writes) cols + 8.
// SPLIT3 rows are three times as long and read the same way: the same two paddings.
// Whole fp32 rows take cols + 4 everywhere: 8, 12 and 16 time the same (within 3 %).
__host__ __device__ constexpr int lds_pitch(int cols) {
  return F32_WHOLE ? cols + 4 : (SPLIT3 ? 3 * cols : cols) + 8;
}
__host__ __device__ constexpr int tile_pitch(int cols, int rows) {
  return SPLIT3 ? 3 * cols + 16
         : !F32_WHOLE && 2 * (4 * rows * (cols + 16) + cols * lds_pitch(cols)) + 1024 <= 160 * 1024
             ? cols + 16
             : lds_pitch(cols);
}
// Pitch (in elem_t) of staged result rows, and between the row groups of a staging tile of its own.
__host__ __device__ constexpr int stage_pitch(int cols) { return ELEM_IS_F32 ? cols + 4 : cols + 8; }
__host__ __device__ constexpr int stage_tile_pitch(int cols, int rows) {
  return SPLIT3 ? stage_pitch(cols) : tile_pitch(cols, rows);
}

// D(16x16) += A(16x32) * B(32x16), fp32 accumulate.
// Lane l = 16*g + r holds  A[row r][k slots of g],  B[k slots of g][col r],
// and D[row 4g+v][col r] in acc[v].  The order of the k slots is free as long as A and B
// use the same one, which several kernels exploit to feed an accumulator tile straight
// back in as an operand.  16-bit elements: one instruction.  SPLIT3: six, the smallest products
// first.  Whole fp32: eight of the 16x16x4 kind, the j-th over the j-th element of every lane's
// fragment (256 flop per cycle and compute unit, a sixteenth of the bf16 rate).
__device__ __forceinline__ f32x4 mma16(frag8 a, frag8 b, f32x4 acc) {
#if defined(COTTN_SPLIT3)
  acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.part[0], b.part[2], acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.part[2], b.part[0], acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.part[1], b.part[1], acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.part[0], b.part[1], acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.part[1], b.part[0], acc, 0, 0, 0);
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.part[0], b.part[0], acc, 0, 0, 0);
#elif defined(COTTN_ELEM_F32)
#pragma unroll
  for (int j = 0; j < 8; ++j) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[j], b[j], acc, 0, 0, 0);
  return acc;
#elif defined(COTTN_ELEM_F16)
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, acc, 0, 0, 0);
#else
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc, 0, 0, 0);
#endif
}

// The kernels of the tile files are written once and are two things.  Kernels; and, with COTTN_REDO defined, functions
// that a workgroup of the same kernel on parts calls to do its work again (Unparted), with their LDS arrays
// where that kernel's are: room[at] for the array numbered `at`.
#undef COTTN_KERNEL
#undef COTTN_LDS_ARRAY
#ifdef COTTN_REDO
constexpr bool REDO = true;
#define COTTN_KERNEL(bounds, name) __device__ __forceinline__ void name(void* const* room,
#define COTTN_LDS_ARRAY(type, name, count, at) type* const name = static_cast<type*>(room[at]);
#else
constexpr bool REDO = false;
#define COTTN_KERNEL(bounds, name) __global__ __launch_bounds__ bounds void COTTN_SYM(name)(
#define COTTN_LDS_ARRAY(type, name, count, at) __shared__ __attribute__((aligned(16))) type name[count];
#endif

// The k slots of lane row g = lane / 16 in a fragment whose k index runs over 32 consecutive
// columns (or rows) of an LDS tile: elements 0..3 at slot_lo(g).., elements 4..7 at
// slot_hi(g)...  16-bit: eight consecutive elements, one 16-byte read; whole fp32: two groups of
// four 16 apart, so that the four lane rows of one 16-byte read cover 64 consecutive bytes.
__device__ __forceinline__ int slot_lo(int g) { return F32_WHOLE ? 4 * g : 8 * g; }
__device__ __forceinline__ int slot_hi(int g) { return F32_WHOLE ? 16 + 4 * g : 8 * g + 4; }

// The products over 32 tokens added to a sum that is longer.  fp32: formed on their own and added
// as one addend, so that the sum is rounded once per 32 tokens and not once per four (causal, N =
// 4000, d = 32: error against 64 bits 3.7e-7 -> 1.9e-7; B8 H12 N1024 d64 151 us either way; 16-bit operands are off by 2^-9 or
// 2^-12 each, and their sums take the products directly).
__device__ __forceinline__ f32x4 mma16_add(frag8 a, frag8 b, f32x4 sum) {
  if (!ELEM_IS_F32) return mma16(a, b, sum);
  const f32x4 t = mma16(a, b, f32x4{0.f, 0.f, 0.f, 0.f});
  return f32x4{sum[0] + t[0], sum[1] + t[1], sum[2] + t[2], sum[3] + t[3]};
}

// Whole fp32 only: the same over half of the k slots, the `half`-th four elements of every
// lane's fragments (what the other half would contract is known to be zero).
__device__ __forceinline__ f32x4 mma16_half_add(frag8 a, frag8 b, f32x4 sum, int half) {
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#ifdef COTTN_F32_WHOLE
  if (half == 0) {
#pragma unroll
    for (int j = 0; j < 4; ++j) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[j], b[j], acc, 0, 0, 0);
  } else {
#pragma unroll
    for (int j = 4; j < 8; ++j) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[j], b[j], acc, 0, 0, 0);
  }
#endif
  return f32x4{sum[0] + acc[0], sum[1] + acc[1], sum[2] + acc[2], sum[3] + acc[3]};
}

// Whole fp32 only: the dot products of 16 rows at x (rows down the result tile) with 16 rows at y (rows
// along it), over columns first_col .. first_col + 16 BLOCKS - 1 of both.  x, y: this lane's
// row (lane % 16 of the 16), g: lane / 16.
template <int BLOCKS>
__device__ __forceinline__ f32x4 row_products(const lds_t* x, const lds_t* y, int first_col, int g) {
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#ifdef COTTN_F32_WHOLE
#pragma unroll
  for (int i = 0; i < BLOCKS; ++i) {
    const f32x4 a = *reinterpret_cast<const f32x4*>(x + first_col + 16 * i + 4 * g);
    const f32x4 b = *reinterpret_cast<const f32x4*>(y + first_col + 16 * i + 4 * g);
#pragma unroll
    for (int j = 0; j < 4; ++j) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[j], b[j], acc, 0, 0, 0);
  }
#endif
  return acc;
}

// Operand fragment whose k index runs along an LDS row; p: the row at the first of the 32
// columns, g: lane / 16.
__device__ __forceinline__ frag8 lds_row_frag(const lds_t* p, int g) {
#if defined(COTTN_SPLIT3)
  frag8 f;
#pragma unroll
  for (int i = 0; i < 3; ++i)
    f.part[i] = __builtin_bit_cast(native8, *reinterpret_cast<const uint4*>(p + PART * i + slot_lo(g)));
  return f;
#elif defined(COTTN_ELEM_F32)
  const f32x4 lo = *reinterpret_cast<const f32x4*>(p + slot_lo(g));
  const f32x4 hi = *reinterpret_cast<const f32x4*>(p + slot_hi(g));
  return frag8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
#else
  return __builtin_bit_cast(frag8, *reinterpret_cast<const uint4*>(p + slot_lo(g)));
#endif
}

// Transposing 8-byte LDS read (gfx950): inside each group of 16 lanes, lane i passes the
// address of 4 consecutive elements, taken as row i/4, columns 4*(i%4).. of a 4x16 block;
// it receives column i of the block's 4 rows.
#ifndef COTTN_F32_WHOLE
__device__ __forceinline__ s16x4 lds_read_tr(const lds_t* p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((COTTN_LDS s16x4*)(p));
}
#endif

// Operand fragment whose k index runs DOWN the rows of a row-major LDS tile (pitch in
// lds_t): the lane with r = lane%16 receives tile[k0 + 0..3][col0 + r] and
// tile[k1 + 0..3][col0 + r].  k0/k1 are the first rows of the two 4-row groups that
// fill this lane's 8 k slots; col0 is a multiple of 16.
__device__ __forceinline__ frag8 lds_col_frag(const lds_t* tile, int pitch, int k0, int k1,
                                               int col0, int r) {
#ifdef COTTN_F32_WHOLE
  // (no transposing read of 4-byte elements: a lane reads its column element by element)
  frag8 v;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    v[j] = tile[(k0 + j) * pitch + col0 + r];
    v[4 + j] = tile[(k1 + j) * pitch + col0 + r];
  }
  return v;
#else
  const int sub_row = r >> 2, sub_col = lds_col(col0) + (r & 3) * 4;
  const auto part = [&](int off) {
    s16x4 lo = lds_read_tr(tile + (k0 + sub_row) * pitch + sub_col + off);
    s16x4 hi = lds_read_tr(tile + (k1 + sub_row) * pitch + sub_col + off);
    s16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    return __builtin_bit_cast(native8, v);
  };
#ifdef COTTN_SPLIT3
  return frag8{{part(0), part(PART), part(2 * PART)}};
#else
  return part(0);
#endif
#endif
}
// The same over rows 32 ks .. 32 ks + 31, in the slot order of lds_row_frag.
__device__ __forceinline__ frag8 lds_col_frag_ks(const lds_t* tile, int pitch, int ks, int g,
                                                  int col0, int r) {
  return lds_col_frag(tile, pitch, 32 * ks + slot_lo(g), 32 * ks + slot_hi(g), col0, r);
}

// Elements <-> fp32; conversions to the element type round to nearest even.
#ifndef COTTN_F32_WHOLE
// two values rounded and packed into one word (low half first): written as one vector
// conversion so that it becomes the packed convert instruction, not two converts and a merge
__device__ __forceinline__ uint32_t pack2(float lo, float hi) {
  typedef __attribute__((ext_vector_type(2))) float f32x2;
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{lo, hi}, elem2));
}
// the two 16-bit values of a word (low half first)
__device__ __forceinline__ void unpack2(uint32_t w, float& lo, float& hi) {
#ifdef COTTN_ELEM_F16
  const elem2 p = __builtin_bit_cast(elem2, w);
  lo = float(p[0]);
  hi = float(p[1]);
#else
  lo = __builtin_bit_cast(float, w << 16);
  hi = __builtin_bit_cast(float, w & 0xFFFF0000u);
#endif
}
#endif
// SPLIT3: whether this wave parted a value that its parts fall short of, or left a result that is not finite.
// The kernels ask at their end whether a wave of the workgroup did, which then does its work again with
// whole products.  (Nothing to note elsewhere.)
//   The lowest bit of a value lies 23 places below its first, and that of a bfloat16 number nowhere below 2^-133
// (the matrix instruction takes subnormal ones as they are): parts are exact from 2^-110 on.  An infinite value,
// and one that rounds to infinity, makes the results that it enters NaN.
//   Four packed 16-bit instructions to four values, written out: the compiler makes the comparisons long before
// it adds them up, in registers that the scans do not have.  With them and what follows from them, against no regard
// to the range, forward + backward: B8 H12 N1024 d64 117 -> 119 us (with a comparison of the rest and a scalar
// instruction to each value 123), 64 units of 2048 rows 145 -> 153, 300 of 1000 at 64 x 128 660 -> 703, whose dQ
// scan in even shares pays most, 200 -> 227.
struct Unparted {
#ifdef COTTN_SPLIT3
  uint32_t least = 0xFFFFFFFFu;   // of each half, 2 |first part| - 1 as bits: 0 is the largest
  bool not_finite = false;
  __device__ __forceinline__ void first_parts(uint2 pairs) {
    uint32_t a, b;
    asm("v_pk_mad_u16 %1, %3, 2, -1 op_sel_hi:[1,0,0]\n\tv_pk_mad_u16 %2, %4, 2, -1 op_sel_hi:[1,0,0]\n\t"
        "v_pk_min_u16 %0, %0, %1\n\tv_pk_min_u16 %0, %0, %2"
        : "+v"(least), "=&v"(a), "=&v"(b) : "v"(pairs.x), "v"(pairs.y));
  }
  template <int TILES>
  __device__ __forceinline__ void results(const f32x4* t, float factor = 1.f) {   // factor times the tiles
    float largest = 0.f;   // NaN if one is
#pragma unroll
    for (int i = 0; i < TILES; ++i)
#pragma unroll
      for (int v = 0; v < 4; ++v) largest = __builtin_elementwise_maximum(largest, fabsf(t[i][v]));
    not_finite |= __any(!(largest * fabsf(factor) < __builtin_inff()));
  }
  // scratch: LDS that no wave reads or writes any more
  template <int NW>
  __device__ __forceinline__ bool in_workgroup(void* scratch) const {
    int* met = static_cast<int*>(scratch);
    constexpr uint32_t LIMIT = 2 * ((127 - 110) << 7) - 1;
    const bool here = __any(not_finite || (least & 0xFFFFu) < LIMIT || (least >> 16) < LIMIT);
    if (threadIdx.x % 64 == 0) met[threadIdx.x / 64] = here;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");   // (no wait for the stores of results)
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    int any = 0;
#pragma unroll
    for (int i = 0; i < NW; ++i) any |= met[i];
    if (__builtin_expect(__builtin_amdgcn_readfirstlane(any) == 0, 1)) return false;
    __threadfence();   // what this workgroup stored is in place before it stores again
    __syncthreads();
    return true;
  }
#else
  template <int TILES>
  __device__ __forceinline__ void results(const f32x4*, float = 1.f) {}
#endif
};
#ifdef COTTN_SPLIT3
// x[0..3] as their three parts, two to a word: parts[i] holds the i-th ones.  SCALED: the parts of f x[0..3], of
// the products as they are before rounding (the last part is rounded).
template <bool SCALED = false>
__device__ __forceinline__ void split4(const float (&x)[4], uint2 (&parts)[3], Unparted& un, float f = 1.f) {
  float rest[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) rest[e] = SCALED ? f * x[e] : x[e];
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    parts[i] = uint2{pack2(rest[0], rest[1]), pack2(rest[2], rest[3])};
    if (i == 2) break;
    float p[4];
    unpack2(parts[i].x, p[0], p[1]);
    unpack2(parts[i].y, p[2], p[3]);
#pragma unroll
    for (int e = 0; e < 4; ++e) rest[e] = SCALED && i == 0 ? __builtin_fmaf(f, x[e], -p[e]) : rest[e] - p[e];
  }
  un.first_parts(parts[0]);
}
#endif
#ifndef COTTN_ELEM_F32
// fp32 sum of squares of the two elements of a word, added to acc
__device__ __forceinline__ float dot2_self(uint32_t w, float acc) {
  const elem2 p = __builtin_bit_cast(elem2, w);
#ifdef COTTN_ELEM_F16
  return __builtin_amdgcn_fdot2(p, p, acc, false);
#else
  return __builtin_amdgcn_fdot2_f32_bf16(p, p, acc, false);
#endif
}
#endif
// four consecutive elements
__device__ __forceinline__ void store4(elem_t* dst, float a, float b, float c, float d) {
#ifdef COTTN_ELEM_F32
  *reinterpret_cast<f32x4*>(dst) = f32x4{a, b, c, d};
#else
  uint2 pk;
  pk.x = pack2(a, b);
  pk.y = pack2(c, d);
  *reinterpret_cast<uint2*>(dst) = pk;
#endif
}
__device__ __forceinline__ void load4(const elem_t* src, float* f) {
#ifdef COTTN_ELEM_F32
  const f32x4 v = *reinterpret_cast<const f32x4*>(src);
#pragma unroll
  for (int i = 0; i < 4; ++i) f[i] = v[i];
#else
  const uint2 raw = *reinterpret_cast<const uint2*>(src);
  unpack2(raw.x, f[0], f[1]);
  unpack2(raw.y, f[2], f[3]);
#endif
}
// The same four in an LDS tile or state copy.
__device__ __forceinline__ void store4_lds(lds_t* dst, float a, float b, float c, float d, Unparted& un) {
#ifdef COTTN_SPLIT3
  const float x[4] = {a, b, c, d};
  uint2 parts[3];
  split4(x, parts, un);
#pragma unroll
  for (int i = 0; i < 3; ++i) *reinterpret_cast<uint2*>(dst + PART * i) = parts[i];
#else
  store4(dst, a, b, c, d);
#endif
}
__device__ __forceinline__ void load4_lds(const lds_t* src, float* f) {
#ifdef COTTN_SPLIT3
  float p[3][4];
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const uint2 raw = *reinterpret_cast<const uint2*>(src + PART * i);
    unpack2(raw.x, p[i][0], p[i][1]);
    unpack2(raw.y, p[i][2], p[i][3]);
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) f[e] = (p[0][e] + p[1][e]) + p[2][e];   // exact
#else
  load4(src, f);
#endif
}
// a 16-byte piece of a row (EPP elements): its sum of squares, and the piece times a factor
__device__ __forceinline__ float piece_sum_sq(uint4 raw) {
  const uint32_t w[4] = {raw.x, raw.y, raw.z, raw.w};
  float ss = 0.f;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
#ifdef COTTN_ELEM_F32
    const float x = __builtin_bit_cast(float, w[e]);
    ss = __builtin_fmaf(x, x, ss);
#else
    ss = dot2_self(w[e], ss);
#endif
  }
  return ss;
}
__device__ __forceinline__ uint4 piece_times(uint4 raw, float f) {
  uint32_t w[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
  for (int e = 0; e < 4; ++e) {
#ifdef COTTN_ELEM_F32
    w[e] = __builtin_bit_cast(uint32_t, f * __builtin_bit_cast(float, w[e]));
#else
    float lo, hi;
    unpack2(w[e], lo, hi);
    w[e] = pack2(f * lo, f * hi);
#endif
  }
  return uint4{w[0], w[1], w[2], w[3]};
}
// such a piece, or the piece times a factor, to its place in an LDS tile
template <bool SCALED>
__device__ __forceinline__ void store_piece_lds(lds_t* dst, uint4 raw, float f, Unparted& un) {
#ifdef COTTN_SPLIT3
  const float x[4] = {__builtin_bit_cast(float, raw.x), __builtin_bit_cast(float, raw.y), __builtin_bit_cast(float, raw.z),
                      __builtin_bit_cast(float, raw.w)};
  uint2 parts[3];
  split4<SCALED>(x, parts, un, f);
#pragma unroll
  for (int i = 0; i < 3; ++i) *reinterpret_cast<uint2*>(dst + PART * i) = parts[i];
#else
  *reinterpret_cast<uint4*>(dst) = SCALED ? piece_times(raw, f) : raw;
#endif
}

// Fills half of an operand fragment with a masked accumulator tile: the tile's element [v] of
// lane row g is k slot 16 half + 4 g + v of the fragment.
__device__ __forceinline__ void put_half(frag8& frag, int half, f32x4 acc, bool k0, bool k1,
                                         bool k2, bool k3, Unparted& un) {
#if defined(COTTN_SPLIT3)
  const float x[4] = {k0 ? acc[0] : 0.f, k1 ? acc[1] : 0.f, k2 ? acc[2] : 0.f, k3 ? acc[3] : 0.f};
  uint2 parts[3];
  split4(x, parts, un);
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    u32x4 words = __builtin_bit_cast(u32x4, frag.part[i]);
    words[2 * half + 0] = parts[i].x;
    words[2 * half + 1] = parts[i].y;
    frag.part[i] = __builtin_bit_cast(native8, words);
  }
#elif defined(COTTN_ELEM_F32)
  frag[4 * half + 0] = k0 ? acc[0] : 0.f;
  frag[4 * half + 1] = k1 ? acc[1] : 0.f;
  frag[4 * half + 2] = k2 ? acc[2] : 0.f;
  frag[4 * half + 3] = k3 ? acc[3] : 0.f;
#else
  u32x4 words = __builtin_bit_cast(u32x4, frag);
  words[2 * half + 0] = pack2(k0 ? acc[0] : 0.f, k1 ? acc[1] : 0.f);
  words[2 * half + 1] = pack2(k2 ? acc[2] : 0.f, k3 ? acc[3] : 0.f);
  frag = __builtin_bit_cast(frag8, words);
#endif
}

// The same with zeros, of a tile that the mask leaves nothing of.
__device__ __forceinline__ void put_no_half(frag8& frag, int half) {
#if defined(COTTN_SPLIT3)
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    u32x4 words = __builtin_bit_cast(u32x4, frag.part[i]);
    words[2 * half + 0] = words[2 * half + 1] = 0u;
    frag.part[i] = __builtin_bit_cast(native8, words);
  }
#endif
}

// x of another lane of the same row of 16 lanes, chosen by a DPP control word: no LDS
// traffic and no extra latency, unlike a general cross-lane permute.
template <int DPP_CTRL>
__device__ __forceinline__ float dpp_read(float x) {
  return __builtin_bit_cast(
      float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), DPP_CTRL, 0xF, 0xF, true));
}

// Sum over the `width` consecutive lanes (a power of two <= 64) that contain this lane; every
// lane of the group ends with the total.  Up to 16 lanes this is DPP only: swap within
// pairs, swap pairs within quads, then mirror the 8-lane half-row and the 16-lane row (after
// the earlier steps every lane of a quad holds the same value, so a mirror pairs each quad
// with a quad of the other half).
template <int width>
__device__ __forceinline__ float group_sum(float x) {
  static_assert(width == 1 || width == 2 || width == 4 || width == 8 || width == 16 ||
                width == 32 || width == 64, "width must be a power of two");
  if (width >= 2) x += dpp_read<0xB1>(x);    // quad_perm [1,0,3,2]
  if (width >= 4) x += dpp_read<0x4E>(x);    // quad_perm [2,3,0,1]
  if (width >= 8) x += dpp_read<0x141>(x);   // row_half_mirror
  if (width >= 16) x += dpp_read<0x140>(x);  // row_mirror
  if (width >= 32) x += __shfl_xor(x, 16, 64);
  if (width >= 64) x += __shfl_xor(x, 32, 64);
  return x;
}

// Orders this wave's earlier LDS writes before its later LDS reads (lanes exchange data
// through LDS without a workgroup barrier).
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Padded batches (sequences of different lengths in one [B][H][N][d] tensor): rows at or
// beyond seq_len[batch] do not exist.  They are never read, contribute to no sum, and the
// rows of every output tensor there are written as zeros.  Without lengths all N rows exist.
__device__ __forceinline__ int valid_rows(const int* __restrict__ seq_len, int unit, const Divisor& H, int N) {
  return seq_len != nullptr ? min(N, max(0, seq_len[quotient(unit, H)])) : N;
}
// The scale is one value per head, or, for padded batches whose stabiliser depends on each
// sequence's own length (Sec. 3.3), one per (batch, head).
__device__ __forceinline__ float unit_scale(const float* __restrict__ s, int unit, const Divisor& H,
                                            int per_unit) {
  return s[per_unit ? unit : unit - quotient(unit, H) * H.n];
}
// Zeros rows row_lo..row_hi-1 of D columns of a [.][LD] tensor of elements (whole workgroup).
template <int D, int LD = D>
__device__ __forceinline__ void zero_rows(elem_t* __restrict__ dst, int row_lo, int row_hi) {
  constexpr int PPR = D / EPP;
  const long pieces = long(max(0, row_hi - row_lo)) * PPR;
  for (long i = threadIdx.x; i < pieces; i += blockDim.x)
    *reinterpret_cast<uint4*>(dst + size_t(row_lo + i / PPR) * LD + (i % PPR) * EPP) = uint4{0u, 0u, 0u, 0u};
}

// 16-byte store of a result that this library does not read again soon: marked non-temporal,
// so that the line does not displace input rows another kernel of the same step re-reads
// from this XCD's L2.
__device__ __forceinline__ void store_streaming(void* dst, uint4 v) {
  __builtin_nontemporal_store(u32x4{v.x, v.y, v.z, v.w}, reinterpret_cast<u32x4*>(dst));
}

// Stores of segment states to the workspace.  A state is read by the next kernel, by
// workgroups of the same (batch, head) unit, which unit_and_segment() puts on this XCD: plain
// stores leave the lines in this XCD's L2 for them (0.5 us of the 52 us step on B8 H12 N1024 d64
// against non-temporal stores).
__device__ __forceinline__ void store_state_words(float* dst, f32x4 v) {
  *reinterpret_cast<f32x4*>(dst) = v;
}

// States that only two kernels of this library hand to each other (workspace arrays that no
// caller reads) need not be row-major.  Stored tile by tile in the order the accumulator
// registers hold them - the 16x16 tile (a, b) as 256 consecutive floats, the four values of
// lane l at 4 l - a wave writes or reads a tile with one instruction that covers 1 KB of
// consecutive addresses.  Row-major, the same four-value pieces lie a matrix row apart and one
// instruction touches 16 to 64 cache lines, which the vector L1 looks up one per cycle: with
// up to three stored states per workgroup that was most of the 2 us by which a scan
// workgroup's first chunk started later than its rows arrived.
__device__ __forceinline__ int tiled_state_offset(int tile_a, int tile_b, int tiles_b, int lane) {
  return (tile_a * tiles_b + tile_b) * 256 + 4 * lane;
}

// Makes the compiler fetch a kernel argument where this stands.  Left alone it fetches each
// argument where it is first used, one scalar load and one wait after the other down the
// kernel's prologue (six or more round trips to the scalar cache before the first row is
// requested); pinned at the top, all of them come with one or two wide loads and one wait.
template <class T>
__device__ __forceinline__ void fetch_argument_now(const T& x) {
  asm volatile("" ::"s"(x));
}
__device__ __forceinline__ void fetch_argument_now(const Divisor& x) { asm volatile("" ::"s"(x.n), "s"(x.scaled)); }
template <class T, class... Rest>
__device__ __forceinline__ void fetch_argument_now(const T& x, const Rest&... rest) {
  fetch_argument_now(x);
  fetch_argument_now(rest...);
}

// Which (batch-head unit, segment) a workgroup of a units * G grid works on.  Workgroups are
// dealt to the 8 XCDs round robin by their index, and each XCD has an L2 of its own.  The
// kernels of one call that share this numbering pass data to each other through that L2: the
// rows a totals workgroup read are there for the scan workgroup of the same (unit, segment),
// and the G segments of a unit all land on one XCD (workgroup indices 8 apart), so the segment
// states that the workgroups of a unit write for each other never cross to another L2.
// (Measured on B8 H12 N1024 d64: 1.6 us of a 56 us step against unit = index / G.)
// Units beyond the last whole group of 8 are numbered plainly.
__device__ __forceinline__ void unit_and_segment(int index, int units, const Divisor& G, int& unit, int& g) {
  const int whole = units & ~7, grouped = whole * G.n;
  if (index < grouped) {
    const int q = quotient(index >> 3, G);   // index / (8 G)
    unit = 8 * q + (index & 7);
    g = (index >> 3) - q * G.n;
  } else {
    const int q = quotient(index - grouped, G);
    unit = whole + q;
    g = index - grouped - q * G.n;
  }
}

// The rows a workgroup of the causal kernels walks, first to last or last to first.
//   One segment of one unit: segment g of seg_rows rows, numbered as above.
//   An even share (EVEN): the units laid end to end, unit_rows (a whole number of chunks) for
//   each, cut every seg_rows rows.  A share may begin in the middle of a unit and go on into the next
//   ones, so that every workgroup has the same number of steps whatever the number of units is.
// The states that workgroups leave for each other (Kh^T V of the last piece of a share, Qh^T dO of the
// first) have one slot per workgroup either way.  Neighbouring shares go to one XCD, as segments do.
struct Span {
  int unit, begin, end;   // the first piece walked: rows begin .. end - 1 of a unit
  int left;               // rows of the share beyond that unit, in the direction walked
  int slot, outermost;    // the workgroup's slot; that of the unit's first (reverse: last) workgroup
  bool mid_unit;          // rows of the unit come before (reverse: after) the piece
};
__device__ __forceinline__ int even_workgroup(int units, const Divisor& seg_rows, int unit_rows) {
  const int workgroups = quotient(units * unit_rows + seg_rows.n - 1, seg_rows);
  const int per_xcd = workgroups / 8, index = blockIdx.x;
  return index < 8 * per_xcd ? index % 8 * per_xcd + index / 8 : index;
}
template <bool REVERSE, bool EVEN>
__device__ __forceinline__ Span span_of_workgroup(int units, int N, const Divisor& G, const Divisor& seg_rows,
                                                  const Divisor& unit_rows) {
  Span s;
  if constexpr (!EVEN) {
    int g;
    unit_and_segment(blockIdx.x, units, G, s.unit, g);
    s.begin = g * seg_rows;
    s.end = min(N, s.begin + seg_rows);
    s.left = 0;
    s.slot = s.unit * G + g;
    s.outermost = REVERSE ? s.unit * G + G - 1 : s.unit * G;
    s.mid_unit = REVERSE ? g < G - 1 : g > 0;
    return s;
  }
  s.slot = even_workgroup(units, seg_rows, unit_rows);
  const int lo = s.slot * seg_rows, hi = min(lo + seg_rows, units * unit_rows);
  s.unit = quotient(REVERSE ? hi - 1 : lo, unit_rows);
  const int start = s.unit * unit_rows, stop = start + unit_rows;
  s.begin = max(lo - start, 0);
  s.end = min(N, min(hi, stop) - start);
  s.left = REVERSE ? max(start - lo, 0) : max(hi - stop, 0);
  s.outermost = quotient(REVERSE ? stop - 1 : start, seg_rows);
  s.mid_unit = REVERSE ? hi < stop : lo > start;
  return s;
}

// How the causal scans walk (a template parameter: chosen at run time, one walk's registers spill in
// another): segments, with the states of earlier ones from the workspace; even shares, of sequences of
// one length or of a padded batch (a piece without rows that exist takes a step of zeros); segments of
// short sequences, whose workgroups form the state of the rows before them by themselves (launch.h:
// own_prefix), the same several steps at a time.
enum Walk { SEGMENTS = 0, EVEN_SHARES = 1, EVEN_PADDED = 2, OWN_PREFIX = 3, OWN_PREFIX_SETS = 4 };
constexpr bool walks_own_prefix(int walk) { return walk == OWN_PREFIX || walk == OWN_PREFIX_SETS; }
// What the last share's slot, which holds no state, begins with in a forward's workspace: whether the states
// there are those of even shares (launch.h: CausalArgs::marked).
constexpr float EVEN_MARK = 1.0f, NO_EVEN_MARK = 0.0f;
constexpr bool walks_even(int walk) { return walk == EVEN_SHARES || walk == EVEN_PADDED; }

// In place, for 4 neighbouring elements of a stack of n matrices `stride` floats apart:
// matrix k (in walking order: first to last, or last to first with `reverse`) <- sum of the
// matrices walked before it.  The last matrix walked never held a value and is not read.  The
// matrices are taken eight at a time with all loads of a batch issued before the first store:
// the sum itself is serial, but a thread then pays one memory latency per eight matrices.
__device__ __forceinline__ void exclusive_running_sum(float* __restrict__ p, int n, size_t stride,
                                                      bool reverse) {
  constexpr int BATCH = 8;
  f32x4 run = {0.f, 0.f, 0.f, 0.f};
  for (int k0 = 0; k0 < n; k0 += BATCH) {
    f32x4 t[BATCH];
#pragma unroll
    for (int i = 0; i < BATCH; ++i) {
      const int k = k0 + i;
      t[i] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (k + 1 < n) t[i] = *reinterpret_cast<const f32x4*>(p + size_t(reverse ? n - 1 - k : k) * stride);
    }
#pragma unroll
    for (int i = 0; i < BATCH; ++i) {
      const int k = k0 + i;
      if (k < n) {
        *reinterpret_cast<f32x4*>(p + size_t(reverse ? n - 1 - k : k) * stride) = run;
        run += t[i];
      }
    }
  }
}

// 1 / max(sqrt(sum_sq), eps)
__device__ __forceinline__ float inv_norm(float sum_sq, float eps) {
  return 1.0f / fmaxf(sqrtf(sum_sq), eps);
}

// The row factors of the tile kernels, out[p] = min(1 / sqrt(sum_sq[p]), inv_eps): the reciprocal
// square root instruction (1 ulp of fp32), for fp32 rows with a Newton step, whose last addition is
// the one rounding that shows.  A square root and a division, correctly rounded, are two, and three
// times the instructions (a seventh of what the fp32 dQ scan issues in a step): left for 0,
// infinity, NaN and what the instruction takes for 0.
template <int PASSES>
__device__ __forceinline__ void row_inv_norms(const float (&sum_sq)[PASSES], float inv_eps, float* out) {
  bool exact_needed = false;
#pragma unroll
  for (int p = 0; p < PASSES; ++p) {
    float y = __builtin_amdgcn_rsqf(sum_sq[p]);
    if (ELEM_IS_F32) {
      const float off = __builtin_fmaf(-sum_sq[p] * y, y, 1.0f);   // 1 - sum_sq y^2
      exact_needed |= !(fabsf(off) < 0.5f);
      y = __builtin_fmaf(0.5f * y, off, y);
    }
    out[p] = fminf(y, inv_eps);
  }
  if (ELEM_IS_F32 && __builtin_expect(__any(exact_needed), 0)) {
#pragma unroll
    for (int p = 0; p < PASSES; ++p) out[p] = fminf(1.0f / sqrtf(sum_sq[p]), inv_eps);
  }
}

}  // namespace COTTN_NS
}  // namespace cottn
