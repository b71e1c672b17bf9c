// Device code of the superkernel (gfx950 / CDNA4 only).
//
// One persistent kernel walks the flat tile table (Section 5.3 of the paper:
// many small kernels repacked into one large execution block).  Every tile
// belongs to one operator in its canonical GEMM view
//     C[Mg,Ng] = A'[Mg,Kg] . Bs[Ng,Kg]^T          (fp32 accumulate)
// with both operands K-contiguous, so a 16-byte piece of a row is at the same
// time one 128-bit load and one MFMA operand (8 halves or 4 floats of K).
//
// Three families of tile code:
//   * skinny (Mg <= 64): weights go HBM -> registers -> MFMA directly; the
//     weight rows are the MFMA's row operand and the few activation rows its
//     column operand, so a lane ends up with four consecutive output columns.
//     Activations are staged through LDS.  The four waves of a workgroup take
//     different 32-row weight groups; long reductions are split over several
//     workgroups whose partial sums the last one to finish adds in fixed order.
//   * LDS tiles (128x128, or 128x64 for operators with at most 64 output
//     columns): staged GEMM with 32x32 MFMAs; the operands go global -> LDS
//     directly (buffer loads with the LDS modifier into a ring of swizzled
//     stage images), through a ring of registers only where an operator is
//     out of reach of 32-bit offsets; the activation operand may be gathered
//     on the fly from an NHWC image (implicit GEMM for convolutions, any stride).
//   * operands that cannot be read in aligned 16-byte pieces, and convolutions
//     on channel-major (NCHW) arrays, whose patch rows and output rows are not
//     contiguous: one output per thread for small rectangles; MFMA blocks whose
//     pieces are read at any address and shifted into place (images in channel
//     planes: element by element, lanes along pixels) for larger ones; only in
//     the kernel instantiations for plans that need them.  Two forms of these have
//     paths of their own: channel-major convolutions that keep the images' width
//     (run_tile_planes) and NHWC ones of few channels, stems (run_tile_rows).
//   * 3x3 convolutions of 64 channels in plans that fill the chip (run_window): weights in registers, pixels through a
//     ring in LDS, every pixel read once for its nine taps.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "sk_internal.h"

namespace sk {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(2)));  // at any element's address
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

// Operand pointers reach the kernel through descriptors in memory, so the compiler cannot
// see that they are global addresses; say so explicitly (global_load instead of flat_load).
#define SK_GLOBAL __attribute__((address_space(1)))
template <class T>
__device__ __forceinline__ const T SK_GLOBAL *as_global(const void *p) {
  return (const T SK_GLOBAL *)(uintptr_t)p;
}
template <class T>
__device__ __forceinline__ T SK_GLOBAL *as_global_mut(void *p) {
  return (T SK_GLOBAL *)(uintptr_t)p;
}

// A record that every lane reads from the same address, in scalar registers, through the scalar cache: for records that
// nothing writes while the kernel runs.  (Handed over through LDS instead, every wave spent two vector instructions per dword on it.)
#define SK_CONSTANT __attribute__((address_space(4)))
template <class S>
__device__ __forceinline__ S load_record(const S *src) {
  static_assert(sizeof(S) % 4 == 0, "whole dwords");
  struct Words {
    uint32_t w[sizeof(S) / 4];
  } v;
  uintptr_t at = (uintptr_t)src;
  // (opaque, so that a record read again later is not kept in registers meanwhile)
  asm volatile("" : "+s"(at));
  const uint32_t SK_CONSTANT *p = (const uint32_t SK_CONSTANT *)at;
#pragma unroll
  for (unsigned i = 0; i < sizeof(S) / 4; ++i) v.w[i] = p[i];
  return __builtin_bit_cast(S, v);
}

constexpr int WORK_DWORDS = (int)(sizeof(TileWork) / 4);
static_assert(WORK_DWORDS <= 64, "one dword of the record per lane");

constexpr int WG_THREADS = 256;
constexpr int LDS_ROW = 144;                  // 128 bytes of K + 16 bytes of padding (bank spread)
constexpr int LDS_TILE_BYTES = 512 * LDS_ROW;  // 72 KB per workgroup: two workgroups share a CU's 160 KB

// Plans of which every tile is a lean 128 x 64 tile ("narrow": the 3x3 layers with at most 64 output channels of many
// tenants) run in a kernel of their own: without the other classes' registers and with two stage images instead of
// three, three workgroups share a CU.  Such a tile spends half its time around its few stages (set-up, first loads,
// outputs, hand-over), which only the CU's other workgroups can fill: the 3x3 64-channel convolutions on 56x56 of 512
// tenants take 214 to 223 us instead of 239 (those of 16 bits run as runs of pixels by now: run_window).  Not every number of tiles gains
// (narrow_pays).
constexpr int NARROW_LDS_BYTES = 2 * (128 + 64) * 128;

// Queue counters of a table: [0] tiles handed out beyond the first grid-full, [1] finished workgroups,
// [16 * (1 + x)] entries handed out from die x's list of LDS tiles (a 64-byte line each).
constexpr int QUEUE_COUNTERS = 16 * 9 + 1;
__device__ __forceinline__ uint32_t *die_list_head(uint32_t *counters, uint32_t x) { return counters + 16u * (1u + x); }

struct KernelArgs {
  uint32_t *counters;   // see QUEUE_COUNTERS
  const TileWork *xwork;  // the LDS tiles' records, die by die (null: tiles are run where their ticket falls)
  const uint32_t *xoff;   // [9] where die x's list starts in xwork
  uint32_t *remaining;  // per operator: tiles not yet retired (null = no stamps)
  uint64_t *stamps;     // [n] completion ticks, [n] = start tick
  uint32_t n_problems;
  uint32_t tile_begin, tile_end;
  uint32_t dynamic;      // 1: tiles come from the atomic counter; 0: static stride over the range
  uint32_t write_start;  // 1: every workgroup lowers the start tick to its own first clock
  f32x4 *ws;             // split-K partial sums
  const uint32_t *ws_off;
  uint32_t *arrive;
};

#ifdef SK_DIAG_CLOCKS
// Diagnostic build (-DSK_DIAG_CLOCKS, a library of its own: see build_diag in build.py and tile_phases.py): thread 0
// of the first SK_DIAG_WGS workgroups stamps the 100 MHz device clock at the phase boundaries of its first
// SK_DIAG_TILES tiles.  Slots per tile: 0 tile taken up, 1 set-up done (before the first operand loads), 2 first
// main-loop step multiplied, 3 main loop done, 4 outputs stored (and split-reduction hand-over done), 5 next
// record handed to all waves, 6 = 1 + tile class + 100 * reduction slices, 7 = the ticket (low half) and the
// flags it was handed over with.
// (first 16 workgroups, 64 tiles each; -DSK_DIAG_WGS_N=512 -DSK_DIAG_TILES_N=24 stamps every workgroup of a launch)
#ifndef SK_DIAG_WGS_N
#define SK_DIAG_WGS_N 16
#endif
#ifndef SK_DIAG_TILES_N
#define SK_DIAG_TILES_N 64
#endif
constexpr int SK_DIAG_WGS = SK_DIAG_WGS_N, SK_DIAG_TILES = SK_DIAG_TILES_N;
__device__ uint64_t g_diag[SK_DIAG_WGS * SK_DIAG_TILES * 8];
#define SK_DIAG(slot_)                                                               \
  do {                                                                               \
    if (blockIdx.x < SK_DIAG_WGS && diag_tile < SK_DIAG_TILES && threadIdx.x == 0)   \
      g_diag[(blockIdx.x * SK_DIAG_TILES + diag_tile) * 8 + (slot_)] = wall_clock64(); \
  } while (0)
#else
#define SK_DIAG(slot_) \
  do {                 \
  } while (0)
#endif

// ---------------------------------------------------------------------------
// element helpers
// ---------------------------------------------------------------------------
template <int DT>
struct Elem;
template <>
struct Elem<SK_F32> {
  static constexpr int ES = 4;
};
template <>
struct Elem<SK_BF16> {
  static constexpr int ES = 2;
};
template <>
struct Elem<SK_F16> {
  static constexpr int ES = 2;
};

__device__ __forceinline__ uint32_t f32_to_bf16_bits(float f) {
  __bf16 h = (__bf16)f;  // v_cvt_pk_bf16_f32: nearest, ties to even; NaN stays NaN
  return (uint32_t)__builtin_bit_cast(uint16_t, h);
}
// Two outputs packed into one dword (lower column in the low half).
template <int DT>
__device__ __forceinline__ uint32_t cvt_pack(float lo, float hi) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  const f32x2 v = {lo, hi};
  if constexpr (DT == SK_BF16) {
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
  } else {
    typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, f16x2));
  }
}
__device__ __forceinline__ uint32_t f32_to_f16_bits(float f) {
  _Float16 h = (_Float16)f;  // v_cvt_f16_f32: nearest, ties to even
  return (uint32_t)__builtin_bit_cast(uint16_t, h);
}

template <int DT>
__device__ __forceinline__ uint32_t cvt_bits(float f) {
  if constexpr (DT == SK_BF16) return f32_to_bf16_bits(f);
  if constexpr (DT == SK_F16) return f32_to_f16_bits(f);
  return __builtin_bit_cast(uint32_t, f);
}

// Outputs of whole tiles are stored past the caches (this bit of a buffer store, nontemporal stores elsewhere) if FLAG_PAST_CACHES is
// set (past_caches in planner.cpp): the launch does not read them again, and what it does read stays (main workload 1028 -> 1000 us).  Not
// the eight-byte stores of the weight-streaming classes: main workload 1002 -> 1019 us.
constexpr int NONTEMPORAL = 2;

// N pieces of 16 bytes, `step` bytes apart.  (One branch around all of them.)
template <int N>
__device__ __forceinline__ void store_out(const u32x4 (&v)[N], __amdgpu_buffer_rsrc_t desc, uint32_t at, uint32_t step, bool past_caches) {
  if (past_caches) {
#pragma unroll
    for (int i = 0; i < N; ++i) __builtin_amdgcn_raw_buffer_store_b128(v[i], desc, at + (uint32_t)i * step, 0, NONTEMPORAL);
  } else {
#pragma unroll
    for (int i = 0; i < N; ++i) __builtin_amdgcn_raw_buffer_store_b128(v[i], desc, at + (uint32_t)i * step, 0, 0);
  }
}

// Store four consecutive outputs of one row (columns n .. n+3, clipped to n_end).
template <int DT>
__device__ __forceinline__ void store4(void *C, int64_t row_off, int n, int n_end, f32x4 v, bool vec_ok) {
  constexpr int ES = Elem<DT>::ES;
  char SK_GLOBAL *p = as_global_mut<char>(C) + (row_off + n) * ES;
  if (vec_ok && n + 3 < n_end) {
    if constexpr (ES == 4) {
      *(f32x4 SK_GLOBAL *)p = v;
    } else {
      u32x2 o;
      o.x = cvt_pack<DT>(v.x, v.y);
      o.y = cvt_pack<DT>(v.z, v.w);
      *(u32x2 SK_GLOBAL *)p = o;
    }
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (n + i < n_end) {
        if constexpr (ES == 4)
          ((float SK_GLOBAL *)p)[i] = v[i];
        else
          ((uint16_t SK_GLOBAL *)p)[i] = (uint16_t)cvt_bits<DT>(v[i]);
      }
    }
  }
}

// The MFMA paths below require both operands to be readable in aligned 16-byte
// pieces (FLAG_VEC_A and FLAG_VEC_B: 16-byte aligned bases and row strides, Kg
// and, for a convolution, Cin multiples of a piece), except where they say so:
// the weight-streaming classes with ANY, and run_tile_any.

// Loads in the MFMA paths are never placed under a branch (a conditional load makes the
// compiler wait for it at the end of the branch, which serialises the loads of a stage)
// and their values are not touched before they are consumed (a select right behind a
// load makes the wave wait for it at once).  So a piece that must read as zero (beyond K,
// in a convolution's padding, rows past Mg, idle slots of a ring) is not masked after the
// load: its address is replaced by that of a piece of zeros in device memory.

// Weight piece: row n of Bs[Ng,Kg], elements k .. k+CE-1; where !ok (beyond K, idle slots of the
// ring) a piece of zeros is read instead, so that a weight row that holds an infinity does
// not meet 0 * inf there.
__device__ __attribute__((aligned(16))) const uint32_t g_zero_piece[4] = {0u, 0u, 0u, 0u};
// Its address in vector registers.  (Given the symbol itself, the compiler selects between the two
// places with a branch and a load in either arm, and then waits for every load in flight.)
__device__ __forceinline__ uintptr_t zero_piece_address() {
  uintptr_t z = (uintptr_t)g_zero_piece;
  asm volatile("" : "+v"(z));
  return z;
}
template <int ES, bool ANY>
__device__ __forceinline__ u32x4 fetch_B(const DevProblem &P, int64_t row_off, int k, bool ok, uintptr_t zeros) {
  using piece_t = typename std::conditional<ANY, u32x4_any, u32x4>::type;
  const uintptr_t p = (uintptr_t)P.B + (uintptr_t)((row_off + k) * ES);
  return __builtin_nontemporal_load((const piece_t SK_GLOBAL *)(ok ? p : zeros));
}

// ---- pieces at any element's address ----
// (The hardware reads 16 bytes from any address in one instruction.)
// Element e of the result is element e + sh of v; what would come from beyond v's ends is zero.
template <int ES>
__device__ __forceinline__ u32x4 shift_piece(const u32x4 &v, int sh) {
  const int n = (sh < 0 ? -sh : sh) * (ES / 2);  // in halves
  const bool d1 = n & 2, d2 = n & 4, gone = n >= 8;
  const uint32_t bits = (n & 1) * 16;
  u32x4 r = v;
  if (__any(sh > 0)) {  // towards lower places
    const u32x4 s = {d1 ? v[1] : v[0], d1 ? v[2] : v[1], d1 ? v[3] : v[2], d1 ? 0u : v[3]};
    const u32x4 t = {d2 ? s[2] : s[0], d2 ? s[3] : s[1], d2 ? 0u : s[2], d2 ? 0u : s[3]};
    const u32x4 u = {__builtin_amdgcn_alignbit(t[1], t[0], bits), __builtin_amdgcn_alignbit(t[2], t[1], bits),
                     __builtin_amdgcn_alignbit(t[3], t[2], bits), t[3] >> bits};
#pragma unroll
    for (int i = 0; i < 4; ++i) r[i] = sh > 0 ? (gone ? 0u : u[i]) : r[i];
  }
  if (__any(sh < 0)) {  // towards higher places
    const u32x4 s = {d1 ? 0u : v[0], d1 ? v[0] : v[1], d1 ? v[1] : v[2], d1 ? v[2] : v[3]};
    const u32x4 t = {d2 ? 0u : s[0], d2 ? 0u : s[1], d2 ? s[0] : s[2], d2 ? s[1] : s[3]};
    // (alignbit shifts right: by 32 - bits, written as a left shift of the pair by `bits`)
    const u32x4 u = {t[0] << bits, bits ? __builtin_amdgcn_alignbit(t[1], t[0], 16) : t[1],
                     bits ? __builtin_amdgcn_alignbit(t[2], t[1], 16) : t[2], bits ? __builtin_amdgcn_alignbit(t[3], t[2], 16) : t[3]};
#pragma unroll
    for (int i = 0; i < 4; ++i) r[i] = sh < 0 ? (gone ? 0u : u[i]) : r[i];
  }
  return r;
}
// Elements below `lo` and from `hi` on become zero.
template <int ES>
__device__ __forceinline__ u32x4 mask_piece(const u32x4 &v, int lo, int hi) {
  u32x4 r = v;
  if constexpr (ES == 4) {
#pragma unroll
    for (int e = 0; e < 4; ++e) r[e] = (e >= lo && e < hi) ? v[e] : 0u;
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const uint32_t m = ((2 * e >= lo && 2 * e < hi) ? 0xffffu : 0u) | ((2 * e + 1 >= lo && 2 * e + 1 < hi) ? 0xffff0000u : 0u);
      r[e] = v[e] & m;
    }
  }
  return r;
}
// The four dwords that start `shift` bits (0 or 16) into v, `end` behind them.
__device__ __forceinline__ u32x4 join_dwords(const u32x4 &v, uint32_t end, uint32_t shift) {
  return u32x4{__builtin_amdgcn_alignbit(v[1], v[0], shift), __builtin_amdgcn_alignbit(v[2], v[1], shift),
               __builtin_amdgcn_alignbit(v[3], v[2], shift), __builtin_amdgcn_alignbit(end, v[3], shift)};
}
__device__ __forceinline__ u32x4 load_any(uintptr_t p) { return *(const u32x4_any SK_GLOBAL *)p; }

// n / d with d given as multiplier and shift (FastDiv), 0 <= n < 2^31.
__device__ __forceinline__ int fast_div(int n, const uint32_t (&d)[2]) {
  return (int)(uint32_t)(((uint64_t)(uint32_t)n * d[0]) >> d[1]);
}

// Where row m of the activation operand starts.
struct RowA {
  int64_t base;  // plain: m*lda.  gather: offset of pixel (b, hb, wb), channel 0, the one under filter tap (0,0); may be negative
  int hb, wb;    // gather: ho*stride-pad_h, wo*stride-pad_w
};

__device__ __forceinline__ RowA row_of(const DevProblem &P, int m) {
  RowA r;
  if (!P.gather) {
    r.base = (int64_t)m * P.lda;
    r.hb = 0;
    r.wb = 0;
  } else {
    const int hw = P.Ho * P.Wo;
    const int b = fast_div(m, P.div_hw);
    const int rem = m - b * hw;
    const int ho = fast_div(rem, P.div_wo);
    const int wo = rem - ho * P.Wo;
    r.hb = ho * P.stride - P.pad_h;
    r.wb = wo * P.stride - P.pad_w;
    if (P.nchw)
      r.base = ((int64_t)b * P.Cin * P.H + r.hb) * P.W + r.wb;  // pixel (b, channel 0, hb, wb)
    else
      r.base = (((int64_t)b * P.H + r.hb) * P.W + r.wb) * P.Cin;
  }
  return r;
}

// Channel-major convolutions: where output (m, n) lives in Y[Nb,Cout,Ho,Wo].
__device__ __forceinline__ int64_t nchw_out_base(const DevProblem &P, int m) {
  const int hw = P.Ho * P.Wo;
  const int b = fast_div(m, P.div_hw);
  return (int64_t)b * P.Ng * hw + (m - b * hw);  // + n * Ho*Wo
}
template <int DT>
__device__ __forceinline__ void store_elem(void *C, int64_t off, float v) {
  char SK_GLOBAL *c = as_global_mut<char>(C) + off * Elem<DT>::ES;
  if constexpr (DT == SK_F32)
    *(float SK_GLOBAL *)c = v;
  else
    *(uint16_t SK_GLOBAL *)c = (uint16_t)cvt_bits<DT>(v);
}

// Activation piece at element `off` of the operand; where !ok the piece of zeros.
template <int ES, bool ANY>
__device__ __forceinline__ u32x4 fetch_A(const DevProblem &P, int64_t off, bool ok, uintptr_t zeros) {
  using piece_t = typename std::conditional<ANY, u32x4_any, u32x4>::type;
  const uintptr_t p = (uintptr_t)P.A + (uintptr_t)(off * ES);
  return *(const piece_t SK_GLOBAL *)(ok ? p : zeros);
}

// Single elements as float, for run_generic.
template <int DT>
__device__ __forceinline__ float load_elem(const void *base, int64_t off) {
  if constexpr (DT == SK_F32) {
    return as_global<float>(base)[off];
  } else if constexpr (DT == SK_BF16) {
    return __builtin_bit_cast(float, (uint32_t)as_global<uint16_t>(base)[off] << 16);
  } else {
    return (float)as_global<_Float16>(base)[off];
  }
}

// ---------------------------------------------------------------------------
// MFMA wrappers: one 16-byte piece per lane and operand.
// 16x16: lane l gives row/column l%16 and K-slot l/16.  32x32: l%32 and l/32.
// The two operands use the same lane -> K-slot map, so which K elements a
// slot really holds does not matter as long as both operands agree.
// ---------------------------------------------------------------------------
template <int DT>
__device__ __forceinline__ void mma16(const u32x4 &a, const u32x4 &b, f32x4 &c) {
  if constexpr (DT == SK_BF16) {
    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0,
                                                0);
  } else if constexpr (DT == SK_F16) {
    c = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
  } else {
    // (whole-vector casts: a bit cast applied to a single vector element reads element 0)
    const f32x4 af = __builtin_bit_cast(f32x4, a), bf = __builtin_bit_cast(f32x4, b);
#pragma unroll
    for (int j = 0; j < 4; ++j) c = __builtin_amdgcn_mfma_f32_16x16x4f32(af[j], bf[j], c, 0, 0, 0);
  }
}

template <int DT>
__device__ __forceinline__ void mma32(const u32x4 &a, const u32x4 &b, f32x16 &c) {
  if constexpr (DT == SK_BF16) {
    c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0,
                                                0);
  } else if constexpr (DT == SK_F16) {
    c = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
  } else {
    const f32x4 af = __builtin_bit_cast(f32x4, a), bf = __builtin_bit_cast(f32x4, b);
#pragma unroll
    for (int j = 0; j < 4; ++j) c = __builtin_amdgcn_mfma_f32_32x32x2f32(af[j], bf[j], c, 0, 0, 0);
  }
}

// ---------------------------------------------------------------------------
// skinny tiles
// ---------------------------------------------------------------------------
// A tile is all Mg (<= 16*RM) activation rows against n_len weight rows and a
// slice [k0, k0+k_len) of the reduction.  The four waves of the workgroup take
// different groups of 32 weight rows (two 16-row MFMA blocks per wave).
//
// Weights never touch LDS: each wave streams its rows HBM -> registers -> MFMA
// through a ring of NB reduction blocks (128 bytes per row each), so NB-1
// blocks of loads stay in flight while one is multiplied, and every wave walks
// along its rows in consecutive 128-byte steps.
//
// The activations (tiny, and gathered from an image for a convolution) are
// staged once per workgroup through LDS in chunks of SKINNY_CHUNK_BYTES,
// double-buffered, one barrier per chunk.
//
// Long reductions are cut into S slices that different workgroups take
// (records with S > 1).  Each slice leaves its fp32 partial sums in a
// workspace in register layout; the workgroup that arrives last adds the S
// partials in slice order (so the result does not depend on arrival order)
// and writes C.
// (8 KB = 4 / 2 / 1 blocks of K per chunk for 1 / 2 / 4 row blocks.  Measured against 16 and 32 KB
// the smaller chunk is faster for every class: fewer staging loads queued between the weight
// loads, less padding of short reductions to whole chunks.)
constexpr int SKINNY_CHUNK_BYTES = 8192;

constexpr int ilog2(int x) { return x <= 1 ? 0 : 1 + ilog2(x >> 1); }

// Two registers loaded with the full-line map hold, for a 16-row MFMA block,
//   first : lanes r16 < 8 -> (row r16, pieces 0..3)      lanes r16 >= 8 -> (row r16-8, pieces 4..7)
//   second: lanes r16 < 8 -> (row r16+8, pieces 0..3)    lanes r16 >= 8 -> (row r16,   pieces 4..7)
// fix_lo gives (row r16, pieces 0..3) in every lane, fix_hi (row r16, pieces 4..7): the halves
// that are in the wrong place come from the other register, rotated by 8 lanes within each row
// of 16 (DPP row_ror:8, written only to the upper resp. lower 8 lanes through the bank mask).
__device__ __forceinline__ u32x4 fix_lo(const u32x4 &first, const u32x4 &second) {
  u32x4 r;
#pragma unroll
  for (int i = 0; i < 4; ++i)
    r[i] = (uint32_t)__builtin_amdgcn_update_dpp((int)first[i], (int)second[i], 0x128, 0xF, 0xC, false);
  return r;
}
__device__ __forceinline__ u32x4 fix_hi(const u32x4 &first, const u32x4 &second) {
  u32x4 r;
#pragma unroll
  for (int i = 0; i < 4; ++i)
    r[i] = (uint32_t)__builtin_amdgcn_update_dpp((int)second[i], (int)first[i], 0x128, 0xF, 0x3, false);
  return r;
}

// One accumulator (16 bytes per lane, 1 KB per wave) written / read at device scope (through
// to memory, not left in or served from an XCD's L2) as two 64-bit relaxed atomics per lane.
// The 1 KB block holds the low halves of all 64 lanes first, then the high halves, so that
// each of the two instructions covers 512 contiguous bytes: a write-through of scattered
// 8-byte pieces would cost a partial-line memory write each.
__device__ __forceinline__ void store_device_scope(f32x4 *block, int lane, const f32x4 &v) {
  unsigned long long *q = (unsigned long long *)block;
  __hip_atomic_store(q + lane, __builtin_bit_cast(unsigned long long, __builtin_shufflevector(v, v, 0, 1)),
                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __hip_atomic_store(q + 64 + lane, __builtin_bit_cast(unsigned long long, __builtin_shufflevector(v, v, 2, 3)),
                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ f32x4 load_device_scope(const f32x4 *block, int lane) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  unsigned long long *q = (unsigned long long *)block;
  const f32x2 lo = __builtin_bit_cast(f32x2, __hip_atomic_load(q + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
  const f32x2 hi =
      __builtin_bit_cast(f32x2, __hip_atomic_load(q + 64 + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
  return f32x4{lo.x, lo.y, hi.x, hi.y};
}

// Memory order of the arrival count that hands split-reduction partials from one workgroup to another.
// The partials themselves are written and read with device-scope accesses that go through to memory
// (see store_device_scope), each wave waits for its own stores to complete (s_waitcnt) and the workgroup
// meets at a barrier before one thread counts it in, so on this hardware a relaxed count suffices.  The
// language memory model asks for release/acquire on the count as well; that variant is
// kept compilable (-DSK_SPLITK_ACQ_REL) and costs a write-back and an invalidate of the XCD's L2 per slice.
#ifdef SK_SPLITK_ACQ_REL
#define SK_ARRIVE_ORDER __ATOMIC_ACQ_REL
#else
#define SK_ARRIVE_ORDER __ATOMIC_RELAXED
#endif
#if defined(__HIP_DEVICE_COMPILE__) && !defined(__gfx950__)
#error "the split-reduction hand-over relies on gfx950's write-through device-scope stores"
#endif

struct SplitK {
  f32x4 *ws;                // partial sums of all split output rectangles
  const uint32_t *ws_off;   // per out_tile_id: offset of its partials in ws, in f32x4 units
  uint32_t *arrive;         // per out_tile_id: slices that have delivered (re-armed by the last one)
};

// The workgroup's next tile: claimed from the queue and its work record fetched while the
// current tile is still streaming, in two steps that each tile class places in its main loop.
//   claim(): thread 0 takes the next index from the queue (an atomic whose answer takes a
//     memory round trip).  Late in the tile, not at its start: a claimed tile cannot start
//     before its workgroup is free, so at the end of the launch tiles claimed early would
//     wait behind long tiles while other workgroups sit idle.
//   issue(): once the answer is there, lane i < WORK_DWORDS of every wave loads dword i of the
//     record (one register per lane).  Only wave 0 has the real index, and only its copy is
//     used.
// CLAIM_LEAD / ISSUE_GAP are counted in steps of the class's main loop (a step is one to two
// microseconds when the memory system is loaded).
struct Prefetch {
  const TileWork *work;
  uint32_t *counter;  // the queue (null: tiles are not handed out by the queue)
  uint32_t base;      // index of the first tile the queue hands out (0 when there is no queue)
  uint32_t next;      // next tile's index minus `base`; meaningful in lane 0 of wave 0 (in all lanes when there
                      // is no queue).  The queue's answer is left untouched until issue() needs it: anything
                      // computed from it at once would make the wave wait for the atomic, and with it for
                      // every load in flight.
  uint32_t last;      // last valid index of the launch
  int tid;            // this tile's copy of the thread index (see the tile loop)
  const TileWork *rec;  // the record of the tile that is running
  uint32_t word = 0;
  // An LDS tile is run by the die whose list holds it (see the tile loop).  While such a tile runs, the
  // workgroup also draws the next entry of its die's list (xhead not null), on the guess that its next
  // ticket falls on an LDS tile again: thread 1 draws beside thread 0 in the same atomic instruction, and
  // the one load of issue() brings the record of that entry (lanes below WORK_DWORDS) and, in lane 63, the
  // dword of the ticket's own record that holds its tile class.  (One atomic and one load as without
  // lists: with two of either in flight the compiler waits, in every step of the LDS-tile loops, until
  // one load at most is outstanding, which also counts the operand loads it does not see.)
  uint32_t *xhead = nullptr;
  const TileWork *xrec = nullptr;  // first record of the die's list
  uint32_t xlen = 0;               // its length (> 0 whenever xhead is set)
#ifdef SK_DIAG_CLOCKS
  int diag_tile = 0;
#endif
  __device__ __forceinline__ void claim() {
    // (lanes other than threads 0 and 1 keep whatever `next` held: it is never used, and any
    // instruction that touched the register here would have to wait for an earlier answer)
    if (counter && tid < (xhead ? 2 : 1)) next = atomicAdd(tid == 0 ? counter : xhead, 1u);
  }
  __device__ __forceinline__ void issue() {
    uint32_t idx = (uint32_t)__builtin_amdgcn_readfirstlane((int)next) + base;
    if (idx > last) idx = last;  // past the end of the table: the workgroup is about to leave
    const int lane = tid & 63;
    const uint32_t SK_GLOBAL *src = as_global<uint32_t>(work + idx) + (lane < WORK_DWORDS ? lane : 0);
    if (xhead) {
      uint32_t k = (uint32_t)__builtin_amdgcn_readlane((int)next, 1);
      if (k >= xlen) k = xlen - 1u;  // the list is used up
      src = lane == 63 ? as_global<uint32_t>(work + idx) + 1 : as_global<uint32_t>(xrec + k) + (lane < WORK_DWORDS ? lane : 0);
    }
    word = *src;
  }
  // step `i` of `total` main-loop steps
  __device__ __forceinline__ void at_step(int i, int total, int lead, int gap) {
    const int claim_at = total > lead ? total - lead : 0;
    const int issue_at = claim_at + gap < total ? claim_at + gap : total - 1;
    if (i == claim_at) claim();
    if (i == issue_at) issue();
  }
};
constexpr int CLAIM_LEAD = 8, ISSUE_GAP = 4;

//
// ANY: operands at any element's address, and GEMMs whose reduction length is not a multiple of a piece.  The
// piece that would reach beyond the end of a row is read so that it ends with the row, and shifted into
// place (shift_piece) when it is used; only the last block of a row has such pieces.  Everything else is
// the same, so aligned operators of a plan that has others too run through this form as well.
template <int DT, int RM, bool ANY, bool GATHER>
__device__ __forceinline__ void run_skinny_form(const DevProblem &P, const sk_tile &T, const SplitK &sp,
                                           unsigned char *lds, uint32_t *s_flag, Prefetch &pf) {
  constexpr int ES = Elem<DT>::ES;
  constexpr int CE = 16 / ES;
  constexpr int KB = 8 * CE;                        // reduction elements per block (128 bytes)
  constexpr int ROWS = 16 * RM;                     // activation rows held in LDS
  constexpr int CHUNK_BYTES = SKINNY_CHUNK_BYTES;
  constexpr int ROWB = CHUNK_BYTES / ROWS;          // bytes of K per row and chunk
  constexpr int LROW = ROWB + 16;                   // padded LDS row (bank spread)
  constexpr int BPC_LOG2 = ilog2(ROWB / 128);
  constexpr int BPC = 1 << BPC_LOG2;                // blocks per chunk: 4, 2, 1
  constexpr int PPR = ROWB / 16;                    // pieces per row and chunk
  constexpr int BUF = ROWS * LROW;                  // bytes per LDS buffer
  // Ring slots (weight blocks in flight plus one) and activation chunks in flight.  Loads come back in order, so a chunk
  // needed one step after it was asked for also makes every weight load issued before it late.  A convolution's
  // chunks are gathered, and its tiles mostly run beside LDS tiles that leave the memory system idle: with one of each in flight a
  // 64-row tile of a 3x3 layer took a memory round trip, 1.8 us, per step; with three and two the ResNet mix x16 takes 85.6
  // instead of 90.4 us.  GEMMs stream: every workgroup of the launch does, the memory system is saturated by far
  // fewer bytes in flight than the launch holds even at one block, and a deeper ring only lengthens every load's
  // wait (BERT mix x8 176 us with one and one, 181 with three and two; main workload 1035, 1041).
  constexpr int NB = GATHER ? 4 : 2;
  constexpr int AD = GATHER && BPC < 4 ? 2 : 1;
  static_assert(AD == 1 || BPC * AD <= NB, "a chunk's registers are told apart by the step within the unrolled loop");
  static_assert(ROWB == BPC * 128, "chunk geometry");
  static_assert(2 * BUF <= LDS_TILE_BYTES, "activation chunks do not fit");

  const int tid = pf.tid;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform: keeps its branches scalar
  const int lane = tid & 63;
  const int r16 = lane & 15, q = lane >> 4;

  const int n_end = (int)T.n0 + (int)T.n_len;
  const int ngroups = ((int)T.n_len + 31) >> 5;
  const int iters = (ngroups + 3) >> 2;

  const int k0 = (int)T.k0, k_stop = (int)T.k0 + (int)T.k_len;
  const int nblocks = ((int)T.k_len + KB - 1) / KB;
  const int nchunks = (nblocks + BPC - 1) >> BPC_LOG2;
  const int nslots = nchunks << BPC_LOG2;  // block slots per wave (blocks past the end read as zero)

  const uintptr_t zeros = zero_piece_address();
  // staging map: thread -> SPT consecutive pieces of one activation row
  constexpr int SPT = CHUNK_BYTES / (WG_THREADS * 16);
  constexpr int TPR = PPR / SPT;  // threads per row
  const int s_row = tid / TPR;
  const int s_piece = (tid % TPR) * SPT;
  const bool s_ok = s_row < P.Mg;
  const RowA srow = row_of(P, s_ok ? s_row : 0);
  const int s_lds = s_row * LROW + s_piece * 16;
  u32x4 ar[AD][SPT];
  int ar_k[AD] = {};  // (ANY) reduction index of the first piece
  const bool ragged = ANY && P.Kg % CE != 0;  // some pieces end beyond their row
  // For a convolution: filter tap (g_r, g_s) and channel g_c of this thread's first piece in the
  // chunk that stage_load will fetch next, and g_off = ((g_r*W + g_s)*Cin + g_c), its distance in
  // elements from the pixel under tap (0,0).  Chunks are fetched in order (0, 1, ..., then 0 again
  // for the next pass), so the position moves on by additions; the divisions happen once per tile.
  int g_r = 0, g_s = 0, g_c = 0;
  int64_t g_off = 0;
  const int64_t next_filter_row = (int64_t)(P.W - P.S) * P.Cin;
  if constexpr (GATHER) {
    const int kk = k0 + s_piece * CE;
    const int tap = fast_div(kk, P.div_cin);
    g_c = kk - tap * P.Cin;
    g_r = fast_div(tap, P.div_s);
    g_s = tap - g_r * P.S;
    g_off = ((int64_t)g_r * P.W + g_s) * P.Cin + g_c;
  }
  const int g_r0 = g_r, g_s0 = g_s, g_c0 = g_c;
  const int64_t g_off0 = g_off;
  auto stage_load = [&](int c, u32x4(&ar)[SPT], int &ar_k) {
    const int k = k0 + ((c << BPC_LOG2) * 8 + s_piece) * CE;
    if constexpr (!GATHER) {
      ar_k = k;
#pragma unroll
      for (int i = 0; i < SPT; ++i) {
        const int at = ANY ? min(k + i * CE, P.Kg - CE) : k + i * CE;
        ar[i] = fetch_A<ES, ANY>(P, srow.base + at, s_ok && k + i * CE < k_stop, zeros);
      }
      return;
    }
    if (c == 0) {
      g_r = g_r0;
      g_s = g_s0;
      g_c = g_c0;
      g_off = g_off0;
    }
    // the thread's pieces follow one another in the patch row (a piece never straddles two taps:
    // Cin is a multiple of a piece); no branch between the loads
    int r = g_r, t = g_s, cc = g_c;
    int64_t off = g_off;
#pragma unroll
    for (int i = 0; i < SPT; ++i) {
      const bool ok = s_ok && k + i * CE < k_stop && (unsigned)(srow.hb + r) < (unsigned)P.H &&
                      (unsigned)(srow.wb + t) < (unsigned)P.W;
      ar[i] = fetch_A<ES, ANY>(P, srow.base + off, ok, zeros);
      cc += CE;
      off += CE;
      const bool next_tap = cc >= P.Cin;
      cc -= next_tap ? P.Cin : 0;
      t += next_tap ? 1 : 0;
      const bool next_row = t == P.S;  // (only ever true right after a step to the next tap)
      t = next_row ? 0 : t;
      r += next_row ? 1 : 0;
      off += next_row ? next_filter_row : 0;
    }
    // on to the next chunk
    constexpr int KC = BPC * 8 * CE;
    g_c += KC;
    g_off += KC;
    while (g_c >= P.Cin) {
      g_c -= P.Cin;
      if (++g_s == P.S) {
        g_s = 0;
        ++g_r;
        g_off += next_filter_row;
      }
    }
  };
  auto stage_store = [&](int c, u32x4(&ar)[SPT], int ar_k) {
    unsigned char *base = lds + (c & 1) * BUF + s_lds;
    if (ragged) {
#pragma unroll
      for (int i = 0; i < SPT; ++i) {
        const int past = ar_k + (i + 1) * CE - P.Kg;  // how far the piece reaches beyond its row (a whole piece: zeros)
        if (__any(past > 0)) ar[i] = shift_piece<ES>(ar[i], max(past, 0));
      }
    }
#pragma unroll
    for (int i = 0; i < SPT; ++i) *(u32x4 *)(base + i * 16) = ar[i];
  };

  const bool vec_c = (P.flags & FLAG_VEC_C) != 0;
  const bool restage_each = nchunks > 1;

  // A wave's work is one stream of block slots: pass 0 (its first weight group) blocks
  // 0..nslots-1, then pass 1, ...  The weight loads run NB-1 slots ahead of the MFMAs and
  // keep running across pass boundaries, so the ring only drains at the end of the tile.
  // --- load stream (ahead) ---
  int p_it = 0, p_blk = 0;
  bool p_act = false;
  // Load map: instruction j of a block covers rows 8j..8j+7 of the 32-row group with their full
  // 128-byte lines: lane (r16, q) reads row 8j + r16%8, piece q + 4*(r16/8).  (Eight whole lines
  // per instruction stream measurably better than sixteen half lines.)  The MFMA wants row
  // r16 in lane r16 with pieces 0..3 resp. 4..7 in slot q; two DPP half-row swaps per pair of
  // registers put the data there when the block is consumed (see fix_lo / fix_hi).
  const int piece = q + 4 * (r16 >> 3);
  int64_t wrow[4] = {0, 0, 0, 0};
  auto set_load_rows = [&](int it) {
    const int g = it * 4 + wave;
    p_act = it < iters && g < ngroups;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      int n = (int)T.n0 + g * 32 + j * 8 + (r16 & 7);
      if (n >= n_end) n = n_end - 1;  // rows past the edge repeat the last row; never stored
      wrow[j] = p_act ? (int64_t)n * P.ldb : 0;
    }
  };
  // The loads are unconditional (see fetch_B): slots past the end re-read the start of a row, and
  // slots that no pass will multiply (past the end of the tile, waves without a group) all read
  // the very first piece of the operand, so that the number of loads in flight at every point
  // of the loop is the same on every path and the waits stay exact.
  auto next_load = [&](u32x4(&w)[4]) {
    const int k = k0 + p_blk * KB + piece * CE;
    const bool in = p_act && k < k_stop;
#pragma unroll
    for (int j = 0; j < 4; ++j) w[j] = fetch_B<ES, ANY>(P, wrow[j], ANY ? min(k, P.Kg - CE) : k, in, zeros);
    if (++p_blk == nslots) {
      p_blk = 0;
      ++p_it;
      set_load_rows(p_it);
    }
  };
  // --- compute stream ---
  int it = 0, blk = 0, buf = 1;
  f32x4 acc[2][RM];
#pragma unroll
  for (int rb = 0; rb < 2; ++rb)
#pragma unroll
    for (int mb = 0; mb < RM; ++mb) acc[rb][mb] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto store_pass = [&]() {
    // lane holds, per (rb, mb): row m = mb*16 + lane%16, columns n_base + rb*16 + (lane/16)*4 + 0..3
    const int g = it * 4 + wave;
    const int n_base = (int)T.n0 + g * 32;
    if (g < ngroups) {
#pragma unroll
      for (int mb = 0; mb < RM; ++mb) {
        const int m = mb * 16 + r16;
        if (m < P.Mg) {
          const int64_t row_off = (int64_t)m * P.ldc;
#pragma unroll
          for (int rb = 0; rb < 2; ++rb) {
            const int n = n_base + rb * 16 + q * 4;
            if (n < n_end) store4<DT>(P.C, row_off, n, n_end, acc[rb][mb], vec_c);
          }
        }
      }
    }
  };

#ifdef SK_DIAG_CLOCKS
  const int diag_tile = pf.diag_tile;
#endif
  SK_DIAG(1);
  set_load_rows(0);
  // the next chunk to fetch: chunk l_c of pass l_it
  int l_c = 0, l_it = 0;
  auto next_chunk = [&](u32x4(&x)[SPT], int &k) {
    if (l_it >= iters) return;
    stage_load(l_c, x, k);
    if (++l_c == nchunks) {
      l_c = 0;
      ++l_it;
    }
  };
  next_chunk(ar[0], ar_k[0]);
  u32x4 w[NB][4];
  next_load(w[0]);
  if (AD == 2 && restage_each) next_chunk(ar[AD - 1], ar_k[AD - 1]);
#pragma unroll
  for (int u = 1; u < NB - 1; ++u) next_load(w[u]);
  if (!restage_each) {
    // the only activation chunk serves every pass
    stage_store(0, ar[0], ar_k[0]);
    buf = 0;
    __syncthreads();
  }

  const int total = iters * nslots;
  for (int i0 = 0; i0 < total; i0 += NB) {
#pragma unroll
    for (int u = 0; u < NB; ++u) {
      const bool live = i0 + u < total;
      pf.at_step(i0 + u, total, CLAIM_LEAD, ISSUE_GAP);
      if (live && restage_each && (blk & (BPC - 1)) == 0) {
        // first block of a chunk: publish it, then start fetching the AD-th after it (of this pass, or of the next).
        // (Chunks and unrolled steps keep step: a pass has whole chunks, so steps u of one parity of u / BPC meet chunks of one.)
        constexpr int set = AD == 2 ? 1 : 0;
        buf ^= 1;
        stage_store(buf, ar[(u / BPC) & set], ar_k[(u / BPC) & set]);
        __syncthreads();
        next_chunk(ar[(u / BPC) & set], ar_k[(u / BPC) & set]);
      }
      next_load(w[(u + NB - 1) % NB]);
      if (live) {
        if (it * 4 + wave < ngroups) {
          const unsigned char *abase = lds + buf * BUF + (blk & (BPC - 1)) * 128 + q * 16 + r16 * LROW;
          // All activation pieces of the block are requested from LDS first, each into registers
          // of its own (read one row block at a time into the same registers, every read would
          // wait for the MFMAs of the row block before it), and before the weights are touched:
          // the LDS round trip then overlaps the wait for the weight block.
          u32x4 a0[RM], a1[RM];
#pragma unroll
          for (int mb = 0; mb < RM; ++mb) {
            a0[mb] = *(const u32x4 *)(abase + mb * 16 * LROW);       // pieces 0..3
            a1[mb] = *(const u32x4 *)(abase + mb * 16 * LROW + 64);  // pieces 4..7
          }
          __builtin_amdgcn_sched_barrier(0);  // (the scheduler would sink the reads back to their uses)
          if (ragged && k0 + (blk + 1) * KB > P.Kg) {  // the last block of the rows
            const int past = k0 + blk * KB + (piece + 1) * CE - P.Kg;
#pragma unroll
            for (int j = 0; j < 4; ++j) w[u][j] = shift_piece<ES>(w[u][j], max(past, 0));
          }
          // rows 16rb..16rb+15: pieces 0..3 (x) and 4..7 (y) in MFMA lane order
          const u32x4 x0 = fix_lo(w[u][0], w[u][1]), y0 = fix_hi(w[u][0], w[u][1]);
          const u32x4 x1 = fix_lo(w[u][2], w[u][3]), y1 = fix_hi(w[u][2], w[u][3]);
#pragma unroll
          for (int mb = 0; mb < RM; ++mb) {
            mma16<DT>(x0, a0[mb], acc[0][mb]);
            mma16<DT>(x1, a0[mb], acc[1][mb]);
            mma16<DT>(y0, a1[mb], acc[0][mb]);
            mma16<DT>(y1, a1[mb], acc[1][mb]);
          }
        }
        if (i0 + u == 0) SK_DIAG(2);
        if (++blk == nslots && it + 1 < iters) {
          // this weight group is done; the next one's loads are already in flight
          store_pass();
#pragma unroll
          for (int rb = 0; rb < 2; ++rb)
#pragma unroll
            for (int mb = 0; mb < RM; ++mb) acc[rb][mb] = f32x4{0.f, 0.f, 0.f, 0.f};
          blk = 0;
          ++it;
        }
      }
    }
  }

  SK_DIAG(3);
  // last pass (the only one of a split rectangle, which has at most four weight groups)
  bool finish = true;
  if (T.S > 1) {
    // Deliver this slice's partial sums; the last slice to arrive adds all of them in slice
    // order.  The partials are written and read with device-scope accesses (they go through
    // to memory, past the per-XCD L2s), so no cache-wide release/acquire is needed: each wave
    // waits for its own stores, the workgroup meets at a barrier, one thread counts it in.
    f32x4 *mine = sp.ws + sp.ws_off[T.out_tile_id];
    const int slot = (wave * 2 * RM) * 64;  // this wave's 2*RM blocks of 64 x 16 bytes within a slice
#pragma unroll
    for (int rb = 0; rb < 2; ++rb)
#pragma unroll
      for (int mb = 0; mb < RM; ++mb)
        store_device_scope(mine + (size_t)T.ks_idx * (4 * 2 * RM * 64) + slot + (rb * RM + mb) * 64, lane,
                           acc[rb][mb]);
    __builtin_amdgcn_s_waitcnt(0);  // all counters to zero: the stores above have completed
    __syncthreads();
    if (tid == 0)
      *s_flag = __hip_atomic_fetch_add(&sp.arrive[T.out_tile_id], 1u, SK_ARRIVE_ORDER, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    const uint32_t prev = *s_flag;
    finish = prev == (uint32_t)T.S - 1;
    if (finish) {
#pragma unroll
      for (int rb = 0; rb < 2; ++rb)
#pragma unroll
        for (int mb = 0; mb < RM; ++mb) acc[rb][mb] = f32x4{0.f, 0.f, 0.f, 0.f};
      // All partial sums of a slice are requested before the first is added, and those of the next AHEAD - 1
      // slices while this one's are added (left to the scheduler the loads went out two at a time, each pair
      // waited for: eight memory round trips per slice, which made an operator cut into dozens of slices
      // several times slower).  The sums are still taken in slice order.
      constexpr int AHEAD = 2;  // slices in flight (four or eight for the classes with fewer rows: measured, no gain)
      f32x4 part[AHEAD][2][RM];
      auto request = [&](int s2, f32x4(&dst)[2][RM]) {
#pragma unroll
        for (int rb = 0; rb < 2; ++rb)
#pragma unroll
          for (int mb = 0; mb < RM; ++mb)
            dst[rb][mb] = load_device_scope(mine + (size_t)s2 * (4 * 2 * RM * 64) + slot + (rb * RM + mb) * 64, lane);
      };
      const int S = (int)T.S;
#pragma unroll
      for (int u = 0; u < AHEAD - 1; ++u)
        if (u < S) request(u, part[u]);
      for (int s0 = 0; s0 < S; s0 += AHEAD) {
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) {
          const int s2 = s0 + u;
          if (s2 + AHEAD - 1 < S) request(s2 + AHEAD - 1, part[(u + AHEAD - 1) % AHEAD]);
          __builtin_amdgcn_sched_barrier(0);
          if (s2 < S) {
#pragma unroll
            for (int rb = 0; rb < 2; ++rb)
#pragma unroll
              for (int mb = 0; mb < RM; ++mb) acc[rb][mb] += part[u][rb][mb];
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      if (tid == 0)  // re-arm for the next launch
        __hip_atomic_store(&sp.arrive[T.out_tile_id], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
  if (finish) store_pass();
  SK_DIAG(4);
}

template <int DT, int RM, bool ANY>
__device__ __forceinline__ void run_skinny(const DevProblem &P, const sk_tile &T, const SplitK &sp, unsigned char *lds,
                                           uint32_t *s_flag, Prefetch &pf) {
  if (P.gather)
    run_skinny_form<DT, RM, ANY, true>(P, T, sp, lds, s_flag, pf);
  else
    run_skinny_form<DT, RM, ANY, false>(P, T, sp, lds, s_flag, pf);
}

// A slice of a split reduction hands its partial sums over; true in the workgroup that arrived last, with the
// sum of all slices (in slice order) in `acc`; false in the others, which have nothing left to do.
template <int FM, int FN>
__device__ __forceinline__ bool split_handover(const sk_tile &T, const SplitK &sp, uint32_t *s_flag, int tid,
                                               f32x16 (&acc)[FN][FM]) {
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63;

    // A slice of a split reduction: same hand-over as in the skinny classes.  Partial sums go to
    // the workspace in register layout with device-scope stores (a slice is FN*FM*4 blocks of
    // 64 x 16 bytes per wave); the last slice to arrive adds all of them in slice order.
    constexpr int PER_WAVE = FN * FM * 4;          // 1 KB blocks per wave and slice
    constexpr int PER_SLICE = 4 * PER_WAVE * 64;   // f32x4 units per slice
    f32x4 *mine = sp.ws + sp.ws_off[T.out_tile_id] + wave * PER_WAVE * 64;
#pragma unroll
    for (int fn = 0; fn < FN; ++fn)
#pragma unroll
      for (int fm = 0; fm < FM; ++fm)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const f32x4 v = {acc[fn][fm][4 * j], acc[fn][fm][4 * j + 1], acc[fn][fm][4 * j + 2], acc[fn][fm][4 * j + 3]};
          store_device_scope(mine + (size_t)T.ks_idx * PER_SLICE + ((fn * FM + fm) * 4 + j) * 64, lane, v);
        }
    __builtin_amdgcn_s_waitcnt(0);  // all counters to zero: the stores above have completed
    __syncthreads();
    if (tid == 0)
      *s_flag = __hip_atomic_fetch_add(&sp.arrive[T.out_tile_id], 1u, SK_ARRIVE_ORDER, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    if (*s_flag != (uint32_t)T.S - 1) return false;
#pragma unroll
    for (int fn = 0; fn < FN; ++fn)
#pragma unroll
      for (int fm = 0; fm < FM; ++fm)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[fn][fm][i] = 0.f;
    // (all partial sums of a slice are requested before the first is added: see run_skinny)
    for (int s2 = 0; s2 < T.S; ++s2) {
      f32x4 part[FN][FM][4];
#pragma unroll
      for (int fn = 0; fn < FN; ++fn)
#pragma unroll
        for (int fm = 0; fm < FM; ++fm)
#pragma unroll
          for (int j = 0; j < 4; ++j)
            part[fn][fm][j] = load_device_scope(mine + (size_t)s2 * PER_SLICE + ((fn * FM + fm) * 4 + j) * 64, lane);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int fn = 0; fn < FN; ++fn)
#pragma unroll
        for (int fm = 0; fm < FM; ++fm)
#pragma unroll
          for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[fn][fm][4 * j + e] += part[fn][fm][j][e];
      __builtin_amdgcn_sched_barrier(0);
    }
    if (tid == 0)  // re-arm for the next launch
      __hip_atomic_store(&sp.arrive[T.out_tile_id], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return true;
}

// What follows the main loop of an LDS tile: the hand-over of a split reduction and the stores.
// lane holds, per (fn, fm): row l32 of the 32x32 block, columns 8*(i/4) + 4*half + (i%4).
template <int DT, int BM, int BN, int WAVES_M, int WAVES_N>
__device__ __forceinline__ void finish_tile(const DevProblem &P, const sk_tile &T, const SplitK &sp, unsigned char *lds,
                                            uint32_t *s_flag, int tid,
                                            f32x16 (&acc)[BN / (32 * WAVES_N)][BM / (32 * WAVES_M)]) {
  constexpr int ES = Elem<DT>::ES;
  constexpr int CE = 16 / ES;
  constexpr int FM = BM / (32 * WAVES_M);
  constexpr int FN = BN / (32 * WAVES_N);
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63;
  const int wm = wave % WAVES_M, wn = wave / WAVES_M;
  const int l32 = lane & 31, half = lane >> 5;
  const int m0 = (int)T.m0, n0 = (int)T.n0;
  const int m_end = m0 + (int)T.m_len, n_end = n0 + (int)T.n_len;
  if (T.S > 1 && !split_handover<FM, FN>(T, sp, s_flag, tid, acc)) return;

  // lane holds, per (fn, fm): row m = l32, columns 8*(i/4) + 4*half + (i%4)
  //
  // Written from the accumulators a store instruction would cover 32 rows with 16 bytes each.
  // Where C allows 16-byte stores the tile goes through LDS instead (free by now: every wave has
  // passed the last stage's barrier) and leaves as whole rows: 16 lanes x 16 bytes side by side.
  constexpr int OROW = BN * ES + 16;  // padded row of the output tile in LDS
  static_assert(BM * OROW <= (BN == 64 ? NARROW_LDS_BYTES : LDS_TILE_BYTES), "output tile does not fit the LDS buffer");
  const bool wide = ((uintptr_t)P.C % 16 == 0) && ((P.ldc * ES) % 16 == 0);
  if (wide) {
#pragma unroll
    for (int fm = 0; fm < FM; ++fm) {
      const int r = (wm * FM + fm) * 32 + l32;
#pragma unroll
      for (int fn = 0; fn < FN; ++fn) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int c = (wn * FN + fn) * 32 + 8 * j + 4 * half;
          unsigned char *q = lds + r * OROW + c * ES;
          if constexpr (ES == 4) {
            *(f32x4 *)q = f32x4{acc[fn][fm][4 * j], acc[fn][fm][4 * j + 1], acc[fn][fm][4 * j + 2], acc[fn][fm][4 * j + 3]};
          } else {
            u32x2 o;
            o.x = cvt_pack<DT>(acc[fn][fm][4 * j], acc[fn][fm][4 * j + 1]);
            o.y = cvt_pack<DT>(acc[fn][fm][4 * j + 2], acc[fn][fm][4 * j + 3]);
            *(u32x2 *)q = o;
          }
        }
      }
    }
    __syncthreads();
    constexpr int PIECES = BN * ES / 16;             // 16-byte pieces per output row
    constexpr int RPI = WG_THREADS / PIECES;         // rows per store instruction
    const int pc = tid % PIECES, pr = tid / PIECES;
    const int n = n0 + pc * CE;
    // 32-bit offsets from the tile's corner; rows past the edge lie outside the descriptor and are not stored
    const int64_t extent = ((int64_t)((int)T.m_len - 1) * P.ldc + (int)T.n_len) * ES;
    if (n + CE <= n_end && (uint64_t)(256 * P.ldc * ES) >> 31 == 0) {
      const __amdgpu_buffer_rsrc_t desc = __builtin_amdgcn_make_buffer_rsrc(
          (void *)((uintptr_t)P.C + (uintptr_t)(((int64_t)m0 * P.ldc + n0) * ES)), 0, (int)extent, 0x00020000);
      const uint32_t ld = (uint32_t)(P.ldc * ES), voff = (uint32_t)pr * ld + (uint32_t)pc * 16u;
      u32x4 v[BM / RPI];
#pragma unroll
      for (int i = 0; i < BM / RPI; ++i) v[i] = *(const u32x4 *)(lds + pr * OROW + pc * 16 + i * (RPI * OROW));
      store_out(v, desc, voff, (uint32_t)RPI * ld, (P.flags & FLAG_PAST_CACHES) != 0);
      return;
    }
#pragma unroll 1
    for (int i = 0; i < BM / RPI; ++i) {
      const int r = pr + i * RPI;
      const int m = m0 + r;
      if (m < m_end && n < n_end) {
        const u32x4 v = *(const u32x4 *)(lds + r * OROW + pc * 16);
        char SK_GLOBAL *dst = as_global_mut<char>(P.C) + ((int64_t)m * P.ldc + n) * ES;
        if (n + CE <= n_end) {
          *(u32x4 SK_GLOBAL *)dst = v;
        } else {
          // ragged right edge: element by element
#pragma unroll
          for (int e = 0; e < CE; ++e) {
            if (n + e < n_end) {
              if constexpr (ES == 4)
                ((uint32_t SK_GLOBAL *)dst)[e] = v[e];
              else
                ((uint16_t SK_GLOBAL *)dst)[e] = (uint16_t)(v[e / 2] >> (16 * (e & 1)));
            }
          }
        }
      }
    }
    // (the barrier at the end of every tile keeps the next tile's LDS writes behind these reads)
    return;
  }
  const bool vec_c = (P.flags & FLAG_VEC_C) != 0;
#pragma unroll
  for (int fm = 0; fm < FM; ++fm) {
    const int m = m0 + (wm * FM + fm) * 32 + l32;
    if (m < m_end) {
      const int64_t row_off = (int64_t)m * P.ldc;
#pragma unroll
      for (int fn = 0; fn < FN; ++fn) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int n = n0 + (wn * FN + fn) * 32 + 8 * j + 4 * half;
          if (n < n_end) {
            f32x4 v = {acc[fn][fm][4 * j], acc[fn][fm][4 * j + 1], acc[fn][fm][4 * j + 2], acc[fn][fm][4 * j + 3]};
            store4<DT>(P.C, row_off, n, n_end, v, vec_c);
          }
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------
// LDS-staged tiles: BM x BN outputs per workgroup, 128 bytes of K per stage
// ---------------------------------------------------------------------------
// Operand pieces travel global memory -> registers -> LDS -> MFMA.  A ring of NS register
// stages keeps NS-1 stages of loads in flight.  LDS holds two stages: while the MFMAs of
// stage s read one buffer, the pieces of stage s+1 are written to the other, and one barrier
// per stage separates "everyone has written s+1 and finished reading s" from the next round.
//
// A stage costs a wave its whole instruction stream (address arithmetic, LDS traffic, MFMAs,
// barrier) back to back, so that stream is kept short: operand row pointers are formed once
// per tile, and the position in the implicit patch matrix (filter tap r,s and channel c of
// this thread's piece) advances by additions only -- no multiply or divide per stage.
template <int DT, int BM, int BN, int WAVES_M, int WAVES_N>
__device__ __forceinline__ void run_tile(const DevProblem &P, const sk_tile &T, const SplitK &sp, unsigned char *lds,
                                         uint32_t *s_flag, Prefetch &pf) {
  constexpr int ES = Elem<DT>::ES;
  constexpr int CE = 16 / ES;
  constexpr int KB = 8 * CE;                  // reduction elements per stage
  constexpr int FM = BM / (32 * WAVES_M);     // 32x32 blocks per wave along m
  constexpr int FN = BN / (32 * WAVES_N);     // ... along n
  constexpr int A_ITERS = BM / 32;            // 16-byte pieces per thread per stage, activations
  constexpr int B_ITERS = BN / 32;            // ... weights
  constexpr int STAGE = (BM + BN) * LDS_ROW;  // bytes of one stage in LDS
  constexpr int NS = 3;
  static_assert(WAVES_M * WAVES_N == 4, "four waves per workgroup");
  static_assert(2 * STAGE <= LDS_TILE_BYTES, "two stages do not fit the LDS buffer");

  const int tid = pf.tid;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63;
  const int wm = wave % WAVES_M, wn = wave / WAVES_M;
  const int l32 = lane & 31, half = lane >> 5;

  const int m0 = (int)T.m0, n0 = (int)T.n0;
  const int m_end = m0 + (int)T.m_len, n_end = n0 + (int)T.n_len;
  const int k_begin = (int)T.k0, k_stop = (int)T.k0 + (int)T.k_len;

  // staging map: thread -> piece c8 of rows (tid/8) + 32*i
  const int c8 = tid & 7;
  const int srow = tid >> 3;
  const bool gvec = P.gather != 0;
  const char SK_GLOBAL *pa[A_ITERS];  // row start (for a convolution: the pixel under filter tap (0,0), may lie outside the image)
  int hb[A_ITERS], wb[A_ITERS];
#pragma unroll
  for (int i = 0; i < A_ITERS; ++i) {
    int m = m0 + srow + 32 * i;
    if (m >= m_end) m = m_end - 1;  // rows past the edge repeat the last row; never stored
    const RowA r = row_of(P, m);
    pa[i] = as_global<char>(P.A) + r.base * ES;
    hb[i] = r.hb;
    wb[i] = r.wb;
  }
  const char SK_GLOBAL *pb[B_ITERS];
#pragma unroll
  for (int i = 0; i < B_ITERS; ++i) {
    int n = n0 + srow + 32 * i;
    if (n >= n_end) n = n_end - 1;
    pb[i] = as_global<char>(P.B) + (int64_t)n * P.ldb * ES;
  }

  f32x16 acc[FN][FM];
#pragma unroll
  for (int fn = 0; fn < FN; ++fn)
#pragma unroll
    for (int fm = 0; fm < FM; ++fm)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[fn][fm][i] = 0.f;

  // position of this thread's piece in the patch row: tap (g_r, g_s), channel g_c;
  // tap_off = ((g_r*W + g_s)*Cin + g_c) elements from the pixel under tap (0,0)
  int g_r = 0, g_s = 0, g_c = 0;
  int64_t tap_off = 0;
  const int64_t next_filter_row = (int64_t)(P.W - P.S) * P.Cin;
  if (gvec) {
    const int k = k_begin + c8 * CE;
    const int tap = fast_div(k, P.div_cin);
    g_c = k - tap * P.Cin;
    g_r = fast_div(tap, P.div_s);
    g_s = tap - g_r * P.S;
    tap_off = ((int64_t)g_r * P.W + g_s) * P.Cin + g_c;
  }
  u32x4 ra[NS][A_ITERS], rb[NS][B_ITERS];
  const uintptr_t zeros = zero_piece_address();
  // Loads are unconditional (stages past the end of the reduction read clamped addresses and
  // are never multiplied), so the number of loads in flight is the same on every path.
  int k_load = k_begin + c8 * CE;  // reduction index of this thread's piece in the next stage to load
  auto gload = [&](u32x4(&xa)[A_ITERS], u32x4(&xb)[B_ITERS]) {
    const bool in = k_load < k_stop;
    if (gvec) {
#pragma unroll
      for (int i = 0; i < A_ITERS; ++i) {
        const bool ok = in && (unsigned)(hb[i] + g_r) < (unsigned)P.H && (unsigned)(wb[i] + g_s) < (unsigned)P.W;
        xa[i] = *(const u32x4 SK_GLOBAL *)(ok ? (uintptr_t)pa[i] + (uintptr_t)(tap_off * ES) : zeros);
      }
      g_c += KB;
      tap_off += KB;
      while (g_c >= P.Cin) {
        g_c -= P.Cin;
        if (++g_s == P.S) {
          g_s = 0;
          ++g_r;
          tap_off += next_filter_row;
        }
      }
    } else {
#pragma unroll
      for (int i = 0; i < A_ITERS; ++i)
        xa[i] = *(const u32x4 SK_GLOBAL *)(in ? (uintptr_t)pa[i] + (uintptr_t)((int64_t)k_load * ES) : zeros);
    }
#pragma unroll
    for (int i = 0; i < B_ITERS; ++i)
      xb[i] = *(const u32x4 SK_GLOBAL *)(in ? (uintptr_t)pb[i] + (uintptr_t)((int64_t)k_load * ES) : zeros);
    k_load += KB;
  };
  auto lstore = [&](int buf, const u32x4(&xa)[A_ITERS], const u32x4(&xb)[B_ITERS]) {
    unsigned char *a = lds + buf * STAGE + srow * LDS_ROW + c8 * 16;
    unsigned char *bb = a + BM * LDS_ROW;
#pragma unroll
    for (int i = 0; i < A_ITERS; ++i) *(u32x4 *)(a + 32 * i * LDS_ROW) = xa[i];
#pragma unroll
    for (int i = 0; i < B_ITERS; ++i) *(u32x4 *)(bb + 32 * i * LDS_ROW) = xb[i];
  };

  const int nstages = (k_stop - k_begin + KB - 1) / KB;
#pragma unroll
  for (int u = 0; u < NS - 1; ++u) gload(ra[u], rb[u]);
  lstore(0, ra[0], rb[0]);
  __syncthreads();
  int buf = 0;
  for (int s0 = 0; s0 < nstages; s0 += NS) {
#pragma unroll
    for (int u = 0; u < NS; ++u) {
      pf.at_step(s0 + u, nstages, CLAIM_LEAD, ISSUE_GAP);
      gload(ra[(u + NS - 1) % NS], rb[(u + NS - 1) % NS]);
      if (s0 + u < nstages) {
        // stage s0+u is in LDS buffer `buf`; put stage s0+u+1 (possibly past the end: zeros
        // times finite weights, never multiplied) into the other one while this one is used
        const unsigned char *la = lds + buf * STAGE;
        const unsigned char *lb = la + BM * LDS_ROW;
        // operand fragments of the first quarter of the stage are requested before the next
        // stage is written, those of quarter kk+1 before the MFMAs of quarter kk
        u32x4 fa[2][FM], fb[2][FN];
        auto frag = [&](int kk, u32x4(&xa)[FM], u32x4(&xb)[FN]) {
          const int piece = (2 * kk + half) * 16;
#pragma unroll
          for (int fm = 0; fm < FM; ++fm)
            xa[fm] = *(const u32x4 *)(la + ((wm * FM + fm) * 32 + l32) * LDS_ROW + piece);
#pragma unroll
          for (int fn = 0; fn < FN; ++fn)
            xb[fn] = *(const u32x4 *)(lb + ((wn * FN + fn) * 32 + l32) * LDS_ROW + piece);
        };
        frag(0, fa[0], fb[0]);
        lstore(buf ^ 1, ra[(u + 1) % NS], rb[(u + 1) % NS]);
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
          if (kk + 1 < 4) frag(kk + 1, fa[(kk + 1) & 1], fb[(kk + 1) & 1]);
#pragma unroll
          for (int fn = 0; fn < FN; ++fn)
#pragma unroll
            for (int fm = 0; fm < FM; ++fm) mma32<DT>(fb[kk & 1][fn], fa[kk & 1][fm], acc[fn][fm]);
        }
        __syncthreads();
        buf ^= 1;
      }
    }
  }

  finish_tile<DT, BM, BN, WAVES_M, WAVES_N>(P, T, sp, lds, s_flag, tid, acc);
}

// ---------------------------------------------------------------------------
// LDS tiles fed by direct global-to-LDS loads
// ---------------------------------------------------------------------------
// The operands are read through buffer descriptors:
//   * one descriptor per operand and tile, based at the tile's first row, its size the extent of
//     the tile's rows: a piece's address is a 32-bit row offset kept in a register for the whole
//     tile plus a scalar offset that advances with the stage, and a piece that lies outside the
//     descriptor reads as zero, so a piece that must not be read gets an offset of 2^31 and more (no sum of a
//     row's offset and a scalar offset reaches 2^31, so the two never wrap, and the scalar offset never exceeds the
//     descriptor's size);
//   * for a convolution whose channel count is a multiple of a stage (64 elements of 2 bytes),
//     all pieces of a stage lie under one filter tap: the tap and its offset are scalar, and
//     whether a row's pixel under that tap lies in the image is one bit of a mask that is
//     worked out once per tile and row.
// It serves operators whose tile extents fit 31 bits of byte offset and, for convolutions,
// those with such channel counts and at most 31 filter taps; the others keep run_tile.
constexpr int DMA_FRONT = 3072;  // the descriptors are based this far in front of the operand's first byte, see dma_stage
struct LeanOperands {
  uintptr_t baseA, baseB;  // first byte the offsets count from
  uint32_t extA, extB;     // bytes from there to the descriptors' ends
  int64_t originA;         // element offset of baseA from P.A
};

// Whether the tile can take the lean path, and its descriptors.  All scalar (P and T are uniform).
template <int ES>
__device__ __forceinline__ bool lean_operands(const DevProblem &P, const sk_tile &T, LeanOperands &L) {
  constexpr int CE = 16 / ES;
  constexpr int KB = 8 * CE;
  // (with DMA_FRONT added still below 2^31; the extents are compared with it by shifts, which are scalar: the 64-bit comparisons' constants
  // were kept in vector registers over the whole tile loop)
  constexpr int64_t LIMIT = ((int64_t)1 << 31) - 4096;
  const int64_t extB = ((int64_t)((int)T.n_len - 1) * P.ldb + P.Kg) * ES;
  L.baseB = (uintptr_t)P.B + (uintptr_t)((int64_t)T.n0 * P.ldb * ES);
  L.extB = (uint32_t)extB;
  if (!P.gather) {
    const int64_t extA = ((int64_t)((int)T.m_len - 1) * P.lda + P.Kg) * ES;
    L.originA = (int64_t)T.m0 * P.lda;
    L.extA = (uint32_t)extA;
    if ((uint64_t)(extA + 4096) >> 31) return false;
  } else {
    if (P.nchw || P.Cin % KB != 0 || P.R * P.S > 31) return false;
    // From the corner of the padded first image of the tile.  The scalar offset of a late tap can lie beyond the array's end
    // (a 3x3 filter on images of one pixel), so the descriptor is as large as an offset can be without the top
    // bit: what is read is inside because its tap is, and NOWHERE is outside whether the hardware compares the offset
    // alone, its sum with the scalar offset, or the offset with the size less the scalar offset.
    const int b0 = fast_div((int)T.m0, P.div_hw);
    const int b1 = fast_div((int)T.m0 + (int)T.m_len - 1, P.div_hw);
    L.originA = (((int64_t)b0 * P.H - P.pad_h) * P.W - P.pad_w) * P.Cin;
    L.extA = (uint32_t)(((int64_t)1 << 31) - DMA_FRONT);
    if (!offsets_below(P, b1 - b0, ES, LIMIT)) return false;
  }
  L.baseA = (uintptr_t)P.A + (uintptr_t)(L.originA * ES);
  return (uint64_t)(extB + 4096) >> 31 == 0;
}

// The operand pieces never pass through registers: a buffer load with the LDS modifier writes the 16
// bytes of lane i at (M0 + 16 i) of the LDS, 1 KB per wave and instruction, and a piece whose offset lies outside
// the descriptor arrives as zeros.
//   * LDS image of a stage: (BM + BN) rows of 128 bytes, no padding (a load instruction fills
//     eight consecutive rows); position p of row r holds the row's piece p ^ ((r >> 1) & 7), so
//     the 16 lanes that a fragment read serves together (rows r .. r+15, one piece) fall into
//     16 different groups of four banks.  The swizzle is applied on the global side: lane i of
//     a load asks for piece (i & 7) ^ swizzle(row of the lane).
//   * a ring of NS such images (as many as fit the kernel's LDS buffer); one barrier per stage, ahead of its last
//     step's MFMAs, says both "everyone's part of stage h+1 has landed" and "everyone has stage h's last fragments
//     in registers", so that stage h+NS may overwrite its image: NS-1 stages are in flight for most of a stage.
//   * the compiler does not see these loads (inline assembly; told about them it would wait for
//     all of them before every LDS read), so the waits are written out: loads complete in order,
//     hence "at most n outstanding" with n the loads of the stages issued later.  Loads and
//     stores of the surrounding code that are also in flight only make these waits, and the
//     compiler's own, wait for more than they need.
//   * the compiler does not look into inline assembly for the wait states the hardware wants between
//     instructions either.  Two matter here: a scalar register written by a vector instruction (the
//     compiler keeps spilled scalars in lanes of a vector register and fetches them with v_readlane
//     wherever it needs them, also right in front of these loads) must not be read by a memory
//     instruction in the next five cycles, and M0 not by an LDS-writing load in the cycle after it
//     was written.  So all loads of a stage sit in ONE statement that opens with the five cycles and
//     hands M0 back as it got it.
//   * with two waves per SIMD a wave's own instruction stream sets the pace of a stage as much as the MFMAs do (one
//     instruction every four cycles at best, the scalar ones included).  So a stage is kept to little more
//     than its MFMAs, fragment reads and loads: the loop is unrolled over the ring's slots (every LDS address is a register of
//     the tile plus a constant), the pieces a wave loads lie 1 KB apart in LDS and are told apart by the
//     instruction's own offset (which counts on both sides, so the lane's global offset is lowered by as
//     much and the descriptor based 3 KB in front), and positions advance by additions only.
//     (About 170 instructions a stage at first, of them 90 scalar, now about 90: 3x3 64-channel convolutions on 56x56 of 512
//     tenants 260 -> 245 us, sixteen 2048-cubed GEMMs 307 -> 302 us.)
// The wave's pieces: NA of activations from M0 on, NBW of weights from M0 + to_b on, each 1 KB after the one before; va and vb are
// offsets from the descriptors' bases (3072 bytes in front of the operand's first byte) less 1024 i.
template <int NA, int NBW>
__device__ __forceinline__ void dma_stage(__amdgpu_buffer_rsrc_t descA, __amdgpu_buffer_rsrc_t descB, const uint32_t (&va)[NA],
                                          const uint32_t (&vb)[NBW], uint32_t soffA, uint32_t soffB, uint32_t lds_addr, uint32_t to_b) {
  static_assert(NA == 4 && (NBW == 4 || NBW == 2), "written out for 128 rows of activations and 128 or 64 of weights");
  if constexpr (NBW == 4) {
    asm volatile("s_nop 4\n\t"
                 "buffer_load_dwordx4 %0, %8, %10 offen lds\n\t"
                 "buffer_load_dwordx4 %1, %8, %10 offen offset:1024 lds\n\t"
                 "buffer_load_dwordx4 %2, %8, %10 offen offset:2048 lds\n\t"
                 "buffer_load_dwordx4 %3, %8, %10 offen offset:3072 lds\n\t"
                 "s_add_u32 m0, m0, %12\n\ts_nop 0\n\t"
                 "buffer_load_dwordx4 %4, %9, %11 offen lds\n\t"
                 "buffer_load_dwordx4 %5, %9, %11 offen offset:1024 lds\n\t"
                 "buffer_load_dwordx4 %6, %9, %11 offen offset:2048 lds\n\t"
                 "buffer_load_dwordx4 %7, %9, %11 offen offset:3072 lds\n\t"
                 "s_sub_u32 m0, m0, %12"
                 :
                 : "v"(va[0]), "v"(va[1]), "v"(va[2]), "v"(va[3]), "v"(vb[0]), "v"(vb[1]), "v"(vb[2]), "v"(vb[3]), "s"(descA),
                   "s"(descB), "s"(soffA), "s"(soffB), "s"(to_b), "{m0}"(lds_addr)
                 : "memory", "scc");
  } else {
    asm volatile("s_nop 4\n\t"
                 "buffer_load_dwordx4 %0, %6, %8 offen lds\n\t"
                 "buffer_load_dwordx4 %1, %6, %8 offen offset:1024 lds\n\t"
                 "buffer_load_dwordx4 %2, %6, %8 offen offset:2048 lds\n\t"
                 "buffer_load_dwordx4 %3, %6, %8 offen offset:3072 lds\n\t"
                 "s_add_u32 m0, m0, %10\n\ts_nop 0\n\t"
                 "buffer_load_dwordx4 %4, %7, %9 offen lds\n\t"
                 "buffer_load_dwordx4 %5, %7, %9 offen offset:1024 lds\n\t"
                 "s_sub_u32 m0, m0, %10"
                 :
                 : "v"(va[0]), "v"(va[1]), "v"(va[2]), "v"(va[3]), "v"(vb[0]), "v"(vb[1]), "s"(descA), "s"(descB), "s"(soffA),
                   "s"(soffB), "s"(to_b), "{m0}"(lds_addr)
                 : "memory", "scc");
  }
}
template <int N>
__device__ __forceinline__ void wait_loads_but() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

template <int DT, int BM, int BN, bool GATHER, int LDS_BYTES>
__device__ __forceinline__ void run_tile_dma(const DevProblem &P, const sk_tile &T, const SplitK &sp, unsigned char *lds,
                                             uint32_t *s_flag, Prefetch &pf, const LeanOperands &L) {
  constexpr int ES = Elem<DT>::ES;
  constexpr int CE = 16 / ES;
  constexpr int KB = 8 * CE;                  // reduction elements per stage (128 bytes per row)
  constexpr int FM = BM / 64, FN = BN / 64;   // 32x32 blocks per wave along m and n (2 x 2 waves)
  constexpr int NA = BM / 32, NBW = BN / 32;  // load instructions per wave and stage: activations, weights
  constexpr int NPW = NA + NBW;
  constexpr int SLOT = (BM + BN) * 128;       // bytes of a stage in LDS
  constexpr int NS = LDS_BYTES / SLOT;        // ring slots
  constexpr uint32_t NOWHERE = 0x80000000u;   // an offset outside every descriptor: the piece arrives as zeros
  static_assert(NS == 2 || NS == 3, "waits below are written for two or three slots");
  static_assert(NPW < 32, "load counter");

  const int tid = pf.tid;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63;
  const int wm = wave & 1, wn = wave >> 1;
  const int l32 = lane & 31, half = lane >> 5;

  const int m0 = (int)T.m0, m_end = m0 + (int)T.m_len;
  const int k_begin = (int)T.k0, k_stop = (int)T.k0 + (int)T.k_len;

  const int nstages = (k_stop - k_begin + KB - 1) / KB;
  // A tile of few stages takes its next ticket at once: taken in its first stage, the answer (a memory round trip) and the record
  // behind it (another) would both be waited for at the tile's end (ResNet mix x16 85.7 -> 84.3 us).
  const int claim_at = nstages > CLAIM_LEAD ? nstages - CLAIM_LEAD : -1;
  if (claim_at < 0) pf.claim();

  constexpr uint32_t FRONT = DMA_FRONT;
  const __amdgpu_buffer_rsrc_t descA = __builtin_amdgcn_make_buffer_rsrc((void *)(L.baseA - FRONT), 0, (int)(L.extA + FRONT), 0x00020000);
  const __amdgpu_buffer_rsrc_t descB = __builtin_amdgcn_make_buffer_rsrc((void *)(L.baseB - FRONT), 0, (int)(L.extB + FRONT), 0x00020000);

  // load map: instruction i of this wave fills rows 8 (NA wave + i) .. + 7 of the operand's block (NBW for the weights);
  // this lane supplies position lane & 7 of row lane / 8 of these, which holds the logical piece c_log[i & 1]
  const int lrow = lane >> 3;
  const int c_log[2] = {(lane & 7) ^ (lane >> 4), (lane & 7) ^ (lane >> 4) ^ 4};
  // what is added to a row's byte offset for piece i
  auto piece_off = [&](int i) { return (uint32_t)c_log[i & 1] * 16u + FRONT - 1024u * (uint32_t)i; };
  uint32_t offA[NA];   // offset of this lane's piece of row i at reduction index 0 (tap (0,0), channel 0), as dma_stage wants it
  uint32_t tapsA[NA];  // convolution: top bit set if the row's pixel under the next stage's tap lies outside the image, then the later taps' bits
  if constexpr (!GATHER) {
    const uint32_t step = 8u * (uint32_t)((int)P.lda * ES) - 1024u;  // from one piece's row to the next, see dma_stage
    const int row = 8 * NA * wave + lrow;
    uint32_t off = (uint32_t)(row * ((int)P.lda * ES)) + FRONT;
#pragma unroll
    for (int i = 0; i < NA; ++i, off += step) {
      offA[i] = row + 8 * i < (int)T.m_len ? off + (uint32_t)c_log[i & 1] * 16u : NOWHERE;  // rows past the edge arrive as zeros; never stored
      tapsA[i] = 0;
    }
  } else {
    // Lane l works out row l of the wave's 8 NA rows (the lanes of a piece's row would all do the same divisions), then
    // every lane fetches those of its NA rows.
    static_assert(8 * NA <= 64, "one row per lane");
    const int g_hw = P.Ho * P.Wo, g_b0 = fast_div(m0, P.div_hw);
    uint32_t g_rows = 0;  // bit rr*S for every filter row rr
    for (int rr = 0; rr < P.R; ++rr) g_rows |= 1u << (rr * P.S);
    // Pixel (b, ho, wo) of the row; its offset from the descriptor's origin (the corner of the padded first
    // image of the tile) in 32 bits: lean_operands has checked that the tile's images lie within 2^31 bytes.
    const int m = m0 + 8 * NA * wave + (lane & (8 * NA - 1));
    const bool in = m < m_end;  // rows past the edge arrive as zeros; never stored
    const int mm = in ? m : m_end - 1;
    const int b = fast_div(mm, P.div_hw);
    const int rem = mm - b * g_hw;
    const int ho = fast_div(rem, P.div_wo);
    const int hs = ho * P.stride, ws = (rem - ho * P.Wo) * P.stride;  // row and column of tap (0,0) in the padded image
    const uint32_t off = (uint32_t)((((b - g_b0) * P.H + hs) * P.W + ws) * P.Cin * ES);
    // filter rows rr with 0 <= hb + rr < H form a range [lo, hi), and so do the filter columns; the
    // columns' bits times the bits rr*S of the rows in range is the mask of all taps in the image (no two
    // products overlap: the columns' bits lie below S; at most 31 taps)
    const int hb = hs - P.pad_h, wb = ws - P.pad_w;
    const int hlo = max(0, -hb), hhi = min(P.R, P.H - hb);
    const int wlo = max(0, -wb), whi = min(P.S, P.W - wb);
    const uint32_t wmk = whi > wlo ? ((1u << whi) - 1u) & ~((1u << wlo) - 1u) : 0u;
    const uint32_t rmk = hhi > hlo ? g_rows & ((1u << (hhi * P.S)) - 1u) & ~((1u << (hlo * P.S)) - 1u) : 0u;
    const uint32_t taps = __builtin_bitreverse32(~(in ? wmk * rmk : 0u));  // tap 0 in the top bit
#pragma unroll
    for (int i = 0; i < NA; ++i) {
      const int from = (8 * i + lrow) * 4;
      offA[i] = (uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)off) + piece_off(i);
      tapsA[i] = (uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)taps);
    }
  }
  uint32_t offB[NBW];
  {
    const uint32_t step = 8u * (uint32_t)((int)P.ldb * ES) - 1024u;
    const int row = 8 * NBW * wave + lrow;
    uint32_t off = (uint32_t)(row * ((int)P.ldb * ES)) + FRONT;
#pragma unroll
    for (int i = 0; i < NBW; ++i, off += step)
      offB[i] = row + 8 * i < (int)T.n_len ? off + (uint32_t)c_log[i & 1] * 16u : NOWHERE;
  }

  f32x16 acc[FN][FM];
#pragma unroll
  for (int fn = 0; fn < FN; ++fn)
#pragma unroll
    for (int fm = 0; fm < FM; ++fm)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[fn][fm][i] = 0.f;

  // scalar position of the next stage to load: reduction index k_next, byte offset from the rows' starts (weights) and
  // from the pixels under tap (0,0) (a convolution's image: consecutive channels and consecutive taps of a filter row follow
  // one another, the next filter row lies row_jump further); stages left under the tap, taps left in the filter row
  int k_next = k_begin;
  uint32_t soffB = (uint32_t)k_begin * ES, soffA = soffB;
  int left_c = 0, left_s = 0;
  const int stages_per_tap = GATHER ? P.Cin / KB : 1;
  const uint32_t row_jump = GATHER ? (uint32_t)((P.W - P.S) * P.Cin * ES) : 0u;
  if constexpr (GATHER) {
    const int tap = fast_div(k_begin, P.div_cin);
    const int t_c = k_begin - tap * P.Cin;
    const int t_r = fast_div(tap, P.div_s);
    const int t_s = tap - t_r * P.S;
    soffA = (uint32_t)(((t_r * P.W + t_s) * P.Cin + t_c) * ES);
    left_c = stages_per_tap - t_c / KB;
    left_s = P.S - t_s;
#pragma unroll
    for (int i = 0; i < NA; ++i) tapsA[i] <<= tap;
  }
  const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)lds;
  const uint32_t my_blocks = lds_base + (uint32_t)wave * (NA * 1024u);  // + slot*SLOT
  const uint32_t to_b = BM * 128 - (uint32_t)wave * ((NA - NBW) * 1024u);
  auto issue = [&](int slot) {
    const uint32_t dst = my_blocks + (uint32_t)slot * SLOT;
    uint32_t va[NA];
    if constexpr (GATHER) {
      // (no reduction tail: the reduction length is a multiple of the channel count, that of a stage)
#pragma unroll
      for (int i = 0; i < NA; ++i) va[i] = offA[i] | (tapsA[i] & NOWHERE);
      dma_stage<NA, NBW>(descA, descB, va, offB, soffA, soffB, dst, to_b);
      soffA += KB * ES;
      if (--left_c == 0) {
        left_c = stages_per_tap;
#pragma unroll
        for (int i = 0; i < NA; ++i) tapsA[i] <<= 1;
        if (--left_s == 0) {
          left_s = P.S;
          soffA += row_jump;
        }
      }
    } else {
      if (k_next + KB <= k_stop) {
        dma_stage<NA, NBW>(descA, descB, offA, offB, soffB, soffB, dst, to_b);
      } else {
        // last stage of a length that is not a multiple of a stage: pieces beyond the end of the reduction come from nowhere
        uint32_t vb[NBW];
#pragma unroll
        for (int i = 0; i < NA; ++i) va[i] = k_next + c_log[i & 1] * CE < k_stop ? offA[i] : NOWHERE;
#pragma unroll
        for (int i = 0; i < NBW; ++i) vb[i] = k_next + c_log[i & 1] * CE < k_stop ? offB[i] : NOWHERE;
        dma_stage<NA, NBW>(descA, descB, va, vb, soffB, soffB, dst, to_b);
      }
      k_next += KB;
    }
    soffB += KB * ES;
  };

  // fragment addresses inside a slot: row (w*F + f)*32 + l32, logical piece 2 kk + half at position
  // (2 kk + half) ^ swizzle(row), and swizzle(row) = (l32 >> 1) & 7 for every block of 32 rows
  int fragA[4], fragB[4];  // piece 2 kk + half of block 0's row, in slot 0
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) {
    const int at = l32 * 128 + (((2 * kk + half) ^ ((l32 >> 1) & 7)) << 4);
    fragA[kk] = wm * FM * 4096 + at;
    fragB[kk] = BM * 128 + wn * FN * 4096 + at;
  }

#ifdef SK_DIAG_CLOCKS
  const int diag_tile = pf.diag_tile;
#endif
  SK_DIAG(1);
  // the fragments of step kk of the stage in slot sl
  u32x4 fa[2][FM], fb[2][FN];
  auto frag = [&](int sl, int kk, u32x4(&xa)[FM], u32x4(&xb)[FN]) {
#pragma unroll
    for (int fm = 0; fm < FM; ++fm) xa[fm] = *(const u32x4 *)(lds + fragA[kk] + (sl * SLOT + fm * 4096));
#pragma unroll
    for (int fn = 0; fn < FN; ++fn) xb[fn] = *(const u32x4 *)(lds + fragB[kk] + (sl * SLOT + fn * 4096));
  };
  auto multiply = [&](const u32x4(&xa)[FM], const u32x4(&xb)[FN]) {
#pragma unroll
    for (int fn = 0; fn < FN; ++fn)
#pragma unroll
      for (int fm = 0; fm < FM; ++fm) mma32<DT>(xb[fn], xa[fm], acc[fn][fm]);
  };
  // (the previous tile's readers of this LDS buffer have passed the barrier at the end of their tile)
#pragma unroll
  for (int u = 0; u < NS; ++u)
    if (u < nstages) issue(u);
  if (nstages >= NS)
    wait_loads_but<(NS - 1) * NPW>();
  else
    wait_loads_but<0>();
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  frag(0, 0, fa[0], fb[0]);
  const int issue_at = claim_at < 0 ? 0 : claim_at + ISSUE_GAP;
  for (int h0 = 0; h0 < nstages; h0 += NS) {
    if (claim_at >= h0 && claim_at < h0 + NS) pf.claim();
    if ((unsigned)(issue_at - h0) < (unsigned)NS) pf.issue();
#pragma unroll
    for (int slot = 0; slot < NS; ++slot) {
      const int h = h0 + slot;
      if (h < nstages) {
        // The fragments of step kk+1 are requested before the MFMAs of step kk (the scheduler is held to
        // that order: left alone it sinks every read to just above its first use).  Requesting all four
        // steps' fragments at the start of the stage was measured slower: the waves of a workgroup leave
        // the barrier together, and their reads then queue at the LDS.
#pragma unroll
        for (int kk = 0; kk < 3; ++kk) {
          frag(slot, kk + 1, fa[(kk + 1) & 1], fb[(kk + 1) & 1]);
          __builtin_amdgcn_sched_barrier(0);
          multiply(fa[kk & 1], fb[kk & 1]);
          __builtin_amdgcn_sched_barrier(0);
        }
        // The stages change hands ahead of the last step's MFMAs, not behind them: its fragments are in registers
        // (so this stage's slot is free once everyone has got here) and stage h+1 has landed, so the barrier, the
        // loads of stage h+NS and the first fragments of stage h+1 all run beside the MFMAs.
        if (h + 1 < nstages) {
          // this wave's loads of stage h+1 have landed: the only ones issued after them are those of the NS - 2 stages behind it
          if (NS > 2 && h + NS - 1 < nstages)
            asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((NS - 2) * NPW) : "memory");
          else
            asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
          __builtin_amdgcn_s_barrier();
          asm volatile("" ::: "memory");
          if (h + NS < nstages) issue(slot);
          __builtin_amdgcn_sched_barrier(0);
          frag(slot + 1 == NS ? 0 : slot + 1, 0, fa[0], fb[0]);
        }
        __builtin_amdgcn_sched_barrier(0);
        multiply(fa[1], fb[1]);
        __builtin_amdgcn_sched_barrier(0);
        if (h == 0) SK_DIAG(2);
      }
    }
  }
  SK_DIAG(3);
  __syncthreads();  // everyone is done with the last stage before the output tile is staged in the same LDS
  // (read again: kept through the stages, what the outputs need of the record cost the loop its scalar registers)
  const TileWork again = load_record(pf.rec);
  finish_tile<DT, BM, BN, 2, 2>(again.prob, again.tile, sp, lds, s_flag, tid, acc);
  SK_DIAG(4);
}

// One LDS tile: the lean path where the operator allows it.
template <int DT, int BM, int BN, bool NARROW>
__device__ __forceinline__ void run_lds_tile(const DevProblem &P, const sk_tile &T, const SplitK &sp, unsigned char *lds,
                                             uint32_t *s_flag, Prefetch &pf) {
  constexpr int BYTES = NARROW ? NARROW_LDS_BYTES : LDS_TILE_BYTES;
  LeanOperands L;
  if (lean_operands<Elem<DT>::ES>(P, T, L)) {
    if (P.gather)
      run_tile_dma<DT, BM, BN, true, BYTES>(P, T, sp, lds, s_flag, pf, L);
    else
      run_tile_dma<DT, BM, BN, false, BYTES>(P, T, sp, lds, s_flag, pf, L);
    return;
  }
  // (the host lets only operators into a narrow plan for which every tile is lean)
  if constexpr (!NARROW) run_tile<DT, BM, BN, 2, 2>(P, T, sp, lds, s_flag, pf);
}

// ---------------------------------------------------------------------------
// 3x3 convolutions of 64 channels with their weights in registers
// ---------------------------------------------------------------------------
// Size-keeping 3x3 NHWC convolutions of 64 channels (16-bit: a pixel is one 128-byte row) into at most 64.  As tiles they spend
// most on bringing every pixel nine times, and the same weights for every tile, from the L2 into LDS and from LDS into registers, with a
// barrier per 24 KB, and on the tiles' ends.  Here a record is a run of an operator's output pixels (window_records), and:
//   * a wave makes 64 pixels x 32 channels at a time and holds its 32 x 576 weights in 144 registers for the whole record;
//   * pixels pass through a ring of three blocks of 128 in LDS, each read once; the nine taps are nine places in
//     the ring (a tap outside the image reads a row of zeros instead: one bit per pixel and tap);
//   * one barrier per 128 pixels (72 MFMAs a wave): the block read next has landed, the one before last is free;
//   * a step's outputs are staged in LDS and stored at the next step's top, so that the wait there is for loads and stores a
//     whole step old; in large plans past the caches, which leaves room there for the pixels (2 to 5 %).  As whole lines of 64
//     channels, out of two waves each (and a barrier in a step's middle, so that their place is free by its end): half lines, a wave's
//     own, made 258 MB of the 206 written to memory (131.7 -> 124.4 us).
// The sums are taken in the tiles' order: the same bits.
// 512 tenants of 56x56, 64 to 64 (0.45 GB, 118 GFLOP), every launch on other operands: 214 to 230 us in the kernel for tiles
// alone, 124 here: 3.6 TB/s of operands and outputs against the 4.8 of a large copy.  (Of 130, with half lines stored and operands the same every
// time, it took 107 without its MFMAs, 120 without its fragment reads, 112 without storing the outputs.)  Bound by memory, with the MFMAs (46 % of the SIMD cycles by SQ_VALU_MFMA_BUSY_CYCLES) not quite beside it.  Fragments two or three steps ahead measure the same.
constexpr int WIN_BLOCK = 128;                          // pixels per step and ring block
constexpr int WIN_RING = 3 * WIN_BLOCK;                 // pixels in the ring
constexpr int WIN_OROW = 144;                              // bytes of a pixel's outputs in LDS, padded
constexpr int WIN_OUT = WIN_RING * 128;                    // where a step's outputs are staged
constexpr int WIN_ZERO = WIN_OUT + WIN_BLOCK * WIN_OROW;   // the row of zeros
static_assert(WIN_ZERO + 128 <= LDS_TILE_BYTES, "the ring, the outputs and the row of zeros do not fit the LDS buffer");
static_assert(WIN_ZERO % 128 == 0, "places in the row of zeros are told apart by the low seven bits");

// Four times 8 pixels side by side, of a wave, to LDS: lane i brings 16 bytes of pixel i / 8.
__device__ __forceinline__ void dma_pixels(__amdgpu_buffer_rsrc_t desc, uint32_t v0, uint32_t v1, uint32_t v2, uint32_t v3, uint32_t lds_addr) {
  // (the instruction's own offset counts in memory and in LDS; for the wait states see dma_stage)
  asm volatile("s_nop 4\n\t"
               "buffer_load_dwordx4 %0, %4, 0 offen lds\n\t"
               "buffer_load_dwordx4 %1, %4, 0 offen offset:1024 lds\n\t"
               "buffer_load_dwordx4 %2, %4, 0 offen offset:2048 lds\n\t"
               "buffer_load_dwordx4 %3, %4, 0 offen offset:3072 lds"
               :
               : "v"(v0), "v"(v1), "v"(v2), "v"(v3), "s"(desc), "{m0}"(lds_addr)
               : "memory");
}

template <int DT>
__device__ __forceinline__ void run_window(const DevProblem &P, const sk_tile &T, unsigned char *lds, Prefetch &pf) {
  constexpr uint32_t NOWHERE = 0x80000000u;
  const int tid = pf.tid;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int wm = wave & 1, wn = wave >> 1, l32 = lane & 31, half = lane >> 5;
  const int m0 = (int)T.m0, m_len = (int)T.m_len;
  const int steps = (m_len + WIN_BLOCK - 1) / WIN_BLOCK;
  const int halo = P.W + 1;  // ring pixel 0 is output pixel m0's tap (0, 0)
  const int pixels = m_len + 2 * halo;  // that any tap of the record names

  // ---- the ring's blocks: pixels m0 - halo + 128 b + (0 .. 127); outside the operand: zeros ----
  const int64_t first = (int64_t)m0 - halo;
  const int64_t have = (int64_t)P.Mg - first;  // (a size-keeping convolution has as many pixels as outputs)
  const __amdgpu_buffer_rsrc_t desc = __builtin_amdgcn_make_buffer_rsrc(
      (void *)((uintptr_t)P.A + (uintptr_t)(first * 128)), 0, (int)((have < pixels ? have : (int64_t)pixels) * 128), 0x00020000);
  const int before = first < 0 ? (int)-first : 0;  // pixels of block 0 in front of the operand (at most halo)
  const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)lds;
  // (what only a step's ends need is worked out there, from a copy of the lane index the compiler cannot see through: kept over the
  // MFMAs beside the weights it would not fit the registers)
  auto lane_again = [&]() {
    int l = lane;
    asm volatile("" : "+v"(l));
    return l;
  };
  // instruction i of this wave: pixels 32 wave + 8 i + lane / 8 of the block; position p of ring row r holds piece p ^ ((r >> 1) & 7)
  auto load_block = [&](int b, int slot) {
    const int l = lane_again(), row = 32 * wave + (l >> 3);
    const uint32_t at = (uint32_t)(b * WIN_BLOCK + row) * 128u, piece = (uint32_t)((l & 7) ^ (l >> 4)) * 16u;
    uint32_t v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = b == 0 && row + 8 * i < before ? NOWHERE : at + (piece ^ (uint32_t)(i & 1) * 64u);
    dma_pixels(desc, v[0], v[1], v[2], v[3], lds_base + (uint32_t)slot * (WIN_BLOCK * 128u) + (uint32_t)wave * 4096u);
  };
  const int blocks = (pixels + WIN_BLOCK - 1) / WIN_BLOCK;
#ifdef SK_DIAG_CLOCKS
  const int diag_tile = pf.diag_tile;
#endif
  SK_DIAG(1);
  if (tid < 8) ((u32x4 *)(lds + WIN_ZERO))[tid] = u32x4{0u, 0u, 0u, 0u};
  load_block(0, 0);
  if (blocks > 1) load_block(1, 1);

  // ---- the weights: piece 2 kk + half of tap t of this lane's output channel ----
  u32x4 w[9][4];
  {
    int n = 32 * wn + l32;
    if (n >= P.Ng) n = P.Ng - 1;  // (never stored)
    const u32x4 SK_GLOBAL *src = as_global<u32x4>((const void *)((uintptr_t)P.B + (uintptr_t)n * (576 * 2))) + half;
#pragma unroll
    for (int t = 0; t < 9; ++t)
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) w[t][kk] = src[t * 8 + 2 * kk];
  }

  __builtin_amdgcn_s_waitcnt(0);  // (the builtin: the compiler, too, takes the weights as arrived and waits for nothing in the loop)

  unsigned char *const out = lds + WIN_OUT;
  const __amdgpu_buffer_rsrc_t descC = __builtin_amdgcn_make_buffer_rsrc(
      (void *)((uintptr_t)P.C + (uintptr_t)((int64_t)m0 * P.Ng * 2)), 0, m_len * P.Ng * 2, 0x00020000);
  // a step's outputs: this wave's 32 pixels, whole lines of 64 channels (pixels past the record's end lie outside the descriptor)
  auto store_step = [&](int i) {
    const int l = lane_again(), r = 32 * wave + (l >> 3), n = (l & 7) * 8;
    u32x4 v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = *(const u32x4 *)(out + (r + 8 * q) * WIN_OROW + n * 2);
    const uint32_t at = n < P.Ng ? (uint32_t)(((i * WIN_BLOCK + r) * P.Ng + n) * 2) : NOWHERE;
    store_out(v, descC, at, (uint32_t)(8 * P.Ng * 2), (P.flags & FLAG_PAST_CACHES) != 0);
  };

  // this lane's two pixels of a step, counted within their image, and how far these move from one step to the next
  const int hw = P.Ho * P.Wo;
  int rem[2];
#pragma unroll
  for (int f = 0; f < 2; ++f) {
    const int m = m0 + 64 * wm + 32 * f + l32;
    rem[f] = m - fast_div(m, P.div_hw) * hw;
  }
  const int by = WIN_BLOCK - fast_div(WIN_BLOCK, P.div_hw) * hw;

  int slot = 0;  // of block i, and with it the ring row of step i's first pixel under tap (0, 0), over 128
  for (int i = 0; i < steps; ++i) {
    // blocks i and i + 1 have landed (all that this wave has in flight was asked for a step ago), block i - 1's readers are done
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if (i + 2 < blocks) load_block(i + 2, slot == 0 ? 2 : slot - 1);
    if (i > 0) store_step(i - 1);
    if (i == steps - 2 || steps == 1) pf.claim();
    if (i == steps - 1) pf.issue();
    // ring row under tap (0, 0), times 128; bit t of `taps`: tap t lies in the image
    uint32_t row128[2], taps[2];
#pragma unroll
    for (int f = 0; f < 2; ++f) {
      const uint32_t r = (uint32_t)(slot * WIN_BLOCK + 64 * wm + 32 * f + l32);
      row128[f] = r << 7;
      const int ho = fast_div(rem[f], P.div_wo), wo = rem[f] - ho * P.Wo;
      const uint32_t rows = 0x038u | (ho > 0 ? 0x007u : 0u) | (ho + 1 < P.Ho ? 0x1c0u : 0u);
      const uint32_t cols = 0x092u | (wo > 0 ? 0x049u : 0u) | (wo + 1 < P.Wo ? 0x124u : 0u);
      taps[f] = rows & cols;
      rem[f] += by;
      if (rem[f] >= hw) rem[f] -= hw;
    }
    f32x16 acc[2];
#pragma unroll
    for (int f = 0; f < 2; ++f)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[f][e] = 0.f;
    // Where piece `half` of the lane's pixel f lies under tap t; piece 2 kk + half: with bits 5 and 6 turned over by kk.  (The ring's
    // length is a multiple of 16 rows: going round does not change the swizzle.)
    auto place = [&](int t, int f) {
      const uint32_t straight = row128[f] + ((uint32_t)((t / 3) * P.W + t % 3) << 7);
      const uint32_t at = min(straight, straight - WIN_RING * 128u) | ((straight >> 4) & 0x70u);
      const uint32_t in = (uint32_t)((int)(taps[f] << (31 - t)) >> 31);
      return ((at & in) | (WIN_ZERO & ~in)) ^ (uint32_t)(half * 16);
    };
    constexpr int AHEAD = 2;  // fragments asked for ahead of their MFMAs, in steps of 16 channels
    u32x4 x[AHEAD + 1][2];
    uint32_t at[2][2];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int f = 0; f < 2; ++f) at[t][f] = place(t, f);
#pragma unroll
    for (int z = 0; z < AHEAD; ++z)
#pragma unroll
      for (int f = 0; f < 2; ++f) x[z][f] = *(const u32x4 *)(lds + (at[z >> 2][f] ^ (uint32_t)((z & 3) << 5)));
#pragma unroll
    for (int z = 0; z < 36; ++z) {
      const int y = z + AHEAD, t = y >> 2, kk = y & 3;
      __builtin_amdgcn_sched_barrier(0);
      if (y < 36) {
#pragma unroll
        for (int f = 0; f < 2; ++f) {
          x[y % (AHEAD + 1)][f] = *(const u32x4 *)(lds + (at[t & 1][f] ^ (uint32_t)(kk << 5)));
          // (places of the tap after the next, as soon as this one's are done with)
          if (kk == 3 && t + 2 < 9) at[t & 1][f] = place(t + 2, f);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int f = 0; f < 2; ++f) mma32<DT>(w[z >> 2][z & 3], x[z % (AHEAD + 1)][f], acc[f]);
      if (z == 17) __builtin_amdgcn_s_barrier();  // every wave has stored its part of the step before: its place is free
    }
    // lane holds, per f: pixel l32, channels 8 j + 4 half + (0 .. 3)
#pragma unroll
    for (int f = 0; f < 2; ++f)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        u32x2 o;
        o.x = cvt_pack<DT>(acc[f][4 * j], acc[f][4 * j + 1]);
        o.y = cvt_pack<DT>(acc[f][4 * j + 2], acc[f][4 * j + 3]);
        const int l = lane_again();
        *(u32x2 *)(out + (64 * wm + 32 * f + (l & 31)) * WIN_OROW + (32 * wn + 8 * j + 4 * (l >> 5)) * 2) = o;
      }
    slot = slot == 2 ? 0 : slot + 1;
    if (i == 0) SK_DIAG(2);
  }
  SK_DIAG(3);
  __syncthreads();
  store_step(steps - 1);
  SK_DIAG(4);
}

// ---------------------------------------------------------------------------
// dispatch and the persistent shell
// ---------------------------------------------------------------------------
// ---------------------------------------------------------------------------
// generic tiles: operands that cannot be read in aligned 16-byte pieces
// (odd K, odd Cin, unaligned pointers or strides).  One output per thread and
// trip, plain fp32 multiply-adds in ascending k.  Correct for everything, fast
// for nothing; used for rectangles with next to no work.
// ---------------------------------------------------------------------------
// (Inlined, like every path of the kernel: as real calls the two slow paths gave the kernel a stack,
// and how well its fast paths then ran changed from build to build.  They exist only in the kernel
// instantiations for plans with such operands: about twice the code.  They
// are given the records' addresses in memory rather than references to the caller's copies, and the
// tile's own copy of the thread index (see the tile loop): taken from threadIdx, what run_tile_any derives from it was
// hoisted out of the tile loop and cost these kernels 1 to 18 spilled vector registers and a stack.)
template <int DT>
__device__ __forceinline__ void run_generic(const DevProblem *P_mem, const sk_tile *T_mem, int tid) {
  const DevProblem P = *P_mem;
  const sk_tile T = *T_mem;
  const int m_len = T.m_len, n_len = T.n_len;
  // a split reduction is done whole by the record of its first slice; the others have nothing to do
  if (T.ks_idx != 0) return;
  for (int idx = tid; idx < m_len * n_len; idx += WG_THREADS) {
    const int m = (int)T.m0 + idx / n_len;
    const int n = (int)T.n0 + idx % n_len;
    const RowA row = row_of(P, m);
    const int64_t wrow = (int64_t)n * P.ldb;
    float acc = 0.f;
    if (!P.gather) {
      for (int k = 0; k < P.Kg; ++k)
        acc = __builtin_fmaf(load_elem<DT>(P.A, row.base + k), load_elem<DT>(P.B, wrow + k), acc);
    } else if (!P.nchw) {
      // taps in the order of the reduction index; those in the padding contribute nothing
      for (int r = 0; r < P.R; ++r) {
        if ((unsigned)(row.hb + r) >= (unsigned)P.H) continue;
        for (int t = 0; t < P.S; ++t) {
          if ((unsigned)(row.wb + t) >= (unsigned)P.W) continue;
          const int64_t xa = row.base + ((int64_t)r * P.W + t) * P.Cin;
          const int64_t wb = wrow + (int64_t)(r * P.S + t) * P.Cin;
          for (int c = 0; c < P.Cin; ++c)
            acc = __builtin_fmaf(load_elem<DT>(P.A, xa + c), load_elem<DT>(P.B, wb + c), acc);
        }
      }
    } else {
      // channel-major: reduction index (c*R + r)*S + t
      const int64_t plane = (int64_t)P.H * P.W;
      for (int c = 0; c < P.Cin; ++c)
        for (int r = 0; r < P.R; ++r) {
          if ((unsigned)(row.hb + r) >= (unsigned)P.H) continue;
          for (int t = 0; t < P.S; ++t) {
            if ((unsigned)(row.wb + t) >= (unsigned)P.W) continue;
            acc = __builtin_fmaf(load_elem<DT>(P.A, row.base + c * plane + (int64_t)r * P.W + t),
                                 load_elem<DT>(P.B, wrow + ((int64_t)c * P.R + r) * P.S + t), acc);
          }
        }
    }
    const int64_t c_off = P.nchw ? nchw_out_base(P, m) + (int64_t)n * P.Ho * P.Wo : (int64_t)m * P.ldc + n;
    store_elem<DT>(P.C, c_off, acc);
  }
}

// ---------------------------------------------------------------------------
// MFMA tiles for operands of any alignment (an image with 3 channels, an odd
// reduction length, unaligned bases) and for channel-major images
// ---------------------------------------------------------------------------
// The LDS image, fragments and MFMAs of run_tile; any output rectangle is walked in blocks of 128 x 128, and
// the slices of a split reduction (always a single block) meet in the workspace like those of the other classes.
// What a stage costs here is getting its 256 rows of 128 bytes into LDS, so:
//   * the hardware reads 16 bytes from any element's address in one instruction.  A reduction is taken as runs
//     of contiguous elements (a GEMM row; for an NHWC convolution the S * Cin elements under one filter row),
//     each padded to whole 16-byte pieces.  A piece that reaches beyond the run, or beyond the part of it that
//     lies in the image, is read from the nearest place inside and shifted, with zeros behind it.
//   * a channel-major image has no contiguous runs along the reduction.  There (where run_tile_planes does not serve it) the lanes of a wave take
//     64 consecutive pixels under one reduction index (channel and tap are scalar; whether a pixel's tap lies in
//     the image is one bit each of a row and a column mask), so a load of single elements is one
//     coalesced access and costs three vector instructions beside it.  The block is computed transposed (output
//     channels as MFMA rows), so that a lane ends up with consecutive pixels of one channel plane.
//   * the loads of a stage are in flight while the one before it is multiplied (two LDS images).
//   * blocks of 64 rows or columns where the record has no more, and where the device's work list cuts long records
//     (refine_tiles): a tile of 51 fp32 stages takes 225 us by itself at 128 x 128.
// Bound by the vector instructions that place a stage's pieces (addresses, shifts, packing of single elements) on
// two waves per SIMD, not by memory.  Measured before / after, against pieces put together element by element with
// one stage at a time and no loads in flight beside the MFMAs: seven stride-2 layers with the 7x7 stem for
// sixteen tenants 167 -> 126 us, the channel-major ResNet layers for eight 208 -> 162 us, 96 operators of odd sizes in
// three types 306 -> 232 us.

// Whether both operands hold at least 16 bytes.  (Channel-major images are read element by element.)
template <int ES>
__device__ __forceinline__ bool holds_a_piece(const DevProblem &P) {
  constexpr int CE = 16 / ES;
  const int64_t a = P.gather ? (int64_t)P.H * P.W * P.Cin : (int64_t)(P.Mg - 1) * P.lda + P.Kg;
  return (P.nchw || a >= CE) && (int64_t)(P.Ng - 1) * P.ldb + P.Kg >= CE;
}

// A slice of a split reduction of run_tile_any or run_tile_planes (see below) hands its partial sums over; true in the workgroup that
// arrived last, with the sum of all slices in `acc`.
template <bool NCHW, int FM, int FN>
__device__ __forceinline__ bool any_handover(const sk_tile &T, const SplitK &sp, unsigned char *lds, uint32_t *s_flag, int tid,
                                             f32x16 (&acc)[FN][FM]) {
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int wm = wave & 1, wn = wave >> 1;
  const int l32 = lane & 31, half = lane >> 5;
  // A slice of a split reduction (such a rectangle is a single block here: at most 128 x 128, or
  // 16, 32 or 64 rows x 128 columns in the skinny classes).  Partial sums go to the rectangle's
  // workspace, which holds per slice `rows` x 128 (64 for the 64-column class) floats, as 16-byte
  // pieces indexed by (quad of consecutive outputs, MFMA row); the last slice to arrive adds
  // all of them in slice order and stores the result.  Same hand-over as in run_tile.
  // The accumulator quads of a thread wait in LDS meanwhile (free by now: the last stage
  // ended with a barrier; a slot per thread and quad), so that the loops below can run rolled up:
  // unrolled over the accumulators they cost this kernel forty registers it does not have.
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  static_assert(FN * FM * 4 * WG_THREADS * 16 <= LDS_TILE_BYTES, "the accumulators do not fit the LDS buffer");
  f32x4 *slot = (f32x4 *)lds + tid;  // quad p of this thread: slot[p * WG_THREADS]
#pragma unroll
  for (int fn = 0; fn < FN; ++fn)
#pragma unroll
    for (int fm = 0; fm < FM; ++fm)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        slot[((fn * FM + fm) * 4 + q) * WG_THREADS] =
            f32x4{acc[fn][fm][4 * q], acc[fn][fm][4 * q + 1], acc[fn][fm][4 * q + 2], acc[fn][fm][4 * q + 3]};
  const int rows = T.cls >= CLS_TILE_128x128 ? 128 : 16 << (T.cls / 3);
  const int cols = T.cls == CLS_TILE_128x64 ? 64 : 128;
  const int lrows = NCHW ? cols : rows, quads = (NCHW ? rows : cols) / 4;
  const size_t per_slice = (size_t)lrows * quads;  // f32x4 units
  unsigned long long *mine = (unsigned long long *)(sp.ws + sp.ws_off[T.out_tile_id]);
  // where quad p = (fn*FM + fm)*4 + q of this thread lies in slice 0, or null if outside the rectangle's rows / columns
  auto place = [&](int p) -> unsigned long long * {
    const int fn = p / (4 * FM), fm = (p >> 2) % FM, q = p & 3;
    const int r = (wm * FM + fm) * 32 + l32, g = (wn * FN + fn) * 8 + q * 2 + half;
    if (r >= lrows || g >= quads) return nullptr;
    return mine + 2 * ((size_t)g * lrows + r);
  };
#pragma unroll 1
  for (int p = 0; p < FN * FM * 4; ++p) {
    unsigned long long *q = place(p);
    if (q) {
      q += 2 * (size_t)T.ks_idx * per_slice;
      const f32x4 v = slot[p * WG_THREADS];
      __hip_atomic_store(q, __builtin_bit_cast(unsigned long long, f32x2{v.x, v.y}), __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(q + 1, __builtin_bit_cast(unsigned long long, f32x2{v.z, v.w}), __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
    }
  }
  __builtin_amdgcn_s_waitcnt(0);  // all counters to zero: the stores above have completed
  __syncthreads();
  if (tid == 0)
    *s_flag = __hip_atomic_fetch_add(&sp.arrive[T.out_tile_id], 1u, SK_ARRIVE_ORDER, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  if (*s_flag != (uint32_t)T.S - 1) return false;
  // Four quads at a time: their partial sums of a slice are requested together (one by one, each quad and slice was a memory round trip).  Quads
  // outside the rectangle read its first one.
  constexpr int TOGETHER = 4;
#pragma unroll 1
  for (int p0 = 0; p0 < FN * FM * 4; p0 += TOGETHER) {
    unsigned long long *q[TOGETHER];
    f32x4 sum[TOGETHER];
#pragma unroll
    for (int u = 0; u < TOGETHER; ++u) {
      q[u] = place(p0 + u);
      if (!q[u]) q[u] = mine;
      sum[u] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll 1
    for (int s2 = 0; s2 < T.S; ++s2) {
      unsigned long long part[TOGETHER][2];
#pragma unroll
      for (int u = 0; u < TOGETHER; ++u) {
        part[u][0] = __hip_atomic_load(q[u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        part[u][1] = __hip_atomic_load(q[u] + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        q[u] += 2 * per_slice;
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < TOGETHER; ++u) {
        const f32x2 lo = __builtin_bit_cast(f32x2, part[u][0]), hi = __builtin_bit_cast(f32x2, part[u][1]);
        sum[u] += f32x4{lo.x, lo.y, hi.x, hi.y};
      }
    }
#pragma unroll
    for (int u = 0; u < TOGETHER; ++u) slot[(p0 + u) * WG_THREADS] = sum[u];
  }
  if (tid == 0)  // re-arm for the next launch
    __hip_atomic_store(&sp.arrive[T.out_tile_id], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
  for (int fn = 0; fn < FN; ++fn)
#pragma unroll
    for (int fm = 0; fm < FM; ++fm)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const f32x4 v = slot[((fn * FM + fm) * 4 + q) * WG_THREADS];
        acc[fn][fm][4 * q] = v.x;
        acc[fn][fm][4 * q + 1] = v.y;
        acc[fn][fm][4 * q + 2] = v.z;
        acc[fn][fm][4 * q + 3] = v.w;
      }
  __syncthreads();  // the slots have been read: the outputs are staged in the same LDS next
  return true;
}

// Outputs of a block of run_tile_any, run_tile_planes or run_tile_rows (rows mb .., columns nb ..): through LDS, so that they leave as runs of consecutive places.
// (WM waves side by side along the rows, 4 / WM along the columns.)
template <int DT, bool NCHW, int ROWS, int COLS, int WM>
__device__ __forceinline__ void any_outputs(const DevProblem *P_mem, const sk_tile *T_mem, int mb, int nb, unsigned char *lds, int tid,
                                            f32x16 (&acc)[COLS * WM / 128][ROWS / (32 * WM)]) {
  constexpr int ES = Elem<DT>::ES;
  constexpr int CE = 16 / ES;
  constexpr int FM = ROWS / (32 * WM), FN = COLS * WM / 128;
  using elem_t = typename std::conditional<ES == 4, uint32_t, uint16_t>::type;
  typedef elem_t piece_t __attribute__((ext_vector_type(CE)));
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int wm = wave % WM, wn = wave / WM;
  const int l32 = lane & 31, half = lane >> 5;
  // (the record is read again: kept through the stages, what the outputs need of it costs the mixed-type kernel a quarter
  // more spilled scalars)
  const DevProblem P = load_record(P_mem);
  const sk_tile T = load_record(T_mem);
  const int m_end = (int)T.m0 + (int)T.m_len, n_end = (int)T.n0 + (int)T.n_len, hw = P.Ho * P.Wo;
  // lane holds, per (fn, fm): MFMA row l32, columns 8*(i/4) + 4*half + (i%4)
  constexpr int OROW = COLS * ES + 16;
  static_assert(ROWS * OROW <= LDS_TILE_BYTES, "output tile does not fit the LDS buffer");
#pragma unroll
  for (int fm = 0; fm < FM; ++fm)
#pragma unroll
    for (int fn = 0; fn < FN; ++fn)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        unsigned char *d = lds + ((wm * FM + fm) * 32 + l32) * OROW + ((wn * FN + fn) * 32 + 8 * q + 4 * half) * ES;
        if constexpr (ES == 4) {
          *(f32x4 *)d = f32x4{acc[fn][fm][4 * q], acc[fn][fm][4 * q + 1], acc[fn][fm][4 * q + 2], acc[fn][fm][4 * q + 3]};
        } else {
          u32x2 o;
          o.x = cvt_pack<DT>(acc[fn][fm][4 * q], acc[fn][fm][4 * q + 1]);
          o.y = cvt_pack<DT>(acc[fn][fm][4 * q + 2], acc[fn][fm][4 * q + 3]);
          *(u32x2 *)d = o;
        }
      }
  __syncthreads();
  constexpr int PIECES = COLS / CE, RPI = WG_THREADS / PIECES;
  const int col = (tid % PIECES) * CE;
  const int row_end = NCHW ? n_end - nb : m_end - mb, col_end = NCHW ? m_end - mb : n_end - nb;
  // NCHW: the piece's pixels (its first one, and whether they lie in one image)
  int64_t pixel0 = 0;
  bool whole = col + CE <= col_end;
  if constexpr (NCHW) {
    if (col < col_end) {
      pixel0 = nchw_out_base(P, mb + col);
      whole = whole && nchw_out_base(P, mb + col + CE - 1) == pixel0 + CE - 1;
    }
  }
  // (the rule for the caches outside the loop: beside each store it cost stride-2 layers x4 to x16 1 to 2 %)
  auto store_rows = [&](auto past_caches) {
#pragma unroll 1
    for (int r = tid / PIECES; r < row_end && r < ROWS; r += RPI) {
      if (col >= col_end) break;
      const u32x4 v = *(const u32x4 *)(lds + r * OROW + col * ES);
      if (whole) {
        const int64_t o = NCHW ? pixel0 + (int64_t)(nb + r) * hw : (int64_t)(mb + r) * P.ldc + nb + col;
        u32x4_any SK_GLOBAL *const dst = (u32x4_any SK_GLOBAL *)((uintptr_t)P.C + (uintptr_t)(o * ES));
        if constexpr (decltype(past_caches)::value)
          __builtin_nontemporal_store(v, dst);
        else
          *dst = v;
      } else {
        const piece_t ev = __builtin_bit_cast(piece_t, v);
#pragma unroll
        for (int e = 0; e < CE; ++e)
          if (col + e < col_end) {
            const int64_t o = NCHW ? nchw_out_base(P, mb + col + e) + (int64_t)(nb + r) * hw : (int64_t)(mb + r) * P.ldc + nb + col + e;
            *(elem_t SK_GLOBAL *)((uintptr_t)P.C + (uintptr_t)(o * ES)) = ev[e];
          }
      }
    }
  };
  if ((P.flags & FLAG_PAST_CACHES) != 0)
    store_rows(std::true_type{});
  else
    store_rows(std::false_type{});
}

template <int DT, bool NCHW, int BM, int BN>
__device__ __forceinline__ void run_tile_any(const DevProblem *P_mem, const sk_tile *T_mem, const SplitK &sp,
                                             unsigned char *lds, uint32_t *s_flag, int tid) {
  constexpr int ES = Elem<DT>::ES;
  constexpr int CE = 16 / ES;
  constexpr int STAGE = (BM + BN) * LDS_ROW;  // pixels (or GEMM rows), then weight rows
  constexpr int NA = BM / 32, NBW = BN / 32;  // pieces per thread and stage
  constexpr int NH = BM / 64;                 // NCHW: pixels per lane
  constexpr int ROWS = NCHW ? BN : BM, COLS = NCHW ? BM : BN;  // of the block as the MFMAs see it
  constexpr int FM = ROWS / 64, FN = COLS / 64;                // 32x32 blocks per wave (2 x 2 waves)
  constexpr uint32_t NOWHERE = 0x80000000u;
  using elem_t = typename std::conditional<ES == 4, uint32_t, uint16_t>::type;
  typedef elem_t piece_t __attribute__((ext_vector_type(CE)));
  static_assert(2 * STAGE <= LDS_TILE_BYTES, "two stages do not fit the LDS buffer");
  const DevProblem P = load_record(P_mem);
  const sk_tile T = load_record(T_mem);
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int wm = wave & 1, wn = wave >> 1;
  const int l32 = lane & 31, half = lane >> 5;
  const int c8 = tid & 7, srow = tid >> 3;
  const int m_end = (int)T.m0 + (int)T.m_len, n_end = (int)T.n0 + (int)T.n_len;
  const int hw = P.Ho * P.Wo;

  // reduction runs and their pieces; this record's slice are the pieces that start in it
  const int run_len = !NCHW && P.gather ? P.S * P.Cin : P.Kg;
  const int ppr = (run_len + CE - 1) / CE;
  auto first_piece = [&](int k) {
    const int run = k / run_len;
    return run * ppr + (k - run * run_len + CE - 1) / CE;
  };
  const int p_begin = first_piece((int)T.k0), p_stop = first_piece((int)T.k0 + (int)T.k_len);
  const int nstages = (p_stop - p_begin + 7) >> 3;

  const int64_t a_run = (int64_t)P.W * P.Cin;  // elements from one filter row's run to the next in the image
  // A piece is read from inside its run's valid elements [lo, hi) and shifted into place, which also leaves zeros
  // where it reaches beyond them.  Runs too short for that (fewer valid elements than a piece somewhere): from
  // the nearest place inside the whole operand, shifted, and masked.
  const int fewest = !P.gather ? P.Kg : min(P.S, min(P.W, max(0, P.S - P.pad_w))) * P.Cin;
  const bool short_a = NCHW || fewest < CE, short_b = run_len < CE;
  const int64_t b_last = (int64_t)(P.Ng - 1) * P.ldb + P.Kg - CE;  // last place a piece may be read from
  const int64_t a_last = (P.gather ? (int64_t)fast_div(P.Mg + hw - 1, P.div_hw) * P.H * P.W * P.Cin
                                   : (int64_t)(P.Mg - 1) * P.lda + P.Kg) - CE;
  const uintptr_t zeros = zero_piece_address();

  for (int mb = (int)T.m0; mb < m_end; mb += BM) {
    // ---- where this thread's rows of the activation operand lie ----
    int64_t a_base[NA];  // GEMM / NHWC: rows srow + 32 i; NCHW: rows lane and lane + 64
    int a_lo[NA], a_hi[NA], a_h[NA];
    uint32_t n_off[NH], n_rows[NH], n_cols[NH];  // NCHW, 32-bit form: byte offset from the descriptor's origin; taps outside
    uintptr_t n_origin = 0;
    bool near = false;
    if constexpr (!NCHW) {
#pragma unroll
      for (int i = 0; i < NA; ++i) {
        int m = mb + srow + 32 * i;
        if (m >= m_end) m = m_end - 1;  // rows past the edge repeat the last row; never stored
        const RowA r = row_of(P, m);
        a_base[i] = r.base;
        a_h[i] = r.hb;
        a_lo[i] = 0;
        a_hi[i] = run_len;
        if (P.gather) {
          // (columns held to 0 .. S before they are multiplied: a padding of many filters' width times the channels does not fit 32 bits)
          a_lo[i] = min(max(0, -r.wb), P.S) * P.Cin;
          a_hi[i] = max(0, min(P.S, P.W - r.wb)) * P.Cin;
        }
      }
    } else {
      const int64_t image = (int64_t)P.Cin * P.H * P.W;
      const int b0 = fast_div(mb, P.div_hw), b1 = fast_div(min(mb + BM, m_end) - 1, P.div_hw);
      const int64_t corner = (int64_t)P.pad_h * P.W + P.pad_w;  // the corner of the padded image lies this far before it
      // (no pixel's offset and tap's offset add up to 2^31, inside the image or not; for the descriptor's size see lean_operands)
      near = offsets_below(P, b1 - b0, ES, (int64_t)1 << 31);
      n_origin = (uintptr_t)P.A + (uintptr_t)((b0 * image - corner) * ES);
#pragma unroll
      for (int h = 0; h < NH; ++h) {
        int m = mb + lane + 64 * h;
        if (m >= m_end) m = m_end - 1;
        const RowA r = row_of(P, m);
        a_base[h] = r.base;
        a_h[h] = r.hb;
        a_lo[h] = r.wb;
        n_off[h] = (uint32_t)((r.base + corner - b0 * image) * ES);
        // bit r of the row mask: filter row r falls outside the image; the same for the filter columns
        const int hlo = max(0, -r.hb), hhi = min(32, max(0, P.H - r.hb)), wlo = max(0, -r.wb), whi = min(32, max(0, P.W - r.wb));
        n_rows[h] = ~((uint32_t)(((uint64_t)1 << hhi) - 1) & ~(uint32_t)(((uint64_t)1 << min(hlo, 32)) - 1));
        n_cols[h] = ~((uint32_t)(((uint64_t)1 << whi) - 1) & ~(uint32_t)(((uint64_t)1 << min(wlo, 32)) - 1));
      }
    }
    const __amdgpu_buffer_rsrc_t descA = __builtin_amdgcn_make_buffer_rsrc((void *)n_origin, 0, (int)NOWHERE, 0x00020000);

    for (int nb = (int)T.n0; nb < n_end; nb += BN) {
      const int64_t b_base = (int64_t)(nb + srow) * P.ldb;  // of this thread's first weight row; the others 32 rows apart
      f32x16 acc[FN][FM];
#pragma unroll
      for (int fn = 0; fn < FN; ++fn)
#pragma unroll
        for (int fm = 0; fm < FM; ++fm)
#pragma unroll
          for (int i = 0; i < 16; ++i) acc[fn][fm][i] = 0.f;

      // ---- the next stage to load: this thread's piece of it ----
      int piece = p_begin + c8;
      int run = piece / ppr, j = piece - run * ppr;
      // NCHW: scalar position of the wave's first reduction index (2 pieces of every stage: 2 wave, 2 wave + 1)
      int ks = (p_begin + 2 * wave) * CE, kc = 0, kr = 0, kt = 0;
      if constexpr (NCHW) {
        const int cr = ks / P.S;
        kt = ks - cr * P.S;
        kc = cr / P.R;
        kr = cr - kc * P.R;
      }
      u32x4 ra[NA], rb[NBW];
      // Where the piece that starts at element e0 of its run is read (`o`: place of the run's start in the operand)
      auto a_from = [&](int i, int e0, int64_t o) {
        if (!short_a) return min(max(e0, a_lo[i]), a_hi[i] - CE);
        int64_t at = o + e0;
        at = at < a_last ? at : a_last;
        return (int)((at > 0 ? at : 0) - o);
      };
      auto b_from = [&](int e0, int64_t o) {
        if (!short_b) return min(e0, run_len - CE);
        const int64_t at = o + e0;
        return (int)((at < b_last ? at : b_last) - o);
      };
      int at_e0 = 0, at_run = 0, at_ks = 0;  // of the stage loaded last
      auto gload = [&]() {
        const bool in = piece < p_stop;
        const int e0 = j * CE;
        at_e0 = e0;
        at_run = run;
        if constexpr (!NCHW) {
#pragma unroll
          for (int i = 0; i < NA; ++i) {
            const bool ok = in && a_hi[i] > a_lo[i] && (!P.gather || (unsigned)(a_h[i] + run) < (unsigned)P.H);
            const int64_t o = a_base[i] + run * a_run;
            const int64_t at = o + a_from(i, e0, o);
            ra[i] = load_any(ok ? (uintptr_t)P.A + (uintptr_t)(at * ES) : zeros);
          }
        } else {
          piece_t el[NH][2];
          const int k_stop = (int)T.k0 + (int)T.k_len;
          // reduction indices ks .. ks + 2 CE - 1 of 64 + 64 pixels; `outside(h, r, t)`: top bit set where the pixel's tap
          // (r, t) lies outside the image
          auto load_elements = [&](auto outside) {
            int k = ks, r = kr, t = kt;
            uint32_t plane = (uint32_t)(kc * P.H * P.W);
#pragma unroll
            for (int pp = 0; pp < 2; ++pp)
#pragma unroll
              for (int e = 0; e < CE; ++e) {
                const bool k_in = k < k_stop;
                const uint32_t soff = k_in ? (plane + (uint32_t)(r * P.W + t)) * ES : 0u;
                const uint32_t k_out = k_in ? 0u : NOWHERE;
#pragma unroll
                for (int h = 0; h < NH; ++h) {
                  const uint32_t off = n_off[h] | ((outside(h, r, t) | k_out) & NOWHERE);
                  if constexpr (ES == 4)
                    el[h][pp][e] = __builtin_amdgcn_raw_buffer_load_b32(descA, off, soff, 0);
                  else
                    el[h][pp][e] = __builtin_amdgcn_raw_buffer_load_b16(descA, off, soff, 0);
                }
                ++k;
                if (++t == P.S) {
                  t = 0;
                  if (++r == P.R) {
                    r = 0;
                    plane += (uint32_t)(P.H * P.W);
                  }
                }
              }
          };
          if (near && P.R <= 32 && P.S <= 32)
            load_elements([&](int h, int r, int t) { return (n_rows[h] << ((31 - r) & 31)) | (n_cols[h] << ((31 - t) & 31)); });
          else if (near)
            load_elements([&](int h, int r, int t) {
              return (unsigned)(a_h[h] + r) < (unsigned)P.H && (unsigned)(a_lo[h] + t) < (unsigned)P.W ? 0u : NOWHERE;
            });
#pragma unroll
          for (int h = 0; h < NH; ++h)
#pragma unroll
            for (int pp = 0; pp < 2; ++pp) ra[2 * h + pp] = __builtin_bit_cast(u32x4, el[h][pp]);
          at_ks = ks;
          // on to the wave's pieces of the next stage: 8 pieces from the first of this one's
          ks += 8 * CE;
          const int cr = ks / P.S;
          kt = ks - cr * P.S;
          kc = cr / P.R;
          kr = cr - kc * P.R;
        }
#pragma unroll
        for (int i = 0; i < NBW; ++i) {
          const bool ok = in && nb + srow + 32 * i < n_end;  // (rows past the edge are never stored)
          const int64_t o = b_base + (int64_t)(32 * i) * P.ldb + (int64_t)run * run_len;
          const int64_t at = o + b_from(e0, o);
          rb[i] = load_any(ok ? (uintptr_t)P.B + (uintptr_t)(at * ES) : zeros);
        }
        piece += 8;
        j += 8;
        while (j >= ppr) {
          j -= ppr;
          ++run;
        }
      };
      // (the checks are for the whole wave: most waves have nothing to shift or mask)
      auto lstore = [&](int buf) {
        unsigned char *s = lds + buf * STAGE;
        const int e0 = at_e0;
#pragma unroll
        for (int i = 0; i < NA; ++i) {
          if constexpr (!NCHW) {
            const int sh = e0 - a_from(i, e0, a_base[i] + at_run * a_run);
            u32x4 v = ra[i];
            if (__any(sh != 0)) v = shift_piece<ES>(v, sh);
            if (short_a) v = mask_piece<ES>(v, a_lo[i] - e0, a_hi[i] - e0);
            *(u32x4 *)(s + (srow + 32 * i) * LDS_ROW + c8 * 16) = v;
          } else if (near) {
            *(u32x4 *)(s + (lane + 64 * (i >> 1)) * LDS_ROW + (2 * wave + (i & 1)) * 16) = ra[i];
          }
        }
        if (NCHW && !near) {  // (images of 2 GiB and more: one element at a time)
          const int k_stop = (int)T.k0 + (int)T.k_len;
#pragma unroll 1
          for (int q = 0; q < 2 * CE * NH; ++q) {
            const int h = q & (NH - 1), k = at_ks + q / NH;
            const int cr = k / P.S, t = k - cr * P.S, c = cr / P.R, r = cr - c * P.R;
            const int hh = (h ? a_h[NH - 1] : a_h[0]) + r, ww = (h ? a_lo[NH - 1] : a_lo[0]) + t;
            const bool ok = k < k_stop && (unsigned)hh < (unsigned)P.H && (unsigned)ww < (unsigned)P.W;
            const int64_t o = (h ? a_base[NH - 1] : a_base[0]) + ((int64_t)c * P.H + r) * P.W + t;
            *(elem_t *)(s + (lane + 64 * h) * LDS_ROW + 2 * wave * 16 + q / NH * ES) =
                *(const elem_t SK_GLOBAL *)(ok ? (uintptr_t)P.A + (uintptr_t)(o * ES) : zeros);
          }
        }
#pragma unroll
        for (int i = 0; i < NBW; ++i) {
          const int sh = e0 - b_from(e0, b_base + (int64_t)(32 * i) * P.ldb + (int64_t)at_run * run_len);
          u32x4 v = rb[i];
          if (__any(sh != 0)) v = shift_piece<ES>(v, sh);
          if (short_b) v = mask_piece<ES>(v, 0, run_len - e0);
          *(u32x4 *)(s + (BM + srow + 32 * i) * LDS_ROW + c8 * 16) = v;
        }
      };

      // (step -1 only loads; an empty slice delivers zeros)
      for (int s = -1; s < nstages; ++s) {
        if (s + 1 < nstages) gload();
        if (s >= 0) {
          // MFMA columns (four consecutive of which a lane holds) come from the operand along whose rows the output is contiguous
          const unsigned char *la = lds + (s & 1) * STAGE + (NCHW ? BM * LDS_ROW : 0);
          const unsigned char *lb = lds + (s & 1) * STAGE + (NCHW ? 0 : BM * LDS_ROW);
#pragma unroll
          for (int kk = 0; kk < 4; ++kk) {
            const int at = (2 * kk + half) * 16;
            u32x4 fa[FM], fb[FN];
#pragma unroll
            for (int f = 0; f < FM; ++f) fa[f] = *(const u32x4 *)(la + ((wm * FM + f) * 32 + l32) * LDS_ROW + at);
#pragma unroll
            for (int f = 0; f < FN; ++f) fb[f] = *(const u32x4 *)(lb + ((wn * FN + f) * 32 + l32) * LDS_ROW + at);
#pragma unroll
            for (int fn = 0; fn < FN; ++fn)
#pragma unroll
              for (int fm = 0; fm < FM; ++fm) mma32<DT>(fb[fn], fa[fm], acc[fn][fm]);
          }
        }
        if (s + 1 < nstages) lstore((s + 1) & 1);
        __syncthreads();  // stage s+1 is written, and everyone has read stage s
      }

      if (T.S > 1 && !any_handover<NCHW, FM, FN>(T, sp, lds, s_flag, tid, acc)) return;
      any_outputs<DT, NCHW, ROWS, COLS, 2>(P_mem, T_mem, mb, nb, lds, tid, acc);
      __syncthreads();  // the output tile has been read before the next block's stages are written
    }
  }
}

// ---------------------------------------------------------------------------
// channel-major convolutions whose pixels lie in the order of their outputs
// ---------------------------------------------------------------------------
// Under one reduction index (channel and tap) of a convolution that keeps its images' width, consecutive outputs read
// consecutive places of one channel plane, from row to row as well.  So (planes_form) instead of single elements:
//   * a thread reads 16 bytes (8 pixels; 4 in fp32) under one reduction index, at whatever address they start, and clears the pixels whose
//     tap lies outside the image (a table in LDS of what each tap keeps of each piece, worked out once per block);
//   * the LDS image of a stage holds a row of pixels per reduction index, pieces turned over (^ 4 per row) so that the rows a fragment
//     takes lie in different banks, and 16-bit fragments are read with the hardware's transposing LDS load (a lane gets four
//     reduction indices of its pixel), fp32 ones element by element.
// The sums are those of run_tile_any: the same bits.  What a stage cost there were the instructions for its single elements (32 loads of
// two bytes a lane and stage, and as many masks and packs; here four loads, and two dozen instructions for each): channel-major
// ResNet layers for eight 98.1 -> 67.6 us (61.8 with the partial sums of slices read together, any_handover).  What binds it now is the
// loads: at places that are no multiples of a dword 16 bytes a lane run one lane a clock (67 clocks for 1 KB, 21 to 24 from any dword's address).
constexpr int PLANES_TAPS = 12;  // the most planes_form lets through
template <int ES>
__device__ __forceinline__ bool planes_tile(const DevProblem &P, const sk_tile &T) {
  constexpr int CE = 16 / ES;
  // (fp32: the host's answer.  The 16-bit kernels ask again: with the flags their other paths took 1 to 2 % longer, see rows_tile.)
  if constexpr (ES == 4) {
    if (!(P.flags & FLAG_PLANES_FORM)) return false;
    if (P.Mg == P.Ho * P.Wo) return true;  // one image
  } else {
    if (!planes_form(P, ES)) return false;
  }
  const int b0 = fast_div((int)T.m0, P.div_hw), b1 = fast_div((int)T.m0 + (int)T.m_len - 1, P.div_hw);
  // (a piece of pixels lies in one image, and all offsets within 2^31 bytes)
  return (b0 == b1 || (P.Ho * P.Wo) % CE == 0) && offsets_below(P, b1 - b0, ES, (int64_t)1 << 31);
}

typedef short s16x4 __attribute__((ext_vector_type(4)));
// Four 16-bit elements of this lane's column out of four rows of a group of 16 lanes.
__device__ __forceinline__ u32x2 read_transposed(const unsigned char *p) {
  return __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)(unsigned char *)p));
}
// Which pixels of a piece to keep under a tap: their bits as the AND of a 16-bit piece takes them, or (fp32) one bit each.
template <int ES>
struct Keep {
  using type = typename std::conditional<ES == 4, uint32_t, u32x4>::type;
  static __device__ __forceinline__ u32x4 apply(const u32x4 &v, const type &k) {
    if constexpr (ES == 4)
      return u32x4{v[0] & (uint32_t)__builtin_amdgcn_sbfe((int)k, 0, 1), v[1] & (uint32_t)__builtin_amdgcn_sbfe((int)k, 1, 1),
                   v[2] & (uint32_t)__builtin_amdgcn_sbfe((int)k, 2, 1), v[3] & (uint32_t)__builtin_amdgcn_sbfe((int)k, 3, 1)};
    else
      return v & k;
  }
};

template <int DT, int BM, int BN>
__device__ __forceinline__ void run_tile_planes(const DevProblem *P_mem, const sk_tile *T_mem, const SplitK &sp, unsigned char *lds,
                                                uint32_t *s_flag, int tid) {
  constexpr int ES = Elem<DT>::ES;
  constexpr int CE = 16 / ES;
  constexpr int KB = 8 * CE;              // reduction elements per stage
  constexpr int PROW = BM * ES;           // bytes of an LDS row of pixels
  constexpr int PPR = BM / CE;            // pieces of such a row
  constexpr int RPP = WG_THREADS / PPR;   // rows that the workgroup fills at a time
  constexpr int NA = KB / RPP, NBW = BN / 32;
  constexpr int WEIGHTS = KB * PROW;      // where the weight rows start
  constexpr int STAGE = WEIGHTS + BN * LDS_ROW;
  constexpr int FM = BN / 64, FN = BM / 64;  // 32x32 blocks per wave: output channels, pixels
  const DevProblem P = load_record(P_mem);
  const sk_tile T = load_record(T_mem);
  const int m_end = (int)T.m0 + (int)T.m_len, n_end = (int)T.n0 + (int)T.n_len;
  const int hw = P.Ho * P.Wo, plane = P.H * P.W, taps = P.R * P.S;
  const int k_stop = (int)T.k0 + (int)T.k_len;
  const int p_begin = ((int)T.k0 + CE - 1) / CE, p_stop = (k_stop + CE - 1) / CE;
  const int nstages = (p_stop - p_begin + 7) >> 3;
  const int stage_c = KB / taps, stage_t = KB - stage_c * taps;  // channels and taps from one stage to the next ...
  const int pass_c = RPP / taps, pass_t = RPP - pass_c * taps;   // ... and from one of a thread's rows to the next
  const bool ragged = P.Kg % CE != 0;                            // the last piece of a weight row reaches beyond it
  const bool masked = taps > 1 || P.pad_h > 0;                   // some taps lie outside the image
  using keep_t = typename Keep<ES>::type;
  keep_t *const keep = (keep_t *)(lds + 2 * STAGE);  // [tap][piece of pixels]
  static_assert(2 * STAGE + PLANES_TAPS * PPR * (int)sizeof(keep_t) <= LDS_TILE_BYTES, "the table of taps does not fit the LDS buffer");

  for (int mb = (int)T.m0; mb < m_end; mb += BM) {
    // (what depends on the thread is worked out again for every block: kept over all of them it would not fit the registers)
    asm volatile("" : "+v"(tid));
    const int b0 = fast_div(mb, P.div_hw), b1 = fast_div(min(mb + BM, m_end) - 1, P.div_hw);
    const char SK_GLOBAL *image = as_global<char>(P.A) + (int64_t)b0 * P.Cin * plane * ES;
    const int a_last = (((b1 - b0 + 1) * P.Cin) * plane - CE) * ES;  // last place a piece may be read from
    if (masked)
      for (int i = tid; i < taps * PPR; i += WG_THREADS) {
        const int t = i / PPR, r = P.S == 3 ? (t * 11) >> 5 : t, s = t - r * P.S;
        const int m = min(mb + (i & (PPR - 1)) * CE, m_end - 1);
        const int rem = m - fast_div(m, P.div_hw) * hw;
        int ho = fast_div(rem, P.div_wo), w = rem - ho * P.Wo + s - P.pad_w, h = ho + r - P.pad_h;
        uint32_t in[CE];  // (of pixels past the edge, which are never stored, whatever follows)
#pragma unroll
        for (int e = 0; e < CE; ++e) {
          in[e] = (unsigned)w < (unsigned)P.W && (unsigned)h < (unsigned)P.H ? ~0u : 0u;
          if (++w == P.Wo + s - P.pad_w) {
            w = s - P.pad_w;
            ++h;
            if (++ho == P.Ho) {
              ho = 0;
              h = r - P.pad_h;
            }
          }
        }
        if constexpr (ES == 4)
          keep[i] = (in[0] & 1u) | (in[1] & 2u) | (in[2] & 4u) | (in[3] & 8u);
        else
#pragma unroll
          for (int e = 0; e < 4; ++e) keep[i][e] = (in[2 * e] & 0xffffu) | (in[2 * e + 1] & 0xffff0000u);
      }
    auto swizzle = [&](int r) { return ES == 4 ? (r << 1) & 8 : BM == 128 ? (r & 3) << 2 : (r << 1) & 4; };

    for (int nb = (int)T.n0; nb < n_end; nb += BN) {
      asm volatile("" : "+v"(tid));
      const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
      const int wm = wave & 1, wn = wave >> 1;
      const int l32 = lane & 31, half = lane >> 5;
      const int c8 = tid & 7, srow = tid >> 3;  // weights: piece c8 of rows srow + 32 i
      const int pc = tid & (PPR - 1), kr = tid / PPR;  // pixels: piece pc of rows kr + RPP i
      f32x16 acc[FN][FM];
#pragma unroll
      for (int fn = 0; fn < FN; ++fn)
#pragma unroll
        for (int fm = 0; fm < FM; ++fm)
#pragma unroll
          for (int i = 0; i < 16; ++i) acc[fn][fm][i] = 0.f;

      // ---- the next stage to load ----
      int ks = p_begin * CE;  // its first reduction index
      uint32_t k_tap[NA];     // this thread's rows of it: tap, and ...
      int k_off[NA];          // ... place under tap (0, 0), in bytes from `image` (may lie in front of it)
      int tap_off;            // lane t: tap t's, from that under tap (0, 0)
      {
        const int tr = P.S == 3 ? (lane * 11) >> 5 : lane;  // (at most PLANES_TAPS taps)
        tap_off = (tr * P.W + lane - tr * P.S) * ES;
        const int m = min(mb + pc * CE, m_end - 1), b = fast_div(m, P.div_hw);
        const int a_off = (b - b0) * P.Cin * plane + m - b * hw - P.pad_h * P.W - P.pad_w;
        int c = (ks + kr) / taps, t = ks + kr - c * taps;
#pragma unroll
        for (int i = 0; i < NA; ++i) {
          k_tap[i] = (uint32_t)t;
          k_off[i] = (a_off + c * plane) * ES;
          c += pass_c;
          t += pass_t;
          if (t >= taps) {
            t -= taps;
            ++c;
          }
          // (opaque, so that the first stage's positions are not worked out apart)
          asm volatile("" : "+v"(k_tap[i]), "+v"(k_off[i]));
        }
      }
      const char SK_GLOBAL *weights = as_global<char>(P.B) + (int64_t)nb * P.ldb * ES;
      uint32_t w_off[NBW];
#pragma unroll
      for (int i = 0; i < NBW; ++i) w_off[i] = (uint32_t)(min(srow + 32 * i, n_end - 1 - nb) * (int)P.ldb) * ES;
      u32x4 ra[NA], rb[NBW];
      uint32_t a_tap[NA];  // of the stage loaded last: its rows' taps; ...
      int a_sh[NA];        // ... how many bytes from their places its pieces were read, ...
      int w_at = 0;        // ... the reduction index of its weight piece
      const int plane_bytes = plane * ES, stage_off = stage_c * plane_bytes;
      auto gload = [&]() {
        int under[NA];
#pragma unroll
        for (int i = 0; i < NA; ++i) under[i] = __builtin_amdgcn_ds_bpermute((int)(k_tap[i] << 2), tap_off);
#pragma unroll
        for (int i = 0; i < NA; ++i) {
          const int off = k_off[i] + under[i], at = min(max(off, 0), a_last);
          a_sh[i] = off - at;
          a_tap[i] = k_tap[i];
          ra[i] = *(const u32x4_any SK_GLOBAL *)(image + (uint32_t)at);
          const uint32_t t = k_tap[i] + (uint32_t)stage_t, u = t - (uint32_t)taps;
          k_off[i] += stage_off + (t >= (uint32_t)taps ? plane_bytes : 0);
          k_tap[i] = min(t, u);  // (t - taps wraps where t < taps)
        }
        w_at = ks + c8 * CE;
        const uint32_t at = (uint32_t)(min(w_at, P.Kg - CE) * ES);
#pragma unroll
        for (int i = 0; i < NBW; ++i) rb[i] = *(const u32x4_any SK_GLOBAL *)(weights + (w_off[i] + at));
        ks += KB;
      };
      auto lstore = [&](int buf) {
        unsigned char *s = lds + buf * STAGE;
        const bool last = ks >= p_stop * CE;  // (zeros beyond the slice, and beyond the weight rows)
        if (masked) {
          keep_t k[NA];
#pragma unroll
          for (int i = 0; i < NA; ++i) k[i] = keep[a_tap[i] * PPR + pc];
          int any = 0;
#pragma unroll
          for (int i = 0; i < NA; ++i) any |= a_sh[i];
          if (__any(any != 0)) {
#pragma unroll
            for (int i = 0; i < NA; ++i) ra[i] = shift_piece<ES>(ra[i], a_sh[i] / ES);
          }
#pragma unroll
          for (int i = 0; i < NA; ++i) ra[i] = Keep<ES>::apply(ra[i], k[i]);
        } else {
#pragma unroll
          for (int i = 0; i < NA; ++i)
            if (__any(a_sh[i] != 0)) ra[i] = shift_piece<ES>(ra[i], a_sh[i] / ES);
        }
        if (last) {
#pragma unroll
          for (int i = 0; i < NA; ++i)
            if (ks - KB + kr + RPP * i >= k_stop) ra[i] = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
          for (int i = 0; i < NBW; ++i) {
            if (ragged) rb[i] = shift_piece<ES>(rb[i], max(w_at - (P.Kg - CE), 0));
            if (w_at >= p_stop * CE) rb[i] = u32x4{0u, 0u, 0u, 0u};
          }
        }
#pragma unroll
        for (int i = 0; i < NA; ++i) {
          const int r = kr + RPP * i;
          *(u32x4 *)(s + r * PROW + ((pc ^ swizzle(r)) << 4)) = ra[i];
        }
#pragma unroll
        for (int i = 0; i < NBW; ++i) *(u32x4 *)(s + WEIGHTS + (srow + 32 * i) * LDS_ROW + c8 * 16) = rb[i];
      };
      // fragment addresses: of block f of this wave's pixels, reduction indices 0 .. of the stage
      int px_at[FN];
#pragma unroll
      for (int f = 0; f < FN; ++f) {
        if constexpr (ES == 2) {
          const int i = lane & 15, r = 8 * half + (i >> 2), px = (wn * FN + f) * 32 + 16 * ((lane >> 4) & 1) + 4 * (i & 3);
          px_at[f] = r * PROW + (((px >> 3) ^ swizzle(r)) << 4) + (px & 7) * 2;
        } else {
          const int px = (wn * FN + f) * 32 + l32;
          px_at[f] = 4 * half * PROW + (((px >> 2) ^ swizzle(4 * half)) << 4) + (px & 3) * 4;
        }
      }
      const int w_frag = WEIGHTS + (wm * FM * 32 + l32) * LDS_ROW + half * 16;

      // (step -1 only loads; an empty slice delivers zeros)
      for (int s = -1; s < nstages; ++s) {
        if (s + 1 < nstages) gload();
        if (s < 0 && masked) __syncthreads();  // the table of taps is written
        if (s >= 0) {
          const unsigned char *l = lds + (s & 1) * STAGE;
          u32x4 fa[2][FM], fb[2][FN];
          auto frag = [&](int kk, u32x4(&xa)[FM], u32x4(&xb)[FN]) {
#pragma unroll
            for (int f = 0; f < FM; ++f) xa[f] = *(const u32x4 *)(l + w_frag + f * 32 * LDS_ROW + kk * 32);
#pragma unroll
            for (int f = 0; f < FN; ++f) {
              if constexpr (ES == 2) {
                const u32x2 lo = read_transposed(l + px_at[f] + kk * 16 * PROW), hi = read_transposed(l + px_at[f] + (kk * 16 + 4) * PROW);
                xb[f] = u32x4{lo.x, lo.y, hi.x, hi.y};
              } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) xb[f][j] = *(const uint32_t *)(l + px_at[f] + (kk * 8 + j) * PROW);
              }
            }
          };
          frag(0, fa[0], fb[0]);
#pragma unroll
          for (int kk = 0; kk < 4; ++kk) {
            if (kk < 3) frag(kk + 1, fa[(kk + 1) & 1], fb[(kk + 1) & 1]);
            __builtin_amdgcn_sched_barrier(0);  // (a step ahead and no further: the registers)
#pragma unroll
            for (int fn = 0; fn < FN; ++fn)
#pragma unroll
              for (int fm = 0; fm < FM; ++fm) mma32<DT>(fb[kk & 1][fn], fa[kk & 1][fm], acc[fn][fm]);
            __builtin_amdgcn_sched_barrier(0);
          }
        }
        if (s + 1 < nstages) lstore((s + 1) & 1);
        __syncthreads();  // stage s+1 is written, and everyone has read stage s
      }
      if (T.S > 1 && !any_handover<true, FM, FN>(T, sp, lds, s_flag, tid, acc)) return;
      any_outputs<DT, true, BN, BM, 2>(P_mem, T_mem, mb, nb, lds, tid, acc);
      __syncthreads();  // the output tile has been read before the next block's stages are written
    }
  }
}

// ---------------------------------------------------------------------------
// NHWC convolutions of few channels: a window of the image in LDS
// ---------------------------------------------------------------------------
// A convolution on an image of few channels (the 7x7 stem on RGB) has runs of S * Cin elements under a filter row that pieces of 16 bytes do not
// divide, and brings every element into LDS once per tap: as patches that was 11.5 us a tile of three stages, nearly all of it vector
// instructions for shifts and addresses and loads at places that are no multiples of a dword.  Here (rows_form):
//   * the rows of the image that a block of 128 output pixels needs are loaded once, with zeros for the padding, 16 bytes a thread wherever they
//     start, and a pixel's patch is read out of them by the MFMA fragments themselves: piece j of filter row r lies r rows and 16 j bytes
//     on from where the patch starts, at a dword's address or (odd strides of odd channel counts of 16 bits) half a dword past one;
//   * what a piece holds beyond its run is cleared (it is some other pixel's);
//   * the weights (at most 64 channels) stay in LDS for all blocks of the record, and the next block's rows are on their way while one
//     is multiplied;
//   * a wave makes 32 pixels x 64 channels, so that each pixel's fragments are read and cleared once.
// Pieces and their order are those of run_tile_any: the same sums, the same bits.  7x7 stems on 224x224x3 of 64 tenants 140 -> 72 us, of 16 beside the
// other down-sampling layers of a residual network 100.4 -> 73.7; with the positions worked out piece by piece in the loop, a hundred scalar
// instructions a step, it gained 19 us of the 66 then.  Not where there is little else in a launch to gain it from: 5x5 filters on one channel (runs shorter than a
// piece, patches as before) 8.7 -> 9.1 us, by what this path costs the kernel's others in scalars.
// Parts of 64 rows, as refine_tiles cuts them where the operators are not marked, go the way of all others in 16-bit types: half a block's waves would
// repeat the last pixel, and every part loads the weights (one, two and four 7x7 stems 10.4, 12.6 and 22.3 us in half blocks, 9.9, 12.0 and 21.1 so, 9.9, 12.0 and 21.1
// before there was this path).  fp32 parts gain either way (3x3 on 60x60 11.6 us as patches, 9.2 here).
// Whether the form serves is the host's answer in fp32, worked out per tile it was 0.4 us of each (the same stem 9.8 us); the 16-bit kernels ask the form itself: with
// the flag the compiler kept 27 scalars more in vector lanes and the paths beside this one took 1 to 2 % longer (odd products of 200 rows x12 59.1 and 60.3 us).
template <int ES>
__device__ __forceinline__ bool rows_tile(const DevProblem &P, const sk_tile &T) {
  if (T.cls < CLS_TILE_128x128 || T.S != 1) return false;
  if (ES == 2 && !(P.flags & FLAG_ROWS) && (int)T.m_len <= 64) return false;
  if (!(ES == 4 ? (P.flags & FLAG_ROWS_FORM) != 0 : rows_form(P, ES).ok)) return false;
  return fast_div((int)T.m0, P.div_hw) == fast_div((int)T.m0 + (int)T.m_len - 1, P.div_hw);
}

// The products of a block: PR pieces per run, `patch` where this lane's starts, `w` this lane's pieces of the weights.
template <int DT, int PR, bool ODD>
__device__ __forceinline__ void multiply_rows(const unsigned char *patch, const unsigned char *w, int R, int image_row, int weight_row, int half,
                                              uint32_t shift, const uint32_t (&tail)[4], f32x16 (&acc)[2][1]) {
  typedef u32x4 u32x4_dword __attribute__((aligned(4)));
  // what this lane keeps where the last piece of a run is that of lanes 0 to 31 (1: of the others, 2: of both; 3: and the others' is none)
  auto keep = [&](int which, int i) { return which == 2 || (which == 1) == (half != 0) ? tail[i] : which == 3 ? 0u : ~0u; };
  auto step = [&](const unsigned char *src, int which) {
    u32x4 x = *(const u32x4_dword *)src;
    if constexpr (ODD) x = join_dwords(x, *(const uint32_t *)(src + 16), shift);
    const u32x4 w0 = *(const u32x4 *)w, w1 = *(const u32x4 *)(w + 32 * weight_row);
    w += 32;
    if (which >= 0) {
#pragma unroll
      for (int i = 0; i < 4; ++i) x[i] &= keep(which, i);
    }
    mma32<DT>(w0, x, acc[0][0]);
    mma32<DT>(w1, x, acc[1][0]);
  };
  if constexpr (PR % 2 == 0) {
    patch += 16 * half;
    for (int r = 0; r < R; ++r, patch += image_row) {
#pragma unroll
      for (int j = 0; j < PR; j += 2) step(patch + 16 * j, j + 2 == PR ? 1 : -1);
    }
  } else {
    // two runs at a time: the middle step has the last piece of one and the first of the other
    const unsigned char *at = patch + 16 * half, *middle = patch + (half ? image_row : 16 * (PR - 1));
    for (int r = 0; r + 1 < R; r += 2, at += 2 * image_row, middle += 2 * image_row) {
#pragma unroll
      for (int j = 0; j < PR - 1; j += 2) step(at + 16 * j, -1);
      step(middle, PR == 1 ? 2 : 0);
#pragma unroll
      for (int j = 1; j < PR; j += 2) step(at + image_row + 16 * j, j + 2 == PR ? 1 : -1);
    }
    if (R & 1) {
#pragma unroll
      for (int j = 0; j < PR - 1; j += 2) step(at + 16 * j, -1);
      step(half ? patch : middle, 3);  // (the weights end with a piece of zeros)
    }
  }
}

template <int DT>
__device__ __forceinline__ void run_tile_rows(const DevProblem *P_mem, const sk_tile *T_mem, unsigned char *lds, Prefetch &pf) {
  constexpr int ES = Elem<DT>::ES;
  constexpr int CE = 16 / ES;
  constexpr int BM = 128;
  static_assert(ROWS_LDS == LDS_TILE_BYTES, "the size rows_form goes by");
  const int tid = pf.tid;
  const DevProblem P = load_record(P_mem);
  const sk_tile T = load_record(T_mem);
  const RowsForm F = rows_form(P, ES);
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int l32 = lane & 31, half = lane >> 5;
  const int m_end = (int)T.m0 + (int)T.m_len, hw = P.Ho * P.Wo;
  const int b = fast_div((int)T.m0, P.div_hw), image_m = b * hw;  // (the record lies in one image)
  const int run_len = P.S * P.Cin, row_len = P.W * P.Cin;
  const int row_pieces = F.image_row / 16;
  const int np = P.R * F.pieces;  // pieces of a patch, and of a weight row
  // pieces of a block's rows per thread, ROWS_LOADS at most; loaded, shifted and cleared in pairs (all six always: 3x3 stems on 112x112 x16 10.8 us, so 9.9; each
  // asked for by itself costs the kernel 40 scalars more in vector lanes, and its other paths 1 to 4 %)
  const int loads = (F.rows * row_pieces + WG_THREADS - 1) / WG_THREADS;
  unsigned char *const window = lds + 64 * F.weight_row;
  const char SK_GLOBAL *const image = as_global<char>(P.A) + (int64_t)b * P.H * row_len * ES;

  // ---- the rows of a block: this thread's pieces tid + 256 i, each always at one place of one of the rows ----
  u32x4 win[ROWS_LOADS];
  int win_row[ROWS_LOADS], win_at[ROWS_LOADS], win_sh[ROWS_LOADS];  // row, byte of an image row it is read from, how far from its place that is
  {
    const uint32_t inv = 0xffffffffu / (uint32_t)row_pieces + 1u;  // i / row_pieces
#pragma unroll
    for (int i = 0; i < ROWS_LOADS; ++i) {
      const int idx = tid + i * WG_THREADS, r = (int)__umulhi((uint32_t)idx, inv), e0 = (idx - r * row_pieces) * CE - P.pad_w * P.Cin;
      const int at = min(max(e0, 0), row_len - CE);
      win_row[i] = r;
      win_at[i] = at * ES;
      win_sh[i] = e0 - at;
    }
  }
  auto first_row = [&](int mb) { return fast_div(mb - image_m, P.div_wo); };
  auto load_window = [&](int mb) {
    const int h0 = first_row(mb) * P.stride - P.pad_h;
#pragma unroll
    for (int i = 0; i < ROWS_LOADS; ++i) {
      if (i % 2 == 0 && i >= loads) break;
      const int h = min(max(h0 + win_row[i], 0), P.H - 1);  // (rows outside the image are cleared when stored)
      win[i] = *(const u32x4_any SK_GLOBAL *)(image + (uint32_t)(h * (row_len * ES) + win_at[i]));
    }
  };
  auto store_window = [&](int mb) {
    const int r0 = first_row(mb), h0 = r0 * P.stride - P.pad_h, rows = (first_row(min(mb + BM, m_end) - 1) - r0) * P.stride + P.R;
#pragma unroll
    for (int i = 0; i < ROWS_LOADS; ++i) {
      if (i % 2 == 0 && i >= loads) break;
      u32x4 v = win[i];
      if (__any(win_sh[i] != 0)) v = shift_piece<ES>(v, win_sh[i]);
      const bool in = (unsigned)(h0 + win_row[i]) < (unsigned)P.H;
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = in ? v[e] : 0u;
      if (win_row[i] < rows) *(u32x4 *)(window + (tid + i * WG_THREADS) * 16) = v;
    }
  };
  load_window((int)T.m0);
  pf.issue();

  // ---- the weights: row n's pieces side by side, and a piece of zeros where they are odd in number ----
  {
    const int per_row = (np + 1) & ~1, n_len = (int)T.n_len;
    const uint32_t inv = 0xffffffffu / (uint32_t)per_row + 1u, inv_run = 0xffffffffu / (uint32_t)F.pieces + 1u;
    const char SK_GLOBAL *const base = as_global<char>(P.B) + (int64_t)T.n0 * P.ldb * ES;
    for (int i0 = 0; i0 < 64 * per_row; i0 += 4 * WG_THREADS) {
      u32x4 v[4];
      int sh[4], to[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int idx = i0 + tid + i * WG_THREADS, n = (int)__umulhi((uint32_t)idx, inv), p = idx - n * per_row, q = min(p, np - 1);
        const int r = F.pieces == 1 ? q : (int)__umulhi((uint32_t)q, inv_run), e0 = (q - r * F.pieces) * CE, at = min(e0, run_len - CE);
        sh[i] = p < np ? e0 - at : CE;  // (shifted by a whole piece: zeros)
        to[i] = n < 64 ? n * F.weight_row + p * 16 : -1;
        // (rows past the edge repeat the last one; never stored)
        v[i] = *(const u32x4_any SK_GLOBAL *)(base + (uint32_t)((min(n, n_len - 1) * (int)P.ldb + r * run_len + at) * ES));
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (__any(sh[i] != 0)) v[i] = shift_piece<ES>(v[i], sh[i]);
        if (to[i] >= 0) *(u32x4 *)(lds + to[i]) = v[i];
      }
    }
  }
  store_window((int)T.m0);
  __syncthreads();

  // what the last piece of a run keeps
  uint32_t tail[4];
  {
    const int keep = run_len - (F.pieces - 1) * CE;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      tail[i] = ES == 4 ? (i < keep ? ~0u : 0u) : (2 * i < keep ? 0xffffu : 0u) | (2 * i + 1 < keep ? 0xffff0000u : 0u);
  }
  const bool odd = ES == 2 && ((P.stride * P.Cin) & 1) != 0;  // some patches start half a dword past one

  for (int mb = (int)T.m0; mb < m_end; mb += BM) {
    const bool more = mb + BM < m_end;
    if (more) load_window(mb + BM);
    // this lane's pixel, and where its patch starts
    const int m = min(mb + 32 * wave + l32, m_end - 1) - image_m, ho = fast_div(m, P.div_wo), wo = m - ho * P.Wo;
    const int start = ((ho - first_row(mb)) * F.image_row + wo * P.Cin * ES) * P.stride;
    const uint32_t shift = (uint32_t)(start & 2) << 3;
    f32x16 acc[2][1];
#pragma unroll
    for (int fn = 0; fn < 2; ++fn)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[fn][0][i] = 0.f;
    const unsigned char *const patch = window + (start & ~3), *const w = lds + l32 * F.weight_row + half * 16;
    auto go = [&](auto odd_c) {
      constexpr bool ODD = decltype(odd_c)::value;
      if (F.pieces == 3)
        multiply_rows<DT, 3, ODD>(patch, w, P.R, F.image_row, F.weight_row, half, shift, tail, acc);
      else if (F.pieces == 2)
        multiply_rows<DT, 2, ODD>(patch, w, P.R, F.image_row, F.weight_row, half, shift, tail, acc);
      else if (F.pieces == 1)
        multiply_rows<DT, 1, ODD>(patch, w, P.R, F.image_row, F.weight_row, half, shift, tail, acc);
      else if (F.pieces == 4)
        multiply_rows<DT, 4, ODD>(patch, w, P.R, F.image_row, F.weight_row, half, shift, tail, acc);
      else
        multiply_rows<DT, 6, ODD>(patch, w, P.R, F.image_row, F.weight_row, half, shift, tail, acc);
    };
    if (ES == 2 && odd)
      go(std::integral_constant<bool, ES == 2>{});
    else
      go(std::false_type{});
    __syncthreads();  // everyone is done with the window: the outputs are staged in its place
    any_outputs<DT, false, BM, 64, 4>(P_mem, T_mem, mb, (int)T.n0, window, tid, acc);
    if (more) {
      __syncthreads();  // the outputs have been read
      store_window(mb + BM);
      __syncthreads();
    }
  }
}

// (A slice of a split reduction must be a single block, so a shape may only be wider than its rectangle.  64 x 128 and 128 x 64
// beside the square ones: without them the channel-major ResNet layers for eight take 173 instead of 152 us, the stride-2
// layers for sixteen 123 instead of 113.)
template <int DT, bool NCHW, bool PLANES, int BM, int BN>
__device__ __forceinline__ void run_block_shape(const DevProblem *P_mem, const sk_tile *T_mem, const SplitK &sp, unsigned char *lds,
                                                uint32_t *s_flag, int tid) {
  if constexpr (PLANES)
    run_tile_planes<DT, BM, BN>(P_mem, T_mem, sp, lds, s_flag, tid);
  else
    run_tile_any<DT, NCHW, BM, BN>(P_mem, T_mem, sp, lds, s_flag, tid);
}
template <int DT, bool NCHW, bool PLANES>
__device__ __forceinline__ void run_block_any(const DevProblem *P_mem, const sk_tile *T_mem, int m_len, int n_len, const SplitK &sp,
                                              unsigned char *lds, uint32_t *s_flag, int tid) {
  if (m_len <= 64 && n_len <= 64)
    run_block_shape<DT, NCHW, PLANES, 64, 64>(P_mem, T_mem, sp, lds, s_flag, tid);
  else if (m_len <= 64)
    run_block_shape<DT, NCHW, PLANES, 64, 128>(P_mem, T_mem, sp, lds, s_flag, tid);
  else if (n_len <= 64)
    run_block_shape<DT, NCHW, PLANES, 128, 64>(P_mem, T_mem, sp, lds, s_flag, tid);
  else
    run_block_shape<DT, NCHW, PLANES, 128, 128>(P_mem, T_mem, sp, lds, s_flag, tid);
}

template <int DT, bool ANY_ALIGNMENT, bool NARROW, bool WINDOW, bool MIXED>
__device__ __forceinline__ void run_class(const DevProblem &P, const sk_tile &T, const DevProblem *P_mem,
                                          const sk_tile *T_mem, const SplitK &sp, unsigned char *lds,
                                          uint32_t *s_flag, Prefetch &pf) {
  if constexpr (NARROW) {
    run_lds_tile<DT, 128, 64, true>(P, T, sp, lds, s_flag, pf);
  } else {
    const int cls = T.cls;
    constexpr int CE = 16 / Elem<DT>::ES;
    bool pieces = true;  // the fast paths can read the operator
    if constexpr (ANY_ALIGNMENT) {
      pieces = (P.flags & (FLAG_VEC_A | FLAG_VEC_B)) == (FLAG_VEC_A | FLAG_VEC_B);
      if (!pieces) {
        // One output per thread costs a thread (outputs / 256) * Kg dependent steps of about 0.1 us; a stage
        // of 64 (fp32: 32) reduction elements through the matrix cores costs a few us whatever the
        // rectangle.  So only rectangles that are done in a few dozen steps go the first way.
        const int per_thread = ((int)T.m_len * (int)T.n_len + WG_THREADS - 1) / WG_THREADS;
        const bool small = (int64_t)per_thread * P.Kg <= 64;
        // The weight-streaming classes read pieces at any element's address; of convolutions those whose pieces never
        // straddle two taps.
        if (!small && cls < CLS_TILE_128x128 && !P.nchw && P.Kg >= CE && (!P.gather || P.Cin % CE == 0)) {
          pieces = true;
        } else {
          pf.claim();
          const bool rows = !small && rows_tile<Elem<DT>::ES>(P, T);
          if (!rows) pf.issue();
          // (an operand of less than one piece also goes the first way: the others read whole pieces from inside it)
          if (small || !holds_a_piece<Elem<DT>::ES>(P))
            run_generic<DT>(P_mem, T_mem, pf.tid);
          // (in the kernel for mixed types the compiler is told that this is rare, and keeps its lane copies of scalars off the other paths: 60 aligned products
          // in three types 148 -> 134 us; said in the others it brings nothing, or 1 % of the stems' own time)
          else if (MIXED ? __builtin_expect_with_probability(rows, 0, 0.999) : rows)
            run_tile_rows<DT>(P_mem, T_mem, lds, pf);
          else if (P.nchw && planes_tile<Elem<DT>::ES>(P, T))
            run_block_any<DT, true, true>(P_mem, T_mem, (int)T.m_len, (int)T.n_len, sp, lds, s_flag, pf.tid);
          else if (P.nchw)
            run_block_any<DT, true, false>(P_mem, T_mem, (int)T.m_len, (int)T.n_len, sp, lds, s_flag, pf.tid);
          else
            run_block_any<DT, false, false>(P_mem, T_mem, (int)T.m_len, (int)T.n_len, sp, lds, s_flag, pf.tid);
        }
      }
    }
    if (ANY_ALIGNMENT && !pieces) {
    } else if (WINDOW && cls == CLS_WINDOW) {
      if constexpr (WINDOW) run_window<DT>(P, T, lds, pf);
    } else if (cls == 0) {
      run_skinny<DT, 1, ANY_ALIGNMENT>(P, T, sp, lds, s_flag, pf);
    } else if (cls == 3) {
      run_skinny<DT, 2, ANY_ALIGNMENT>(P, T, sp, lds, s_flag, pf);
    } else if (cls == 6) {
      run_skinny<DT, 4, ANY_ALIGNMENT>(P, T, sp, lds, s_flag, pf);
    } else if (cls == CLS_TILE_128x64) {
      run_lds_tile<DT, 128, 64, false>(P, T, sp, lds, s_flag, pf);
    } else {
      run_lds_tile<DT, 128, 128, false>(P, T, sp, lds, s_flag, pf);
    }
  }
}

// ONLY_DT >= 0: every operator of the plan has that element type (one third of the
// code, fewer registers); ONLY_DT < 0: operators of mixed types.
// ANY_ALIGNMENT false: every operator can be read in aligned 16-byte pieces, and the kernel
// does not carry the paths for the others (their calls cost the fast paths registers and a
// stack); true: operators of either kind.
// NARROW: every tile of the plan is a lean 128 x 64 tile (see NARROW_LDS_BYTES).
template <int ONLY_DT, bool ANY_ALIGNMENT, bool NARROW>
__global__ void __launch_bounds__(WG_THREADS, NARROW ? 3 : 2) sk_superkernel(const TileWork *__restrict__ work, KernelArgs a) {
  __shared__ __attribute__((aligned(16))) unsigned char lds[NARROW ? NARROW_LDS_BYTES : LDS_TILE_BYTES];
  // By parity: [0] the next record's ticket, [1] flags (MAIL_*), [2] its index in xwork, [3] the ticket that waits while it runs.
  // (Wave 0 has fetched the record itself ahead of time, which brings it into the L2 for everyone's load_record.)
  __shared__ __attribute__((aligned(16))) uint32_t s_mail[2][4];
  __shared__ uint32_t s_flag;
  const SplitK sp{a.ws, a.ws_off, a.arrive};
  enum : uint32_t { MAIL_RUN = 1, MAIL_FROM_LIST = 2, MAIL_PENDING = 4, MAIL_OWES = 8 };

  // Start of the launch = the earliest first clock of any workgroup (the host has set the slot to all ones).
  if (a.write_start && a.stamps && threadIdx.x == 0)
    __hip_atomic_fetch_min((unsigned long long *)&a.stamps[a.n_problems], (unsigned long long)wall_clock64(),
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);

  // Tickets and lists.  The queue hands out positions of the table in order ("tickets"); the first ticket of
  // a workgroup is its block index.  A ticket that falls on a skinny tile is that tile.  A ticket that
  // falls on an LDS tile only says that one LDS tile is due: which one, the workgroup takes from the list
  // of its die (the host has sorted every LDS tile of the table into one of eight lists so that tiles
  // sharing operand panels meet behind one L2; workgroups go to the dies round robin by block index), and
  // from the other dies' lists once its own is used up.  While an LDS tile runs, the next entry of the
  // list is drawn together with the next ticket (Prefetch), on the guess that the ticket falls on an LDS
  // tile again; if it falls on a skinny tile instead, the entry runs first and the ticket's tile right after
  // it (its record is fetched while the entry runs, no new ticket is taken).  Work that is bound to a
  // workgroup is thus always its very next tile: an entry held back until the workgroup's next LDS ticket
  // left dozens of workgroups with a tile still to run when the tickets ran out, and cost mixed plans a
  // tenth of their time.  Such an entry ran without a ticket: the workgroup owes one, and the next ticket of
  // its own that falls on an LDS tile stands for nothing (it takes another ticket at once, and draws nothing
  // in advance while it owes).  Without that the LDS tiles as a whole ran ahead of their tickets by one tile
  // per wrong guess, and the launch ended on long skinny tiles with nothing short left to fill in.  What is
  // still owed when the tickets run out shows as tickets that find every list empty.  Every entry is drawn
  // exactly once and run by the workgroup that drew it, so every tile of the table runs exactly once.
  const uint32_t last = a.tile_end - 1u;
  const bool lists = a.xoff != nullptr;
  const uint32_t die = blockIdx.x & 7u;
  uint32_t xbeg = 0, xlen = 0;
  if (lists) {
    xbeg = a.xoff[die];
    xlen = a.xoff[die + 1] - xbeg;
  }
  uint32_t used_up = xlen == 0 ? 1u << die : 0u;  // lists seen empty (wave 0's copy is the one that counts)
  bool owes = false;                               // an entry of a list has run without a ticket

  const int wave0 = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) == 0;
  const int lane0 = (int)(threadIdx.x & 63u);
  const int wlane = lane0 < WORK_DWORDS ? lane0 : 0;
  // What the tile just run fetched for the next one (Prefetch): lane 0 of `got` holds the ticket (less
  // `got_base`), lane 1 the entry drawn from the die's list if `drew`; `got_word` the record of the ticket,
  // or, if `drew`, the record of that entry with the ticket's tile class in lane 63.
  uint32_t got = blockIdx.x, got_base = a.tile_begin;
  uint32_t got_word = 0;
  if (wave0) got_word = as_global<uint32_t>(work + (a.tile_begin + blockIdx.x <= last ? a.tile_begin + blockIdx.x : last))[wlane];
  bool drew = false;
  bool have_done = false;  // a tile has just been run: its operator and that operator's tile count
  uint32_t done_problem = 0, done_count = 0;
  int par = 0;
#ifdef SK_DIAG_CLOCKS
  int diag_tile = 0;
#endif
  for (;;) {
    if (wave0) {
      // wave 0 decides what runs next and hands the record to the other waves
      uint32_t idx = (uint32_t)__builtin_amdgcn_readfirstlane((int)got) + got_base;
      uint32_t word = got_word, flags = 0, xi = 0, waits = 0;
      if (!lists) {
        flags = idx <= last ? MAIL_RUN : 0u;
      } else {
        const uint32_t k = drew ? (uint32_t)__builtin_amdgcn_readlane((int)got, 1) : 0u;
        bool drawn = drew && k < xlen;  // `word` is the record of entry k of the die's list
        if (drew && !drawn) used_up |= 1u << die;
        bool have_record = !drew;       // `word` is the table's record at the ticket
        for (;;) {
          const bool ticket = idx <= last;
          // the ticket's tile class: sk_tile's dword 1, low half
          const uint32_t cls = (uint32_t)__builtin_amdgcn_readlane((int)word, have_record ? 1 : 63) & 0xffffu;
          if (ticket && cls >= CLS_TILE_128x128) {
            if (owes) {  // this ticket pays for the entry that ran without one
              owes = false;
              uint32_t n2 = 0;
              if (lane0 == 0) n2 = atomicAdd(&a.counters[0], 1u);
              idx = (uint32_t)__builtin_amdgcn_readfirstlane((int)n2) + a.tile_begin + gridDim.x;
              word = as_global<uint32_t>(work + (idx <= last ? idx : last))[wlane];
              have_record = true;
              continue;
            }
            if (drawn) {
              xi = xbeg + k;
              flags = MAIL_RUN | MAIL_FROM_LIST;
              break;
            }
            // nothing in hand: draw now, from the own list first
            bool found = false;
            for (uint32_t d = 0; d < 8u && !found; ++d) {
              const uint32_t x2 = (die + d) & 7u;
              if ((used_up >> x2) & 1u) continue;
              const uint32_t b2 = a.xoff[x2], l2 = a.xoff[x2 + 1] - b2;
              uint32_t k2 = l2;
              if (l2 != 0 && lane0 == 0) k2 = atomicAdd(die_list_head(a.counters, x2), 1u);
              k2 = (uint32_t)__builtin_amdgcn_readfirstlane((int)k2);
              if (k2 < l2) {
                xi = b2 + k2;
                found = true;
              } else {
                used_up |= 1u << x2;
              }
            }
            if (found) {
              word = as_global<uint32_t>(a.xwork + xi)[wlane];
              flags = MAIL_RUN | MAIL_FROM_LIST;
              break;
            }
            // every list is empty: the tile this ticket stood for has run already; take the next ticket
            uint32_t n2 = 0;
            if (lane0 == 0) n2 = atomicAdd(&a.counters[0], 1u);
            idx = (uint32_t)__builtin_amdgcn_readfirstlane((int)n2) + a.tile_begin + gridDim.x;
            word = as_global<uint32_t>(work + (idx <= last ? idx : last))[wlane];
            have_record = true;
            continue;
          }
          if (ticket) {  // a skinny tile: the ticket is the tile
            if (drawn) {  // the entry drawn in advance runs first; the ticket's tile follows it
              xi = xbeg + k;
              waits = idx;
              owes = true;
              flags = MAIL_RUN | MAIL_FROM_LIST | MAIL_PENDING;
            } else {
              flags = MAIL_RUN;
              // (a draw that found the list used up has left no record of the ticket)
              if (!have_record) word = as_global<uint32_t>(work + idx)[wlane];
            }
            break;
          }
          // the tickets are used up: run what is still in hand
          idx = last;
          if (drawn) {
            xi = xbeg + k;
            flags = MAIL_RUN | MAIL_FROM_LIST;
          }
          break;
        }
        if (owes) flags |= MAIL_OWES;
      }
      if (lane0 == 0) {
        s_mail[par][0] = idx;
        s_mail[par][1] = flags;
        s_mail[par][2] = xi;
        s_mail[par][3] = waits;
      }
    }
    __syncthreads();
    if (a.remaining && have_done && threadIdx.x == 0) {
      // the workgroup that retires an operator's last tile stamps it and re-arms the count
      const uint32_t left = atomicSub(&a.remaining[done_problem], 1u);
      if (left == 1u) {
        a.stamps[done_problem] = wall_clock64();
        a.remaining[done_problem] = done_count;
      }
    }
    const uint32_t flags = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_mail[par][1]);
#ifdef SK_DIAG_CLOCKS
    if (have_done) {
      SK_DIAG(5);
      ++diag_tile;
    }
#endif
    if (!(flags & MAIL_RUN)) break;
    const uint32_t t = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_mail[par][0]);
    const TileWork *cur =
        (flags & MAIL_FROM_LIST) ? a.xwork + (uint32_t)__builtin_amdgcn_readfirstlane((int)s_mail[par][2]) : work + t;
    // (wave 0 has fetched the record ahead of time: it is in this die's L2)
    const TileWork W = load_record(cur);
    const bool pending = (flags & MAIL_PENDING) != 0;  // a ticket waits: this tile takes no new one
    owes = (flags & MAIL_OWES) != 0;
    const uint32_t waits = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_mail[par][3]);
    par ^= 1;

    // Everything a tile derives from the thread index is derived again for each tile, from a
    // copy the compiler cannot see through: hoisted out of this loop those values would stay
    // live across all tile classes, spill, and every reload of a spilled register waits for all
    // the loads and stores in flight.
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const bool queue = a.dynamic && !pending;
    Prefetch pf{work, queue ? &a.counters[0] : nullptr, queue ? a.tile_begin + gridDim.x : 0u,
                pending ? waits : t + gridDim.x, last, tid, cur};
    const sk_tile &T = W.tile;
    drew = lists && T.cls >= CLS_TILE_128x128 && !pending && !owes && !((used_up >> die) & 1u);
    if (drew) {
      pf.xhead = die_list_head(a.counters, die);
      pf.xrec = a.xwork + xbeg;
      pf.xlen = xlen;
    }
#ifdef SK_DIAG_CLOCKS
    pf.diag_tile = diag_tile;
#endif
    SK_DIAG(0);
#ifdef SK_DIAG_CLOCKS
    if (blockIdx.x < SK_DIAG_WGS && diag_tile < SK_DIAG_TILES && threadIdx.x == 0)
      g_diag[(blockIdx.x * SK_DIAG_TILES + diag_tile) * 8 + 6] = 1 + T.cls + 100ull * T.S;
    if (blockIdx.x < SK_DIAG_WGS && diag_tile < SK_DIAG_TILES && threadIdx.x == 0)
      g_diag[(blockIdx.x * SK_DIAG_TILES + diag_tile) * 8 + 7] = ((uint64_t)flags << 32) | t;  // how it was handed over, and the ticket
#endif
    const DevProblem &P = W.prob;
    if constexpr (ONLY_DT >= 0) {
      run_class<ONLY_DT, ANY_ALIGNMENT, NARROW, !ANY_ALIGNMENT && !NARROW && ONLY_DT != SK_F32, false>(P, T, &cur->prob, &cur->tile, sp, lds, &s_flag, pf);
    } else {
      switch (P.dtype) {
        case SK_BF16: run_class<SK_BF16, ANY_ALIGNMENT, NARROW, false, true>(P, T, &cur->prob, &cur->tile, sp, lds, &s_flag, pf); break;
        case SK_F16: run_class<SK_F16, ANY_ALIGNMENT, NARROW, false, true>(P, T, &cur->prob, &cur->tile, sp, lds, &s_flag, pf); break;
        default: run_class<SK_F32, ANY_ALIGNMENT, NARROW, false, true>(P, T, &cur->prob, &cur->tile, sp, lds, &s_flag, pf); break;
      }
    }

    if (a.remaining) __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    got = pf.next;
    got_base = pf.base;
    got_word = pf.word;
    have_done = true;
    if (a.remaining) {
      const TileWork again = load_record(cur);
      done_problem = again.tile.problem;
      done_count = (uint32_t)again.prob.tile_count;
    }
  }

  // the last workgroup to leave re-arms the queue for the next launch
  if (a.dynamic && threadIdx.x == 0) {
    const uint32_t done = atomicAdd(&a.counters[1], 1u);
    if (done == gridDim.x - 1) {
      a.counters[0] = 0u;
      a.counters[1] = 0u;
      if (lists)
        for (uint32_t x = 0; x < 8u; ++x) *die_list_head(a.counters, x) = 0u;
      __threadfence();
    }
  }
}

}  // namespace sk
