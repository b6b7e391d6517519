// Batched lookup kernels (gfx950) for packed layout 3: several to many activation rows (batched
// decode, prefill mpGEMM).
//
// Section 3.2 of the paper argues that the tables must sit in fast on-chip memory and that a large
// tile over M lets many weight rows reuse one table.  Here the tables of a K-slice and of NT = 4 or
// 8 activation rows live in LDS, laid out [table][entry][n] (NT fp16 values = 8 or 16 bytes per
// entry), and every LANE owns one weight row: a wavefront looks one table up for 64 rows at a
// time.  All lanes of a read address the same table, whose 16 entries cover the LDS banks evenly,
// so lanes that want the same entry are served by broadcast and lanes that want different entries
// hit different banks: the lookups are free of bank conflicts, and one lookup feeds NT
// activation rows.
//
//   * Weight permutation / interleaving (Section 3.2): a lane reads the `bits` index dwords of its
//     row and of one 32-k chunk with one load (16 bytes at 4 bit); the eight nibbles of a dword are
//     the indices of eight consecutive tables, and two mask-and-shift operations turn them into
//     the byte offsets of the entries (even and odd tables) four at a time.
//   * Aggregation: the eight entries of a chunk and plane are added as packed 16-bit pairs, two
//     activation rows per instruction, then widened.  Exact for integer tables (32-bit additions of
//     biased pairs, two entries per instruction: rows_int_bias).  For fp16 tables
//     this is this library's own choice and it is lossy (three fp16 roundings per chunk sum: about
//     1.5e-4 -> 3.4e-4 relative error, still a sixth of the 2e-3 bar); it is not the paper's "fast
//     8-bit aggregation" (Section 4), an integer averaging trick that is not built here.
//   * Bit-plane shift-accumulate (Eq. 1): the widening v_fma_mix_f32 takes the fp16 chunk sum and
//     multiplies by 2^i.
//   * Scale, zero and bias once per quantisation group (Section 4, bit-serial linear transform).
//     In the many-row kernel with fp16 tables the group's scale rides on the plane weights
//     (s/2 * 2^i, four multiplies when a group starts) and the bias term s * (mid - z) * S is
//     added at the same moment, so a group costs 12 instructions instead of 32 and the finished
//     group sums need no registers of their own; integer tables keep exact integer group sums
//     and convert once per group.
//   * Axis order (Section 3.2 "axis reordering"): K is walked slice by slice inside the
//     workgroup, so only a 32 KB slice of the tables is live in LDS; the sums of a row stay
//     in the lane's registers: fixed order.
//   * Few activation rows (batched decode) leave too few (row block, n tile) pairs to fill the
//     chip: K is then also split over gridDim.z workgroups, whose partial sums meet in the
//     workspace; rows_sum_kernel, the next kernel on the stream, adds them in slice order (fixed
//     order again) and writes the result.  Where that asks for slices of eight chunks (a handful
//     of activation rows), mpgemm_rows8_kernel further down takes the call instead.
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <type_traits>

#include "tmac.h"
#include "tmac_internal.h"

namespace tmac {

typedef uint32_t ru32x4v __attribute__((ext_vector_type(4)));
typedef uint32_t ru32x2v __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) char rows_lds_char;
// wave-uniform data that no running kernel writes: read through scalar loads into scalar registers
typedef __attribute__((address_space(4))) const float rows_const_float;
__device__ __forceinline__ rows_const_float* rows_const(const void* p) { return (rows_const_float*)(uintptr_t)p; }
typedef __attribute__((address_space(3))) const ru32x2v rows_lds_u32x2;
typedef __attribute__((address_space(3))) const ru32x4v rows_lds_u32x4;

#ifndef TMAC_ROWS_WAVES
#define TMAC_ROWS_WAVES 4
#endif
#ifndef TMAC_ROWS_TARGET_WGS
#define TMAC_ROWS_TARGET_WGS 4096
#endif
constexpr int ROWS_WAVES = TMAC_ROWS_WAVES;  // 64-row tiles per workgroup
constexpr int ROWS_TARGET_WGS = TMAC_ROWS_TARGET_WGS;  // K is split until a call has about this many workgroups
constexpr int ROWS_LDS = 32768;     // bytes of tables per LDS slice: 1024 k for 4 activation rows, 512 k for 8
constexpr int ROWS_RUN_WGS = 1024;         // four workgroups (one wavefront per SIMD each) per CU: what the chip holds at once
constexpr int ROWS_RUN_LONG = 163840;      // chunks from which there are twice as many
constexpr int ROWS_RUN_INT_CHUNKS = 12288; // chunks of pairs (RowsShare) from which the run serves a call: integer tables,
constexpr int ROWS_RUN_ACT_CHUNKS = 5000;  // ... fp16 tables built from activations, more than 32 rows,
constexpr int ROWS_RUN_ACT_BITS = 15000;   // ... times the bits,
constexpr int ROWS_RUN_ACT_FEW = 24576;    // ... up to 32 rows,
constexpr double ROWS_RUN_LUT_LOOKUPS = 0.75e9;  // ... fp16 tables from a LUT buffer: look-ups,
constexpr int ROWS_RUN_LUT_ROWS = 1536;    // ... and weight rows times bits (rows_plan)
constexpr int ROWS_NT_WIDE = 8;     // activation rows per workgroup when there are enough of them
constexpr int ROWS_NT_NARROW = 4;   // ... and otherwise
constexpr int64_t ROWS_SUM_WIDE = 1 << 19;  // outputs from which the slice sums go four to a thread (two wavefronts per SIMD)

typedef _Float16 rh2v __attribute__((ext_vector_type(2)));
typedef short rs2v __attribute__((ext_vector_type(2)));

// The call as one run of chunks, dealt out evenly.  A pair is a block of 256 weight rows and a set of 16
// activation rows; the pairs' chunks follow each other, weight rows fastest, and workgroup w takes the chunks
// [w total / wgs, (w + 1) total / wgs) of the run, whatever pairs they belong to.  What it has of one pair is
// one part of that pair's sums; a pair's parts are numbered from its first workgroup.  (Workgroups with one chunk
// more spread evenly over the run instead of its first ones: 0.95 to 1.02 times as fast, 0.985 on average of 22 calls.)
struct RowsShare {
  uint32_t wgs, per, more;      // workgroups, chunks of each; the first `more` take one more
  uint32_t row_blocks, chunks;  // blocks of 256 weight rows, chunks of a pair
  uint32_t inv_row_blocks, inv_chunks;  // rows_inverse() of the two
  __device__ uint32_t start(uint32_t wg) const { return wg * per + min(wg, more); }
  __device__ uint32_t owner(uint32_t chunk) const {
    const uint32_t head = more * (per + 1);
    return chunk < head ? chunk / (per + 1) : more + (chunk - head) / per;
  }
  __device__ uint32_t first(uint32_t pair) const { return owner(pair * chunks); }
  __device__ int parts(uint32_t pair) const { return (int)(owner((pair + 1) * chunks - 1) - first(pair)) + 1; }
};
// n / d = the high half of n * rows_inverse(d, n) for n d < 2^32 and d > 1; 0 else, for a division
inline uint32_t rows_inverse(uint32_t d, uint64_t n) { return d > 1 && n * d < 0x100000000ull ? (uint32_t)((0x100000000ull + d - 1) / d) : 0u; }
__device__ __forceinline__ uint32_t rows_div(uint32_t n, uint32_t d, uint32_t inverse) { return inverse ? __umulhi(n, inverse) : n / d; }

// Grid of the eight-chunk kernel (n tiles, row blocks, K slices): slices of whole quantisation groups, of equal length
// but for one.
struct Rows8Grid {
  int per, more;          // groups (chunks, where there are none) of a slice; the first `more` take one more
  uint32_t inv_x, inv_y;  // rows_inverse() of n tiles and row blocks
};

struct RowsParams {
  const uint32_t* idx;     // [n_tiles][n_chunks][64][bits] dwords
  const uint32_t* sz;      // [n_tiles][nq][64] {fp16 scale, fp16 zero}
  const uint16_t* tables;  // [n tile][KG][2^g][NT] fp16 or int16: the LDS layout, n tile by n tile
  const void* S;           // [N][nq] fp32 / int32 group sums
  void* out;
  const float* act_scale;
  int64_t ldo;
  int M, N, KG, n_tiles, n_chunks, nq;
  int cpg;                 // 32-k chunks per quantisation group (grouped mode)
  int cpg_log2;            // its logarithm when it is a power of two (the eight-chunk kernel needs one)
  int cps;                 // 32-k chunks per workgroup along K (a multiple of cpg); gridDim.z slices
  int slices;              // K slices of the eight-chunk kernel (gridDim.z)
  Rows8Grid grid8;
  int Mp;                  // M rounded up to 64
  float* ws_part;          // split K: [slices][N][Mp] partial sums (fp32, or int32 bit patterns)
  float* ws_srow;          // fused table build, one scale per row or tensor: [slices][N] sums of the
                           // activations of a K slice (fp32, or int32 bit patterns)
  int grouped;             // 1: group scales, 0: one scale per row or per tensor
  int per_tensor, int_exact, icoef;
  float wscale, zero_point, mid;
  const void* A;           // fused table build: activations [N][lda], fp16 or int8 (else unused)
  int64_t lda;
  int K;
  float pw[4];             // plane weights 1, 2, 4, 8: kernel arguments, so that plane 0 also takes the
                           // fused convert-multiply-add (a literal 1.0 would be folded into cvt + add)
  int out_t;
  const float* fix_scale;  // fixed-point tables: [set of 16 rows][chunk >> fix_shift][16] value of one unit (-0: entries not finite)
  int fix_shift;           // 2: one unit per 128-k block, 0: one per chunk (see rows_fix_kernel)
  uint16_t* raw;           // ... and the fp16 tables, as in a LUT buffer, where a unit is -0
  int lut_nt, raw_nt;      // activation rows of an n tile of the LUT buffer, 4 or 8 (rows_nt), and of raw
  RowsShare share;         // mpgemm_run_kernel and its sums: which part of the call a workgroup serves (the other kernels, which
                           // take K slices of equal length, do not read it)
};

// 32-k chunks of tables one LDS slice holds, for LUT group size g and nt activation rows
constexpr int rows_lds_chunks(int g, int nt) { return ROWS_LDS / ((32 / g) * (1 << g) * 2 * nt); }

// a[0] = sum of a[0..N), added pairwise: ((a0 + a1) + (a2 + a3)) + ...
template <typename T, int N>
__device__ __forceinline__ void tree_sum(T (&a)[N]) {
#pragma unroll
  for (int s = 1; s < N; s *= 2) {
#pragma unroll
    for (int i = 0; i + s < N; i += 2 * s) a[i] += a[i + s];
  }
}


// PAD: bytes from table to table beyond its own, for kernels that build the tables a table per lane: without them
// all tables start at the same LDS bank and the lanes' stores come one after the other.  A look-up reads one table,
// wherever it starts.
template <int NT, int G, int PAD = 0>
struct RowsShape {
  static constexpr int ENT = 1 << G;          // entries per table
  static constexpr int ES = 2 * NT;           // bytes per entry: NT 16-bit values
  static constexpr int TB = ENT * ES + PAD;   // bytes per table
  static constexpr int TPC = 32 / G;          // tables, i.e. lookups per plane, of a 32-k chunk
  static constexpr int CB = (TPC * TB + 255) / 256 * 256;  // bytes per chunk
  static constexpr int HD = NT / 2;           // dwords per entry
};


// Integer tables in LDS hold their entries plus 128 g, which makes them non-negative 16-bit values
// (|entry| <= 128 g), so that two of them side by side in a dword are added by plain 32-bit additions
// without a carry from one to the other: v_add3_u32 adds two entries' pairs in the time v_pk_add_i16
// takes for one (1.8 ns per wavefront and SIMD each).  The 32 / g entries of a chunk and plane add up to
// their sum plus ROWS_CHUNK_BIAS, at most twice that; planes 0..2 fit 16 bits together with their
// weights 1, 2, 4 (7 * 8192 < 65536).
constexpr int rows_int_bias(int g) { return 128 * g; }
constexpr int ROWS_CHUNK_BIAS = 4096;  // (32 / g) * 128 g

// l += (one half of pair) * W: the widening of a 16-bit sum, one instruction
template <int W>
__device__ __forceinline__ void rows_widen(int& l0, int& l1, uint32_t pair) {
  asm("v_mad_u32_u16 %0, %1, %2, %0" : "+v"(l0) : "v"(pair), "n"(W));
  asm("v_mad_u32_u16 %0, %1, %2, %0 op_sel:[1,0,0,0]" : "+v"(l1) : "v"(pair), "n"(W));
}

// l = start + (one half of pair) * W
template <int W>
__device__ __forceinline__ void rows_widen_from(int& l0, int& l1, uint32_t pair, int start) {
  asm("v_mad_u32_u16 %0, %1, %2, %3" : "=v"(l0) : "v"(pair), "n"(W), "s"(start));
  asm("v_mad_u32_u16 %0, %1, %2, %3 op_sel:[1,0,0,0]" : "=v"(l1) : "v"(pair), "n"(W), "s"(start));
}

// Algorithm 1 Precompute for one (activation row, LUT group of four) inside a lookup kernel:
// entries 0..7 of the table, as four dwords of two 16-bit entries, with the arithmetic
// of the stand-alone precompute kernel ((+-a0 +- a1) + (+-a2 - a3), every addition in fp16;
// entries 8..15 are the negated entries 7..0: mirror consolidation, Section 3.3).  Integer entries come
// with their bias (rows_int_bias).  a: the four activations, int8 in the first dword.
template <bool IS_INT>
__device__ __forceinline__ void rows_half_table(ru32x2v a, uint32_t (&low)[4]) {
  if constexpr (IS_INT) {
    const int a0 = (int8_t)(a.x & 0xff), a1 = (int8_t)((a.x >> 8) & 0xff), a2 = (int8_t)((a.x >> 16) & 0xff), a3 = (int8_t)(a.x >> 24);
    int e[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) e[q] = ((q & 1) ? a0 : -a0) + ((q & 2) ? a1 : -a1) + ((q & 4) ? a2 : -a2) - a3;
#pragma unroll
    for (int d = 0; d < 4; ++d) low[d] = ((uint32_t)e[2 * d] + ((uint32_t)e[2 * d + 1] << 16)) + (uint32_t)rows_int_bias(4) * 0x10001u;
  } else {
    half_table_f16(a.x, a.y, low);
  }
}

// Stage a K slice of tables into LDS: the LUT buffer holds them in the LDS layout, so this is a copy,
// `per` 16-byte pieces per thread, all loads requested before the first store; consecutive lanes
// write consecutive 16 bytes (no bank conflicts).  Tables from kg_end on are written as zeros.
// Integer entries get their bias on the way.
template <bool IS_INT, int NT, int G, int BYTES>
__device__ __forceinline__ void rows_stage_copy(const RowsParams& p, char* tab, int ntile, int kg0, int kg_end) {
  using Sh = RowsShape<NT, G>;
  constexpr int THREADS = 64 * ROWS_WAVES, PER = BYTES / 16 / THREADS;
  static_assert(PER >= 1 && BYTES % (16 * THREADS) == 0, "whole pieces per thread");
  const char* src = reinterpret_cast<const char*>(p.tables) + ((size_t)ntile * p.KG + (size_t)kg0) * Sh::TB;
  // (pieces of tables from kg_end on read the slice's first piece instead and are zeroed afterwards:
  // no branches between the loads)
  const int live_bytes = max(kg_end - kg0, 0) * Sh::TB;
  ru32x4v v[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int off = (i * THREADS + (int)threadIdx.x) * 16;
    v[i] = *reinterpret_cast<const ru32x4v*>(src + (off < live_bytes ? off : 0));
  }
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int off = (i * THREADS + (int)threadIdx.x) * 16;
    const ru32x4v z = {0u, 0u, 0u, 0u};
    ru32x4v e = off < live_bytes ? v[i] : z;
    if constexpr (IS_INT) {
      constexpr short be = (short)rows_int_bias(G);
#pragma unroll
      for (int d = 0; d < 4; ++d) e[d] = __builtin_bit_cast(uint32_t, (rs2v)(__builtin_bit_cast(rs2v, (uint32_t)e[d]) + rs2v{be, be}));
    }
    *reinterpret_cast<ru32x4v*>(tab + off) = e;
  }
}

// Build and stage tables in one go (tables from the activations, g = 4): item `it` is a table, counted from table
// kg0, of four activation rows (of eight, the first or second four), written entry-major [table][entry][n], eight bytes
// an entry.  Tables from kg_end on are written as zeros.
// First the activations are requested, without a branch in between (clamped addresses): loads behind a
// branch each come one after the other.  us from the start of the kernel until all tables are there, 16 rows x 11008 x
// 4096, 4 bit: 9.5 with a branch before each load, half a table of eight rows for each lane and the tables' first
// entries in the same LDS bank, 3.4 like this.
template <int NT, bool IS_INT>
__device__ __forceinline__ void rows_item_load(const RowsParams& p, ru32x2v (&a)[4], int it, int n0, int kg0) {
  const int k = min(4 * (kg0 + it / (NT / 4)), p.K - 4), n = n0 + it % (NT / 4) * 4;
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int64_t at = min(n + t, p.N - 1) * p.lda + k;
    if constexpr (IS_INT) a[t] = ru32x2v{*reinterpret_cast<const uint32_t*>(static_cast<const int8_t*>(p.A) + at), 0u};
    else a[t] = *reinterpret_cast<const ru32x2v*>(static_cast<const __half*>(p.A) + at);
  }
}

template <int NT, bool IS_INT, int PAD>
__device__ __forceinline__ void rows_stage_item(const RowsParams& p, char* tab, const ru32x2v (&a)[4], int it, int n0, int kg0, int kg_end) {
  using Sh = RowsShape<NT, 4, PAD>;
  const int table = it / (NT / 4), kg = kg0 + table, n = n0 + it % (NT / 4) * 4;
  uint32_t low[4][4];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const bool live = n + t < p.N && kg < kg_end && 4 * kg < p.K;
    rows_half_table<IS_INT>(live ? a[t] : ru32x2v{0u, 0u}, low[t]);
  }
  char* const dst = tab + table / Sh::TPC * Sh::CB + table % Sh::TPC * Sh::TB + it % (NT / 4) * 8;
#pragma unroll
  for (int d = 0; d < 4; ++d) {  // dword d of every row holds entries 2d, 2d+1
    const ru32x2v even = {__builtin_amdgcn_perm(low[1][d], low[0][d], 0x05040100u), __builtin_amdgcn_perm(low[3][d], low[2][d], 0x05040100u)};
    const ru32x2v odd = {__builtin_amdgcn_perm(low[1][d], low[0][d], 0x07060302u), __builtin_amdgcn_perm(low[3][d], low[2][d], 0x07060302u)};
    // entry 15 - e = -(entry e): sign bits flipped, or subtracted from twice the bias
    auto mirror = [](ru32x2v e) {
      if constexpr (IS_INT) return (2u * (uint32_t)rows_int_bias(4) * 0x10001u) - e;
      else return e ^ 0x80008000u;
    };
    *reinterpret_cast<ru32x2v*>(dst + (2 * d) * Sh::ES) = even;
    *reinterpret_cast<ru32x2v*>(dst + (2 * d + 1) * Sh::ES) = odd;
    *reinterpret_cast<ru32x2v*>(dst + (15 - 2 * d) * Sh::ES) = mirror(even);
    *reinterpret_cast<ru32x2v*>(dst + (14 - 2 * d) * Sh::ES) = mirror(odd);
  }
}

// The lookups of one 32-k chunk: x = the lane's `BITS` index dwords, cbase = LDS byte address of
// the chunk's first table (low byte zero); L += sum over planes of 2^plane * (sum of the looked-up
// entries), per activation row.
// With OCT = 2 the workgroup serves two sets of NT activation rows whose tables sit OSTRIDE bytes
// apart in LDS: one address (one permute) then feeds two reads, and L holds 2 NT sums.
template <bool IS_INT, int BITS, int NT, int G, typename AccT, int OCT = 1, int OSTRIDE = 0, int PAD = 0>
__device__ __forceinline__ void rows_chunk(const uint32_t (&x)[BITS], uint32_t cbase, AccT (&L)[NT * OCT],
                                           const float (&pw)[4]) {
  using Sh = RowsShape<NT, G, PAD>;
  constexpr int TPC = Sh::TPC, HD = Sh::HD, TB = Sh::TB;
  static_assert(OCT == 1 || (OCT == 2 && NT == 8 && TPC * OCT <= 16), "two row sets: eight rows each, g = 4");
  // rounds of 16 LDS reads (one, two or four planes at g = 2, 4, 8): the hardware counts at
  // most 15 outstanding LDS operations exactly, so a round's reads can be consumed as they return
  constexpr int PL = 16 / (TPC * OCT);
  uint32_t c[OCT * HD];  // integer tables: the planes of a widening with their weights, as biased 16-bit pairs
#pragma unroll
  for (int b0 = 0; b0 < BITS; b0 += PL) {
    uint32_t e[PL][TPC][OCT * HD];
#pragma unroll
    for (int bb = 0; bb < PL; ++bb) {
      const int b = b0 + bb;
      if (b >= BITS) break;
      // byte offsets of the entries inside their tables (entry * ES), four tables per dword
      uint32_t off[4];
      if constexpr (G == 4) {
        off[0] = (NT == 4) ? (x[b] << 3) & 0x78787878u : (x[b] << 4) & 0xF0F0F0F0u;  // even tables
        off[1] = (NT == 4) ? (x[b] >> 1) & 0x78787878u : x[b] & 0xF0F0F0F0u;         // odd tables
      } else if constexpr (G == 2) {
        // field r of byte i is table 4 i + r
        if constexpr (NT == 4) {
          off[0] = (x[b] << 3) & 0x18181818u; off[1] = (x[b] << 1) & 0x18181818u;
          off[2] = (x[b] >> 1) & 0x18181818u; off[3] = (x[b] >> 3) & 0x18181818u;
        } else {
          off[0] = (x[b] << 4) & 0x30303030u; off[1] = (x[b] << 2) & 0x30303030u;
          off[2] = x[b] & 0x30303030u;        off[3] = (x[b] >> 2) & 0x30303030u;
        }
      }
#pragma unroll
      for (int j = 0; j < TPC; ++j) {
        uint32_t a;
        if constexpr (G == 8) {
          a = cbase + ((x[b] >> (8 * j)) & 0xffu) * (uint32_t)Sh::ES;
        } else {
          // address = {0, cbase byte 2, cbase byte 1, one byte of the offsets}: one byte permute;
          // the table's own TB * j goes into the instruction's offset field
          constexpr int FPB = 8 / G;  // index fields per byte
          a = __builtin_amdgcn_perm(off[j % FPB], cbase, 0x0C020100u + 4u + (uint32_t)(j / FPB));
        }
        if constexpr (NT == 4) {
          const ru32x2v r = *reinterpret_cast<rows_lds_u32x2*>(a + j * TB);
          e[bb][j][0] = r.x; e[bb][j][1] = r.y;
        } else {
#pragma unroll
          for (int o = 0; o < OCT; ++o) {
            const ru32x4v r = *reinterpret_cast<rows_lds_u32x4*>(a + j * TB + o * OSTRIDE);
            e[bb][j][4 * o + 0] = r.x; e[bb][j][4 * o + 1] = r.y; e[bb][j][4 * o + 2] = r.z; e[bb][j][4 * o + 3] = r.w;
          }
        }
      }
    }
    __builtin_amdgcn_sched_barrier(0);  // keep the reads above the accumulation
    // fp16 tables: the entries of a plane (one per table of the chunk) are added pairwise as packed
    // fp16 values, two activation rows per instruction: log2(32/g) roundings to fp16 (lossy, this
    // library's choice: the widening happens once per chunk and plane); the chunk sum then enters the
    // 32-bit sum of the quantisation group times 2^plane.  Integer tables: exact, see rows_int_bias; the
    // biases of a chunk, ROWS_CHUNK_BIAS * (2^BITS - 1), are in L's start value.
#pragma unroll
    for (int bb = 0; bb < PL; ++bb) {
      const int b = b0 + bb;
      if (b >= BITS) break;
#pragma unroll
      for (int u = 0; u < OCT * HD; ++u) {
        if constexpr (IS_INT) {
          uint32_t q = e[bb][0][u];
#pragma unroll
          for (int j = 1; j < TPC; ++j) q += e[bb][j][u];
          // (four planes: two and two, so that no sum stays in registers through the next round of reads; three and one made
          // the eight-chunk kernel spill 13 registers)
          constexpr int PLANES = BITS == 4 ? 2 : 3;
          c[u] = b % PLANES == 0 ? q : c[u] + (q << (b % PLANES));
          if (b == PLANES - 1 || (b < PLANES && b == BITS - 1)) rows_widen<1>(L[2 * u], L[2 * u + 1], c[u]);
          else if (b == BITS - 1) rows_widen<1 << PLANES>(L[2 * u], L[2 * u + 1], c[u]);
        } else {
          rh2v q[TPC];
#pragma unroll
          for (int j = 0; j < TPC; ++j) q[j] = __builtin_bit_cast(rh2v, e[bb][j][u]);
          tree_sum(q);
          const float w = pw[b];
          L[2 * u] = fmaf((float)q[0].x, w, L[2 * u]);
          L[2 * u + 1] = fmaf((float)q[0].y, w, L[2 * u + 1]);
        }
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  }
}

// The same for integer tables in the many-row kernel's usual shape (eight activation rows, g = 4), in
// rounds of the eight reads of one plane and row set instead of sixteen: a round's entries take 32
// registers, which leaves room for more wavefronts, and a SIMD's wavefronts cover each other's reads.
// Bound by the look-up rate of LDS and the vector ALUs about equally: per plane and 16 activation rows
// sixteen reads (110 ns with four wavefronts on the CU's four SIMDs) and 11 address, 32 adding and 8 to
// 16 widening instructions (95 ns).  128 rows x 8640 x 3200 at 2 bit: 67.8 us with packed 16-bit adds,
// 60.4 with rounds of sixteen reads, 53.8 like this (next round's reads ahead of a round's sums: 60.0).
// fp16 tables gain nothing from the shorter rounds (the vector ALUs bind there).
template <int BITS, int OCT, int OSTRIDE>
__device__ __forceinline__ void rows_chunk_int(const uint32_t (&x)[BITS], uint32_t cbase, int (&L)[8 * OCT]) {
  using Sh = RowsShape<8, 4>;
  constexpr int TPC = Sh::TPC, HD = Sh::HD, TB = Sh::TB;
  uint32_t c[OCT * HD];  // planes 0..2 with their weights, as biased 16-bit pairs
#pragma unroll
  for (int b = 0; b < BITS; ++b) {
    const uint32_t even = (x[b] << 4) & 0xF0F0F0F0u, odd = x[b] & 0xF0F0F0F0u;
    uint32_t a[TPC];
#pragma unroll
    for (int j = 0; j < TPC; ++j) a[j] = __builtin_amdgcn_perm(j & 1 ? odd : even, cbase, 0x0C020100u + 4u + (uint32_t)(j / 2));
#pragma unroll
    for (int o = 0; o < OCT; ++o) {
      ru32x4v e[TPC];
#pragma unroll
      for (int j = 0; j < TPC; ++j) e[j] = *reinterpret_cast<rows_lds_u32x4*>(a[j] + j * TB + o * OSTRIDE);
      __builtin_amdgcn_sched_barrier(0);  // keep the reads above the accumulation
#pragma unroll
      for (int u = 0; u < HD; ++u) {
        uint32_t q = e[0][u];
#pragma unroll
        for (int j = 1; j < TPC; ++j) q += e[j][u];
        int& l0 = L[8 * o + 2 * u];
        int& l1 = L[8 * o + 2 * u + 1];
        uint32_t& cc = c[o * HD + u];
        if (b < 3) {
          cc = b == 0 ? q : cc + (q << b);
          if (b == (BITS < 3 ? BITS - 1 : 2)) rows_widen<1>(l0, l1, cc);
        } else {
          rows_widen<8>(l0, l1, q);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

// Scale of activation row n (int8 activations quantised per token), 1 where there is none.
__device__ __forceinline__ float rows_act_scale(const RowsParams& p, int n) { return p.act_scale ? p.act_scale[n] : 1.0f; }

// Sum of activation row n from the LUT buffer (one scale per row or per tensor: nq = 1).
template <bool IS_INT>
__device__ __forceinline__ void rows_row_sum(const RowsParams& p, int n, float& Sf, int& Si) {
  Sf = 0.f;
  Si = 0;
  if (p.grouped) return;
  if constexpr (IS_INT) Si = static_cast<const int*>(p.S)[n];
  else Sf = static_cast<const float*>(p.S)[n];
}

// Last step for output (n, m): vf = finished group sums (group scales) or the raw look-up sum (fp
// tables), vi = the raw integer look-up sum; s, z = scale and zero of row m when there is one
// scale per row or per tensor; Sf / Si = the sum of activation row n in that case.  Returns the bits
// to store as fp32, or as int32 for TMAC_OUT_I32.
template <bool IS_INT>
__device__ __forceinline__ uint32_t rows_result(const RowsParams& p, float vf, int vi, float s, float z, float Sf, int Si,
                                                float as) {
  float res;
  int ires = 0;
  if (p.grouped) {
    res = vf * as;
  } else if constexpr (IS_INT) {
    const int St = Si;
    if (p.int_exact) {
      ires = (vi + p.icoef * St) >> 1;  // numerator is always even
      res = ((float)ires * as) * s;     // two roundings, left to right
    } else {
      res = (fmaf(p.mid - z, (float)St, 0.5f * (float)vi) * as) * s;
    }
  } else {
    const float St = Sf;
    res = (s * fmaf(p.mid - z, St, 0.5f * vf)) * as;
  }
  return p.out_t == TMAC_OUT_I32 ? (uint32_t)ires : __float_as_uint(res);
}

template <bool IS_INT>
__device__ __forceinline__ void rows_finish(const RowsParams& p, int n, int m, float vf, int vi, float s, float z,
                                            float Sf, int Si, float as) {
  const uint32_t r = rows_result<IS_INT>(p, vf, vi, s, z, Sf, Si, as);
  const size_t o = (size_t)n * p.ldo + m;
  if (p.out_t == TMAC_OUT_F16) static_cast<__half*>(p.out)[o] = __float2half_rn(__uint_as_float(r));
  else static_cast<uint32_t*>(p.out)[o] = r;
}


// OCT = 2: the workgroup serves two n tiles of NT = 8 activation rows (their tables side by side in
// the two halves of the LDS slice), so that one address permute feeds two reads; the LUT buffer's
// n tiles stay eight rows wide.
template <bool IS_INT, int BITS, int NT, int G, int OCT>
__global__ __launch_bounds__(64 * ROWS_WAVES) void mpgemm_rows_kernel(const RowsParams p) {
  using Sh = RowsShape<NT, G>;
  constexpr int TPC = Sh::TPC, CB = Sh::CB;
  constexpr int CPS = rows_lds_chunks(G, NT) / OCT;  // 32-k chunks per slice
  constexpr int NTT = NT * OCT;                      // activation rows of the workgroup
  constexpr int OSTRIDE = ROWS_LDS / OCT;            // bytes between the two row sets' tables
  static_assert(CPS >= 1 && CB % 256 == 0, "chunk bases must keep a zero low byte");
  __shared__ __attribute__((aligned(2048))) char tab[ROWS_LDS];  // byte-permuted addresses need the alignment
  using AccT = typename std::conditional<IS_INT, int, float>::type;

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n0 = blockIdx.x * NTT;                      // activation rows of this workgroup
  const int tile_raw = blockIdx.y * ROWS_WAVES + wave;  // 64-row tile of this wave
  const bool tile_ok = tile_raw < p.n_tiles;
  const int tile = tile_ok ? tile_raw : p.n_tiles - 1;  // clamped: loads stay in range, stores are masked
  const uint32_t* my_idx = p.idx + ((size_t)tile * p.n_chunks * 64 + lane) * BITS;
  const uint32_t* my_sz = p.sz + (size_t)tile * p.nq * 64 + lane;
  const uint32_t lds0 = (uint32_t)(uintptr_t)((rows_lds_char*)tab);  // a multiple of 1024

  // fp tables: L is the running result, the plane weights w carry half the current group's scale and
  // the group's bias term is added when the group starts; integer tables (and one scale per row or
  // tensor): L is the raw look-up sum of the group (row), finished in acc at the group's end
  float acc[NTT];
  AccT L[NTT];
#pragma unroll
  for (int t = 0; t < NTT; ++t) acc[t] = 0.f;
  float w[4] = {p.pw[0], p.pw[1], p.pw[2], p.pw[3]};

  auto load_idx = [&](int c, uint32_t (&x)[BITS]) {
    const uint32_t* src = my_idx + (size_t)c * 64 * BITS;
    if constexpr (BITS == 4) {
      const ru32x4v v = *reinterpret_cast<const ru32x4v*>(src);
      x[0] = v.x; x[1] = v.y; x[2] = v.z; x[3] = v.w;
    } else if constexpr (BITS == 2) {
      const ru32x2v v = *reinterpret_cast<const ru32x2v*>(src);
      x[0] = v.x; x[1] = v.y;
    } else {
#pragma unroll
      for (int b = 0; b < BITS; ++b) x[b] = src[b];
    }
  };

  // this workgroup's share of K: chunks [cz0, cz1)
  const int cz0 = blockIdx.z * p.cps, cz1 = min(cz0 + p.cps, p.n_chunks);
  const int kg_end = min(cz1 * TPC, p.KG);  // tables beyond it are read as zero
  int gq = p.grouped ? cz0 / p.cpg : 0, cg = 0;  // current quantisation group, chunks done in it (wave-uniform)
  // {scale, zero} of the lane's row and the activation sums of a group (wave-uniform: scalar registers):
  // requested one group ahead for fp tables, which need them when the group starts, and when the group
  // starts for integer tables, which need them when it ends
  uint32_t szv = 0, szv_next = 0;
  AccT Sg[NTT], Sg_next[NTT];
  auto load_group = [&](int g) {
    const int gc = min(g, p.nq - 1);
    szv_next = my_sz[(size_t)gc * 64];
#pragma unroll
    for (int t = 0; t < NTT; ++t) {
      const int n = min(n0 + t, p.N - 1);
      Sg_next[t] = static_cast<const AccT*>(p.S)[(size_t)n * p.nq + gc];
    }
  };
#pragma unroll
  for (int t = 0; t < NTT; ++t) Sg[t] = Sg_next[t] = 0;
  if (p.grouped && !IS_INT) load_group(gq);
  // (integer tables: minus the biases of the chunks that enter one sum, a group's or this workgroup's)
  const AccT L0 = IS_INT ? (AccT)(-ROWS_CHUNK_BIAS * ((1 << BITS) - 1) * (p.grouped ? p.cpg : cz1 - cz0)) : (AccT)0;
#pragma unroll
  for (int t = 0; t < NTT; ++t) L[t] = L0;
  uint32_t xn[BITS];
  load_idx(cz0, xn);

  for (int c0 = cz0; c0 < cz1; c0 += CPS) {
    // stage the tables of this K-slice for the NT activation rows: item = (table, half) reads the
    // 8 entries of the four rows and writes them entry-major
    __syncthreads();
    {
      const int last8 = (p.N + NT - 1) / NT - 1;  // last n tile of the LUT buffer (a second row set past it repeats it)
#pragma unroll
      for (int o = 0; o < OCT; ++o)
        rows_stage_copy<IS_INT, NT, G, OSTRIDE>(p, tab + o * OSTRIDE, min((int)blockIdx.x * OCT + o, last8), c0 * TPC, kg_end);
    }
    __syncthreads();

    const int c_end = min(c0 + CPS, cz1);
    // Per chunk and pair of bit planes: 16 LDS reads are issued first, then accumulated in issue
    // order, so that the reads overlap each other and the accumulation of the earlier ones; the
    // other waves of the SIMD cover the start of every round.
    for (int c = c0; c < c_end; ++c) {
      uint32_t x[BITS];
#pragma unroll
      for (int b = 0; b < BITS; ++b) x[b] = xn[b];
      if (c + 1 < cz1) load_idx(c + 1, xn);  // next chunk's indices, one chunk ahead
      if (p.grouped && cg == 0 && gq < p.nq) {  // (chunks in the K padding belong to no group)
        if constexpr (IS_INT) load_group(gq);
        // (fp tables: the group's scale/zero and activation sums have been requested a group ago)
        szv = szv_next;
#pragma unroll
        for (int t = 0; t < NTT; ++t) Sg[t] = Sg_next[t];
        if constexpr (!IS_INT) {
          const float s = __half2float(__ushort_as_half((uint16_t)(szv & 0xffffu)));
          const float z = __half2float(__ushort_as_half((uint16_t)(szv >> 16)));
          const float hs = 0.5f * s, bz = s * (p.mid - z);
#pragma unroll
          for (int b = 0; b < 4; ++b) w[b] = hs * p.pw[b];
#pragma unroll
          for (int t = 0; t < NTT; ++t) L[t] = fmaf(bz, Sg[t], L[t]);  // bias term of Section 4's linear transform
        }
        // (the requests for the next group come after the last use of this group's values, so that they
        // can land in the same registers and nobody has to wait for them before the next group starts)
        if constexpr (!IS_INT) {
          __builtin_amdgcn_sched_barrier(0);
          load_group(gq + 1);
        }
      }
      const uint32_t cbase = lds0 + (uint32_t)(c - c0) * (uint32_t)CB;
      if constexpr (IS_INT && NT == 8 && G == 4) rows_chunk_int<BITS, OCT, OSTRIDE>(x, cbase, L);
      else rows_chunk<IS_INT, BITS, NT, G, AccT, OCT, OSTRIDE>(x, cbase, L, w);
      if (p.grouped && gq < p.nq && ++cg == p.cpg) {
        if constexpr (IS_INT) {
          const float s = __half2float(__ushort_as_half((uint16_t)(szv & 0xffffu)));
          const float z = __half2float(__ushort_as_half((uint16_t)(szv >> 16)));
#pragma unroll
          for (int t = 0; t < NTT; ++t) {
            acc[t] = fmaf(s, fmaf(p.mid - z, (float)Sg[t], 0.5f * (float)L[t]), acc[t]);
            L[t] = L0;
          }
        }
        cg = 0;
        ++gq;
      }
    }
  }

  // finish and store: lanes of a wave write 64 consecutive outputs of one activation row
  const int m = tile_raw * 64 + lane;
  const bool row_ok = tile_ok && m < p.M;
  float s = p.wscale, z = p.zero_point;
  if (!p.grouped && !p.per_tensor) {
    const uint32_t v = my_sz[0];
    s = __half2float(__ushort_as_half((uint16_t)(v & 0xffffu)));
    z = __half2float(__ushort_as_half((uint16_t)(v >> 16)));
  }
  auto finish = [&](int n, float vf, int vi) {
    float Sf;
    int Si;
    rows_row_sum<IS_INT>(p, n, Sf, Si);
    rows_finish<IS_INT>(p, n, m, vf, vi, s, z, Sf, Si, rows_act_scale(p, n));
  };
  constexpr bool RAW_INT = IS_INT;  // ungrouped integer tables: partial sums are exact integers
  const int nz = gridDim.z;
  if (nz == 1) {
    if (!row_ok) return;
#pragma unroll
    for (int t = 0; t < NTT; ++t) {
      if (n0 + t >= p.N) break;
      finish(n0 + t, (IS_INT && p.grouped) ? acc[t] : (float)L[t], IS_INT ? (int)L[t] : 0);
    }
    return;
  }

  // Split K: publish the partial sums with plain stores; rows_sum_kernel, launched behind this
  // kernel on the same stream, adds the slices in slice order and finishes.  The kernel boundary
  // orders the stores before the loads on every XCD (one L2 each); handing over inside the kernel
  // instead (release fence, arrival counter, acquire fence in the last workgroup) makes every
  // workgroup write back its L2, which cost more than the second launch at every size tried.
  const bool raw_int = RAW_INT && !p.grouped;
  if (tile_ok) {
#pragma unroll
    for (int t = 0; t < NTT; ++t) {
      const int n = n0 + t;
      if (n < p.N) {
        const size_t o = ((size_t)blockIdx.z * p.N + n) * p.Mp + (size_t)tile_raw * 64 + lane;
        p.ws_part[o] = (IS_INT && p.grouped) ? acc[t] : (raw_int ? __int_as_float((int)L[t]) : (float)L[t]);
      }
    }
  }
}

template <bool IS_INT, bool RUN = false>
static hipError_t launch_rows_sum(const RowsParams& p, int nz, hipStream_t st);

template <bool IS_INT, int BITS, int NT, int G, int OCT>
static hipError_t launch_rows_one(const RowsParams& p, hipStream_t st) {
  RowsParams local = p;
  void* args[] = {&local};
  const dim3 grid((p.N + NT * OCT - 1) / (NT * OCT), (p.n_tiles + ROWS_WAVES - 1) / ROWS_WAVES,
                  (p.n_chunks + p.cps - 1) / p.cps);
  hipError_t e = hipLaunchKernel(reinterpret_cast<const void*>(mpgemm_rows_kernel<IS_INT, BITS, NT, G, OCT>), grid,
                                 dim3(64 * ROWS_WAVES), args, 0, st);
  if (e != hipSuccess || grid.z == 1) return e;
  return launch_rows_sum<IS_INT>(p, (int)grid.z, st);
}

template <bool IS_INT, int NT, int G, int OCT = 1>
static hipError_t launch_rows_bits(const RowsParams& p, int bits, hipStream_t st) {
  switch (bits) {
    case 1: return launch_rows_one<IS_INT, 1, NT, G, OCT>(p, st);
    case 2: return launch_rows_one<IS_INT, 2, NT, G, OCT>(p, st);
    case 3: return launch_rows_one<IS_INT, 3, NT, G, OCT>(p, st);
    case 4: return launch_rows_one<IS_INT, 4, NT, G, OCT>(p, st);
  }
  return hipErrorInvalidValue;
}

// oct: n tiles per workgroup (2 only with g = 4 and eight-row n tiles)
template <bool IS_INT>
static hipError_t launch_rows_nt(const RowsParams& p, int g, int nt, int oct, int bits, hipStream_t st) {
  if (g == 8) return launch_rows_bits<IS_INT, ROWS_NT_NARROW, 8>(p, bits, st);  // (rows_nt: always narrow)
  if (g == 2)
    return nt == ROWS_NT_WIDE ? launch_rows_bits<IS_INT, ROWS_NT_WIDE, 2>(p, bits, st)
                              : launch_rows_bits<IS_INT, ROWS_NT_NARROW, 2>(p, bits, st);
  if (oct == 2) return launch_rows_bits<IS_INT, ROWS_NT_WIDE, 4, 2>(p, bits, st);
  return nt == ROWS_NT_WIDE ? launch_rows_bits<IS_INT, ROWS_NT_WIDE, 4>(p, bits, st)
                            : launch_rows_bits<IS_INT, ROWS_NT_NARROW, 4>(p, bits, st);
}


// ------------------------------------------------------------------------------------------
// Few activation rows: a slice of at most sixteen chunks per workgroup, sums finished by a second kernel
// ------------------------------------------------------------------------------------------
// With few activation rows a call is a chain of latencies, not a stream: the general kernel above
// asks for a chunk's indices one chunk ahead.  Here a workgroup's slice is at most sixteen chunks (512 k, g = 4;
// rows8_slices): all tables and the indices of eight chunks are requested in one go at the start, the
// partial sums are written with plain stores, and rows_sum_kernel, the
// next kernel on the stream, adds the slices in slice order and finishes.
// Slices of at most eight chunks are straight-line code; longer ones have a variant of their own that requests the other
// chunks' indices as places get free.  Where one variant with scales one group ahead served both, its waits for scales and
// the registers of its loop made short slices slow.  us, that variant and now (before there were longer slices): 2 x 1680 x
// 6112, 3 bit in groups of 32 12.8, 10.9 (10.7); 2 x 3692 x 6976, 2 bit in groups of 32 13.0, 11.2 (11.7); 4 x 4096 x 4096, 4
// bit 11.7, 10.7 (11.6).  A copy of the straight-line code inside the variant with the loop spills registers.
// Bound by the vector ALUs once the tables are there: 47 instructions per plane and chunk of eight rows, of which 28
// add and 11 make addresses.  16 rows x 11008 x 4096, 4 bit, from the activations, us after the start of the kernel
// (median of the wavefronts): tables there 3.4, half the look-ups 11, end 19 (21.7 for the last); with a branch before
// each activation load, 128-byte steps between the lanes' LDS stores and a spilled register, tables were there at 9.5.
// A SIMD serves its oldest wavefront first; priorities that fall with the chunks done keep a CU's four level (28.8 us
// for the call without, 26.8 with; slices of eight chunks, 27 random calls 0.97 of the time on average).  Where workgroups
// come in several rounds they would let the new ones overtake those about to end (63 calls: 1.02 on average; 64 x 3125 x
// 8064, int8, 4 bit 52.3 us, 48.6 without).  Row blocks with a slice more, so that 1024 instead of 946 workgroups share the
// work, and a high priority while the tables are built change nothing.
constexpr int R8_CH = 8;     // chunks whose indices a wavefront holds at once
// variants: slices of at most eight chunks that the chip holds all at once, or in several rounds; longer slices
enum { R8_ONCE, R8_ROUNDS, R8_LONG };
constexpr int R8_MOST = 16;  // most chunks of a slice: four workgroups' tables of eight activation rows take 147 KB of LDS
// LDS bytes of a chunk's tables (those built in the kernel lie further apart: RowsShape)
constexpr int rows8_chunk_bytes(int nt, bool fused) {
  return nt == 8 ? (fused ? RowsShape<8, 4, 16>::CB : RowsShape<8, 4>::CB) : (fused ? RowsShape<4, 4, 8>::CB : RowsShape<4, 4>::CB);
}
// ... of a workgroup whose slice has `len` chunks: the group sums, then the tables (those of a LUT buffer are copied
// eight chunks at a time, whatever the slice's length)
constexpr int rows8_lds_bytes(int nt, bool fused, int len) {
  return R8_MOST * nt * 4 + (fused ? len : (len + R8_CH - 1) / R8_CH * R8_CH) * rows8_chunk_bytes(nt, fused);
}

// ... and how many such workgroups a CU holds.  (With the larger of both kinds of tables: how a call is split does not
// depend on who builds them.)
constexpr int rows8_wgs(int nt, int bits, int len) {
  const int own = rows8_lds_bytes(nt, true, len), copied = rows8_lds_bytes(nt, false, len);
  const int by_lds = 163840 / (own > copied ? own : copied), by_regs = rows8_wgs_by_registers(nt, bits, len > R8_CH);
  return by_regs < by_lds ? by_regs : by_lds;
}

// Which (n tile, row block, K slice) a workgroup serves.  The hardware hands workgroups to the
// chip's eight XCDs (one L2 each) round-robin by linear id; with the plain blockIdx mapping the
// n tiles that share a block of packed indices would sit on eight different L2s and each would
// fetch the block from memory.  Here the (row block, K slice) groups go round-robin over the XCDs
// and the n tiles of a group follow each other on one XCD, so a block of indices is fetched once
// (measured: 74 -> 26 MB fetched at 64 activation rows of a 4096 x 4096 4-bit matrix, same time;
// the general kernel keeps the plain order, where the same remapping trades index re-reads for
// table re-reads and changes neither bytes nor time).
struct RowsUnit {
  int nt, rb, kz;
};
__device__ __forceinline__ RowsUnit rows_unit(const Rows8Grid& g) {
  const uint32_t gx = gridDim.x, gy = gridDim.y, groups = gy * gridDim.z;
  const uint32_t lin = (blockIdx.z * gy + blockIdx.y) * gx + blockIdx.x;
  const uint32_t whole = (groups & ~7u) * gx;  // ids of the groups that fill all eight XCDs evenly
  const bool even = lin < whole;               // the few groups left over keep the plain order
  const uint32_t n = even ? lin >> 3 : lin, quot = rows_div(n, gx, g.inv_x), grp = even ? (lin & 7u) + 8u * quot : quot;
  RowsUnit r;
  r.nt = (int)(n - quot * gx);
  r.kz = (int)rows_div(grp, gy, g.inv_y);
  r.rb = (int)(grp - (uint32_t)r.kz * gy);
  return r;
}


template <bool IS_INT, int BITS, int NT, bool FUSED, int KIND>
__global__ __launch_bounds__(64 * ROWS_WAVES, rows8_wgs_by_registers(NT, BITS, KIND == R8_LONG)) void mpgemm_rows8_kernel(const RowsParams p) {
  static_assert(64 * 8 >= 32 * R8_MOST, "a lane for eight activations of a row's slice");
  constexpr bool LONG = KIND == R8_LONG;
  constexpr int G = 4, PAD = FUSED ? 2 * NT : 0;
  using Sh = RowsShape<NT, G, PAD>;
  extern __shared__ __attribute__((aligned(2048))) char rows8_lds[];  // as many chunks as the longest slice has (launch_rows8_one)
  float (*const sS)[NT] = reinterpret_cast<float (*)[NT]>(rows8_lds);  // [chunk]: sum of activations for the bias term added after it (see 2.)
  char* const tab = rows8_lds + R8_MOST * NT * 4;
  using AccT = typename std::conditional<IS_INT, int, float>::type;

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const RowsUnit un = rows_unit(p.grid8);
  const int n0 = un.nt * NT;
  const int tile_raw = un.rb * ROWS_WAVES + wave;
  const bool tile_ok = tile_raw < p.n_tiles;
  const int tile = tile_ok ? tile_raw : p.n_tiles - 1;  // clamped: loads stay in range, stores are masked
  const uint32_t* my_idx = p.idx + ((size_t)tile * p.n_chunks * 64 + lane) * BITS;
  const uint32_t* my_sz = p.sz + (size_t)tile * p.nq * 64 + lane;
  const uint32_t lds0 = (uint32_t)(uintptr_t)((rows_lds_char*)tab);
  const int cz0 = (un.kz * p.grid8.per + min(un.kz, p.grid8.more)) << p.cpg_log2;
  const int nc = (p.grid8.per + (un.kz < p.grid8.more ? 1 : 0)) << p.cpg_log2;  // chunks of this workgroup, 1 to R8_MOST

  // 1. all global loads, unconditional (clamped addresses): activations and indices of the first eight chunks
  constexpr int ITEMS = Sh::TPC * NT / 4;  // tables of four rows in a chunk
  static_assert(!FUSED || R8_MOST * ITEMS <= 64 * ROWS_WAVES, "one item for each thread");
  constexpr int SUM_ROWS = (NT + ROWS_WAVES - 1) / ROWS_WAVES;  // rows whose sums a wavefront makes: wave, wave + 4
  using SumT = typename std::conditional<IS_INT, ru32x2v, ru32x4v>::type;
  ru32x2v build[4];
  SumT act[SUM_ROWS];  // eight activations for each lane
  if constexpr (FUSED) {
    rows_item_load<NT, IS_INT>(p, build, threadIdx.x, n0, cz0 * Sh::TPC);
#pragma unroll
    for (int i = 0; i < SUM_ROWS; ++i) {
      const int64_t at = min(n0 + wave + i * ROWS_WAVES, p.N - 1) * p.lda + min((cz0 << 5) + 8 * lane, p.K - 8);
      act[i] = *reinterpret_cast<const SumT*>(static_cast<const char*>(p.A) + at * (IS_INT ? 1 : 2));
    }
  }
  const int cmask = (1 << p.cpg_log2) - 1;
  uint32_t x[R8_CH][BITS];
  auto load_chunk = [&](int c, uint32_t (&xc)[BITS]) {
    const uint32_t* src = my_idx + (size_t)min(cz0 + c, p.n_chunks - 1) * 64 * BITS;
    if constexpr (BITS == 4) {
      const ru32x4v v = *reinterpret_cast<const ru32x4v*>(src);
      xc[0] = v.x; xc[1] = v.y; xc[2] = v.z; xc[3] = v.w;
    } else if constexpr (BITS == 2) {
      const ru32x2v v = *reinterpret_cast<const ru32x2v*>(src);
      xc[0] = v.x; xc[1] = v.y;
    } else {
#pragma unroll
      for (int b = 0; b < BITS; ++b) xc[b] = src[b];
    }
  };
  // {scale, zero} of a chunk's group, or of the row (per tensor: there are none; not used), two chunks ahead.  (All eight at
  // the start cost calls with one scale 3 to 5 %; a branch around them costs more elsewhere, because waits after it count as
  // if there were no loads in it: 4 x 4096 x 4096, 4 bit, one call 11.5 us, 10.7 like this.)
  auto load_sz = [&](int c) { return *(p.per_tensor ? my_idx : p.grouped ? my_sz + (size_t)min((cz0 + c) >> p.cpg_log2, p.nq - 1) * 64 : my_sz); };
  auto ends_group = [&](int c) { return ((c + 1) & cmask) == 0; };
  constexpr int SZ = 2;  // (a divisor of R8_CH)
  uint32_t szv[SZ];
  load_chunk(0, x[0]);
#pragma unroll
  for (int c = 0; c < SZ; ++c) szv[c] = load_sz(c);
#pragma unroll
  for (int c = 1; c < R8_CH; ++c) load_chunk(c, x[c]);

  // 2. tables of the chunks, and the group sums, into LDS
  const int kg_end = min((cz0 + nc) * Sh::TPC, p.KG);
  if constexpr (FUSED) {
    if ((int)threadIdx.x < nc * ITEMS) rows_stage_item<NT, IS_INT, PAD>(p, tab, build, threadIdx.x, n0, cz0 * Sh::TPC, kg_end);
    // lane: eight activations of a row, four lanes a chunk, whose sum by butterfly; then the sums up to each chunk from
    // its group's start
    float ssum[SUM_ROWS];
    const int k0 = (cz0 << 5) + 8 * lane, c = lane >> 2;
#pragma unroll
    for (int r = 0; r < SUM_ROWS; ++r) {
      const SumT v = act[r];
      if constexpr (IS_INT) {
        int si = __builtin_amdgcn_sdot4((int)v.x, 0x01010101, 0, false);
        si = __builtin_amdgcn_sdot4((int)v.y, 0x01010101, si, false);
        ssum[r] = (float)si;  // sums of a group stay below 2^24: exact
      } else {
        float f[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) f[i] = __half2float(__ushort_as_half((uint16_t)(v[i >> 1] >> (16 * (i & 1)))));
        ssum[r] = ((f[0] + f[1]) + (f[2] + f[3])) + ((f[4] + f[5]) + (f[6] + f[7]));
      }
      if (n0 + wave + r * ROWS_WAVES >= p.N || c >= nc || k0 >= p.K) ssum[r] = 0.f;
      ssum[r] += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(ssum[r]), 0xB1, 0xf, 0xf, true));  // lane ^ 1
      ssum[r] += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(ssum[r]), 0x4E, 0xf, 0xf, true));  // lane ^ 2
    }
    if (p.grouped) {
      const int back = c & cmask;  // chunks before c in the same group (slices hold whole groups)
      for (int o = 1; o <= cmask; o <<= 1) {
#pragma unroll
        for (int r = 0; r < SUM_ROWS; ++r) {
          const float before = __shfl_up(ssum[r], 4 * o);
          if (o <= back) ssum[r] += before;
        }
      }
      if ((lane & 3) == 0) {
#pragma unroll
        for (int r = 0; r < SUM_ROWS; ++r) sS[c][wave + r * ROWS_WAVES] = ssum[r];
      }
    } else if (un.rb == 0) {
      // (one scale per row or tensor: the whole slice's sum per row, for rows_sum_kernel)
#pragma unroll
      for (int r = 0; r < SUM_ROWS; ++r) {
#pragma unroll
        for (int o = 4; o < 64; o <<= 1) ssum[r] += __shfl_xor(ssum[r], o);
        const int n = n0 + wave + r * ROWS_WAVES;
        if (n < p.N && lane == 0) p.ws_srow[(size_t)un.kz * p.N + n] = IS_INT ? __int_as_float((int)ssum[r]) : ssum[r];
      }
    }
  } else {
    // (the group sums are requested before the tables; after them they were a round trip to memory of their own: 48 x 11008 x
    // 4096, 1 bit, two calls 35.3 us, 34.7 like this)
    const int c = threadIdx.x / NT, t = threadIdx.x % NT;
    const bool sums = p.grouped && c < R8_MOST;
    float sum = 0.f;
    if (sums) {
      const size_t at = (size_t)min(n0 + t, p.N - 1) * p.nq + min((cz0 + c) >> p.cpg_log2, p.nq - 1);
      if constexpr (IS_INT) sum = (float)static_cast<const int*>(p.S)[at];
      else sum = static_cast<const float*>(p.S)[at];
    }
    rows_stage_copy<IS_INT, NT, G, R8_CH * Sh::CB>(p, tab, un.nt, cz0 * Sh::TPC, kg_end);
    if (LONG && nc > R8_CH) rows_stage_copy<IS_INT, NT, G, R8_CH * Sh::CB>(p, tab + R8_CH * Sh::CB, un.nt, (cz0 + R8_CH) * Sh::TPC, kg_end);
    if (sums) sS[c][t] = sum;
  }
  __syncthreads();

  // 3. the chunks, eight of them straight-line
  float acc[NT];
  AccT L[NT];
  // (integer tables: minus the biases of the chunks that enter one sum, a group's or this workgroup's)
  const AccT L0 = IS_INT ? (AccT)(-ROWS_CHUNK_BIAS * ((1 << BITS) - 1) * (p.grouped ? 1 << p.cpg_log2 : nc)) : (AccT)0;
#pragma unroll
  for (int t = 0; t < NT; ++t) { acc[t] = 0.f; L[t] = L0; }
  auto eight = [&](int c0) {
#pragma unroll
    for (int i = 0; i < R8_CH; ++i) {
      const int c = c0 + i;
      if (c < nc) {
        // wavefronts that are behind come first (see mpgemm_run_kernel)
        if (KIND != R8_ROUNDS && c0 == 0) {
          if (i == 0) __builtin_amdgcn_s_setprio(3);
          if (i == 3) __builtin_amdgcn_s_setprio(2);
          if (i == 6) __builtin_amdgcn_s_setprio(1);
        } else if (LONG && i == 0) {
          __builtin_amdgcn_s_setprio(0);
        }
        rows_chunk<IS_INT, BITS, NT, G, AccT, 1, 0, PAD>(x[i], lds0 + (uint32_t)c * (uint32_t)Sh::CB, L, p.pw);
        // a quantisation group ends with this chunk (chunks in the K padding belong to no group)
        if (p.grouped && ends_group(c) && ((cz0 + c) >> p.cpg_log2) < p.nq) {
          const float s = __half2float(__ushort_as_half((uint16_t)(szv[i % SZ] & 0xffffu)));
          const float z = __half2float(__ushort_as_half((uint16_t)(szv[i % SZ] >> 16)));
#pragma unroll
          for (int t = 0; t < NT; ++t) {
            acc[t] = fmaf(s, fmaf(p.mid - z, sS[c][t], 0.5f * (float)L[t]), acc[t]);
            L[t] = L0;
          }
        }
        if (p.grouped && (LONG || i + SZ < R8_CH) && ends_group(c + SZ) && c + SZ < nc) szv[i % SZ] = load_sz(c + SZ);
        if constexpr (LONG) {
          if (c + R8_CH < nc) load_chunk(c + R8_CH, x[i]);
        }
      }
    }
  };
  if constexpr (LONG) {
#pragma unroll 1
    for (int c0 = 0; c0 < nc; c0 += R8_CH) eight(c0);
  } else {
    eight(0);
  }

  // 4. one slice: finish here; several: publish the partial sums for rows_sum_kernel
  const int m = tile_raw * 64 + lane;
  if (gridDim.z == 1) {
    if (!tile_ok || m >= p.M) return;
    float s = p.wscale, z = p.zero_point;
    if (!p.grouped && !p.per_tensor) {
      s = __half2float(__ushort_as_half((uint16_t)(szv[0] & 0xffffu)));
      z = __half2float(__ushort_as_half((uint16_t)(szv[0] >> 16)));
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      if (n0 + t >= p.N) break;
      float Sf;
      int Si;
      rows_row_sum<IS_INT>(p, n0 + t, Sf, Si);
      rows_finish<IS_INT>(p, n0 + t, m, p.grouped ? acc[t] : (float)L[t], IS_INT ? (int)L[t] : 0, s, z, Sf, Si,
                          rows_act_scale(p, n0 + t));
    }
    return;
  }
  if (!tile_ok) return;
  const bool raw_int = IS_INT && !p.grouped;  // ungrouped integer tables: partial sums are exact integers
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const int n = n0 + t;
    if (n < p.N) {
      const size_t o = ((size_t)un.kz * p.N + n) * p.Mp + (size_t)m;
      p.ws_part[o] = p.grouped ? acc[t] : (raw_int ? __int_as_float((int)L[t]) : (float)L[t]);
    }
  }
}

// Adds the partial sums [nz][N][Mp] of the K slices in slice order and finishes: VEC outputs per
// thread.  Bound by memory traffic.  Everything the thread needs is requested before the first wait
// (scales and zeros, the activation scale, the row sum or its per-slice parts, the partial sums of a
// round of slices), so that a call pays one round trip to memory, not one per operand.  Many outputs go
// four to a thread (one 16-byte load per slice and one store) in rounds of eight or four slices, few one
// to a thread in rounds of sixteen.  Four against one, us: 511 x 8640 outputs from two slices 10.2 against
// 16.3, from four 14.4 against 17.9; 256 x 3200 from nine to seventeen 7.4 to 10.8 against 7.5 to 11.2;
// 64 x 8640 from thirteen 7.0 against 8.5; 100 x 5504 from 22 9.6 against 10.3.  The number of slices decides
// nothing: of sixteen shapes with two to 34 one lost, 128 x 8640 from thirteen (11.8 against 11.2, also
// with the last five taken as four and one).  96 x 3200, below the line, is even at 8.9.
// RUN: the parts of a run of chunks, whose number changes from pair to pair (nz is not used).
template <bool IS_INT, int VEC, bool RUN>
__global__ __launch_bounds__(256) void rows_sum_kernel(const RowsParams p, int nz) {
  const uint32_t id = blockIdx.x * 256u + threadIdx.x;   // (launch_rows_sum checks that the ids fit)
  const uint32_t per_row = (uint32_t)p.Mp / VEC;
  const int n = (int)(id / per_row), m0 = (int)(id % per_row) * VEC;
  if (n >= p.N || m0 >= p.M) return;
  if constexpr (RUN) nz = p.share.parts((uint32_t)(n >> 4) * p.share.row_blocks + (uint32_t)(m0 >> 8));
  const bool raw_int = IS_INT && !p.grouped;
  const float* src = p.ws_part + (size_t)n * p.Mp + m0;
  const size_t stride = (size_t)p.N * p.Mp;
  const bool own_sz = !p.grouped && !p.per_tensor;
  uint32_t szv[VEC];
#pragma unroll
  for (int i = 0; i < VEC; ++i) szv[i] = own_sz ? p.sz[(size_t)(m0 >> 6) * p.nq * 64 + (m0 & 63) + i] : 0u;
  const float as = rows_act_scale(p, n);
  // fused table build: the row sum is the sum of the slices' sums, taken in slice order below
  const bool slice_sums = !p.grouped && p.ws_srow != nullptr;
  float Sf = 0.f;
  int Si = 0;
  if (!p.grouped && !slice_sums) rows_row_sum<IS_INT>(p, n, Sf, Si);
  float sf[VEC];
  int si[VEC];
#pragma unroll
  for (int i = 0; i < VEC; ++i) { sf[i] = 0.f; si[i] = 0; }
  // R slices from sl0 on, requested without branches in between (slices past the last repeat it)
  auto round = [&](int sl0, auto rc) {
    constexpr int R = decltype(rc)::value;
    float v[R][VEC], r[R];
#pragma unroll
    for (int u = 0; u < R; ++u) {
      const int sl = min(sl0 + u, nz - 1);
      const float* at = src + (size_t)sl * stride;
      if constexpr (VEC == 4) {
        const ru32x4v q = *reinterpret_cast<const ru32x4v*>(at);
#pragma unroll
        for (int i = 0; i < VEC; ++i) v[u][i] = __uint_as_float(q[i]);
      } else {
        v[u][0] = at[0];
      }
      r[u] = slice_sums ? p.ws_srow[(size_t)sl * p.N + n] : 0.f;
    }
#pragma unroll
    for (int u = 0; u < R; ++u) {
      if (sl0 + u < nz) {
#pragma unroll
        for (int i = 0; i < VEC; ++i) {
          if (raw_int) si[i] += __float_as_int(v[u][i]);
          else sf[i] += v[u][i];
        }
        if constexpr (IS_INT) Si += __float_as_int(r[u]);
        else Sf += r[u];
      }
    }
  };
  for (int sl0 = 0; sl0 < nz;) {
    const int left = nz - sl0;
    if (VEC == 1 && left > 8) { round(sl0, std::integral_constant<int, 16>()); sl0 += 16; }
    else if (left > 4) { round(sl0, std::integral_constant<int, 8>()); sl0 += 8; }
    else { round(sl0, std::integral_constant<int, 4>()); sl0 += 4; }
  }
  uint32_t res[VEC];
#pragma unroll
  for (int i = 0; i < VEC; ++i) {
    float s = p.wscale, z = p.zero_point;
    if (own_sz) {
      s = __half2float(__ushort_as_half((uint16_t)(szv[i] & 0xffffu)));
      z = __half2float(__ushort_as_half((uint16_t)(szv[i] >> 16)));
    }
    res[i] = rows_result<IS_INT>(p, sf[i], si[i], s, z, Sf, Si, as);
  }
  // one store where all four outputs exist and their address allows it (any output pointer and leading
  // dimension is accepted), else one by one
  const size_t o = (size_t)n * p.ldo + m0;
  const bool half = p.out_t == TMAC_OUT_F16;
  char* const dst = static_cast<char*>(p.out) + o * (half ? 2 : 4);
  if constexpr (VEC == 4) {
    if (m0 + 4 <= p.M && (reinterpret_cast<uintptr_t>(dst) & (half ? 7u : 15u)) == 0) {
      if (half) {
        uint32_t h[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) h[i] = __half_as_ushort(__float2half_rn(__uint_as_float(res[i])));
        *reinterpret_cast<ru32x2v*>(dst) = ru32x2v{h[0] | (h[1] << 16), h[2] | (h[3] << 16)};
      } else {
        *reinterpret_cast<ru32x4v*>(dst) = ru32x4v{res[0], res[1], res[2], res[3]};
      }
      return;
    }
  }
#pragma unroll
  for (int i = 0; i < VEC; ++i) {
    if (m0 + i >= p.M) break;
    if (half) reinterpret_cast<__half*>(dst)[i] = __float2half_rn(__uint_as_float(res[i]));
    else reinterpret_cast<uint32_t*>(dst)[i] = res[i];
  }
}

template <bool IS_INT, bool RUN>
static hipError_t launch_rows_sum(const RowsParams& p, int nz, hipStream_t st) {
  RowsParams local = p;
  void* args[] = {&local, &nz};
  const int64_t outs = (int64_t)p.N * p.Mp;
  const bool wide = outs >= ROWS_SUM_WIDE;
  const int64_t blocks = (outs / (wide ? 4 : 1) + 255) / 256;  // (Mp is a multiple of 64)
  if (blocks > 0x00ffffff) return hipErrorInvalidValue;        // (ids of 32 bits; their partial sums alone would be 64 GB)
  const void* fn = wide ? reinterpret_cast<const void*>(rows_sum_kernel<IS_INT, 4, RUN>)
                        : reinterpret_cast<const void*>(rows_sum_kernel<IS_INT, 1, RUN>);
  return hipLaunchKernel(fn, dim3((unsigned)blocks), dim3(256), args, 0, st);
}

// ------------------------------------------------------------------------------------------
// fp16 tables as fixed-point numbers
// ------------------------------------------------------------------------------------------
// With fp16 tables and many look-ups the vector ALUs bind: v_pk_add_f16 takes 1.8 ns per wavefront and
// SIMD for one entry of two activation rows, and a plane's sum takes three fp16 roundings.  Large calls
// therefore turn the tables into 16-bit integers first, with one unit for each (activation row,
// quantisation group of at most 128 k): the unit is the largest sum that one chunk's eight entries can
// reach, divided by ROWS_FIX_MAX, so that the eight entries of any chunk and plane add up within 16 bits,
// exactly, with two entries per v_add3_u32.  What is rounded is each entry, once, to 2^-15 of the largest
// sum of a chunk, where fp16 sums round to 2^-11 of every partial sum: 256 rows x 5120 x 5120 at 4 bit is
// off by 2.3e-4 instead of 3.5e-4.
// Where every entry of a unit's chunks is a multiple of the least power of two that is at least as large, that is the
// unit, and no entry is rounded: fp16 sums of whole numbers, fractions of a power of two and subnormal numbers are
// exact, and with the other unit such rows were off by up to 1e-4.  (Looking for it: 0.5 us of a call with 256 rows x
// 5120 x 5120, 4 bit, 132.0 -> 132.5.)
// A unit never spans two groups: with group scales that undo the size of the activations (one group's
// activations 30 times its neighbours', its scales a thirtieth) one unit for the four groups of a
// 128-k block was off by 2.3e-3, one for each is by 2.4e-4, like groups of one size.  Groups of whole 128-k
// blocks (or none) have one unit per block; others have one stored per chunk, the same for the chunks of a
// block that one group holds.
// In memory and LDS an entry pair is the number (hi + B) * 65536 + lo + B modulo 2^32 (B =
// ROWS_FIX_BIAS): additions of whole dwords are exact, and the sum of a chunk's eight pairs has two
// clean halves, sum + 32768.
// Where an activation row's entries are not all finite, the chunks of that unit hold zeros for this row and
// the unit is -0; mpgemm_run_kernel adds what their fp16 entries give, with fp16 additions, so that
// infinities and NaNs come out as they do in the general kernel (rows_add_raw).  Other rows do not notice.
// The fp16 entries are read from the LUT buffer; a call that builds the integers from the activations writes
// those blocks into the buffer's place in its workspace.
constexpr int ROWS_FIX_BIAS = 4096;
constexpr float ROWS_FIX_MAX = 32700.f;  // + 8 roundings of half a unit stays below 32767

// One workgroup: the 32 tables of a 128-k block for 16 activation rows; thread = the table of a pair of
// rows, wavefront = the eight tables of a chunk, so that a chunk's largest sum is three exchanges away.
// Entries 0..7 are looked at, the others are their negatives (Section 3.3).  FROM_ACT: entries from the
// activations (with the fp16 additions of the precompute kernel: both routes hold the same numbers), and
// further workgroups for the group sums; else from the LUT buffer, whose group sums are copied into the
// order the look-up kernel reads, [set of 16 rows][group][16].  Bound by launch and memory: 21 MB of
// tables written at 511 rows of K = 5120, 9.5 us (one thread per entry of a table: 21).
template <bool FROM_ACT>
__global__ __launch_bounds__(256) void rows_fix_kernel(const RowsParams p, uint32_t* __restrict__ fix, float* __restrict__ scale,
                                                       float* __restrict__ sums, int Geff, int n_fix) {
  if constexpr (FROM_ACT) {
    if ((int)blockIdx.x >= n_fix) {
      group_sums_wave<false, true>(p.A, p.N, p.lda, sums, Geff, p.nq, ((int)blockIdx.x - n_fix) * 4 + (threadIdx.x >> 6));
      return;
    }
  }
  typedef unsigned short us2v __attribute__((ext_vector_type(2)));
  constexpr int TD = 64 + 4, OD = 32 * TD + 32;    // dwords from table to table and set half to set half: conflict-free writes
  __shared__ __attribute__((aligned(16))) uint32_t stage[2 * OD];
  __shared__ float smax[4][16];                    // [chunk][row]: largest sum of the chunk's eight entries
  __shared__ uint32_t off_grid[4];                 // [chunk]: rows with an entry that is no multiple of the power of two
  const int nblk = p.KG / 32;
  const int set = blockIdx.x / nblk, blk = blockIdx.x % nblk;
  const int u = threadIdx.x & 7, tb = threadIdx.x >> 3, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int kg = blk * 32 + tb, n = set * 16 + 2 * u;
  uint32_t v[8];                                   // entries 0..7 of rows n (low half) and n + 1
  if constexpr (FROM_ACT) {
    uint32_t t0[4], t1[4];
    ru32x2v a0 = {0u, 0u}, a1 = {0u, 0u};
    if (4 * kg < p.K) {
      const __half* const at = static_cast<const __half*>(p.A) + 4 * kg;
      if (n < p.N) a0 = *reinterpret_cast<const ru32x2v*>(at + n * p.lda);
      if (n + 1 < p.N) a1 = *reinterpret_cast<const ru32x2v*>(at + (n + 1) * p.lda);
    }
    half_table_f16(a0.x, a0.y, t0);
    half_table_f16(a1.x, a1.y, t1);
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      v[2 * d] = __builtin_amdgcn_perm(t1[d], t0[d], 0x05040100u);
      v[2 * d + 1] = __builtin_amdgcn_perm(t1[d], t0[d], 0x07060302u);
    }
  } else {
    const int tile = n / p.lut_nt;
    const uint16_t* const at = p.tables + ((size_t)tile * p.KG + kg) * (16 * p.lut_nt) + (n & (p.lut_nt - 1));
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = tile * p.lut_nt < p.N ? *reinterpret_cast<const uint32_t*>(at + e * p.lut_nt) : 0u;
    const int r = set * 16 + (int)threadIdx.x;
    if (threadIdx.x < 16 && r < p.N)
      for (int gq = blk; gq < p.nq; gq += nblk) sums[((size_t)set * p.nq + gq) * 16 + threadIdx.x] = static_cast<const float*>(p.S)[(size_t)r * p.nq + gq];
  }
  // fp16 magnitudes compare as integers, infinities and NaNs on top
  us2v m = __builtin_bit_cast(us2v, v[0] & 0x7fff7fffu);
#pragma unroll
  for (int e = 1; e < 8; ++e) m = __builtin_elementwise_max(m, __builtin_bit_cast(us2v, v[e] & 0x7fff7fffu));
  float b0 = __half2float(__ushort_as_half(m.x)), b1 = __half2float(__ushort_as_half(m.y));
#pragma unroll
  for (int o = 8; o < 64; o <<= 1) {
    b0 += __shfl_xor(b0, o);
    b1 += __shfl_xor(b1, o);
  }
  if ((threadIdx.x & 63) < 8) {
    smax[wave][2 * u] = b0;
    smax[wave][2 * u + 1] = b1;
  }
  // the chunks of the block that share the unit of this wavefront's chunk: those of its group
  int u0 = 0, u1 = 4;
  if (p.fix_shift == 0) {
    u0 = (blk * 4 + wave) / p.cpg * p.cpg - blk * 4;
    u1 = u0 + p.cpg;
  }
  __syncthreads();
  float f[2];
  bool any_bad = false;  // in any chunk of the block
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    float b = 0.f;
    bool bad = false;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const float sum = smax[c][2 * u + h];
      const bool fin = sum <= 1e30f;
      any_bad |= !fin;
      if (c >= u0 && c < u1) {
        bad |= !fin;
        b = fmaxf(b, sum);
      }
    }
    f[h] = bad ? -1.f : b;
  }
  // the unit: the least power of two that is large enough, if all entries of these chunks are multiples of it, else the
  // least number (entries 0..3 of the chunk's eight tables tell most rows that they are not; the other entries are looked
  // at only if a row may be)
  float unit[2], factor[2], rest[2] = {0.f, 0.f};
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    unit[h] = __uint_as_float((__float_as_uint(fmaxf(f[h], 0.f) * (1.f / ROWS_FIX_MAX)) + 0x7fffffu) & 0x7f800000u);
    factor[h] = __uint_as_float(0x7f000000u - __float_as_uint(unit[h]));
  }
  uint32_t off = 0u;  // bit 8 h + u: row 2 u + h
#pragma unroll
  for (int part = 0; part < 2; ++part) {
    if (off == 0xffffu) break;
#pragma unroll
    for (int e = 4 * part; e < 4 * part + 4; ++e) {
      const rh2v x = __builtin_bit_cast(rh2v, v[e]);
      rest[0] = fmaxf(rest[0], __builtin_amdgcn_fractf(fmaf((float)x.x, factor[0], 0.f)));
      rest[1] = fmaxf(rest[1], __builtin_amdgcn_fractf(fmaf((float)x.y, factor[1], 0.f)));
    }
    uint64_t lo = __ballot(rest[0] != 0.f), hi = __ballot(rest[1] != 0.f);  // bit 8 table + u
    lo |= lo >> 32; lo |= lo >> 16; lo |= lo >> 8;
    hi |= hi >> 32; hi |= hi >> 16; hi |= hi >> 8;
    off = ((uint32_t)lo & 0xffu) | ((uint32_t)hi & 0xffu) << 8;
  }
  if ((threadIdx.x & 63) == 0) off_grid[wave] = off;
  __syncthreads();
  off = 0u;
#pragma unroll
  for (int c = 0; c < 4; ++c) off |= c >= u0 && c < u1 ? off_grid[c] : 0u;
#pragma unroll
  for (int h = 0; h < 2; ++h)
    if (off >> (8 * h + u) & 1u) {
      unit[h] = f[h] / ROWS_FIX_MAX;
      factor[h] = ROWS_FIX_MAX / f[h];
    }
  if ((threadIdx.x & 63) < 8 && (wave == 0 || p.fix_shift == 0)) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
      scale[((size_t)set * (p.n_chunks >> p.fix_shift) + ((blk * 4 + wave) >> p.fix_shift)) * 16 + 2 * u + h] = f[h] < 0.f ? -0.f : unit[h];
  }
  const float f0 = factor[0], f1 = factor[1];
  const uint32_t keep = (f[0] < 0.f ? 0u : 0xffffu) | (f[1] < 0.f ? 0u : 0xffff0000u);
  uint32_t* const dst = stage + (u >> 2) * OD + tb * TD + (u & 3);
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    // nearest integer, ties to even: the low bits of x f + 1.5 * 2^23
    const rh2v x = __builtin_bit_cast(rh2v, v[e]);
    const uint32_t i0 = __float_as_uint(fmaf((float)x.x, f0, 12582912.f)), i1 = __float_as_uint(fmaf((float)x.y, f1, 12582912.f));
    // two signed halves side by side -> hi * 65536 + lo, then the bias of both
    const uint32_t d = ((__builtin_amdgcn_perm(i1, i0, 0x05040100u) & keep) ^ 0x8000u) + ((uint32_t)ROWS_FIX_BIAS * 0x10001u - 0x8000u);
    dst[e * 4] = d;
    dst[(15 - e) * 4] = 2u * ROWS_FIX_BIAS * 0x10001u - d;
  }
  auto store = [&](uint32_t* to) {
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int o = i >> 1, q = (i & 1) * 256 + (int)threadIdx.x;  // 16-byte piece of the half's 32 tables
      const int t8 = set * 2 + o;
      if (t8 * 8 < p.N)
        *reinterpret_cast<ru32x4v*>(to + ((size_t)t8 * p.KG + blk * 32) * 64 + q * 4) =
            *reinterpret_cast<const ru32x4v*>(stage + o * OD + (q >> 4) * TD + (q & 15) * 4);
    }
  };
  store(fix);
  if constexpr (FROM_ACT) {
    if (__any(any_bad)) {  // (the same in all wavefronts: each sees the sums of every row and chunk)
      __syncthreads();
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        dst[e * 4] = v[e];
        dst[(15 - e) * 4] = v[e] ^ 0x80008000u;
      }
      store(reinterpret_cast<uint32_t*>(p.raw));
    }
  }
}

// A sum of at most four chunks, |sum| < 2^21, that starts from ROWS_FLOAT_ZERO is the bit pattern of 1.5 2^23 plus it:
// as a number by one subtraction (1.1 ns per wavefront and SIMD; a conversion takes 1.8)
constexpr int ROWS_FLOAT_ZERO = 0x4B400000;
__device__ __forceinline__ float rows_float(int l) { return __int_as_float(l) - 12582912.f; }

// The look-ups of one 32-k chunk for two sets of eight activation rows, in rounds of the eight reads of
// one plane and row set (see rows_chunk_int): L += the planes' sums, and their biases, times the planes'
// weights.  START: L begins at `start`.
template <int BITS, int OSTRIDE, bool START>
__device__ __forceinline__ void rows_chunk_fix(const uint32_t (&x)[BITS], uint32_t cbase, int (&L)[16], int start = 0) {
  using Sh = RowsShape<8, 4>;
  constexpr int TPC = Sh::TPC, HD = Sh::HD, TB = Sh::TB;
  auto plane = [&](auto bc) {
    constexpr int b = decltype(bc)::value;
    const uint32_t even = (x[b] << 4) & 0xF0F0F0F0u, odd = x[b] & 0xF0F0F0F0u;
    uint32_t a[TPC];
#pragma unroll
    for (int j = 0; j < TPC; ++j) a[j] = __builtin_amdgcn_perm(j & 1 ? odd : even, cbase, 0x0C020100u + 4u + (uint32_t)(j / 2));
#pragma unroll
    for (int o = 0; o < 2; ++o) {
      ru32x4v e[TPC];
#pragma unroll
      for (int j = 0; j < TPC; ++j) e[j] = *reinterpret_cast<rows_lds_u32x4*>(a[j] + j * TB + o * OSTRIDE);
      __builtin_amdgcn_sched_barrier(0);  // keep the reads above the accumulation
#pragma unroll
      for (int u = 0; u < HD; ++u) {
        uint32_t q = e[0][u];
#pragma unroll
        for (int j = 1; j < TPC; ++j) q += e[j][u];
        if constexpr (START && b == 0) rows_widen_from<1>(L[8 * o + 2 * u], L[8 * o + 2 * u + 1], q, start);
        else rows_widen<1 << b>(L[8 * o + 2 * u], L[8 * o + 2 * u + 1], q);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  plane(std::integral_constant<int, 0>());
  if constexpr (BITS > 1) plane(std::integral_constant<int, 1>());
  if constexpr (BITS > 2) plane(std::integral_constant<int, 2>());
  if constexpr (BITS > 3) plane(std::integral_constant<int, 3>());
}

// What the chunks whose unit is -0 (see above) contribute to activation rows n0 .. n0 + 15 of the lane's
// weight row, added to its own partial sums: the fp16 entries of eight rows at a time, with the additions of
// the general kernel.  Only a wavefront that met such a unit comes here.  A row is done once its sum is NaN
// in all lanes, which a NaN anywhere takes one chunk for and infinities usually not many more, since the
// planes' signs differ.
// 256 rows x 5120 x 5120 at 4 bit: 142 us with finite rows, 143 with one NaN, 151 with one row of NaNs, 168 with
// all rows (fp16 tables throughout: 165); 511 x 13824 x 5120 at 2 bit: 366, 370, 408, 421 (454).
template <int BITS>
__device__ __forceinline__ void rows_add_raw(const RowsParams& p, const float* unit, const uint32_t* idx, const uint32_t* sz, int n0,
                                             int cz0, int cz1, float* part, bool live) {
  const int lane = threadIdx.x & 63, shift = p.fix_shift;
  const int units = ((cz1 + (1 << shift) - 1) >> shift) - (cz0 >> shift);  // (the first and last may be other workgroups' in part)
  unit += (size_t)(cz0 >> shift) * 16;
#pragma unroll 1
  for (int o = 0; o < 2 && n0 + 8 * o < p.N; ++o) {
    // (a LUT buffer's n tiles may be four rows wide: then the second half comes from the next tile)
    const bool narrow = p.raw_nt == 4;
    const uint16_t* const tables = p.raw + (size_t)((n0 >> 3) + o) * p.KG * 128;
    const uint16_t* const upper = (n0 >> 2) + 2 * o + 1 < (p.N + 3) >> 2 ? tables + (size_t)p.KG * 64 : tables;
    uint32_t open = (1u << min(p.N - n0 - 8 * o, 8)) - 1u, some = 0;  // rows not NaN everywhere yet, rows with such units
    float sum[8];
#pragma unroll
    for (int r = 0; r < 8; ++r) sum[r] = 0.f;
#pragma unroll 1
    for (int u0 = 0; u0 < units && open; u0 += 8) {
      const int u = u0 + (lane >> 3);
      uint64_t marks = __ballot(u < units && __float_as_int(unit[(size_t)min(u, units - 1) * 16 + 8 * o + (lane & 7)]) < 0);
#pragma unroll 1
      for (int c = ((cz0 >> shift) + u0) << shift, left = 1 << shift; marks; ++c) {
        const uint32_t rows = c >= cz0 && c < cz1 ? (uint32_t)marks & open : 0u;
        if (p.grouped && c / p.cpg >= p.nq) break;  // chunks in the K padding belong to no group
        if (rows) {
          some |= rows;
          const float hs = p.grouped ? 0.5f * __half2float(__ushort_as_half((uint16_t)(sz[(size_t)(c / p.cpg) * 64] & 0xffffu))) : 1.f;
#pragma unroll 1
          for (int b = 0; b < BITS; ++b) {
            const uint32_t x = idx[(size_t)c * 64 * BITS + b];
            const float w = (float)(1 << b);
            ru32x4v e[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
              const size_t entry = (size_t)(c * 8 + j) * 16 + ((x >> (4 * j)) & 15u);
              if (narrow) {
                const ru32x2v lo = *reinterpret_cast<const ru32x2v*>(tables + entry * 4), hi = *reinterpret_cast<const ru32x2v*>(upper + entry * 4);
                e[j] = ru32x4v{lo.x, lo.y, hi.x, hi.y};
              } else {
                e[j] = *reinterpret_cast<const ru32x4v*>(tables + entry * 8);
              }
            }
#pragma unroll
            for (int d = 0; d < 4; ++d) {
              rh2v q[8];
#pragma unroll
              for (int j = 0; j < 8; ++j) q[j] = __builtin_bit_cast(rh2v, (uint32_t)e[j][d]);
              tree_sum(q);
              if (rows >> (2 * d) & 1u) sum[2 * d] = fmaf((float)q[0].x, hs * w, sum[2 * d]);
              if (rows >> (2 * d + 1) & 1u) sum[2 * d + 1] = fmaf((float)q[0].y, hs * w, sum[2 * d + 1]);
            }
          }
#pragma unroll
          for (int r = 0; r < 8; ++r)
            if (__all(sum[r] != sum[r] || !live)) open &= ~(1u << r);
        }
        if (--left == 0) {
          left = 1 << shift;
          marks >>= 8;
        }
      }
    }
#pragma unroll
    for (int r = 0; r < 8; ++r)
      if (some >> r & 1u) part[(size_t)(8 * o + r) * p.Mp] += sum[r];
  }
}

// Which tables a run of chunks looks up: integer ones (one scale per row or tensor), or fixed-point ones with a unit
// for each 128-k block, for each chunk where a group is one, or for each chunk else.
enum { RUN_INT, RUN_BLOCK, RUN_SOLO, RUN_CHUNK };

// Look-ups in fixed-point tables (from the workspace, written by rows_fix_kernel), and in integer tables with one scale
// per row or tensor: two sets of eight activation rows per workgroup, the call as one run of chunks (RowsShare), an
// equal share for each of the 1024 workgroups that the chip holds at once; results through the workspace to
// rows_sum_kernel even where a pair has one part only (finishing here as well costs 40 registers).  The integer sums
// of a quantisation group and 128-k block are converted once and multiplied by their unit and half the group's scale;
// RUN_SOLO starts every chunk's sum from the constant and asks for units and group sums before its look-ups.
// Bound by the look-up rate of LDS (rows_chunk_int): with tables and indices at hand the loop runs at 84 % of it at 4
// bit (81 at 2 bit) with four wavefronts per SIMD, 86 with five, and neither earlier reads nor fewer additions change
// that; what a call takes beyond it is the start of the stream (9 us of a 16 row call without any look-up), the tables
// and the slice sums.
// Shares alone are slower than two to four rounds of workgroups with K slices of equal length (256 rows x 5120 x 5120,
// 4 bit: 148 us against 137; 511 x 13824 x 5120, 2 bit: 388 against 365; no matter how the pairs are ordered): a SIMD
// serves its oldest wavefront first, so one workgroup of a CU is done after three quarters of the time and its place
// stays empty (12.2 wavefronts per CU on average, of 16).  Wavefronts that are behind therefore get a higher priority.
// Indices are requested two chunks ahead, at one and two bits, whose chunks are over sooner, four (511 x 13824 x 5120:
// 351 us, two 356).
// Us, K slices of equal length and now: 256 x 5120 x 5120, 4 bit 135.8, 132.3; 511 x 13824 x 5120, 2 bit 373, 356,
// groups of 32 436, 417; 256 x 5120 x 5120 in groups of 32, 2 bit 102.1, 95.7; ternary 128 x 8640 x 3200 56.4, 50.2,
// 256 x 3200 x 8640 99.1, 94.2; against fp16 sums 48 x 11008 x 4096, 4 bit 75.0, 57.9, in groups of 32 79.4, 60.5, 64 x
// 4096 x 4096 43.5, 36.1, 300 x 700 x 8192 71.8, 59.5.
// (The chunk loop not unrolled, indices handed from register to register: 53 and 382 us for the ternary and the 2-bit
// call of 511 rows; a copy of it without the bounds of a share: 53.7 and 353.)
// The fixed-point variants keep 60 to 67 of their scalars (parameters, 16 units, addresses) in lanes of a vector register
// (integer tables: none, two at 3 bit); they are read back once per 128-k block or part, not within a chunk's look-ups.
template <int BITS, int MODE>
__global__ __launch_bounds__(64 * ROWS_WAVES, 4) void mpgemm_run_kernel(const RowsParams p) {
  constexpr bool IS_INT = MODE == RUN_INT;
  using Sh = RowsShape<8, 4>;
  constexpr int CB = Sh::CB, OSTRIDE = 4 * CB;
  constexpr int BIAS = IS_INT ? ROWS_CHUNK_BIAS : 32768;  // of a chunk's sum, per plane weight
  __shared__ __attribute__((aligned(2048))) char tab[2 * OSTRIDE];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // (gridDim.x is a multiple of 8: neighbours in the run share an XCD and its L2)
  const uint32_t wg = (blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3);
  if (wg >= p.share.wgs) return;
  const uint32_t at0 = p.share.start(wg);
  const int todo = (int)(p.share.start(wg + 1) - at0);
  if (todo <= 0) return;
  const int chunks = (int)p.share.chunks, row_blocks = (int)p.share.row_blocks;
  const int pair0 = (int)rows_div(at0, p.share.chunks, p.share.inv_chunks), c00 = (int)(at0 - (uint32_t)pair0 * p.share.chunks);
  const uint32_t lds0 = (uint32_t)(uintptr_t)((rows_lds_char*)tab);
  const int last8 = (p.N + 7) / 8 - 1;  // (a second row set past it repeats it)
  const int bpg = p.cpg >> 2;           // blocks per quantisation group

  auto tile_of = [&](int rb) { return min(rb * ROWS_WAVES + wave, p.n_tiles - 1); };  // (clamped: loads stay in range, stores are masked)
  auto load_idx = [&](const uint32_t* base, uint32_t (&x)[BITS]) {
    const uint32_t* src = base + (uint32_t)lane * BITS;
    if constexpr (BITS == 4) {
      const ru32x4v v = *reinterpret_cast<const ru32x4v*>(src);
      x[0] = v.x; x[1] = v.y; x[2] = v.z; x[3] = v.w;
    } else if constexpr (BITS == 2) {
      const ru32x2v v = *reinterpret_cast<const ru32x2v*>(src);
      x[0] = v.x; x[1] = v.y;
    } else {
#pragma unroll
      for (int b = 0; b < BITS; ++b) x[b] = src[b];
    }
  };
  // the tables of a 128-k block, 8 KB for each set of eight rows, are requested while the block before it is
  // looked up, a chunk's indices two chunks ahead
  ru32x4v next[4];
  auto request = [&](int set, int blk) {
    const char* const b0 = reinterpret_cast<const char*>(p.tables) + ((size_t)(set * 2) * p.KG + blk * 32) * Sh::TB;
    const char* const b1 = reinterpret_cast<const char*>(p.tables) + ((size_t)min(set * 2 + 1, last8) * p.KG + blk * 32) * Sh::TB;
    const uint32_t o = threadIdx.x * 16;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      next[i] = *reinterpret_cast<const ru32x4v*>(b0 + o + i * 4096);
      next[2 + i] = *reinterpret_cast<const ru32x4v*>(b1 + o + i * 4096);
    }
  };
  int set = (int)rows_div((uint32_t)pair0, p.share.row_blocks, p.share.inv_row_blocks), rb = pair0 - set * row_blocks, c = c00, left = todo, flag = 0;
  const uint32_t* idx = p.idx + ((size_t)tile_of(rb) * chunks + (c & ~3)) * 64 * BITS;
  constexpr int AHEAD = BITS <= 2 ? 4 : 2;
  uint32_t x[AHEAD][BITS];
#pragma unroll
  for (int i = 0; i < AHEAD; ++i) load_idx(idx + ((c & (4 - AHEAD)) + i) * 64 * BITS, x[i]);
  request(set, c >> 2);  // (after the indices: before them 1.005 to 1.02 times the time)
  while (true) {  // the parts of this workgroup, pair by pair
    const int end = min(chunks, c + left);
    left -= end - c;
    const int n0 = set * 16, tile_raw = rb * ROWS_WAVES + wave;
    const uint32_t* const my_sz = p.sz + (size_t)tile_of(rb) * p.nq * 64 + lane;
    constexpr int SHIFT = MODE == RUN_BLOCK ? 2 : 0;  // a unit for each block, or for each chunk
    rows_const_float* fix_scale = rows_const(p.fix_scale) + ((size_t)set * (chunks >> SHIFT) + (c >> SHIFT)) * 16;
    rows_const_float* const sums = rows_const(p.S) + (size_t)set * p.nq * 16;
    const int rb_n = rb + 1 == row_blocks ? 0 : rb + 1, set_n = rb + 1 == row_blocks ? set + 1 : set;  // the next pair
    const uint32_t* const idx_n = p.idx + (size_t)tile_of(rb_n) * chunks * 64 * BITS;
    float acc[16];
    int L[16];
#pragma unroll
    for (int t = 0; t < 16; ++t) {
      acc[t] = 0.f;
      L[t] = -(end - c) * (BIAS * ((1 << BITS) - 1));  // (fixed point: set anew in every block)
    }
    int gq = 0, bg = 0;  // quantisation group, its block or chunk
    float hs = 1.f;      // half the group's scale (1: one scale per row or tensor, applied at the end)
    uint32_t szv = 0;
    bool enter = !IS_INT && p.grouped != 0;
    if (enter) {
      const int at = MODE == RUN_BLOCK ? c >> 2 : c, per = MODE == RUN_BLOCK ? bpg : p.cpg;
      gq = at / per;  // (RUN_CHUNK: chunks in the K padding belong to no group)
      bg = at - gq * per;
      szv = my_sz[(size_t)min(gq, p.nq - 1) * 64];
    }
    bool first = true;  // RUN_CHUNK: a sum starts
    for (; c < end;) {
      const int lo = c & 3, hi = min(end - (c & ~3), 4);
      c = (c & ~3) + hi;
      __syncthreads();
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        ru32x4v e = next[i];
        if constexpr (IS_INT) {
          constexpr short be = (short)rows_int_bias(4);
#pragma unroll
          for (int d = 0; d < 4; ++d) e[d] = __builtin_bit_cast(uint32_t, (rs2v)(__builtin_bit_cast(rs2v, (uint32_t)e[d]) + rs2v{be, be}));
        }
        *reinterpret_cast<ru32x4v*>(tab + (i >> 1) * OSTRIDE + (i & 1) * 4096 + threadIdx.x * 16) = e;
      }
      __syncthreads();
      if (c < end) request(set, c >> 2);
      else if (left > 0) request(set_n, 0);
      const uint32_t* const here = idx;
      idx = c < end ? idx + 4 * 64 * BITS : left > 0 ? idx_n : idx;
      // wavefronts that are behind come first (see above)
      const int done4 = 4 * (todo - left - (end - c));
      if (done4 <= todo) __builtin_amdgcn_s_setprio(3);
      else if (done4 <= 2 * todo + 1) __builtin_amdgcn_s_setprio(2);
      else if (done4 <= 3 * todo + 2) __builtin_amdgcn_s_setprio(1);
      else __builtin_amdgcn_s_setprio(0);
      // half the scale of the group; its bias term (Section 4's linear transform) goes with its first chunk
      auto enter_group = [&](bool starts) {
        enter = false;
        const float s = __half2float(__ushort_as_half((uint16_t)(szv & 0xffffu)));
        const float z = __half2float(__ushort_as_half((uint16_t)(szv >> 16)));
        hs = 0.5f * s;
        if (starts) {
          const float bz = s * (p.mid - z);
#pragma unroll
          for (int t = 0; t < 16; ++t) acc[t] = fmaf(bz, sums[(size_t)gq * 16 + t], acc[t]);
        }
      };
      float unit[16];  // value of one unit (wave-uniform); -0 where entries are not finite
      if constexpr (MODE == RUN_BLOCK) {
        if (enter) enter_group(bg == 0 && lo == 0);  // a group starts, or the part starts inside one
#pragma unroll
        for (int t = 0; t < 16; ++t) unit[t] = fix_scale[t];
        fix_scale += 16;
        if (lo != 0) {  // (else the first chunk starts the sums)
#pragma unroll
          for (int t = 0; t < 16; ++t) L[t] = ROWS_FLOAT_ZERO + (lo - hi) * (BIAS * ((1 << BITS) - 1));
        }
      }
      auto chunk = [&](auto ic) {
        constexpr int i = decltype(ic)::value;
        if (i >= lo && i < hi) {
          const uint32_t cbase = lds0 + (uint32_t)i * CB;
          uint32_t (&xi)[BITS] = x[i & (AHEAD - 1)];
          if constexpr (IS_INT) {
            rows_chunk_int<BITS, 2, OSTRIDE>(xi, cbase, L);
          } else if constexpr (MODE == RUN_BLOCK) {
            rows_chunk_fix<BITS, OSTRIDE, i == 0>(xi, cbase, L, ROWS_FLOAT_ZERO - hi * (BIAS * ((1 << BITS) - 1)));
          } else if constexpr (MODE == RUN_SOLO) {
            if (gq < p.nq) {  // (chunks in the K padding belong to no group)
              const float s = __half2float(__ushort_as_half((uint16_t)(szv & 0xffffu)));
              const float z = __half2float(__ushort_as_half((uint16_t)(szv >> 16)));
              szv = my_sz[(size_t)min(gq + 1, p.nq - 1) * 64];
              float sum[16];
#pragma unroll
              for (int t = 0; t < 16; ++t) {
                unit[t] = fix_scale[t];
                sum[t] = sums[(size_t)gq * 16 + t];
              }
              fix_scale += 16;
              rows_chunk_fix<BITS, OSTRIDE, true>(xi, cbase, L, ROWS_FLOAT_ZERO - BIAS * ((1 << BITS) - 1));
              const float bz = 2.f * (p.mid - z);
              hs = 0.5f * s;
#pragma unroll
              for (int t = 0; t < 16; ++t) {
                flag |= __float_as_int(unit[t]);
                acc[t] = fmaf(hs, fmaf(rows_float(L[t]), unit[t], bz * sum[t]), acc[t]);
              }
              ++gq;
            }
          } else if (gq < p.nq) {
            if (enter) {
              enter_group(bg == 0);
              szv = my_sz[(size_t)min(gq + 1, p.nq - 1) * 64];
            }
            if (first) {  // the chunks of this group left in this block and part
#pragma unroll
              for (int t = 0; t < 16; ++t) unit[t] = fix_scale[t];
              const int n = min(hi - i, p.cpg - bg);
#pragma unroll
              for (int t = 0; t < 16; ++t) L[t] = ROWS_FLOAT_ZERO - n * (BIAS * ((1 << BITS) - 1));
            }
            fix_scale += 16;
            rows_chunk_fix<BITS, OSTRIDE, false>(xi, cbase, L);
            const bool ends = ++bg == p.cpg;
            first = ends || i + 1 == hi;
            if (first) {
#pragma unroll
              for (int t = 0; t < 16; ++t) {
                flag |= __float_as_int(unit[t]);
                acc[t] = fmaf(rows_float(L[t]), unit[t] * hs, acc[t]);
              }
            }
            if (ends) {
              bg = 0;
              ++gq;
              enter = true;
            }
          }
        }
        if (i >= (lo & (4 - AHEAD))) load_idx(i + AHEAD < 4 ? here + (i + AHEAD) * 64 * BITS : idx + (i + AHEAD - 4) * 64 * BITS, x[i & (AHEAD - 1)]);
        __builtin_amdgcn_sched_barrier(0);
      };
      chunk(std::integral_constant<int, 0>());
      chunk(std::integral_constant<int, 1>());
      chunk(std::integral_constant<int, 2>());
      chunk(std::integral_constant<int, 3>());
      if constexpr (MODE == RUN_BLOCK) {
#pragma unroll
        for (int t = 0; t < 16; ++t) {
          flag |= __float_as_int(unit[t]);
          acc[t] = fmaf(rows_float(L[t]), unit[t] * hs, acc[t]);
        }
        if (p.grouped && ++bg == bpg) {
          bg = 0;
          ++gq;
          enter = true;
          szv = my_sz[(size_t)min(gq, p.nq - 1) * 64];
        }
      }
    }
    if (tile_raw < p.n_tiles) {
      const uint32_t slot = wg - p.share.first((uint32_t)(set * row_blocks + rb));
      float* const part = p.ws_part + ((size_t)slot * p.N + n0) * p.Mp + tile_raw * 64 + lane;
#pragma unroll
      for (int t = 0; t < 16; ++t)
        if (n0 + t < p.N) part[(size_t)t * p.Mp] = IS_INT ? __int_as_float(L[t]) : acc[t];
    }
    if (left <= 0) break;
    c = 0;
    rb = rb_n;
    set = set_n;
  }
  if constexpr (!IS_INT) {
    if (flag >= 0) return;
    // the parts again, for the blocks whose entries are not finite
    left = todo;
    set = pair0 / row_blocks;
    rb = pair0 - set * row_blocks;
    c = c00;
    while (left > 0) {
      const int end = min(chunks, c + left), tile_raw = rb * ROWS_WAVES + wave;
      if (tile_raw < p.n_tiles) {
        const uint32_t slot = wg - p.share.first((uint32_t)(set * row_blocks + rb));
        rows_add_raw<BITS>(p, p.fix_scale + (size_t)set * (chunks >> p.fix_shift) * 16, p.idx + ((size_t)tile_raw * chunks * 64 + lane) * BITS,
                           p.sz + (size_t)tile_raw * p.nq * 64 + lane, set * 16, c, end,
                           p.ws_part + ((size_t)slot * p.N + set * 16) * p.Mp + tile_raw * 64 + lane, tile_raw * 64 + lane < p.M);
      }
      left -= end - c;
      c = 0;
      if (++rb == row_blocks) {
        rb = 0;
        ++set;
      }
    }
  }
}

static RowsShare rows_share(int wgs, int total, int row_blocks, int chunks) {
  return RowsShare{(uint32_t)wgs, (uint32_t)(total / wgs), (uint32_t)(total % wgs), (uint32_t)row_blocks, (uint32_t)chunks,
                   rows_inverse((uint32_t)row_blocks, (uint64_t)(total / chunks)), rows_inverse((uint32_t)chunks, (uint64_t)total)};
}

template <int MODE>
static const void* rows_run_kernel(int bits) {
  if constexpr (MODE == RUN_INT) {
    if (bits == 1) return reinterpret_cast<const void*>(mpgemm_run_kernel<1, MODE>);
  }
  return bits == 2   ? reinterpret_cast<const void*>(mpgemm_run_kernel<2, MODE>)
         : bits == 3 ? reinterpret_cast<const void*>(mpgemm_run_kernel<3, MODE>)
                     : reinterpret_cast<const void*>(mpgemm_run_kernel<4, MODE>);
}

// Tables to fixed point, look-ups, slice sums.
static hipError_t launch_rows_fix(const RowsParams& p, const RowsPlan& pl, int bits, bool from_act, int Geff,
                                  uint32_t* fix, float* scale, float* sums, hipStream_t st) {
  RowsParams local = p;
  local.raw = const_cast<uint16_t*>(p.tables);  // (written only where the tables are built here)
  int n_fix = pl.fix_tiles * (p.KG / 32);
  const int64_t blocks = n_fix + (from_act ? (group_sums_waves(p.N, p.nq, Geff) + 3) / 4 : 0);
  if (blocks > 0x7fffffff) return hipErrorInvalidValue;
  void* args[] = {&local, &fix, &scale, &sums, &Geff, &n_fix};
  hipError_t e = hipLaunchKernel(from_act ? reinterpret_cast<const void*>(rows_fix_kernel<true>)
                                          : reinterpret_cast<const void*>(rows_fix_kernel<false>),
                                 dim3((unsigned)blocks), dim3(256), args, 0, st);
  if (e != hipSuccess) return e;
  local.tables = reinterpret_cast<const uint16_t*>(fix);
  local.fix_scale = scale;
  local.S = sums;
  local.share = rows_share(pl.fix_wgs, pl.fix_total, pl.row_blocks, p.n_chunks);
  const void* fn = pl.fix_shift == 2 ? rows_run_kernel<RUN_BLOCK>(bits) : p.cpg == 1 ? rows_run_kernel<RUN_SOLO>(bits) : rows_run_kernel<RUN_CHUNK>(bits);
  void* args2[] = {&local};
  e = hipLaunchKernel(fn, dim3((pl.fix_wgs + 7) / 8 * 8), dim3(64 * ROWS_WAVES), args2, 0, st);
  if (e != hipSuccess) return e;
  return launch_rows_sum<false, true>(local, 0, st);
}

template <bool IS_INT, int BITS, int NT, bool FUSED>
static hipError_t launch_rows8_one(const RowsParams& p, hipStream_t st) {
  RowsParams local = p;
  const int nz = p.slices;
  void* args[] = {&local};
  const dim3 grid((p.N + NT - 1) / NT, (p.n_tiles + ROWS_WAVES - 1) / ROWS_WAVES, nz);
  const uint64_t wgs = (uint64_t)grid.x * grid.y * grid.z;
  const int units = p.n_chunks >> p.cpg_log2;  // (n_chunks is a multiple: K is one of the group's size, and padded to 128)
  local.grid8 = Rows8Grid{units / nz, units % nz, rows_inverse(grid.x, wgs), rows_inverse(grid.y, wgs / grid.x)};
  const int len = (local.grid8.per + (local.grid8.more > 0)) << p.cpg_log2;  // chunks of the longest slice
  const int lds = rows8_lds_bytes(NT, FUSED, len);
  const void* const kernel = len > R8_CH ? reinterpret_cast<const void*>(mpgemm_rows8_kernel<IS_INT, BITS, NT, FUSED, R8_LONG>)
                             : wgs > 256u * (unsigned)rows8_wgs(NT, BITS, len)
                                 ? reinterpret_cast<const void*>(mpgemm_rows8_kernel<IS_INT, BITS, NT, FUSED, R8_ROUNDS>)
                                 : reinterpret_cast<const void*>(mpgemm_rows8_kernel<IS_INT, BITS, NT, FUSED, R8_ONCE>);
  hipError_t e = hipLaunchKernel(kernel, grid, dim3(64 * ROWS_WAVES), args, lds, st);
  if (e != hipSuccess || nz == 1) return e;
  return launch_rows_sum<IS_INT>(p, nz, st);
}

template <bool IS_INT, int NT, bool FUSED>
static hipError_t launch_rows8_bits(const RowsParams& p, int bits, hipStream_t st) {
  switch (bits) {
    case 1: return launch_rows8_one<IS_INT, 1, NT, FUSED>(p, st);
    case 2: return launch_rows8_one<IS_INT, 2, NT, FUSED>(p, st);
    case 3: return launch_rows8_one<IS_INT, 3, NT, FUSED>(p, st);
    case 4: return launch_rows8_one<IS_INT, 4, NT, FUSED>(p, st);
  }
  return hipErrorInvalidValue;
}

template <bool IS_INT, bool FUSED = false>
static hipError_t launch_rows8_nt(const RowsParams& p, int nt, int bits, hipStream_t st) {
  return nt == ROWS_NT_WIDE ? launch_rows8_bits<IS_INT, ROWS_NT_WIDE, FUSED>(p, bits, st)
                            : launch_rows8_bits<IS_INT, ROWS_NT_NARROW, FUSED>(p, bits, st);
}

// K slices of the eight-chunk kernel, whole groups each, eight to sixteen chunks long: the most of which a CU gets at most
// five workgroups (further wavefronts do not pay for their partial sums), else the most that the chip holds at once, and
// slices of eight chunks if there is no such number.  Measured with every split of 90 random calls of 4 to 100 rows: where
// this takes longer slices, ones of eight chunks take 0.94 to 1.19 times as long, 1.07 on average (40 calls; 25 x 3859 x 5600,
// 4 bit 23.0 us, 27.2 with eight, 36 x 2267 x 4096, 2 bit 20.1, 18.8); where no split fits, longer ones take 0.99 to 1.14 times as long
// as eight, 1.04 on average (29 calls; 100 x 1890 x 8704, 1 bit 30.3, 34.7 with sixteen).  The fastest split of each call is another 1.8 %
// faster.  `fewest`: see rows_plan_oct.
static int rows8_slices(int64_t pairs, int n_chunks, int cpg, int nt, int bits, int fewest) {
  const int most = (n_chunks + R8_CH - 1) / R8_CH, least = std::max((n_chunks + R8_MOST - 1) / R8_MOST, fewest);
  for (const int per_cu : {5, 8}) {
    for (int s = most; s >= least; --s) {
      const int len = (n_chunks / cpg + s - 1) / s * cpg;
      if (len > R8_MOST) break;
      if (pairs * s <= 256 * std::min(rows8_wgs(nt, bits, len), per_cu)) return s;
    }
  }
  return most;
}

// Calls that may build their tables inside the eight-chunk kernel, where it serves them (rows_builds_tables).
static bool rows_may_build(const tmac_wdesc* desc, int N) { return N <= 32 && desc->K % 8 == 0; }

// How a call is split: workgroups along N and M, and the number of K slices (1 when the (row block,
// n tile) pairs alone fill the chip; otherwise enough slices of at least 256 k, whole quantisation
// groups each, to give about two workgroups per CU).
// The plan with `oct` n tiles per workgroup.
static RowsPlan rows_plan_oct(const tmac_wdesc* desc, int N, int oct) {
  const Geometry ge = geometry(desc);
  RowsPlan pl;
  pl.row_blocks = (ge.n_tiles + ROWS_WAVES - 1) / ROWS_WAVES;
  pl.nt = rows_nt(N, desc->g);
  pl.oct = oct;
  pl.n_tiles_n = (N + pl.nt * pl.oct - 1) / (pl.nt * pl.oct);
  const bool one_group = (desc->group == 0 || desc->group == desc->K);
  const int cpg = (one_group || desc->group < 32) ? 1 : desc->group / 32;  // (sizes below 32 are rejected at launch)
  const int min_cps = (8 + cpg - 1) / cpg * cpg;  // at least 256 k, whole groups
  const int64_t pairs = (int64_t)pl.n_tiles_n * pl.row_blocks;
  int64_t want = pairs >= ROWS_TARGET_WGS ? 1 : (ROWS_TARGET_WGS + pairs - 1) / pairs;
  const int max_slices = (ge.n_chunks + min_cps - 1) / min_cps;
  if (want > max_slices) want = max_slices;
  int cps = (int)((ge.n_chunks + want - 1) / want);
  // whole LDS slices where a workgroup gets at least one (nothing staged in vain), whole groups always
  const int lds_chunks = rows_lds_chunks(desc->g, pl.nt) / pl.oct;
  int unit = cpg;
  if (want > 1 && cps >= lds_chunks) {
    unit = lds_chunks;
    while (unit % cpg) unit += lds_chunks;
  }
  cps = (cps + unit - 1) / unit * unit;
  if (cps < min_cps) cps = min_cps;
  pl.cps = cps;
  // eight-chunk slices, several of them, g = 4, a group size that divides 256 (or no groups):
  // the kernel pair for few activation rows.  (Workspace sizes stay those of such slices also where rows8_slices takes fewer: which
  // calls tmac_mpgemm_noalloc has room for and where a run of chunks fits (rows_plan) does not move with the split.)
  pl.eight = pl.oct == 1 && desc->g == 4 && cps == R8_CH && ge.n_chunks > R8_CH && (one_group || R8_CH % cpg == 0);
  pl.slices = (ge.n_chunks + cps - 1) / cps;
  pl.part_bytes = pl.slices > 1 ? ((size_t)pl.slices * N * ge.Mp * 4 + 255) / 256 * 256 : 0;
  pl.ctr_bytes = 0;  // (no arrival counters: the slices meet in rows_sum_kernel)
  pl.fix = false;
  pl.fix_tiles = pl.fix_shift = pl.fix_wgs = pl.fix_total = pl.run_wgs = pl.run_total = 0;
  pl.fix_part_bytes = pl.fix_tab_bytes = pl.fix_scale_bytes = pl.fix_sums_bytes = 0;
  pl.srow_bytes = pl.eight ? ((size_t)pl.slices * N * 4 + 255) / 256 * 256 : 0;
  // (tables built in the kernel and one scale per row or tensor: the sums of the activations are in ws_srow, a part from
  // each slice, for rows_sum_kernel to add, which is launched from two slices on)
  if (pl.eight) pl.slices = rows8_slices(pairs, ge.n_chunks, cpg, pl.nt, desc->bits, one_group && rows_may_build(desc, N) ? 2 : 1);
  return pl;
}

// Many activation rows at g = 4: a workgroup takes two n tiles (16 rows), one address permute per two
// reads.  Measured against one n tile per workgroup (precompute + lookup, 4 bit): 13824 x 5120 even
// at 48 rows, 7 % ahead at 64, 9 % at 96, 6 % at 128 and beyond; 4096 x 4096, where the eight-chunk
// kernel pair serves up to 192 rows, behind below 96 rows, even at 96, 4 % ahead at 128.
static RowsPlan rows_plan_plain(const tmac_wdesc* desc, int N) {
  const RowsPlan one = rows_plan_oct(desc, N, 1);
  const bool can = desc->g == 4 && one.nt == ROWS_NT_WIDE;
  if (can && (N >= 128 || (N >= 64 && !one.eight))) return rows_plan_oct(desc, N, 2);
  return one;
}

// The run of chunks (RowsShare) for a call of `pairs` pairs: workgroups, chunks in all, most parts of a pair.
struct RunPlan {
  int wgs, total, parts;
};
static RunPlan rows_run(int64_t pairs, int n_chunks) {
  RunPlan r = {0, 0, 0};
  const int64_t total = pairs * n_chunks;
  if (total >= (1 << 30)) return r;  // (32-bit arithmetic in the kernel)
  // (a second round of workgroups for long runs, whose shares drift apart all the same.  Times as fast as one round: of 17
  // calls of 65536 to 138240 chunks 16 at 0.98 to 1.00, one at 1.005; of 14 of 163840 to 276480 nine at 1.004 to 1.05 (511 x 13824
  // x 5120, 2 bit 356.5 -> 352.8 us, in groups of 32 435 -> 414), five at 0.99 to 1.00)
  const int wgs = total >= ROWS_RUN_LONG ? 2 * ROWS_RUN_WGS : ROWS_RUN_WGS;
  r.wgs = (int)(total < wgs ? total : wgs);
  r.total = (int)total;
  const int per = r.total / r.wgs;  // at least this many chunks each
  r.parts = r.total % r.wgs == 0 && n_chunks % per == 0 ? n_chunks / per : (n_chunks - 1) / per + 2;
  return r;
}

// Which calls are served by a run of chunks (RowsShare), and which fp16 tables become fixed-point numbers.
//
// Run of chunks, integer tables (one scale per row or tensor, more than 32 rows): from ROWS_RUN_INT_CHUNKS on, twelve
// for each workgroup.  Times as fast as K slices of equal length: 1.10 at 12288 chunks (96 rows x 4096 x 4096), 1.16 at
// 16512 (48 x 11008 x 4096), 1.05 to 1.18 at 14000 to 57000; below, 1.00 at 8192 (64 x 4096 x 4096), 1.00 at 6144
// (33 x 4096 x 4096), 0.96 at 5504 (16 x 11008 x 4096).
// Run of chunks, fp16 tables and 2 to 4 bits, as fixed-point numbers (groups of 128 unless said otherwise):
//   * built from activations (tmac_mpgemm_fused; the conversion takes the place of the precompute): from
//     ROWS_RUN_ACT_CHUNKS on, and ROWS_RUN_ACT_BITS chunks times bits.  Of 41 random calls up to twice that line 39 are
//     faster than with fp16 sums, 1.08 times on average (0.97 to 1.20; 0.93 at 511 x 1024 x 2048, 2 bit, and 40 x 4096 x
//     4096, 3 bit; 1.31 at 48 x 11008 x 4096, 4 bit); of 19 below it, from 10000 on, six, 0.97 times as fast (0.83 to 1.07;
//     40 x 4096 x 4096, 2 bit 26.4 us against 22.0).  Up to 32 rows the other side builds its tables in the look-up
//     kernel and saves a launch: chunks times bits from ROWS_RUN_ACT_FEW on, 1.18 times on average (11 calls from 32768 on,
//     1.00 to 1.42: 32 x 8192 x 4096, 4 bit 1.00, 16 x 13824 x 5120 1.20), 0.95 at the line (16 x 16384 x 4096, 3 bit in
//     groups of 64) and below it 0.78 to 0.94 (32 x 4096 x 4096, 16 x 8192 x 4096, 16 x 11008 x 4096, 4 bit), 1.17 once
//     (32 x 11008 x 4096, 2 bit).  For time alone the line would be 32768; results between are closer with fixed point.
//   * from a LUT buffer the conversion is one more launch: look-ups from ROWS_RUN_LUT_LOOKUPS on, 1.4 times as many up to 32
//     rows, twice as many there where more than 15 % of the sets' rows do not exist; ROWS_RUN_LUT_ROWS weight rows times bits
//     for each table; and ROWS_RUN_ACT_CHUNKS, in sets that are not full ROWS_RUN_INT_CHUNKS.  Of 64 random calls that these lines take 55 are faster than with fp16
//     sums, 1.06 times on average (0.94 to 1.21); of 46 that they leave, from 0.4e9 look-ups on, 14, 0.95 (0.72 to 1.08).
//     At the lines: 1.05 and 1.07 at 0.8e9 and 1.07e9 look-ups (64 x 4096 x 4096, 3 and 4 bit), 0.94 and 0.96 at 0.6e9 (48 x
//     4096 x 4096 and 64 x 3072 x 4096, 3 bit); up to 32 rows 0.80 to 0.98 below (32 x 4096 x
//     4096, 16 x 11008 x 4096, 4 bit, 20 x 12000 x 5120, 3 bit; 1.11 and 1.25 at 2 bit: 32 x 11008 x 4096, 28 x 16384 x 4096 in
//     groups of 32), between 1.4 and 2 times the line 1.07 on average in sets that are full (25 calls, 0.99 to 1.20; 16 x
//     13824 x 5120 and 32 x 8192 x 4096, 4 bit 1.04 and 1.05) and 0.97 in others (18 calls, 0.91 to 1.07; 20 x 28512 x 1856, 4 bit
//     46.8 us against 51.7), 1.26 above (16 x 28672 x 4096, 4 bit); weight rows times bits 1.05 at 2100 (300 x 700 x
//     8192, 3 bit), 0.90 to 1.07 at 1200 to 1536 (eleven calls, seven below 1), 0.88 at 768 (511 x 256 x 13824, 3 bit);
//     sets that are not full 0.92, 1.00 and 1.05 at 8448, 11264 and 10240 chunks (40 x 2700 x 8192, 52 x 2800 x 8192, 65 x 2048
//     x 8192).  Within the library's own array where the plain plan is, because tmac_mpgemm_noalloc gives tmac_mpgemm's
//     results bit for bit.
// At 1 bit fixed point is 0.93 to 1.05 times as fast as fp16 sums: tables and launches weigh four times as much there.
RowsPlan rows_plan(const tmac_wdesc* desc, int N, bool from_act) {
  RowsPlan pl = rows_plan_plain(desc, N);
  if (desc->g != 4 || N <= 8) return pl;
  const size_t room = pl.part_bytes + pl.ctr_bytes + pl.srow_bytes;
  const Geometry ge = geometry(desc);
  const bool one_group = (desc->group == 0 || desc->group == desc->K);
  const int cpg = (one_group || desc->group < 32) ? 1 : desc->group / 32;
  const int tiles = (N + 15) / 16;
  const int64_t pairs = (int64_t)tiles * pl.row_blocks;
  const size_t slice = (size_t)N * ge.Mp * 4;
  const RunPlan run = rows_run(pairs, ge.n_chunks);
  if (one_group && N > 32 && pl.nt == ROWS_NT_WIDE && run.total >= ROWS_RUN_INT_CHUNKS && (size_t)run.parts * slice <= room) {
    pl.run_wgs = run.wgs;
    pl.run_total = run.total;
  }
  if (desc->bits < 2) return pl;
  // units: one per 128-k block where no block holds parts of two groups, else one per chunk
  const int shift = (one_group || cpg % 4 == 0) ? 2 : 0;
  const size_t tab = rows_raw_bytes(desc, N), scale = (size_t)tiles * (ge.n_chunks >> shift) * 64;
  const size_t sums = (size_t)tiles * (one_group ? 1 : desc->K / desc->group) * 64;
  const double lookups = (double)N * ge.Mp * (ge.Kp / 4) * desc->bits;
  const size_t run_parts = ((size_t)run.parts * slice + 255) / 256 * 256;
  if (!run.wgs) return pl;
  bool take;
  if (from_act) {
    const int64_t by_bits = (int64_t)run.total * desc->bits;
    take = N > 32 ? run.total >= ROWS_RUN_ACT_CHUNKS && by_bits >= ROWS_RUN_ACT_BITS : by_bits >= ROWS_RUN_ACT_FEW;
  } else {
    const bool part_full = N * 20 < tiles * 16 * 17;  // sets with many rows that do not exist
    take = lookups >= (N > 32 ? 1. : part_full ? 2. : 1.4) * ROWS_RUN_LUT_LOOKUPS && (int64_t)desc->M * desc->bits >= ROWS_RUN_LUT_ROWS &&
           run.total >= (part_full && pl.nt == ROWS_NT_WIDE ? ROWS_RUN_INT_CHUNKS : ROWS_RUN_ACT_CHUNKS);
    const size_t own = (size_t)TMAC_NOALLOC_MAX_WORKSPACE;  // within the library's own array where the plain plan is
    if (room <= own && run_parts + tab + scale + sums > own) take = false;
  }
  if (!take) return pl;
  pl.fix = true;
  pl.fix_wgs = run.wgs;
  pl.fix_total = run.total;
  pl.fix_tiles = tiles;
  pl.fix_shift = shift;
  pl.fix_part_bytes = run_parts;
  pl.fix_tab_bytes = tab;
  pl.fix_scale_bytes = scale;
  pl.fix_sums_bytes = sums;
  return pl;
}

// (as many as the fixed-point tables themselves take)
size_t rows_raw_bytes(const tmac_wdesc* desc, int N) { return (size_t)((N + 7) / 8) * (geometry(desc).Kp / 4) * 256; }

bool rows_fixed_from_act(const tmac_wdesc* desc, int N) { return desc->g == 4 && rows_plan(desc, N, true).fix; }

// Whether the eight-chunk kernel could build the tables of a call that brings activations; such calls need a
// leading dimension that is a multiple of eight, whichever kernel serves them.
bool rows_reads_eight(const tmac_wdesc* desc, int N) {
  return rows_may_build(desc, N) && rows_plan_plain(desc, N).eight;  // (activations are summed eight at a time)
}

// Whether a call builds its tables inside the lookup kernel when it is given activations instead
// of a LUT buffer: the eight-chunk kernel, up to 32 activation rows (every
// block of 256 weight rows builds the tables again: from 64 rows on that costs more than the
// launch of the precompute kernel it saves).
bool rows_builds_tables(const tmac_wdesc* desc, int N, bool is_int) {
  return rows_reads_eight(desc, N) && (is_int || !rows_fixed_from_act(desc, N));  // (activations are summed eight at a time)
}

// lut_dev: buffer of tmac_precompute_lut, or NULL with A_dev / lda given (only where
// rows_builds_tables says so), or with fixed_from_act room for such a buffer, and A_dev / lda.
int launch_rows_gemm(const tmac_wdesc* desc, const void* packed_dev, const void* lut_dev, const void* A_dev,
                     int64_t lda, int lut_t, int N, const float* act_scale_dev, float weight_scale, void* out_dev,
                     int out_t, int64_t ldo, void* workspace_dev, size_t workspace_bytes, void* stream, bool fixed_from_act) {
  if (lut_t != TMAC_LUT_F16 && lut_t != TMAC_LUT_I16) return TMAC_EUNSUPPORTED;
  const bool from_act = fixed_from_act;  // fixed-point tables from the activations; lut_dev: room for a LUT buffer
  const bool fused = (lut_dev == nullptr);
  if (fused && (!A_dev || !rows_builds_tables(desc, N, lut_t == TMAC_LUT_I16))) return TMAC_EUNSUPPORTED;
  if (from_act && (!lut_dev || !A_dev || lut_t != TMAC_LUT_F16 || !rows_fixed_from_act(desc, N))) return TMAC_EUNSUPPORTED;
  const Geometry ge = geometry(desc);
  LutGeom lg;
  if (!lut_geom(N, desc->K, desc->g, desc->group, lut_t, &lg)) return TMAC_EINVAL;
  const bool is_int = (lut_t == TMAC_LUT_I16);
  const bool one_group = (desc->group == 0 || desc->group == desc->K);
  const RowsPlan pl = rows_plan(desc, N, from_act);
  if (fused && one_group && pl.slices < 2) return TMAC_EUNSUPPORTED;  // (no buffer of row sums to finish from)
  if (pl.n_tiles_n > 0x7fffffff || pl.row_blocks > 65535 || pl.slices > 65535) return TMAC_EUNSUPPORTED;
  if (pl.bytes() > 0) {
    if (!workspace_dev) return TMAC_EINVAL;
    if (workspace_bytes < pl.bytes()) return TMAC_ESIZE;
  }
  // int32 accumulators: |L| <= 128 * (2^b - 1) * K must stay below 2^31
  if (is_int && (double)128.0 * ((1 << desc->bits) - 1) * desc->K >= 2147483647.0) return TMAC_EUNSUPPORTED;

  RowsParams p;
  const char* blob = static_cast<const char*>(packed_dev);
  p.idx = reinterpret_cast<const uint32_t*>(blob + ge.idx_off);
  p.sz = reinterpret_cast<const uint32_t*>(blob + ge.sz_off);
  p.tables = static_cast<const uint16_t*>(lut_dev);
  p.S = lut_dev == nullptr ? nullptr : static_cast<const char*>(lut_dev) + lg.s_off;
  p.A = A_dev;
  p.lda = lda;
  p.K = desc->K;
  p.out = out_dev;
  p.act_scale = act_scale_dev;
  p.ldo = ldo;
  p.M = desc->M; p.N = N; p.KG = lg.KG; p.n_tiles = ge.n_tiles; p.n_chunks = ge.n_chunks; p.nq = lg.nq;
  p.grouped = one_group ? 0 : 1;
  p.cpg = one_group ? 1 : desc->group / 32;
  p.cpg_log2 = 0;
  while ((2 << p.cpg_log2) <= p.cpg) ++p.cpg_log2;
  p.cps = pl.cps;
  p.slices = pl.slices;
  p.Mp = ge.Mp;
  p.ws_part = static_cast<float*>(workspace_dev);
  p.ws_srow = (fused && one_group) ? reinterpret_cast<float*>(static_cast<char*>(workspace_dev) + pl.part_bytes + pl.ctr_bytes)
                                   : nullptr;
  p.per_tensor = (desc->group == 0);
  p.wscale = weight_scale;
  p.mid = 0.5f * (float)((1 << desc->bits) - 1);
  p.zero_point = p.per_tensor ? desc->zero_point : 0.f;
  p.int_exact = 0;
  p.icoef = 0;
  p.out_t = out_t;
  p.pw[0] = 1.f; p.pw[1] = 2.f; p.pw[2] = 4.f; p.pw[3] = 8.f;
  if (p.per_tensor && is_int) {
    const float z = desc->zero_point;
    if (z == rintf(z) && fabsf(z) < 64.f) {
      p.int_exact = 1;
      p.icoef = ((1 << desc->bits) - 1) - 2 * (int)z;
    }
  }
  if (out_t == TMAC_OUT_I32 && !p.int_exact) return TMAC_EINVAL;
  hipStream_t st = static_cast<hipStream_t>(stream);
  hipError_t e;
  p.fix_scale = nullptr;
  p.lut_nt = pl.nt;
  p.raw_nt = from_act ? 8 : pl.nt;
  p.share = RowsShare{};
  p.fix_shift = pl.fix_shift;
  p.raw = nullptr;
  if (pl.fix && !is_int && !fused) {
    char* const tab = static_cast<char*>(workspace_dev) + pl.fix_part_bytes;
    e = launch_rows_fix(p, pl, desc->bits, from_act, lg.Geff, reinterpret_cast<uint32_t*>(tab),
                        reinterpret_cast<float*>(tab + pl.fix_tab_bytes),
                        reinterpret_cast<float*>(tab + pl.fix_tab_bytes + pl.fix_scale_bytes), st);
  } else if (pl.run_wgs && is_int) {
    p.share = rows_share(pl.run_wgs, pl.run_total, pl.row_blocks, p.n_chunks);
    void* args[] = {&p};
    e = hipLaunchKernel(rows_run_kernel<RUN_INT>(desc->bits), dim3((pl.run_wgs + 7) / 8 * 8), dim3(64 * ROWS_WAVES), args, 0, st);
    if (e == hipSuccess) e = launch_rows_sum<true, true>(p, 0, st);
  } else if (fused) e = is_int ? launch_rows8_nt<true, true>(p, pl.nt, desc->bits, st) : launch_rows8_nt<false, true>(p, pl.nt, desc->bits, st);
  else if (pl.eight) e = is_int ? launch_rows8_nt<true>(p, pl.nt, desc->bits, st) : launch_rows8_nt<false>(p, pl.nt, desc->bits, st);
  else e = is_int ? launch_rows_nt<true>(p, desc->g, pl.nt, pl.oct, desc->bits, st) : launch_rows_nt<false>(p, desc->g, pl.nt, pl.oct, desc->bits, st);
  if (e != hipSuccess) {
    note_hip_error((int)e);
    return TMAC_EHIP;
  }
  return TMAC_OK;
}

}  // namespace tmac
