// bf16 GEMM on the gfx950 matrix cores (v_mfma_f32_32x32x16_bf16, fp32
// accumulate) for the VJP and parameter-gradient contractions.
//
// Shape of the kernel
//   workgroup   8 wavefronts, output tile 256 x 256, one workgroup per CU; a
//               wavefront owns 128 x 64 = 4 x 2 MFMA blocks of 32 x 32 (128
//               accumulator registers per lane).  The 256 x 256 tile keeps the
//               global -> LDS stream, which is what bounds the kernel (measured:
//               the copies alone take 0.6 of the time the MFMAs alone take),
//               at 128 flop per byte copied.
//   persistent  one workgroup per CU walks a list of tiles.  The K slices of all
//               its tiles form one stream through a ring of 4 LDS stages, so the
//               first slices of the next tile are already in flight while the
//               current tile's epilogue runs: no per-tile fill latency.
//   two phases  the wavefronts form two groups of four (one wavefront of each
//               group per SIMD).  A wavefront alternates between a load phase
//               (issue its share of the global -> LDS copy of the slice three
//               ahead, read all fragments of the current slice from LDS, store
//               a finished tile) and a compute phase (16 MFMAs back to back
//               at raised priority), with a workgroup barrier after each
//               phase.  The second group runs one barrier behind the first, so
//               on every SIMD one wavefront multiplies while the other one
//               loads: the LDS latency is paid once per slice, in bulk, and
//               hidden behind the other group's MFMAs.  A wavefront issues at
//               most one instruction every four cycles, so the load phase has to
//               be short in instructions to fit under the 512 MFMA cycles of the
//               other group: the lean kernel's is about 50.
//   K pipeline  slices of 32 (32 KB per stage); a slice is copied global -> LDS
//               directly (global_load_lds_dwordx4, no staging registers), issued
//               from inline assembly so that the waits can be counted by hand.
//   LDS layout  an operand tile sits in LDS in the orientation it has in memory:
//                 KC  contraction index contiguous, [rows][32 k]: a lane's 8
//                     k-values are one 16-byte ds_read;
//                 RC  row index contiguous, [32 k][rows]: the lane's 8 k-values
//                     are strided and fetched with the LDS transpose read
//                     ds_read_b64_tr_b16 (two per fragment; within 16 lanes it
//                     returns to lane j, element r, element j%4 of the 8 bytes
//                     addressed by lane 4r + j/4).
//               A direct-to-LDS copy writes 1 KB per wavefront contiguously, so
//               rows cannot be padded; the 64 LDS banks are spread by an XOR
//               swizzle of the 16-byte chunk index instead, applied on the
//               global-address side of the copy and again by the readers.
//   pairings    NN (A KC, B RC)  da = g W2, dn = da W1   (weights as stored)
//               TN (A RC, B RC)  dW2 = g^T z, dW1 = da^T y, dU
//               NT (A KC, B KC)  forward  a = y W1^T, out = z W2^T
//   accumulator the MFMAs are issued with the operands exchanged (B fragment
//               first), which leaves a lane with one output row and groups of
//               four consecutive output columns.
//   lean        every tile inside the matrix, K a multiple of 32, the hot
//               epilogues.  Straight-line: its epilogues issue a
//               known number of memory operations, so the copies stay counted
//               across them.  bf16 tiles leave through 4 KB of wave-private LDS
//               so that every global access covers whole 128-byte lines; fp32
//               tiles (parameter gradients, one per 256+ slices) are stored
//               from the registers, 16 bytes per lane.  Every other size, the
//               remaining epilogues and launches with few tiles go to
//               gemm_tile.hip; launch_gemm_mfma at the end of this file decides.
//   tile order  workgroup ids are dealt round-robin to the 8 XCDs (one L2
//               each): id % 8 selects a contiguous eighth of the tile list,
//               the workgroups of an XCD take consecutive tiles of it, and the
//               list walks 8 x 8 blocks of tiles, so the tiles an XCD works on
//               at one time share operand panels.
#include "gemm_device.h"
#include <type_traits>

namespace hbp {

namespace {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float float2v __attribute__((ext_vector_type(2)));

constexpr int BM = 256, BN = 256, BK = 32, NW = 8, NTHR = 64 * NW;
constexpr int A_BYTES = BM * BK * 2;            // 16 KB
constexpr int B_BYTES = BN * BK * 2;            // 16 KB
constexpr int STAGE_BYTES = A_BYTES + B_BYTES;  // 32 KB
constexpr int GROUP_M = 8;                      // tile rows per block of the tile walk
constexpr int PER_SLICE = 4;                    // copies per wave per slice (2 for A, 2 for B)

// Byte offset of this lane's chunk of copy i (of 2) relative to the first
// element of the tile's slice (the same for every slice and tile of a launch).
template <bool KC>
__device__ __forceinline__ unsigned lane_src_offset(long ld, int i, int wave, int lane) {
  const int j = wave + NW * i;
  if (KC) {
    const int r = 16 * j + (lane >> 2);
    const int c = (lane & 3) ^ ((r >> 2) & 3);
    return (unsigned)(r * ld + 8 * c) * 2u;
  } else {
    const int k = 2 * j + (lane >> 5);
    const int c = (lane & 31) ^ (4 * (k & 3));
    return (unsigned)(k * ld + 8 * c) * 2u;
  }
}
// 32 rows x 16 k fragment: lane l holds row (l % 32), k = kk + 8*(l/32) .. +7
template <bool KC>
__device__ __forceinline__ bf16x8 frag(const unsigned char* tile, int row0, int kk, int lane) {
  if (KC) {
    const int r = row0 + (lane & 31);
    const int c = (kk >> 3) + (lane >> 5);
    const uint4 v = *reinterpret_cast<const uint4*>(tile + r * 64 + ((c ^ ((r >> 2) & 3)) << 4));
    return __builtin_bit_cast(bf16x8, v);
  } else {
    typedef __attribute__((address_space(3))) short4v* lds_p;
    const int s = lane & 15;
    const int e = row0 + 16 * ((lane >> 4) & 1) + 4 * (s & 3);
    const int k = kk + 8 * (lane >> 5) + (s >> 2);          // k & 3 == s >> 2 for both halves
    const int sw = 4 * (s >> 2);
    const unsigned char* p = tile + k * 512 + (((e >> 3) ^ sw) << 4) + (e & 7) * 2;
    const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_p)(p));
    const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_p)(p + 4 * 512));
    const short8v v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, v);
  }
}

// 4 consecutive elements <-> 4 floats
__device__ __forceinline__ unsigned pack2(float a, float b) {   // round to nearest even (v_cvt_pk_bf16_f32)
  const float2v v = {a, b};
  return __builtin_bit_cast(unsigned, __builtin_convertvector(v, bf16x2));
}
__device__ __forceinline__ void unpack4(uint2 r, float (&o)[4]) {
  o[0] = __uint_as_float(r.x << 16); o[1] = __uint_as_float(r.x & 0xFFFF0000u);
  o[2] = __uint_as_float(r.y << 16); o[3] = __uint_as_float(r.y & 0xFFFF0000u);
}

// Division of numbers below 2^31 by a fixed d: (n m) >> sh with m = floor(2^sh / d) + 1, sh = 31 + ceil(log2 d) (the method
// of Granlund and Montgomery).  The hardware has no integer division, and a tile's coordinates took two 64-bit and five
// 32-bit ones, twice per tile: about 1.5 us of a tile that takes 18.
struct FastDiv {
  unsigned m, sh;
  __device__ __forceinline__ unsigned operator()(unsigned n) const { return (unsigned)(((unsigned long long)n * m) >> sh); }
};
inline FastDiv fast_div(unsigned d) {
  unsigned s = 0;
  while ((1ull << s) < d) ++s;
  return {(unsigned)((1ull << (31 + s)) / d + 1), 31 + s};
}
// the tile walk of a launch: a tile's share of the contraction is KT slices, one more in the first `longer` of the shares
struct Walk {
  FastDiv by_mn, by_grp, by_split;
  unsigned tiles_mn, grp_tiles;      // tiles per matrix, and per block of GROUP_M tile rows
  int tiles_m, split, KT, longer, total, per_xcd;
};
inline Walk make_walk(const GemmArgs& g) {
  Walk w;
  const unsigned tm = (unsigned)(g.M / BM), tn = (unsigned)(g.N / BN);
  w.tiles_m = (int)tm;
  w.tiles_mn = tm * tn;
  w.grp_tiles = GROUP_M * tn;
  w.split = g.split_k;
  w.by_mn = fast_div(w.tiles_mn);
  w.by_grp = fast_div(w.grp_tiles);
  w.by_split = fast_div((unsigned)g.split_k);
  w.KT = (int)(g.K / BK / g.split_k);
  w.longer = (int)(g.K / BK % g.split_k);
  w.total = (int)((long)w.tiles_mn * g.batch * g.split_k);
  w.per_xcd = (w.total + 7) / 8;
  return w;
}

// coordinates of one output tile, its share of the contraction: the start and the number of slices
struct TileCoord {
  long batch, m0, n0, k_begin;
  int split, kt;
};

__device__ __forceinline__ TileCoord decode_tile(const Walk& w, int t) {
  TileCoord c;
  const unsigned zb = w.by_mn((unsigned)t);              // batch * split_k + split
  const unsigned rem = (unsigned)t - zb * w.tiles_mn;
  const unsigned grp = w.by_grp(rem);
  const unsigned in_grp = rem - grp * w.grp_tiles;
  const unsigned left = (unsigned)w.tiles_m - grp * GROUP_M;
  unsigned col = in_grp / GROUP_M, row = in_grp % GROUP_M;
  if (left < (unsigned)GROUP_M) { col = in_grp / left; row = in_grp - col * left; }   // the last, lower block
  c.m0 = (long)(grp * GROUP_M + row) * BM;
  c.n0 = (long)col * BN;
  const unsigned batch = w.by_split(zb);
  c.batch = batch;
  c.split = (int)(zb - batch * (unsigned)w.split);
  c.kt = w.KT + (c.split < w.longer);
  c.k_begin = ((long)c.split * w.KT + (c.split < w.longer ? c.split : w.longer)) * BK;
  return c;
}

// Epilogues of the lean kernel
enum FastEpi {
  FAST_STORE = 1,      // C(bf16) = acc
  FAST_STORE_F32 = 2,  // C(fp32) = acc, also the split-K partial sums
  FAST_MUL_AUX = 3,    // C(bf16) = acc * aux
  FAST_MUL_1MZ2 = 4,   // C(bf16) = acc * (1 - aux^2)
  FAST_ADD_AUX = 5,    // C(bf16) = acc + aux
  FAST_RESID = 6,      // C(bf16) = acc + lambda[n] * aux   (forward: x_{l+1}; lambda NULL = 1)
  FAST_ACT_GELU = 7    // C(bf16) = gelu(acc), out2(bf16) = gelu'(acc)   (forward: z and act')
};

// Straight-line epilogue from the registers for a tile fully inside the matrix (fp32 output).
__device__ __forceinline__ void epilogue_f32(const GemmArgs& g, const TileCoord& tc, const float16v (&acc)[4][2], int wm0, int wn0,
                                             int lane) {
  const long cb = g.split_k > 1 ? ((long)tc.split * g.batch + tc.batch) * g.c_sb : tc.batch * g.c_sb;
  float* c = reinterpret_cast<float*>(g.C) + cb + (tc.m0 + wm0 + (lane & 31)) * g.ldc + tc.n0 + wn0 + 4 * (lane >> 5);
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        *reinterpret_cast<float4*>(c + (long)(32 * i) * g.ldc + 32 * j + 8 * q) =
            make_float4(acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]);
}

// The lean form of the kernel, for launches in which every tile lies inside the
// matrix and every tile's contraction range is a multiple of 4 slices: the LDS
// stage of every step is then a compile-time constant (four steps are written
// out), the copies need two scalar pointers that advance by a constant, and a
// step is ~40 instructions next to its 16 MFMAs.  (A wavefront issues at most
// one instruction every four cycles, so the instruction count of the load phase
// is what decides whether it fits under the other group's 512 MFMA cycles.)
template <int C>
__device__ __forceinline__ void dma16_c(unsigned off, const void* sbase, unsigned lds_wave_base) {
  asm volatile("s_add_u32 m0, %2, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1\n"
               :: "v"(off), "s"(sbase), "s"(lds_wave_base), "n"(C) : "memory", "scc");
}

// Epilogue of a bf16 tile through 4 KB of wave-private LDS, 32 rows x 64 columns at a time: the
// accumulators (and the fused operand) change between the MFMA layout (a lane owns one row and
// groups of 4 columns) and a row layout (8 lanes cover the 128 bytes of a row), so that every
// global access of a wave covers whole 128-byte lines: 8 rows per instruction.  The 16-byte chunk
// k of row r sits at chunk k ^ (r/2 % 8) of the row (bank spread for both access shapes).
// Lanes of one wave exchange data through LDS here: the hardware executes a wave's LDS instructions in
// order, and a wave barrier between the two access shapes keeps the compiler from moving a read of one
// shape above the writes of the other (it emits no instruction).
typedef unsigned uint4v __attribute__((ext_vector_type(4)));   // (a first-class vector: stays in registers)
struct Quad16 { uint4v x0, x1, x2, x3; };   // 4 x 16 bytes per lane: 32 rows of the row layout
template <int FAST> constexpr bool has_aux() {
  return FAST == FAST_MUL_AUX || FAST == FAST_MUL_1MZ2 || FAST == FAST_ADD_AUX || FAST == FAST_RESID;
}
// the fused operand's 32 rows of a round (of 4) in the row layout
__device__ __forceinline__ void fetch_aux(Quad16& q, const GemmArgs& g, const TileCoord& tc, int wm0, int wn0, int lane, int round) {
  const bf16_t* a = reinterpret_cast<const bf16_t*>(g.aux) + tc.batch * g.aux_sb +
                    (tc.m0 + wm0 + (lane >> 3) + 32 * round) * g.ldc + tc.n0 + wn0 + 8 * (lane & 7);
  const long ld8 = 8 * g.ldc;
  // (streamed once: non-temporal, so that it does not push the operand panels out of L2)
  q.x0 = __builtin_nontemporal_load(reinterpret_cast<const uint4v*>(a));
  q.x1 = __builtin_nontemporal_load(reinterpret_cast<const uint4v*>(a + ld8));
  q.x2 = __builtin_nontemporal_load(reinterpret_cast<const uint4v*>(a + 2 * ld8));
  q.x3 = __builtin_nontemporal_load(reinterpret_cast<const uint4v*>(a + 3 * ld8));
}
// qa, qb: the first two rounds' fused operand, fetched during the tile's last slices
template <int FAST>
__device__ __forceinline__ void epilogue_staged_fn(const GemmArgs& g, const TileCoord& tc, const float16v (&acc)[4][2],
                                                   int wm0, int wn0, int lane, unsigned char* stg, const Quad16& qa, const Quad16& qb) {
  constexpr bool HAS_AUX = has_aux<FAST>();
  constexpr bool TWO_OUT = FAST == FAST_ACT_GELU;
  // row layout: this lane's row within a group of 8 rows, and its chunk of the row
  const int rr = lane >> 3, rk = lane & 7;
  // MFMA layout: this lane's row within the 32, half-chunk (4 columns) within a chunk
  const int mr = lane & 31, mh = lane >> 5;
  const long off_row = (tc.m0 + wm0 + rr) * g.ldc + tc.n0 + wn0 + 8 * rk;     // row layout, first row group
  bf16_t* cp = reinterpret_cast<bf16_t*>(g.C) + tc.batch * g.c_sb + off_row;
  bf16_t* cp2 = TWO_OUT ? reinterpret_cast<bf16_t*>(g.out2) + tc.batch * g.out2_sb + off_row : nullptr;
  const long ld8 = 8 * g.ldc;
  // FAST_RESID: the coefficients of this lane's columns in the MFMA layout (chunk k: columns 8 k + 4 mh .. + 3)
  float lam[8][4];
  if (FAST == FAST_RESID) {
    const float* lp = g.lambda ? g.lambda + tc.batch * g.lambda_sb + tc.n0 + wn0 + 4 * mh : nullptr;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      if (lp) {
        const float4 t = *reinterpret_cast<const float4*>(lp + 8 * k);
        lam[k][0] = t.x; lam[k][1] = t.y; lam[k][2] = t.z; lam[k][3] = t.w;
      } else {
        lam[k][0] = lam[k][1] = lam[k][2] = lam[k][3] = 1.f;
      }
    }
  }
  // staging addresses, row layout: rows rr, rr + 8, rr + 16, rr + 24
  auto row_at = [&](int r) { return stg + r * 128 + ((rk ^ ((r >> 1) & 7)) << 4); };
  unsigned char* const p0 = row_at(rr);
  unsigned char* const p1 = row_at(rr + 8);
  unsigned char* const p2 = row_at(rr + 16);
  unsigned char* const p3 = row_at(rr + 24);
  unsigned char* const m_base = stg + mr * 128 + 8 * mh;
  const int m_sw = (mr >> 1) & 7;
  // 32 rows x 64 columns now in the staging tile (MFMA layout written): read as rows, store whole lines
  auto flush = [&](bf16_t* c) {
    __builtin_amdgcn_wave_barrier();
    const uint4v o0 = *reinterpret_cast<const uint4v*>(p0);
    const uint4v o1 = *reinterpret_cast<const uint4v*>(p1);
    const uint4v o2 = *reinterpret_cast<const uint4v*>(p2);
    const uint4v o3 = *reinterpret_cast<const uint4v*>(p3);
    __builtin_amdgcn_wave_barrier();      // the next round's writes stay behind these reads
    __builtin_nontemporal_store(o0, reinterpret_cast<uint4v*>(c));
    __builtin_nontemporal_store(o1, reinterpret_cast<uint4v*>(c + ld8));
    __builtin_nontemporal_store(o2, reinterpret_cast<uint4v*>(c + 2 * ld8));
    __builtin_nontemporal_store(o3, reinterpret_cast<uint4v*>(c + 3 * ld8));
  };
  auto round = [&](auto ic, const Quad16& q) {
    constexpr int i = decltype(ic)::value;
    uint2 auxm[8];
    uint2 second[8];        // TWO_OUT: the second output's values, packed, until the first has left the staging tile
    if (HAS_AUX) {
      *reinterpret_cast<uint4v*>(p0) = q.x0;
      *reinterpret_cast<uint4v*>(p1) = q.x1;
      *reinterpret_cast<uint4v*>(p2) = q.x2;
      *reinterpret_cast<uint4v*>(p3) = q.x3;
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int k = 0; k < 8; ++k) auxm[k] = *reinterpret_cast<const uint2*>(m_base + ((k ^ m_sw) << 4));
    }
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int qd = 0; qd < 4; ++qd) {
        float v[4];
#pragma unroll
        for (int x = 0; x < 4; ++x) v[x] = acc[i][j][4 * qd + x];
        if (HAS_AUX) {
          float t[4];
          unpack4(auxm[4 * j + qd], t);
#pragma unroll
          for (int x = 0; x < 4; ++x) {
            if (FAST == FAST_MUL_AUX) v[x] *= t[x];
            else if (FAST == FAST_ADD_AUX) v[x] += t[x];
            else if (FAST == FAST_RESID) v[x] = fmaf(lam[4 * j + qd][x], t[x], v[x]);
            else v[x] *= (1.f - t[x] * t[x]);
          }
        }
        if (TWO_OUT) {
          float dz[4];
#pragma unroll
          for (int x = 0; x < 4; ++x) gelu_both(v[x], v[x], dz[x]);
          second[4 * j + qd] = make_uint2(pack2(dz[0], dz[1]), pack2(dz[2], dz[3]));
        }
        *reinterpret_cast<uint2*>(m_base + (((4 * j + qd) ^ m_sw) << 4)) = make_uint2(pack2(v[0], v[1]), pack2(v[2], v[3]));
      }
    flush(cp + (long)(32 * i) * g.ldc);
    if (TWO_OUT) {
#pragma unroll
      for (int k = 0; k < 8; ++k) *reinterpret_cast<uint2*>(m_base + ((k ^ m_sw) << 4)) = second[k];
      flush(cp2 + (long)(32 * i) * g.ldc);
    }
  };
  // (the residual sum's 32 coefficients per lane leave registers for one more round at a time only)
  constexpr bool TIGHT = FAST == FAST_RESID;
  Quad16 qc = {}, qd = {};
  if (HAS_AUX) fetch_aux(qc, g, tc, wm0, wn0, lane, 2);
  if (HAS_AUX && !TIGHT) fetch_aux(qd, g, tc, wm0, wn0, lane, 3);
  round(std::integral_constant<int, 0>(), qa);
  if (TIGHT) fetch_aux(qd, g, tc, wm0, wn0, lane, 3);
  round(std::integral_constant<int, 1>(), qb);
  round(std::integral_constant<int, 2>(), qc);
  round(std::integral_constant<int, 3>(), qd);
}
template <int FAST> struct StagedOps {   // vector-memory operations per wave of one epilogue (a lower bound: the
  static constexpr int value = FAST == FAST_STORE_F32 ? 32 : FAST == FAST_STORE ? 16 : 32;   // waits stay safe with more)
};

constexpr int PAIR_AREA = 2 * A_BYTES;                   // 256 rows x 128 bytes: two slices of a K-contiguous operand
// Byte offset of this lane's 16 bytes of the first of a wave's four copies of a pair (rows 8 wave .. + 7 of the
// first 64; the lane's LDS place l % 8 in row l / 8 holds chunk (l % 8) ^ (row / 2 % 8) of the row's 128 bytes)
__device__ __forceinline__ unsigned pair_src_offset(long ld, int wave, int lane) {
  const int r = 8 * wave + (lane >> 3);
  const int c = (lane & 7) ^ ((r >> 1) & 7);
  return (unsigned)(r * ld + 8 * c) * 2u;
}
// 32 rows x 16 k fragment out of a pair area: lane l holds row (l % 32), chunk c0 + l / 32 of the row's eight
__device__ __forceinline__ bf16x8 frag_pair(const unsigned char* area, int row0, int c0, int lane) {
  const int r = row0 + (lane & 31);
  const int c = c0 + (lane >> 5);
  const uint4 v = *reinterpret_cast<const uint4*>(area + r * 128 + ((c ^ ((r >> 1) & 7)) << 4));
  return __builtin_bit_cast(bf16x8, v);
}

constexpr int LEAN_NST = 4;                              // 4 x 32 KB, + 4 KB per wave for the epilogue
constexpr int LEAN_LDS = LEAN_NST * STAGE_BYTES + NW * 4096;

// PAIR (A contiguous along K, every tile's range an even number of slices): A is copied two slices at a time, 128
// bytes of every row, so that each request for A takes a whole 128-byte line out of L2 (a 64-byte row segment costs
// L2 a whole line as well, and the other half is asked for again one slice later: half as much again in L2 reads
// for the pairing with one K-contiguous operand, which is bound by them).  LDS then holds two areas of 256 rows x
// 128 bytes for A (chunk k of row r at chunk k ^ (r/2 % 8)), refilled at every even step with the pair two steps
// ahead, and the ring of four 16 KB stages for B behind them; everything else is as without it.
template <bool A_KC, bool B_KC, int FAST, bool ONE_AT_A_TIME, bool PAIR>
__global__ __launch_bounds__(NTHR, 1) void gemm_mfma_lean_kernel(GemmArgs g, Walk walk) {
  static_assert(!PAIR || A_KC, "pairs of slices are copied for a K-contiguous A only");
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int grp = wave >> 2;
  const int wm0 = grp * 128, wn0 = (wave & 3) * 64;
  const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;
  const unsigned lds_wave = lds0 + (unsigned)wave * 1024u;

  const int xcd = blockIdx.x & 7;
  // Plain walk: every XCD takes a contiguous eighth of the tile list (small matrices: an XCD's L2 keeps a
  // matrix's panels to itself).  ONE_AT_A_TIME: blocks of (workgroups per XCD) consecutive tiles are dealt to the
  // XCDs in turn, so that at any time the whole chip works on neighbouring blocks of ONE matrix of the batch:
  // with operands too large for the caches, what the eight L2s miss is then the same panels at the same time
  // (one trip to memory instead of eight, the rest served by the memory-side cache).
  const int wpx = gridDim.x >> 3;
  const int t_stride = ONE_AT_A_TIME ? (int)gridDim.x : wpx;
  int t = (ONE_AT_A_TIME ? xcd * wpx : xcd * walk.per_xcd) + (int)(blockIdx.x >> 3);
  const int t_end = !ONE_AT_A_TIME && (xcd + 1) * walk.per_xcd < walk.total ? (xcd + 1) * walk.per_xcd : walk.total;
  if (t >= t_end) return;
  // Shares of unequal length are met by the parameter gradients alone (the only split launches); elsewhere a launch's one
  // length stays in a scalar register.
  constexpr bool SHARES = !A_KC;
  auto slices_of = [&](const TileCoord& c) { return SHARES ? c.kt : walk.KT; };

  const long lda = A_KC ? g.a_sm : g.a_sk;
  const long ldb = B_KC ? g.b_sn : g.b_sk;
  const long step_a = (A_KC ? BK : BK * lda) * 2, step_b = (B_KC ? BK : BK * ldb) * 2;   // bytes per slice
  // per-lane byte offsets of the wave's two copies per operand (the second is 128 rows / 16 k rows further)
  // (PAIR: copy i of 4 covers rows 64 i + 8 wave .. + 7, 8 lanes to a row; its offset is added to the scalar base)
  const unsigned offA0 = PAIR ? pair_src_offset(lda, wave, lane) : lane_src_offset<A_KC>(lda, 0, wave, lane);
  const unsigned offB0 = lane_src_offset<B_KC>(ldb, 0, wave, lane);
  const unsigned offA1 = offA0 + (unsigned)((A_KC ? 128 : 16) * lda * 2);
  const unsigned offB1 = offB0 + (unsigned)((B_KC ? 128 : 16) * ldb * 2);
  const long pair_rows64 = 64 * lda * 2;                  // bytes between the rows of consecutive copies of a pair

  // ---- producer (wave-uniform): first byte of the next slice to copy per operand, slices left in
  // the tile it copies from, that tile's index, the stage the slice goes to ----
  const unsigned char* qa;
  const unsigned char* qb;
  int p_left, pt = t;
  bool p_more = true;
  unsigned p_off = 0;      // byte offset of the producer's stage in the ring (PAIR: of its B stage behind the A areas)
  unsigned p_aoff = 0;     // PAIR: byte offset of the A area the next pair goes to
  auto aim = [&](const TileCoord& c) {
    qa = reinterpret_cast<const unsigned char*>(reinterpret_cast<const bf16_t*>(g.A) + c.batch * g.a_sb +
                                                (A_KC ? c.m0 * lda + c.k_begin : c.m0 + c.k_begin * lda));
    qb = reinterpret_cast<const unsigned char*>(reinterpret_cast<const bf16_t*>(g.B) + c.batch * g.b_sb +
                                                (B_KC ? c.n0 * ldb + c.k_begin : c.n0 + c.k_begin * ldb));
    p_left = slices_of(c);
  };
  auto copy_slice = [&]() {
    if (PAIR) {
      // an odd slice of its tile (an odd number of slices left): first the pair of A it completes, then its B
      if (p_left & 1) {
        const unsigned dsta = lds_wave + p_aoff;
        dma16_c<0>(offA0, qa, dsta);
        dma16_c<NW * 1024>(offA0, qa + pair_rows64, dsta);
        dma16_c<2 * NW * 1024>(offA0, qa + 2 * pair_rows64, dsta);
        dma16_c<3 * NW * 1024>(offA0, qa + 3 * pair_rows64, dsta);
        qa += 2 * step_a;
        p_aoff ^= (unsigned)PAIR_AREA;
      }
      const unsigned dst = lds_wave + 2 * PAIR_AREA + p_off;
      dma16_c<0>(offB0, qb, dst);
      dma16_c<NW * 1024>(offB1, qb, dst);
      qb += step_b;
      p_off = p_off == (LEAN_NST - 1) * B_BYTES ? 0u : p_off + B_BYTES;
    } else {
      const unsigned dst = lds_wave + p_off;
      dma16_c<0>(offA0, qa, dst);
      dma16_c<NW * 1024>(offA1, qa, dst);
      dma16_c<A_BYTES>(offB0, qb, dst);
      dma16_c<A_BYTES + NW * 1024>(offB1, qb, dst);
      qa += step_a;
      qb += step_b;
      p_off = p_off == (LEAN_NST - 1) * STAGE_BYTES ? 0u : p_off + STAGE_BYTES;
    }
    if (--p_left == 0) {
      pt += t_stride;
      if (pt < t_end) aim(decode_tile(walk, pt));
      else p_more = false;
    }
  };

  float16v acc[4][2];
  bf16x8 fa[4][2], fb[2][2];
  Quad16 aux0 = {}, aux1 = {};   // the first half of a tile's fused operand
  TileCoord cc = decode_tile(walk, t);   // the consumer's tile
  unsigned c_off = 0;      // byte offset of the consumer's stage
  int epi_recent = 0;      // waits that still see the last epilogue's operations
  constexpr int E = StagedOps<FAST>::value;
  constexpr int AHEAD = LEAN_NST - 1;                      // slices copied ahead of the one being multiplied
  constexpr int W_PLAIN = (AHEAD - 1) * PER_SLICE;
  constexpr int W_EPI = W_PLAIN + E > 63 ? 63 : W_PLAIN + E;
  // EARLY: half of the fused operand is asked for before the tile's end, and the groups' epilogues run together (below).
  // Not on the one-at-a-time walk, where the stream of copies is the limit: a backward pass over 96 blocks of 16384 x 8192
  // x 2048 took 316 ms with it and with its second test of epi_recent in every slice, 311 without (before either: 311).
  constexpr bool EARLY = has_aux<FAST>() && !ONE_AT_A_TIME;
  // the slice that the second step of a tile waits for was copied after the 8 early loads of the epilogue before
  constexpr int E2 = EARLY ? E - 8 : E, W_EPI2 = W_PLAIN + E2 > 63 ? 63 : W_PLAIN + E2;
  // PAIR: a wave issues 4 copies of A and 2 of B in an even step, 2 of B in an odd one.  At the end of an even
  // step c the B of slice c + 1 (issued two steps before) must have landed: what may be outstanding is what was
  // issued after it, 2 + 4 + 2 copies (and a recent epilogue's operations); at the end of an odd step the pair
  // that holds slice c + 1, issued in the step before: 2 + 2 copies.
  constexpr int W_EVEN = 8, W_EVEN_EPI = W_EVEN + E > 63 ? 63 : W_EVEN + E, W_ODD = 4;
  unsigned c_aoff = 0;     // PAIR: byte offset of the A area being read

  // One slice: load phase, barrier, compute phase, barrier.
  // Barrier intervals ("ticks"): group 0 loads slice c in tick 2c and multiplies it in tick 2c+1;
  // group 1 does the same one tick later.  Slice c+3 is issued in the load phase of slice c into
  // the stage of slice c-1, which its last reader (group 1, tick 2c-1) has left.  Every wave waits
  // for its own share of slice c+1 at the end of its load phase of slice c, a barrier or more
  // before the first reader of slice c+1 starts.
  // AUX 1: the tile's last slice but one, where the first half of the epilogue's fused operand is asked for (8 loads after
  // the step's copies); AUX 2: the last slice: both steps' waits may leave those loads outstanding.
  // last: a tile's last slice.  With a long epilogue (a fused operand, GELU) group 1 leaves out the barrier after it and
  // meets it after its epilogue instead: the two groups' epilogues, chains of LDS and memory latencies, then run in
  // the same tick, not one after the other.  Measured: 16384 x 4096 x 1024 with GELU 183 -> 174 us, 32768 x 1024 x 256 47 -> 41,
  // 12 x 32768 x 1024 x 256 with act' 329 -> 325; plain stores 1 % slower, so not there.
  constexpr bool TOGETHER = EARLY || FAST == FAST_ACT_GELU;
  auto step = [&](auto first_c, auto odd_c, auto aux_c, bool last) {
    constexpr bool FIRST = decltype(first_c)::value;
    constexpr int AUX = decltype(aux_c)::value, X = AUX ? 8 : 0;
    constexpr bool ODD = decltype(odd_c)::value;         // (PAIR only: the slice's place in its pair)
    const bool copying = p_more;
    if (copying) copy_slice();
    if (AUX == 1) { fetch_aux(aux0, g, cc, wm0, wn0, lane, 0); fetch_aux(aux1, g, cc, wm0, wn0, lane, 1); }
    if (PAIR) {
      const unsigned char* stb = smem + 2 * PAIR_AREA + c_off;
      const unsigned char* sta = smem + c_aoff;
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int j = 0; j < 2; ++j) fb[j][h] = frag<B_KC>(stb, wn0 + 32 * j, 16 * h, lane);
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int i = 0; i < 4; ++i) fa[i][h] = frag_pair(sta, wm0 + 32 * i, (ODD ? 4 : 0) + 2 * h, lane);
      c_off = c_off == (LEAN_NST - 1) * B_BYTES ? 0u : c_off + B_BYTES;
      if (ODD) c_aoff ^= (unsigned)PAIR_AREA;
      if (!copying) wait_vm_lds<X>();
      else if (ODD) wait_vm_lds<W_ODD + X>();
      else if (epi_recent > 0) { wait_vm_lds<W_EVEN_EPI>(); epi_recent = 0; }
      else wait_vm_lds<W_EVEN + X>();
    } else {
      const unsigned char* st = smem + c_off;
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int j = 0; j < 2; ++j) fb[j][h] = frag<B_KC>(st + A_BYTES, wn0 + 32 * j, 16 * h, lane);
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int i = 0; i < 4; ++i) fa[i][h] = frag<A_KC>(st, wm0 + 32 * i, 16 * h, lane);
      c_off = c_off == (LEAN_NST - 1) * STAGE_BYTES ? 0u : c_off + STAGE_BYTES;
      // this wave's share of the next slice has landed once only what it issued for the slices after
      // that one (and a recent epilogue's operations, which lie among them) is outstanding
      if (!copying) wait_vm_lds<X>();
      else if (EARLY && epi_recent > 1) { wait_vm_lds<W_EPI>(); --epi_recent; }
      else if (epi_recent > 0) { wait_vm_lds<W_EPI2>(); --epi_recent; }
      else wait_vm_lds<W_PLAIN + X>();
    }
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(1);
    const float16v zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[j][0], fa[i][0], FIRST ? zero : acc[i][j], 0, 0, 0);
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[j][1], fa[i][1], acc[i][j], 0, 0, 0);
    __builtin_amdgcn_s_setprio(0);
    __builtin_amdgcn_sched_barrier(0);
    if (!TOGETHER || !last || grp == 0) __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
  };

  aim(cc);
  int pro = 0;             // slices copied before the first step
#pragma unroll 1
  for (; pro < AHEAD && p_more; ++pro) copy_slice();
  // slice 0 has landed once at most the pro - 1 slices after it are outstanding
  if (PAIR) {              // (issued: B of slice 0, the first pair of A, B of slices 1 and 2)
    if (pro == 3) wait_vm<4>(); else wait_vm<0>();
  } else if (pro == 3) wait_vm<2 * PER_SLICE>();
  else if (pro == 2) wait_vm<PER_SLICE>(); else wait_vm<0>();
  __builtin_amdgcn_s_barrier();                 // slice 0 is in LDS
  if (grp == 1) __builtin_amdgcn_s_barrier();   // group 1 runs one tick behind

  constexpr std::integral_constant<bool, false> no{};
  constexpr std::integral_constant<bool, true> yes{};
  constexpr std::integral_constant<int, 0> a0{};
  constexpr std::integral_constant<int, EARLY ? 1 : 0> a1{};
  constexpr std::integral_constant<int, EARLY ? 2 : 0> a2{};
  while (true) {
    const int KT = slices_of(cc);
    if (!EARLY) {
      step(yes, no, a0, !PAIR && KT == 1);
      if (PAIR) step(no, yes, a0, KT == 2);
#pragma unroll 1
      for (int k = PAIR ? 2 : 1; k < KT; k += PAIR ? 2 : 1) {
        step(no, no, a0, !PAIR && k + 1 == KT);
        if (PAIR) step(no, yes, a0, k + 2 == KT);
      }
    } else {                 // (at least four slices: the launcher sees to it)
      step(yes, no, a0, false);
      if (PAIR) step(no, yes, a0, false);
#pragma unroll 1
      for (int k = PAIR ? 4 : 3; k < KT; k += PAIR ? 2 : 1) {
        step(no, no, a0, false);
        if (PAIR) step(no, yes, a0, false);
      }
      step(no, no, a1, false);
      if (PAIR) step(no, yes, a2, true); else step(no, no, a2, true);
    }
    if (has_aux<FAST>() && !EARLY) { fetch_aux(aux0, g, cc, wm0, wn0, lane, 0); fetch_aux(aux1, g, cc, wm0, wn0, lane, 1); }
    if (FAST == FAST_STORE_F32) epilogue_f32(g, cc, acc, wm0, wn0, lane);
    else epilogue_staged_fn<FAST>(g, cc, acc, wm0, wn0, lane, smem + LEAN_NST * STAGE_BYTES + wave * 4096, aux0, aux1);
    if (TOGETHER && grp == 1) {
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_sched_barrier(0);
    }
    epi_recent = AHEAD - 1;
    t += t_stride;
    if (t >= t_end) break;
    cc = decode_tile(walk, t);
  }
  if (grp == 0) __builtin_amdgcn_s_barrier();   // matches group 1's last barrier
}

template <bool A_KC, bool B_KC, int FAST, bool ONE_AT_A_TIME, bool PAIR>
hipError_t launch_lean_walk(const GemmArgs& g, hipStream_t s) {
  static std::atomic<bool> attr_set[MAX_DEVICES];
  auto kern = gemm_mfma_lean_kernel<A_KC, B_KC, FAST, ONE_AT_A_TIME, PAIR>;
  {
    hipError_t e = raise_lds_limit(reinterpret_cast<const void*>(kern), LEAN_LDS, attr_set);
    if (e != hipSuccess) return e;
  }
  const Walk walk = make_walk(g);
  const int wg_per_xcd = walk.per_xcd < 32 ? walk.per_xcd : 32;
  hipLaunchKernelGGL(kern, dim3((unsigned)(wg_per_xcd * 8)), dim3(NTHR), LEAN_LDS, s, g, walk);
  return hipGetLastError();
}
template <bool A_KC, bool B_KC, int FAST>
hipError_t launch_lean(const GemmArgs& g, hipStream_t s) {
  // a batch of matrices whose operands run to tens of megabytes each: the chip takes them one at a time (measured
  // on 96 blocks of 16384 x 8192 x 2048: 8-10 % faster; on 32 blocks of 8192 x 2048 x 512: 10 % slower)
  const bool one_at_a_time = g.batch > 1 && (g.M + g.N) * g.K * 2 >= (64L << 20);
  if constexpr (A_KC) {
    // Every tile's share of K an even number of slices: A in pairs of slices.  Measured: 2-10 % on matrices that
    // the caches hold (L2 reads down by a third); on the one-at-a-time walk over 96 blocks of 16384 x 8192 x 2048
    // the same time (fewer cycles at a lower clock: the chip is at its power limit there) with twice the fills from
    // memory, the pairs being asked for closer to their use: not taken there.
    if (!one_at_a_time && g.K % ((long)g.split_k * 2 * BK) == 0)
      return launch_lean_walk<A_KC, B_KC, FAST, false, true>(g, s);
  }
  return one_at_a_time ? launch_lean_walk<A_KC, B_KC, FAST, true, false>(g, s)
                       : launch_lean_walk<A_KC, B_KC, FAST, false, false>(g, s);
}
// 128 x 128 tiles once they give most compute units one, else 64 x 64.  Measured, 128 / 64: 24 tiles of 128 (1000 x 328 x
// 1304) 18.9 / 10.1 us, 128 tiles (2048 x 1024 x 4096) 42.3 / 28.0, 192 tiles (4096 x 768 x 3072) 36.4 / 37.2, 288 tiles
// (1000 x 328 x 1304, batch 12) 27.1 / 33.4, 768 tiles (3000 x 1000 x 4000, batch 4) 122 / 222.
// The smallest launches: the smaller tiles, whose wavefronts share the contraction, as long as every compute unit has at most
// one.  Measured, 64 x 64 / 64 x 32 / 32 x 32: 1000 x 328 x 1304 (176 tiles of 64 x 32, 352 of 32 x 32) 10.2 / 8.2 / 10.6 us,
// 512 x 768 x 3072 (192, 384) 15.9 / 11.9 / 16.0, 1024 x 256 x 1200 (128, 256) 8.3 / 7.9 / 6.6, 100 x 512 x 2048 (32, 64)
// 12.5 / 7.6 / 6.3; not for a handful of rows and columns over one slice, which has nothing to share out (exact backpropagation of 6
// blocks of 8 x 64 x 64 44.3 / - / 48.8 us, of 30 rows 47.6 / - / 49.9; their forward 37.3 / - / 39.9 and 43.6 / - / 40.3, of 3 x 16 x
// 256 47.5 / - / 41.0); beyond: 600 x 1000 x 4000 (320, 608) 21.9 / 26.8 / 25.7, 1200 x 768 x 256 (456, 912) 4.7 / 6.8 / 10.1.
inline hipError_t launch_tile_for(const GemmArgs& g, hipStream_t s) {
  auto tiles = [&g](long tm, long tn) { return (g.M + tm - 1) / tm * ((g.N + tn - 1) / tn) * g.batch * g.split_k; };
  if (tiles(128, 128) >= 192) return launch_gemm_tile(g, 128, 128, s);
  if (g.M <= 16 && g.N <= 64 && g.K <= 64) return launch_gemm_tile(g, 64, 64, s);
  if (tiles(32, 32) <= 256) return launch_gemm_tile(g, 32, 32, s);
  return tiles(64, 32) <= 256 ? launch_gemm_tile(g, 64, 32, s) : launch_gemm_tile(g, 64, 64, s);
}

// does the lean kernel have this pairing's epilogue?
inline bool has_lean(const GemmArgs& g, bool a_kc, bool b_kc) {
  if (!a_kc) return g.mode == EPI_STORE && !g.addf && (g.c_is_f32 || g.split_k > 1);     // parameter gradients
  if (g.addf || g.split_k > 1) return false;
  if (g.c_is_f32) return b_kc && g.mode == EPI_STORE;                                    // the recurrent kinds' U xin
  if (g.mode == EPI_STORE) return true;
  if (!b_kc) return g.mode == EPI_MUL_AUX || g.mode == EPI_MUL_1MZ2 || g.mode == EPI_ADD_AUX;   // block VJPs
  if (g.mode == EPI_ACT_GELU) return g.out2;                                             // forward
  return g.mode == EPI_RESID && g.aux && !g.lambda_mn;
}
hipError_t launch_lean_nn(const GemmArgs& g, hipStream_t s) {
  switch (g.mode) {
    case EPI_STORE: return launch_lean<true, false, FAST_STORE>(g, s);
    case EPI_MUL_AUX: return launch_lean<true, false, FAST_MUL_AUX>(g, s);
    case EPI_MUL_1MZ2: return launch_lean<true, false, FAST_MUL_1MZ2>(g, s);
    case EPI_ADD_AUX: return launch_lean<true, false, FAST_ADD_AUX>(g, s);
    default: return hipErrorInvalidValue;
  }
}
hipError_t launch_lean_nt(const GemmArgs& g, hipStream_t s) {
  if (g.c_is_f32) return launch_lean<true, true, FAST_STORE_F32>(g, s);
  switch (g.mode) {
    case EPI_STORE: return launch_lean<true, true, FAST_STORE>(g, s);
    case EPI_ACT_GELU: return launch_lean<true, true, FAST_ACT_GELU>(g, s);
    case EPI_RESID: return launch_lean<true, true, FAST_RESID>(g, s);
    default: return hipErrorInvalidValue;
  }
}
hipError_t launch_lean_for(const GemmArgs& g, bool a_kc, bool b_kc, hipStream_t s) {
  if (!a_kc) return launch_lean<false, false, FAST_STORE_F32>(g, s);
  return b_kc ? launch_lean_nt(g, s) : launch_lean_nn(g, s);
}

// rows m0 .. m1 and columns n0 .. n1 of a product
GemmArgs part_of(const GemmArgs& g, long m0, long m1, long n0, long n1) {
  GemmArgs p = g;
  p.M = m1 - m0;
  p.N = n1 - n0;
  p.A = reinterpret_cast<const bf16_t*>(g.A) + m0 * g.a_sm;
  p.B = reinterpret_cast<const bf16_t*>(g.B) + n0 * g.b_sn;
  const long o = m0 * g.ldc + n0;
  if (g.c_is_f32 || g.split_k > 1) p.C = reinterpret_cast<float*>(g.C) + o;
  else p.C = reinterpret_cast<bf16_t*>(g.C) + o;
  if (g.aux) p.aux = reinterpret_cast<const bf16_t*>(g.aux) + o;
  if (g.out2) p.out2 = reinterpret_cast<bf16_t*>(g.out2) + o;
  if (g.addf) p.addf = g.addf + o;
  if (g.lambda) p.lambda = g.lambda + n0;
  if (g.lambda_mn) p.lambda_mn = reinterpret_cast<const bf16_t*>(g.lambda_mn) + o;
  return p;
}

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

}  // namespace

namespace {
// the layouts, sizes and alignments that the bf16 kernels take
bool covered(const GemmArgs& g) {
  const bool a_kc = g.a_sk == 1, a_rc = g.a_sm == 1;
  const bool b_kc = g.b_sk == 1, b_rc = g.b_sn == 1;
  if (!(a_kc || a_rc) || !(b_kc || b_rc)) return false;
  const long lda = a_kc ? g.a_sm : g.a_sk, ldb = b_kc ? g.b_sn : g.b_sk;
  // 16-byte accesses everywhere: contiguous extents, leading dimensions and batch strides in multiples of 8
  if ((a_kc ? g.K : g.M) % 8 || (b_kc ? g.K : g.N) % 8 || g.N % 8) return false;
  if (lda % 8 || ldb % 8 || g.ldc % 8 || g.a_sb % 8 || g.b_sb % 8 || g.c_sb % 8) return false;
  if (g.aux_sb % 8 || g.out2_sb % 8 || g.addf_sb % 8 || g.lambda_sb % 8) return false;
  if (!aligned16(g.A) || !aligned16(g.B) || !aligned16(g.C) || !aligned16(g.aux) || !aligned16(g.out2) ||
      !aligned16(g.addf) || !aligned16(g.lambda) || !aligned16(g.lambda_mn))
    return false;
  if (lda > (1L << 22) || ldb > (1L << 22)) return false;   // per-lane source offsets are 32-bit
  if (g.split_k > 1 && g.mode != EPI_STORE) return false;
  if (g.M <= 0 || g.N <= 0 || g.K <= 0 || g.batch <= 0 || g.split_k <= 0) return false;
  const bool act = g.mode == EPI_ACT_GELU || g.mode == EPI_ACT_TANH;
  return (a_kc && (b_kc || (b_rc && !act))) || (a_rc && b_rc && !act);
}
// whether the 256 x 256 kernel takes the launch: whole, or (sizes that are no multiple of its tile) the whole tiles of it
enum Lean { LEAN_NOT, LEAN_WHOLE, LEAN_PART };
Lean lean_share(const GemmArgs& g) {
  const bool a_kc = g.a_sk == 1, b_kc = g.b_sk == 1;
  // (a fused operand is asked for two slices before a tile's end, the first two being waited for otherwise: four at least)
  if (!has_lean(g, a_kc, b_kc) || g.K % BK != 0 || g.K / BK < g.split_k || (g.mode != EPI_STORE && g.K < 4 * BK)) return LEAN_NOT;
  const long hm = g.M / BM * BM, hn = g.N / BN * BN;
  const long tiles = (hm / BM) * (hn / BN) * g.batch * g.split_k;
  if (hm == g.M && hn == g.N) return gemm_fills_chip(tiles) ? LEAN_WHOLE : LEAN_NOT;
  return tiles >= GEMM_SPLIT_FROM ? LEAN_PART : LEAN_NOT;
}
}  // namespace

bool launch_gemm_mfma(const GemmArgs& g, hipStream_t s, hipError_t* err) {
  *err = hipSuccess;
  if (!covered(g)) return false;
  const bool a_kc = g.a_sk == 1, b_kc = g.b_sk == 1;
  const Lean lean = lean_share(g);
  if (lean == LEAN_WHOLE) {
    *err = launch_lean_for(g, a_kc, b_kc, s);
  } else if (lean == LEAN_PART) {
    // the whole tiles, then the remaining columns of all rows, then the remaining rows (disjoint blocks of C)
    const long hm = g.M / BM * BM, hn = g.N / BN * BN;
    *err = launch_lean_for(part_of(g, 0, hm, 0, hn), a_kc, b_kc, s);
    if (*err == hipSuccess && hn < g.N) *err = launch_tile_for(part_of(g, 0, g.M, hn, g.N), s);
    if (*err == hipSuccess && hm < g.M) *err = launch_tile_for(part_of(g, hm, g.M, 0, hn), s);
  } else {
    *err = launch_tile_for(g, s);
  }
  return true;
}

namespace {
long tiles_of(const GemmArgs& g, long tm, long tn) { return (g.M + tm - 1) / tm * ((g.N + tn - 1) / tn) * g.batch * g.split_k; }
}  // namespace
// The tiles as for one product with all of their tiles (launch_tile_for).  Not where a product is long enough for itself: parameter
// gradients in tiles of 128 go together if that takes fewer rounds of the 512 that run at a time, or is short, up to 2048 tiles (two
// products) or 4096 (a transformer's four).  Measured, passes of one or two iterations, us, apart / together: two products, 8 blocks of 1000
// x 360 x 1440 (288 + 288 tiles) 156.7 / 163.4, 24 of 1000 x 200 x 800 (336 each) 126.6 / 131.4, 20 of 100 x 328 x 1304 (660) 74.0 / 68.2, 12 of
// 200 x 520 x 2080 (1020, short) 107.7 / 103.9, 8 of 141 x 1152 x 4608 (2592) 152 / 159; four, 6 layers of 2736 x 512 (1152 in all) 847 / 753
// with the VJPs', 3 of 1740 x 1024 (2304) 974 / 885.
// Block VJPs in tiles of 128 go together but where contractions are long and a compute unit has as many tiles either way (256 at a time,
// a remainder counting as 256): then two or three share one longer.  From contractions of 1536 on that is so past 512 tiles, from 4096 on at
// any number; a wide and a narrow product (the first contractions) fill each other's last round at any length.  Measured,
// gradients of k = 2, us, second contractions apart / together (the first iteration's tiles, the second's): 2 layers of 8900 x 256 (contractions
// of 1024 and 768; 280 + 280, 140 + 280) 387 / 366, of 15300 x 256 (480 + 480, 240 + 480) 586 / 580; of 2400 x 512 (2048 and 1536; 152 + 152, 76 +
// 152) 251 / 229, of 4400 x 512 (280 + 280, 140 + 280) 443 / 421, of 7168 x 512 (448 + 448, 224 + 448) 597 / 625; of 2200 x 1024 (2048 and 3072; 288
// + 288, 144 + 288) 532 / 515, of 3000 x 1024 (384 + 384, 192 + 384) 622 / 640, 4 of 1500 (384 + 384, 288 + 384) 692 / 685; 4096 and more: 4 of 256 x
// 1536 (96 + 96) 657 / 603, 2 of 500 x 2048 (128 + 128) 744 / 698, 4 of 500 x 1536 (192 + 192) 851 / 893, 4 of 384 x 2048 (192 + 192) 1051 / 1103,
// 2 of 1500 x 1536 (288 + 288) 954 / 949.  First ones alone: 2 of 3000 x 768 (1152 + 288) 516 / 488, of 4000 x 1024 (2048 + 512) 1100 / 1062.
bool gemm_mfma_group_ok(const GemmArgs* g, int n) {
  if (n < 2 || n > GEMM_GROUP) return false;
  long t128 = 0, rounds = 0, per_cu = 0, longest = 0;
  bool wide = false;                       // one wide, one narrow
  for (int i = 0; i < n; ++i) {
    if (!covered(g[i]) || lean_share(g[i]) != LEAN_NOT || g[i].b_sn != 1 || (g[i].a_sk == 1) != (g[0].a_sk == 1)) return false;
    if (g[i].b_sk == 1 || (g[i].a_sk == 1 && g[i].a_sm == 1)) return false;       // (a single column: either layout)
    const long t = tiles_of(g[i], 128, 128);
    t128 += t;
    rounds += (t + 511) / 512;
    per_cu += (t + 255) / 256;
    longest = g[i].K > longest ? g[i].K : longest;
    wide = wide || g[i].N != g[0].N;
  }
  if (g[0].a_sk == 1)
    return t128 <= (1L << 24) &&
           (longest < 1536 || wide || (longest < 4096 && t128 <= 512) || (t128 + 255) / 256 < per_cu);
  return t128 < 192 || (t128 <= (n == 2 ? 2048 : 4096) && ((t128 + 511) / 512 < rounds || longest <= 256));
}
hipError_t launch_gemm_mfma_group(const GemmArgs* g, int n, hipStream_t s) {
  long t128 = 0, t3232 = 0, t6432 = 0;
  for (int i = 0; i < n; ++i) { t128 += tiles_of(g[i], 128, 128); t3232 += tiles_of(g[i], 32, 32); t6432 += tiles_of(g[i], 64, 32); }
  return t128 >= 192     ? launch_gemm_tile_group(g, n, 128, 128, s)
         : t3232 <= 256  ? launch_gemm_tile_group(g, n, 32, 32, s)
         : t6432 <= 256  ? launch_gemm_tile_group(g, n, 64, 32, s)
                         : launch_gemm_tile_group(g, n, 64, 64, s);
}

}  // namespace hbp
