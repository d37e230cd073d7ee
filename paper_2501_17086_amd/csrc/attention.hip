// Multi-head self-attention between the two matrices of an attention sub-block (appendix, GPT-2 paragraph: every
// transformer layer is split into its self-attention and feed-forward sub-layers): forward o = softmax(q k^T / sqrt(dh)) v
// and its vector-Jacobian product  dv = P^T do,  dP = do v^T,  dS = P (.) (dP - rowsum(do (.) o)),  dq = dS k / sqrt(dh),
// dk = dS^T q / sqrt(dh).  P is never stored: the forward keeps one number per (head, query), the base-2 logarithm of
// the row's sum of exp2(s log2 e), and the backward kernels rebuild P tile by tile from q and k.
//
// bf16 storage with heads of up to 128 columns runs on the matrix cores (v_mfma_f32_32x32x16_bf16; the width is padded
// to 32, 64 or 128).  A workgroup of four wavefronts owns four tiles of 32 queries (forward, dq) or 32 keys (dk, dv), one per
// wavefront, and streams the other side's tiles through a ring of LDS buffers that all four read; or, where there are few
// problems, it owns one tile, and each wavefront streams every fourth tile of the other side through a ring of its own:
//   - the MFMA is issued so that a lane owns one query (dk/dv kernel: one key) and its 16 accumulator registers run
//     over 16 of the streamed tile's 32 keys (queries): row statistics, the running rescale of the output and the
//     factor dP - D are per-lane scalars (D and the row statistic enter as the accumulators' start values);
//   - the scores of a lane, rounded to bf16 (64-wide heads) or cut into three bf16 parts that hold all of them (every other
//     width, which plain kernels with fp32 scores served before), are fed back as the second product's operand straight from the
//     registers: the contraction index of an MFMA is a dummy, so it is enough that the other operand is fetched
//     in the same (permuted) order of keys, which the transposing LDS read ds_read_b64_tr_b16 does from the tile;
//   - tiles reach LDS by direct copies (global_load_lds_dwordx4, no staging registers) issued steps ahead; the loop holds no
//     other global load, so a counted s_waitcnt tells a wavefront that its copies of the next pair of tiles have landed.  Of
//     a shared ring each wavefront copies a quarter of every pair, three steps ahead, and one barrier per step completes the
//     hand-over.  A wavefront with a ring of its own copies whole pairs, one or two steps ahead, and meets no barrier in the
//     loop; the four wavefronts' sums (forward: and the rows' maxima and sums) meet in LDS at the end;
//   - dq on one side and dk, dv on the other are two kernels that each rebuild S: seven products instead of five,
//     no atomics, results bitwise repeatable.
// Everything else (fp32 storage, wider heads) takes plain one-wavefront-per-query (per-key) kernels.
#include "hbp_common.h"

#include <cfloat>
#include <type_traits>

namespace hbp {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short short4v __attribute__((ext_vector_type(4)));
typedef short short8v __attribute__((ext_vector_type(8)));
typedef float float16v __attribute__((ext_vector_type(16)));

constexpr float LOG2E = 1.4426950408889634f;

__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// ------------------------------------------------------------------------------------------------------------
// plain kernels: one wavefront per query (forward, dq) or per key (dk, dv); any storage type, any head width
// ------------------------------------------------------------------------------------------------------------
template <typename T>
__device__ __forceinline__ float dot_rows(const T* a, const T* b, int n) {
  float s = 0.f;
  for (int c = 0; c < n; ++c) s = fmaf(Elem<T>::load(a + c), Elem<T>::load(b + c), s);
  return s;
}

template <typename T>
__global__ __launch_bounds__(64) void attn_fwd_plain_kernel(AttnArgs a) {
  extern __shared__ float sh[];                  // T floats: the query's scores, then probabilities
  const int lane = threadIdx.x;
  const long p = blockIdx.x;                     // (sequence, head)
  const int i = blockIdx.y;
  const int h = (int)(p % a.heads);
  const long seq = p / a.heads;
  const long d = (long)a.heads * a.dh, ld = 3 * d;
  const T* base = reinterpret_cast<const T*>(a.qkv) + seq * a.T * ld + (long)h * a.dh;
  const T* q = base + (long)i * ld;
  const int jn = a.causal ? i + 1 : (int)a.T;
  const float c = a.scale * LOG2E;
  float m = -INFINITY;
  for (int j = lane; j < jn; j += 64) {
    const float s = c * dot_rows(q, base + (long)j * ld + d, a.dh);
    sh[j] = s;
    m = fmaxf(m, s);
  }
  m = wave_max(m);
  float sum = 0.f;
  for (int j = lane; j < jn; j += 64) {
    const float pr = exp2f(sh[j] - m);
    sh[j] = pr;
    sum += pr;
  }
  sum = wave_sum(sum);
  __syncthreads();
  T* o = reinterpret_cast<T*>(a.o) + (seq * a.T + i) * d + (long)h * a.dh;
  for (int cc = lane; cc < a.dh; cc += 64) {
    float acc = 0.f;
    for (int j = 0; j < jn; ++j) acc = fmaf(sh[j], Elem<T>::load(base + (long)j * ld + 2 * d + cc), acc);
    Elem<T>::store(o + cc, acc / sum);
  }
  if (lane == 0) a.lse[p * a.T + i] = m + log2f(sum);
}

// dq of one query; also leaves D = sum_c do[c] o[c] for the dk/dv kernel
template <typename T>
__global__ __launch_bounds__(64) void attn_bwd_q_plain_kernel(AttnArgs a) {
  extern __shared__ float sh[];                  // T floats: dS of this query
  const int lane = threadIdx.x;
  const long p = blockIdx.x;
  const int i = blockIdx.y;
  const int h = (int)(p % a.heads);
  const long seq = p / a.heads;
  const long d = (long)a.heads * a.dh, ld = 3 * d;
  const T* base = reinterpret_cast<const T*>(a.qkv) + seq * a.T * ld + (long)h * a.dh;
  const T* q = base + (long)i * ld;
  const T* dout = reinterpret_cast<const T*>(a.dout) + (seq * a.T + i) * d + (long)h * a.dh;
  const T* o = reinterpret_cast<const T*>(a.o) + (seq * a.T + i) * d + (long)h * a.dh;
  float dpart = 0.f;
  for (int cc = lane; cc < a.dh; cc += 64) dpart = fmaf(Elem<T>::load(dout + cc), Elem<T>::load(o + cc), dpart);
  const float D = wave_sum(dpart);
  const float L2 = a.lse[p * a.T + i];
  const int jn = a.causal ? i + 1 : (int)a.T;
  const float c = a.scale * LOG2E;
  for (int j = lane; j < jn; j += 64) {
    const T* k = base + (long)j * ld + d;
    const float pr = exp2f(c * dot_rows(q, k, a.dh) - L2);
    const float dp = dot_rows(dout, k + d, a.dh);
    sh[j] = pr * (dp - D);
  }
  __syncthreads();
  T* dq = reinterpret_cast<T*>(a.dqkv) + (seq * a.T + i) * ld + (long)h * a.dh;
  for (int cc = lane; cc < a.dh; cc += 64) {
    float acc = 0.f;
    for (int j = 0; j < jn; ++j) acc = fmaf(sh[j], Elem<T>::load(base + (long)j * ld + d + cc), acc);
    Elem<T>::store(dq + cc, acc * a.scale);
  }
  if (lane == 0) a.dsum[p * a.T + i] = D;
}

// dk, dv of one key (after the dq kernel: reads D)
template <typename T>
__global__ __launch_bounds__(64) void attn_bwd_kv_plain_kernel(AttnArgs a) {
  extern __shared__ float sh[];                  // 2 T floats: P and dS of this key's column
  const int lane = threadIdx.x;
  const long p = blockIdx.x;
  const int j = blockIdx.y;
  const int h = (int)(p % a.heads);
  const long seq = p / a.heads;
  const long d = (long)a.heads * a.dh, ld = 3 * d;
  const T* base = reinterpret_cast<const T*>(a.qkv) + seq * a.T * ld + (long)h * a.dh;
  const T* k = base + (long)j * ld + d;
  const T* dbase = reinterpret_cast<const T*>(a.dout) + seq * a.T * d + (long)h * a.dh;
  float* shp = sh;
  float* shs = sh + a.T;
  const int i0 = a.causal ? j : 0;
  const float c = a.scale * LOG2E;
  for (int i = i0 + lane; i < a.T; i += 64) {
    const float pr = exp2f(c * dot_rows(base + (long)i * ld, k, a.dh) - a.lse[p * a.T + i]);
    const float dp = dot_rows(dbase + (long)i * d, k + d, a.dh);
    shp[i] = pr;
    shs[i] = pr * (dp - a.dsum[p * a.T + i]);
  }
  __syncthreads();
  T* dk = reinterpret_cast<T*>(a.dqkv) + (seq * a.T + j) * ld + d + (long)h * a.dh;
  for (int cc = lane; cc < a.dh; cc += 64) {
    float ak = 0.f, av = 0.f;
    for (int i = i0; i < a.T; ++i) {
      ak = fmaf(shs[i], Elem<T>::load(base + (long)i * ld + cc), ak);
      av = fmaf(shp[i], Elem<T>::load(dbase + (long)i * d + cc), av);
    }
    Elem<T>::store(dk + cc, ak * a.scale);
    Elem<T>::store(dk + d + cc, av);
  }
}

// ------------------------------------------------------------------------------------------------------------
// matrix-core kernels: bf16, dh <= 128
// ------------------------------------------------------------------------------------------------------------
// mfma(X, Y, acc): lane l, element r of acc  +=  sum_k X[8 (r/4) + 4 (l/32) + r%4][k] * Y[l % 32][k], where for one
// step of 16 k-values a lane's 8 operand elements are k = 8 (l/32) .. + 7 of row l % 32 of X and of Y.  Only the
// pairing matters: element i of lane half hh of X meets element i of lane half hh of Y.
__device__ __forceinline__ float16v mfma(bf16x8 x, bf16x8 y, float16v acc) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(x, y, acc, 0, 0, 0);
}
__device__ __forceinline__ int tile_row_of(int r, int hh) { return 8 * (r >> 2) + 4 * hh + (r & 3); }
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }   // v_exp_f32: exp2(-inf) = 0

// An LDS tile: 32 rows of one head, DHP columns of bf16 (DHP = 32, 64 or 128: the head width rounded up).  The 16-byte
// chunks of a row are spread over the 64 banks by an XOR: within any four consecutive rows the XOR (with the row's
// place in the 256 bytes that the banks span) moves a group of four chunks to four different places, which is what a
// transposing read of four rows touches at once, and within any sixteen rows it moves a single chunk to all places, for
// the reads along a row.
template <int DHP>
struct Geo {
  static constexpr int RB = 2 * DHP;                 // bytes per row
  static constexpr int TB = 32 * RB;                 // ... per tile
  static constexpr int CPR = RB / 16;                // chunks per row
  static constexpr int RPC = 64 / CPR;               // rows per copy of 1 KB
  static constexpr int COPIES = TB / 1024;           // copies per tile
  static constexpr int PW = 2 * COPIES / 4;          // copies per wavefront of a pair of tiles, four wavefronts sharing it
  static constexpr int KK = DHP / 16;                // steps of 16 columns
  static constexpr int MB = DHP / 32;                // blocks of 32 columns
  static __device__ __forceinline__ int swz(int r) {
    if (DHP == 32) return (r >> 2) & 3;
    if (DHP == 64) return (((r >> 1) & 1) << 2) | ((r >> 2) & 3);
    return ((r & 3) << 2) | ((r >> 2) & 3);
  }
};

// Addresses: a wavefront-uniform pointer to row 0 of the 32-row tile plus one 32-bit byte offset per lane, which is
// the same for every whole tile (computed once); a tile that runs past the last row re-reads that row instead.  A head
// narrower than DHP: the chunks past its width repeat its last one (finite wherever the head is) and meet zeros in the
// other operand of every product that contracts over them; results in those columns are not stored.
//
// Tiles reach LDS by direct copies (global_load_lds_dwordx4: 16 bytes per lane from memory to lds_base + 16 lane,
// no staging registers), issued steps ahead into a ring of buffers.  The chunk swizzle is applied on the memory side:
// LDS position (row r, slot c) receives chunk c ^ swz(r) of the row.  The compiler sees neither the LDS write nor when
// it lands: a counted wait (copies_in_flight) and the workgroup's barrier (workgroup_handover) come before the reads.
__device__ __forceinline__ void copy16_to_lds(unsigned off, const void* sbase_in, unsigned lds_base) {
  // (the base is uniform by construction; say so where the register allocator has moved it to vector registers)
  const unsigned long long b = reinterpret_cast<unsigned long long>(sbase_in);
  const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)b);
  const unsigned hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(b >> 32));
  const void* sbase = reinterpret_cast<const void*>((unsigned long long)lo | ((unsigned long long)hi << 32));
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1\n"
               :: "v"(off), "s"(sbase), "s"(lds_base) : "memory");
}
// 4 bytes per lane from a per-lane address to lds_base + 4 lane
__device__ __forceinline__ void copy4_to_lds(const void* gptr, unsigned lds_base) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %0, off\n" :: "v"(gptr), "s"(lds_base) : "memory");
}
// this lane's byte offset into a tile (row stride ldb) for copy u, rows from rows_left on repeating the last one;
// dh8: chunks that the head has
template <int DHP>
__device__ __forceinline__ unsigned copy_offset(unsigned ldb, int u, int rows_left, int dh8, int lane) {
  typedef Geo<DHP> G;
  const int r = G::RPC * u + lane / G::CPR;
  int c = (lane % G::CPR) ^ G::swz(r);
  c = c < dh8 ? c : dh8 - 1;
  return (unsigned)(r < rows_left ? r : rows_left - 1) * ldb + (unsigned)c * 16u;
}
// a whole tile by one wavefront
template <int DHP>
__device__ __forceinline__ void copy_tile(const unsigned char* base, unsigned ldb, int rows_left, int dh8, unsigned lds_tile,
                                          int lane) {
#pragma unroll
  for (int u = 0; u < Geo<DHP>::COPIES; ++u)
    copy16_to_lds(copy_offset<DHP>(ldb, u, rows_left, dh8, lane), base, lds_tile + 1024u * u);
}
// A pair of tiles filled by the four wavefronts of a workgroup together, PW copies each: half of them of either tile
// (32 columns: one copy each, of the first tile by wavefronts 0 and 1).
template <int DHP>
struct PairCopy {
  typedef Geo<DHP> G;
  static constexpr int H = G::PW < 2 ? 1 : G::PW / 2;
  unsigned off[G::PW];
  static __device__ __forceinline__ int tile(int w, int i) { return G::PW == 1 ? w >> 1 : i / H; }
  static __device__ __forceinline__ int part(int w, int i) { return G::PW == 1 ? w & 1 : w * H + i % H; }
  static __device__ __forceinline__ unsigned offset(unsigned ldb0, unsigned ldb1, int rows_left, int dh8, int w, int i, int lane) {
    return copy_offset<DHP>(tile(w, i) ? ldb1 : ldb0, part(w, i), rows_left, dh8, lane);
  }
  __device__ __forceinline__ PairCopy(unsigned ldb0, unsigned ldb1, int dh8, int w, int lane) {
#pragma unroll
    for (int i = 0; i < G::PW; ++i) off[i] = offset(ldb0, ldb1, 32, dh8, w, i, lane);
  }
  // rows_left < 32: the tile that runs past the last row
  __device__ __forceinline__ void issue(const unsigned char* t0, const unsigned char* t1, unsigned ldb0, unsigned ldb1, int rows_left,
                                        int dh8, unsigned lds_pair, int w, int lane) const {
    const unsigned dst = lds_pair + (unsigned)(G::PW == 1 ? w : w * H) * 1024u;
    if (rows_left >= 32) {
#pragma unroll
      for (int i = 0; i < G::PW; ++i)
        copy16_to_lds(off[i], tile(w, i) ? t1 : t0, dst + (G::PW == 1 ? 0u : (unsigned)(i / H) * G::TB + (unsigned)(i % H) * 1024u));
    } else {
#pragma unroll
      for (int i = 0; i < G::PW; ++i)
        copy16_to_lds(offset(ldb0, ldb1, rows_left, dh8, w, i, lane), tile(w, i) ? t1 : t0,
                      dst + (G::PW == 1 ? 0u : (unsigned)(i / H) * G::TB + (unsigned)(i % H) * 1024u));
    }
  }
};
// at most N of this wavefront's copies still in flight (they land in issue order)
template <int N>
__device__ __forceinline__ void copies_in_flight() {
  __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
}
// ... and no LDS read either: the buffer that the next copies go to has been read
template <int N>
__device__ __forceinline__ void copies_in_flight_read() {
  __builtin_amdgcn_s_waitcnt(0x0070 | (N & 15) | ((N >> 4) << 14));
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}
// A value loaded from memory before the loop is made to arrive here.  Without this the compiler places its own counted
// waits for such loads at their first use inside the loop, and since it does not know of the direct copies, those
// waits would also drain the copies that were just issued for three steps ahead, on every step.
template <typename V>
__device__ __forceinline__ void landed(V& v) {
  asm volatile("" : "+v"(v));
}
// every wavefront of the workgroup has passed its wait: the tile is complete, and the buffer of the step before is free
__device__ __forceinline__ void workgroup_handover() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("" ::: "memory");
}
__device__ __forceinline__ unsigned lds_address(const void* p) {
  return (unsigned)(uintptr_t)(__attribute__((address_space(3))) const unsigned char*)p;
}
// operand fragment with the contraction along the tile's columns (step kk of 16 columns): lane holds row l % 32
template <int DHP>
__device__ __forceinline__ bf16x8 frag_cols_lds(const unsigned char* tile, int kk, int lane) {
  typedef Geo<DHP> G;
  const int r = lane & 31, ch = 2 * kk + (lane >> 5);
  return __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(tile + r * G::RB + ((ch ^ G::swz(r)) << 4)));
}
// the same, zero past the head's width (the operand that is kept in registers)
template <int DHP>
__device__ __forceinline__ bf16x8 own_cols_lds(const unsigned char* tile, int kk, int dh8, int lane) {
  const uint4 v = __builtin_bit_cast(uint4, frag_cols_lds<DHP>(tile, kk, lane));
  const bool in = 2 * kk + (lane >> 5) < dh8;
  return __builtin_bit_cast(bf16x8, make_uint4(in ? v.x : 0u, in ? v.y : 0u, in ? v.z : 0u, in ? v.w : 0u));
}
// this lane's piece of a fragment into its place in the tile
template <int DHP>
__device__ __forceinline__ void put_cols_lds(unsigned char* tile, int kk, int lane, bf16x8 v) {
  typedef Geo<DHP> G;
  const int r = lane & 31, ch = 2 * kk + (lane >> 5);
  *reinterpret_cast<uint4*>(tile + r * G::RB + ((ch ^ G::swz(r)) << 4)) = __builtin_bit_cast(uint4, v);
}
// the same straight from memory; rows from rows_left on repeat the last one
__device__ __forceinline__ bf16x8 own_cols_mem(const unsigned char* base, unsigned ldb, int rows_left, int kk, int dh8, int lane) {
  const int r = lane & 31, ch = 2 * kk + (lane >> 5);
  const bool in = ch < dh8;
  const uint4 v = *reinterpret_cast<const uint4*>(base + (unsigned)(r < rows_left ? r : rows_left - 1) * ldb + 16u * (in ? ch : 0));
  return __builtin_bit_cast(bf16x8, make_uint4(in ? v.x : 0u, in ? v.y : 0u, in ? v.z : 0u, in ? v.w : 0u));
}
// operand fragment with the contraction along the tile's ROWS, in the order the accumulator of the first product
// holds them: lane holds column 32 m + l % 32; its element i of step t is tile row 16 t + 8 (i/4) + 4 (l/32) + i%4
// (= tile_row_of(8 t + i, l/32)).  ds_read_b64_tr_b16: within 16 lanes, lane j receives as element r' element j%4 of
// the 8 bytes addressed by lane 4 r' + j/4.
template <int DHP>
__device__ __forceinline__ bf16x8 frag_rows_lds(const unsigned char* tile, int m, int t, int lane) {
  typedef Geo<DHP> G;
  typedef __attribute__((address_space(3))) short4v* lds_p;
  const int s = lane & 15;
  const int e = 32 * m + 16 * ((lane >> 4) & 1) + 4 * (s & 3);
  const int r_lo = 16 * t + 4 * (lane >> 5) + (s >> 2), r_hi = r_lo + 8;
  const unsigned char* p_lo = tile + r_lo * G::RB + (((e >> 3) ^ G::swz(r_lo)) << 4) + (e & 7) * 2;
  const unsigned char* p_hi = tile + r_hi * G::RB + (((e >> 3) ^ G::swz(r_hi)) << 4) + (e & 7) * 2;
  const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_p)(p_lo));
  const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_p)(p_hi));
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}
// 8 accumulator elements (r = 8 t .. 8 t + 7) rounded to bf16 as the second product's operand
__device__ __forceinline__ bf16x8 pack8(const float* v) {
  const uint4 w = make_uint4(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]), pack_bf16x2(v[4], v[5]),
                             pack_bf16x2(v[6], v[7]));
  return __builtin_bit_cast(bf16x8, w);
}
// The second products' operand, 16 probabilities (or dS) of a lane.  Rounded to bf16 once, or (EXACT) cut into three bf16
// parts of 8 bits each that add up to the value itself: the products and sums are then those of fp32 operands.
template <bool EXACT>
struct Scores {
  static constexpr int PARTS = EXACT ? 3 : 1;
  bf16x8 part[PARTS][2];
  __device__ __forceinline__ explicit Scores(const float (&v)[16]) {
    if (!EXACT) {
#pragma unroll
      for (int t = 0; t < 2; ++t) part[0][t] = pack8(v + 8 * t);
      return;
    }
    float rest[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) rest[r] = v[r];
#pragma unroll
    for (int p = 0; p < PARTS; ++p)
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        unsigned w[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          float& x = rest[8 * t + 2 * i];
          float& y = rest[8 * t + 2 * i + 1];
          w[i] = __builtin_amdgcn_perm(__float_as_uint(y), __float_as_uint(x), 0x07060302u);   // the upper halves
          x -= __uint_as_float(__float_as_uint(x) & 0xFFFF0000u);                             // (exact)
          y -= __uint_as_float(__float_as_uint(y) & 0xFFFF0000u);
        }
        part[p][t] = __builtin_bit_cast(bf16x8, make_uint4(w[0], w[1], w[2], w[3]));
      }
  }
  // acc += tile rows 16 t .. of `x` times their scores
  __device__ __forceinline__ float16v times(bf16x8 x, int t, float16v acc) const {
#pragma unroll
    for (int p = 0; p < PARTS; ++p) acc = mfma(x, part[p][t], acc);
    return acc;
  }
};
__device__ __forceinline__ void store4b(bf16_t* p, float a, float b, float c, float d) {
  *reinterpret_cast<uint2*>(p) = make_uint2(pack_bf16x2(a, b), pack_bf16x2(c, d));
}
// A tile's results, scaled (a lane holds columns 32 m + tile_row_of(r, hh) of row l % 32), dh columns of them, to `base`, the
// tile's first row (stride ld elements); rows from rows_left on are not there.  They pass through 2 KB of LDS of the
// wavefront's own, 32 columns at a time, so that a store covers 64 bytes of a row and not 16: straight from the
// accumulators a tile is 8 instructions of 32 pieces of lines each, and the L2 takes one piece a clock (dk, dv of 768 problems of
// 1024: 323 -> 301 us).
template <int MB>
__device__ __forceinline__ void store_tile(bf16_t* base, long ld, int rows_left, const float16v (&acc)[MB], float f, int dh,
                                           unsigned char* stg, int lane) {
  const int r = lane & 31, hh = lane >> 5, rr = lane >> 2, ch = lane & 3;
#pragma unroll
  for (int m = 0; m < MB; ++m) {
    if (32 * m >= dh) break;
#pragma unroll
    for (int g = 0; g < 4; ++g)
      store4b(reinterpret_cast<bf16_t*>(stg + r * 64 + ((g ^ ((r >> 2) & 3)) << 4) + 8 * hh), acc[m][4 * g] * f,
              acc[m][4 * g + 1] * f, acc[m][4 * g + 2] * f, acc[m][4 * g + 3] * f);
    __builtin_amdgcn_wave_barrier();                       // (a wavefront's LDS operations execute in order)
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int row = rr + 16 * u;
      const uint4 v = *reinterpret_cast<const uint4*>(stg + row * 64 + ((ch ^ ((row >> 2) & 3)) << 4));
      if (row < rows_left && 32 * m + 8 * ch < dh) *reinterpret_cast<uint4*>(base + row * ld + 32 * m + 8 * ch) = v;
    }
    __builtin_amdgcn_wave_barrier();
  }
}
template <int MB>
__device__ __forceinline__ void zero_acc(float16v (&acc)[MB]) {
#pragma unroll
  for (int m = 0; m < MB; ++m)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[m][r] = 0.f;
}
__device__ __forceinline__ float dot8(bf16x8 a, bf16x8 b) {
  const uint4 x = __builtin_bit_cast(uint4, a), y = __builtin_bit_cast(uint4, b);
  const unsigned xs[4] = {x.x, x.y, x.z, x.w}, ys[4] = {y.x, y.y, y.z, y.w};
  float acc = 0.f;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    acc = fmaf(__uint_as_float(xs[i] << 16), __uint_as_float(ys[i] << 16), acc);
    acc = fmaf(__uint_as_float(xs[i] & 0xFFFF0000u), __uint_as_float(ys[i] & 0xFFFF0000u), acc);
  }
  return acc;
}

constexpr int AT_WAVES = 4;    // wavefronts per workgroup: 4 tiles of 32 queries (dk/dv kernel: keys) that share the streamed tiles
constexpr int AT_NST = 4;      // stages of the ring of streamed tile pairs: copies run AT_NST - 1 steps ahead

// Which (sequence, head) problem and which block of AT_WAVES tiles a workgroup takes.  Consecutive workgroup ids go to
// the eight XCDs in turn, each with an L2 of its own, and all blocks of one problem stream the same k / v (q / do)
// tiles.  by_problem (large grids): the blocks of a problem get ids that land on ONE XCD, next to each other in its
// dispatch order, so they start together, stream in step and the tiles come from memory once per problem instead of
// once per block.  Otherwise (a grid of a few rounds of workgroups, where the tail decides): every problem's
// longest block first, then the next longest.  The grid holds 8 ceil(P / 8) nblk workgroups; one whose problem does
// not exist leaves at once (the whole workgroup, before any barrier).
struct BlockOf { unsigned p; int slot; bool exists; };
__device__ __forceinline__ BlockOf block_of(const AttnArgs& a, int nblk) {
  const unsigned P = (unsigned)(a.seqs * a.heads), id = blockIdx.x;
  BlockOf b;
  if (a.by_problem) {
    const unsigned xcd = id & 7u, turn = id >> 3, j = turn / (unsigned)nblk;
    b.p = xcd + 8u * j;
    b.slot = (int)(turn - j * (unsigned)nblk);
  } else {
    const unsigned Pr = (P + 7u) & ~7u;
    b.slot = (int)(id / Pr);
    b.p = id - (unsigned)b.slot * Pr;
  }
  b.exists = b.p < P;
  return b;
}
// grids from about four rounds of resident workgroups per XCD on: problem by problem
constexpr long BY_PROBLEM_FROM = 4 * 1024;
inline long attn_grid(const AttnArgs& a, bool shared = false) {
  const long P = a.seqs * a.heads, nt = (a.T + 31) / 32, nblk = shared ? nt : (nt + AT_WAVES - 1) / AT_WAVES;
  return 8 * ((P + 7) / 8) * nblk;
}

// Few problems (SHARED): a workgroup takes ONE tile of 32 queries (keys) and its four wavefronts share the tiles of the other side
// out, every fourth each, through rings of their own: no barrier in the loop, a quarter of its steps, four times the workgroups.
// Their results, the sums of the second products (and in the forward pass the rows' maxima and sums), meet in LDS at the end.
// Every workgroup streams for 32 rows then, not 128.
template <int DHP, bool SHARED> constexpr int ring_stages() { return !SHARED ? AT_NST : DHP == 128 ? 2 : 3; }
template <bool SHARED> constexpr int rings() { return SHARED ? AT_WAVES : 1; }
// tiles first, first + 4, .. below end
__device__ __forceinline__ int every_fourth(int end, int first) { return end > first ? (end - first + AT_WAVES - 1) / AT_WAVES : 0; }
// acc of wavefront 0 becomes the sum of the four wavefronts', each times its f; `sums`: 256 bytes per accumulator and wavefront
// (the rings, which everyone has left)
template <int MB>
__device__ __forceinline__ void meet_sums(float16v (&acc)[MB], float* sums, int wave, int lane, const float (&f)[AT_WAVES]) {
#pragma unroll
  for (int m = 0; m < MB; ++m)
#pragma unroll
    for (int r = 0; r < 16; ++r) sums[((wave * MB + m) * 16 + r) * 64 + lane] = acc[m][r];
  __syncthreads();
#pragma unroll
  for (int i = 0; i < MB * 4; ++i) {                       // a quarter of the accumulators each
    const int e = wave * MB * 4 + i;
    float t = f[0] * sums[e * 64 + lane];
#pragma unroll
    for (int w = 1; w < AT_WAVES; ++w) t = fmaf(f[w], sums[(w * MB * 16 + e) * 64 + lane], t);
    sums[e * 64 + lane] = t;
  }
  __syncthreads();
  if (wave == 0) {
#pragma unroll
    for (int m = 0; m < MB; ++m)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[m][r] = sums[(m * 16 + r) * 64 + lane];
  }
}

// One (sequence, head): wavefront-uniform byte pointers to row 0 of q, k, v (row stride 6 d bytes) and of the
// d-wide arrays (row stride 2 d bytes), all at the head's columns.
struct Head {
  const unsigned char* q; const unsigned char* k; const unsigned char* v;
  long wide_off;         // byte offset of row 0 of the head in a [tokens, d] array
  long tok0, d, ld;
  unsigned h;
};
__device__ __forceinline__ Head head_of(const AttnArgs& a, unsigned p) {
  Head hd;
  const unsigned heads = (unsigned)a.heads;
  hd.h = p % heads;
  const unsigned seq = p / heads;
  hd.d = (long)heads * a.dh;
  hd.ld = 3 * hd.d;
  hd.tok0 = (long)seq * a.T;
  hd.q = reinterpret_cast<const unsigned char*>(a.qkv) + (hd.tok0 * hd.ld + (long)hd.h * a.dh) * 2;
  hd.k = hd.q + hd.d * 2;
  hd.v = hd.k + hd.d * 2;
  hd.wide_off = (hd.tok0 * hd.d + (long)hd.h * a.dh) * 2;
  return hd;
}

// 64-wide heads (PAD = false) round P and dS to bf16 once for the second products; every other width is held to the plain
// kernels, which keep them in fp32: there they enter whole, in three parts, at three times the second products.
template <int DHP, bool PAD> constexpr bool exact_scores() { return !(DHP == 64 && !PAD); }

// Infinities and NaNs.  A product on the matrix cores meets every element of a tile, also those that the mask, the sequence's
// end or the head's width leave out, and there 0 times an infinity is NaN; so are the second and third part of an infinite
// score.  Where the scores are held whole, a row of a result that did not come out finite is therefore computed once more,
// term by term over what it sees, as the plain kernels do: one wavefront, the columns over its lanes.  Finite data never
// comes here; the test costs a product per accumulator and tile.
template <int MB>
__device__ __forceinline__ float not_finite(const float16v (&acc)[MB], float t) {     // NaN if any of them is not finite
#pragma unroll
  for (int m = 0; m < MB; ++m)
#pragma unroll
    for (int r = 0; r < 16; ++r) t = fmaf(acc[m][r], 0.f, t);
  return t;
}
// rows (bits) of this wavefront's tile in which a lane's t is NaN, rows_left of them
__device__ __forceinline__ unsigned rows_to_redo(float t, int rows_left) {
  const unsigned long long b = __ballot(t != t);
  const unsigned rows = (unsigned)b | (unsigned)(b >> 32);
  return rows_left < 32 ? rows & ((1u << rows_left) - 1u) : rows;
}
// out[c] += sum over 64 rows of w (lane j: row j) times column c of `rows`; a lane holds columns lane and lane + 64
struct TwoColumns {
  float v[2] = {0.f, 0.f};
  __device__ __forceinline__ void add(float w, int n, const bf16_t* rows, long ld, int dh, int lane) {
    for (int j = 0; j < n; ++j) {
      const float wj = __shfl(w, j, 64);
#pragma unroll
      for (int u = 0; u < 2; ++u)
        if (lane + 64 * u < dh) v[u] = fmaf(wj, Elem<bf16_t>::load(rows + j * ld + lane + 64 * u), v[u]);
    }
  }
  __device__ __forceinline__ void store(bf16_t* out, float f, int dh, int lane) const {
#pragma unroll
    for (int u = 0; u < 2; ++u)
      if (lane + 64 * u < dh) Elem<bf16_t>::store(out + lane + 64 * u, v[u] * f);
  }
};
__device__ __forceinline__ void redo_fwd(const AttnArgs& a, const Head& hd, unsigned p, int i, int lane) {
  const bf16_t* k = reinterpret_cast<const bf16_t*>(hd.k);
  const bf16_t* q = reinterpret_cast<const bf16_t*>(hd.q) + i * hd.ld;
  const int jn = a.causal ? i + 1 : (int)a.T;
  const float c = a.scale * LOG2E;
  float m = -INFINITY, sum = 0.f;
  for (int j = lane; j < jn; j += 64) m = fmaxf(m, c * dot_rows(q, k + j * hd.ld, a.dh));
  m = wave_max(m);
  TwoColumns o;
  for (int j0 = 0; j0 < jn; j0 += 64) {
    float pr = 0.f;
    if (j0 + lane < jn) {
      pr = exp2f(c * dot_rows(q, k + (j0 + lane) * hd.ld, a.dh) - m);
      sum += pr;
    }
    o.add(pr, jn - j0 < 64 ? jn - j0 : 64, k + j0 * hd.ld + hd.d, hd.ld, a.dh, lane);
  }
  sum = wave_sum(sum);
#pragma unroll
  for (int u = 0; u < 2; ++u) o.v[u] /= sum;
  o.store(reinterpret_cast<bf16_t*>(reinterpret_cast<unsigned char*>(a.o) + hd.wide_off) + i * hd.d, 1.f, a.dh, lane);
  if (lane == 0) a.lse[(long)p * a.T + i] = m + log2f(sum);
}
// D: of this query
__device__ __forceinline__ void redo_q(const AttnArgs& a, const Head& hd, unsigned p, int i, float D, int lane) {
  const bf16_t* k = reinterpret_cast<const bf16_t*>(hd.k);
  const bf16_t* q = reinterpret_cast<const bf16_t*>(hd.q) + i * hd.ld;
  const bf16_t* dout = reinterpret_cast<const bf16_t*>(reinterpret_cast<const unsigned char*>(a.dout) + hd.wide_off) + i * hd.d;
  const int jn = a.causal ? i + 1 : (int)a.T;
  const float c = a.scale * LOG2E, L2 = a.lse[(long)p * a.T + i];
  TwoColumns dq;
  for (int j0 = 0; j0 < jn; j0 += 64) {
    float ds = 0.f;
    if (j0 + lane < jn) {
      const bf16_t* kj = k + (j0 + lane) * hd.ld;
      ds = exp2f(c * dot_rows(q, kj, a.dh) - L2) * (dot_rows(dout, kj + hd.d, a.dh) - D);
    }
    dq.add(ds, jn - j0 < 64 ? jn - j0 : 64, k + j0 * hd.ld, hd.ld, a.dh, lane);
  }
  dq.store(reinterpret_cast<bf16_t*>(a.dqkv) + (q - reinterpret_cast<const bf16_t*>(a.qkv)), a.scale, a.dh, lane);
}
// D_of(i): D of query i
template <typename F>
__device__ __forceinline__ void redo_kv(const AttnArgs& a, const Head& hd, unsigned p, int j, F D_of, int lane) {
  const bf16_t* q = reinterpret_cast<const bf16_t*>(hd.q);
  const bf16_t* kj = reinterpret_cast<const bf16_t*>(hd.k) + j * hd.ld;
  const bf16_t* dout = reinterpret_cast<const bf16_t*>(reinterpret_cast<const unsigned char*>(a.dout) + hd.wide_off);
  const int T = (int)a.T;
  const float c = a.scale * LOG2E;
  TwoColumns dk, dv;
  for (int i0 = a.causal ? j : 0; i0 < T; i0 += 64) {
    float pr = 0.f, ds = 0.f;
    const int i = i0 + lane, n = T - i0 < 64 ? T - i0 : 64;
    if (i < T) {
      pr = exp2f(c * dot_rows(q + i * hd.ld, kj, a.dh) - a.lse[(long)p * a.T + i]);
      ds = pr * (dot_rows(dout + i * hd.d, kj + hd.d, a.dh) - D_of(i));
    }
    dk.add(ds, n, q + i0 * hd.ld, hd.ld, a.dh, lane);
    dv.add(pr, n, dout + i0 * hd.d, hd.d, a.dh, lane);
  }
  bf16_t* out = reinterpret_cast<bf16_t*>(a.dqkv) + (kj - reinterpret_cast<const bf16_t*>(a.qkv));
  dk.store(out, a.scale, a.dh, lane);
  dv.store(out + hd.d, 1.f, a.dh, lane);
}
// f(row) for every row of the tile that came out not finite, after the tile's own stores
template <typename F>
__device__ __forceinline__ void redo_rows(float t, int rows_left, F f) {
  unsigned rows = rows_to_redo(t, rows_left);
  if (rows == 0) return;
  copies_in_flight<0>();                                   // (stores too: what follows overwrites some of them)
  for (; rows != 0; rows &= rows - 1) f(__ffs((int)rows) - 1);
}

// The three kernels share one shape (SHARED: as described there).  A workgroup of four wavefronts owns four consecutive tiles of
// 32 queries (dk/dv kernel: keys), one per wavefront, and streams the tiles of the other side through a ring of AT_NST buffer
// pairs that all four read: at step t each wavefront waits for its own share of pair t, the workgroup meets at a
// barrier (pair t complete; everyone done with pair t-1), its copies of pair t + AT_NST - 1 go out into the
// buffer just freed, and the wavefront computes on pair t (or skips it when the causal mask hides the whole tile from
// its rows).  No global load is issued inside the loop other than these copies, so the counted wait is exact.

template <int DHP, bool PAD, bool CAUSAL, bool SHARED>
__global__ __launch_bounds__(64 * AT_WAVES, SHARED ? 1 : 2) void attn_fwd_mfma_kernel(AttnArgs a) {
  constexpr int NST = ring_stages<DHP, SHARED>();
  typedef Geo<DHP> G;
  constexpr bool EXACT = exact_scores<DHP, PAD>();
  __shared__ __attribute__((aligned(1024))) unsigned char smem[rings<SHARED>() * NST][2][G::TB];   // [stage][k | v]
  __shared__ __attribute__((aligned(256))) unsigned char staging[AT_WAVES][2048];   // [wave]: results on their way out
  const int lane = threadIdx.x & 63, hh = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int T = (int)a.T, nt = (T + 31) >> 5;
  const int nblk = SHARED ? nt : (nt + AT_WAVES - 1) / AT_WAVES;
  const BlockOf bo = block_of(a, nblk);
  if (!bo.exists) return;
  const int blk = nblk - 1 - bo.slot;                              // long rows first
  const int qt = SHARED ? blk : AT_WAVES * blk + wave;
  const bool live = qt < nt;                                       // a ragged workgroup's spare wavefronts only copy
  const unsigned p = bo.p;
  const Head hd = head_of(a, p);
  const unsigned ldb = (unsigned)(hd.ld * 2);
  const int dh = PAD ? a.dh : DHP, dh8 = dh >> 3;
  unsigned char (*const ring)[2][G::TB] = smem + (SHARED ? wave * NST : 0);
  const unsigned lds0 = (unsigned)__builtin_amdgcn_readfirstlane((int)lds_address(ring));
  const bool ragged = (T & 31) != 0;
  const int q0 = 32 * qt, qi = q0 + (lane & 31);
  const float c = a.scale * LOG2E;
  const int last_q = SHARED ? qt : AT_WAVES * blk + AT_WAVES - 1 < nt - 1 ? AT_WAVES * blk + AT_WAVES - 1 : nt - 1;
  const int nkt = CAUSAL ? last_q + 1 : nt;                        // key tiles the workgroup streams
  const int own_nkt = CAUSAL ? qt + 1 : nt;                        // ... and those this wavefront's rows see
  const PairCopy<DHP> pc(ldb, ldb, dh8, wave, lane);
  // the i-th pair of the ring: key tile i, this wavefront's share of its copies, or (SHARED) the wavefront's i-th key tile, whole
  const int n_ring = SHARED ? every_fourth(nkt, wave) : nkt;
  auto tile_of = [&](int i) __attribute__((always_inline)) { return SHARED ? wave + AT_WAVES * i : i; };
  auto issue = [&](int i) __attribute__((always_inline)) {
    const int kt = tile_of(i), left = ragged && kt == nt - 1 ? T - 32 * kt : 32;
    const unsigned char* kb = hd.k + (long)(32 * kt) * ldb;
    const unsigned dst = lds0 + (unsigned)(i % NST) * (2u * G::TB);
    if (SHARED) {
      copy_tile<DHP>(kb, ldb, left, dh8, dst, lane);
      copy_tile<DHP>(kb + hd.d * 2, ldb, left, dh8, dst + G::TB, lane);
    } else {
      pc.issue(kb, kb + hd.d * 2, ldb, ldb, left, dh8, dst, wave, lane);
    }
  };
  for (int i = 0; i < NST - 1 && i < n_ring; ++i) issue(i);
  bf16x8 fq[G::KK];
#pragma unroll
  for (int kk = 0; kk < G::KK; ++kk) fq[kk] = own_cols_mem(hd.q + (long)(live ? q0 : 0) * ldb, ldb, live ? T - q0 : 1, kk, dh8, lane);
#pragma unroll
  for (int kk = 0; kk < G::KK; ++kk) landed(fq[kk]);
  float16v o[G::MB];
  zero_acc(o);
  // (the row's maximum starts from the lowest finite number: a first tile whose scores are all minus infinity weighs nothing then)
  float m = -FLT_MAX, l = 0.f;
  // one tile of 32 keys; MASKED: the tile on the diagonal (causal) or the one that runs past the last key
  auto step = [&](int i, auto masked_c) __attribute__((always_inline)) {
    constexpr bool MASKED = decltype(masked_c)::value;
    const int k0 = 32 * tile_of(i);
    const unsigned char* tk = ring[i % NST][0];
    const unsigned char* tv = ring[i % NST][1];
    float16v s;
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] = 0.f;
    // every operand read of the step goes out here: those of the second product land while the scores are reduced
    bf16x8 fk[G::KK], fv[G::MB][2];
#pragma unroll
    for (int kk = 0; kk < G::KK; ++kk) fk[kk] = frag_cols_lds<DHP>(tk, kk, lane);
#pragma unroll
    for (int mb = 0; mb < G::MB; ++mb)
#pragma unroll
      for (int t = 0; t < 2; ++t) fv[mb][t] = frag_rows_lds<DHP>(tv, mb, t, lane);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int kk = 0; kk < G::KK; ++kk) s = mfma(fk[kk], fq[kk], s);
    float sv[16];
    float tmax = -INFINITY;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      sv[r] = s[r] * c;
      if (MASKED) {
        const int kj = k0 + tile_row_of(r, hh);
        if (!(CAUSAL ? kj <= qi : kj < T)) sv[r] = -INFINITY;
      }
      tmax = fmaxf(tmax, sv[r]);
    }
    tmax = fmaxf(tmax, __shfl_xor(tmax, 32, 64));
    const float mn = fmaxf(m, tmax);
    const float alpha = fast_exp2(m - mn);
    float ps = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) { sv[r] = fast_exp2(sv[r] - mn); ps += sv[r]; }
    ps += __shfl_xor(ps, 32, 64);
    l = l * alpha + ps;
    m = mn;
#pragma unroll
    for (int mb = 0; mb < G::MB; ++mb)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[mb][r] *= alpha;
    const Scores<EXACT> pq(sv);
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int mb = 0; mb < G::MB; ++mb) o[mb] = pq.times(fv[mb][t], t, o[mb]);
  };
  // pair i complete and visible to those that read it, the buffer of pair i - 1 free and refilled
  auto advance = [&](int i) __attribute__((always_inline)) {
    if (SHARED) {
      if (i + NST - 2 < n_ring) copies_in_flight_read<2 * G::COPIES * (NST - 2)>();
      else copies_in_flight_read<0>();
    } else {
      if (i + NST - 2 < n_ring) copies_in_flight<G::PW * (NST - 2)>();
      else copies_in_flight<0>();
      workgroup_handover();
    }
    if (i + NST - 1 < n_ring) issue(i + NST - 1);
  };
  // whole tiles, then the masked one (SHARED: of the wavefront that has it), then (causal) the tiles the workgroup streams for its
  // later rows only
  const int n_own = SHARED ? n_ring : live ? own_nkt : 0;
  const bool masked_own = (CAUSAL || ragged) && (!SHARED || (nkt - 1) % AT_WAVES == wave);
  const int n_plain = masked_own ? n_own - 1 : n_own;
  int i = 0;
  for (; i < n_plain; ++i) { advance(i); step(i, std::false_type()); }
  if (i < n_own) { advance(i); step(i, std::true_type()); ++i; }
  for (; i < n_ring; ++i) advance(i);
  if (SHARED) {
    __syncthreads();                                               // everyone has left the rings
    float* const rows = reinterpret_cast<float*>(smem) + AT_WAVES * G::MB * 16 * 64;       // behind the sums: [wave][m | l][lane]
    rows[2 * wave * 64 + lane] = m;
    rows[(2 * wave + 1) * 64 + lane] = l;
    __syncthreads();
    float f[AT_WAVES], top = rows[lane];
#pragma unroll
    for (int w = 1; w < AT_WAVES; ++w) top = fmaxf(top, rows[2 * w * 64 + lane]);
    l = 0.f;
#pragma unroll
    for (int w = 0; w < AT_WAVES; ++w) {                           // (a wavefront without a tile: sums of zero)
      f[w] = fast_exp2(rows[2 * w * 64 + lane] - top);
      l = fmaf(f[w], rows[(2 * w + 1) * 64 + lane], l);
    }
    m = top;
    meet_sums(o, reinterpret_cast<float*>(smem), wave, lane, f);
  }
  if (!(l > 0.f)) l = NAN;                                         // no score above minus infinity: NaN, as the plain kernel has it
  if (SHARED ? wave == 0 : live) {
    store_tile(reinterpret_cast<bf16_t*>(reinterpret_cast<unsigned char*>(a.o) + hd.wide_off) + (long)q0 * hd.d, hd.d, T - q0, o,
               1.f / l, dh, staging[wave], lane);
    if (hh == 0 && qi < T) a.lse[(long)p * a.T + qi] = m + log2f(l);
    if (EXACT) redo_rows(not_finite(o, 0.f), T - q0, [&](int r) { redo_fwd(a, hd, p, q0 + r, lane); });
  }
}

// dq of four tiles of 32 queries (SHARED: of one); also leaves D = rowsum(do (.) o) of their queries for the dk/dv kernel
template <int DHP, bool PAD, bool CAUSAL, bool SHARED>
__global__ __launch_bounds__(64 * AT_WAVES, SHARED ? 1 : 2) void attn_bwd_q_mfma_kernel(AttnArgs a) {
  constexpr int NST = ring_stages<DHP, SHARED>();
  typedef Geo<DHP> G;
  constexpr bool EXACT = exact_scores<DHP, PAD>();
  __shared__ __attribute__((aligned(1024))) unsigned char smem[rings<SHARED>() * NST][2][G::TB];   // [stage][k | v]
  __shared__ __attribute__((aligned(256))) unsigned char staging[AT_WAVES][2048];   // [wave]: results on their way out
  const int lane = threadIdx.x & 63, hh = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int T = (int)a.T, nt = (T + 31) >> 5;
  const int nblk = SHARED ? nt : (nt + AT_WAVES - 1) / AT_WAVES;
  const BlockOf bo = block_of(a, nblk);
  if (!bo.exists) return;
  const int blk = nblk - 1 - bo.slot;
  const int qt = SHARED ? blk : AT_WAVES * blk + wave;
  const bool live = qt < nt;
  const unsigned p = bo.p;
  const Head hd = head_of(a, p);
  const unsigned ldb = (unsigned)(hd.ld * 2), ldw = (unsigned)(hd.d * 2);
  const int dh = PAD ? a.dh : DHP, dh8 = dh >> 3;
  unsigned char (*const ring)[2][G::TB] = smem + (SHARED ? wave * NST : 0);
  const unsigned lds0 = (unsigned)__builtin_amdgcn_readfirstlane((int)lds_address(ring));
  const bool ragged = (T & 31) != 0;
  const int q0 = live ? 32 * qt : 0, qi = 32 * qt + (lane & 31);
  const int qc = qi < T ? qi : T - 1;
  const float c = a.scale * LOG2E;
  const int last_q = SHARED ? qt : AT_WAVES * blk + AT_WAVES - 1 < nt - 1 ? AT_WAVES * blk + AT_WAVES - 1 : nt - 1;
  const int nkt = CAUSAL ? last_q + 1 : nt;
  const int own_nkt = CAUSAL ? qt + 1 : nt;
  const PairCopy<DHP> pc(ldb, ldb, dh8, wave, lane);
  // the i-th pair of the ring: key tile i, this wavefront's share of its copies, or (SHARED) the wavefront's i-th key tile, whole
  const int n_ring = SHARED ? every_fourth(nkt, wave) : nkt;
  auto tile_of = [&](int i) __attribute__((always_inline)) { return SHARED ? wave + AT_WAVES * i : i; };
  auto issue = [&](int i) __attribute__((always_inline)) {
    const int kt = tile_of(i), left = ragged && kt == nt - 1 ? T - 32 * kt : 32;
    const unsigned char* kb = hd.k + (long)(32 * kt) * ldb;
    const unsigned dst = lds0 + (unsigned)(i % NST) * (2u * G::TB);
    if (SHARED) {
      copy_tile<DHP>(kb, ldb, left, dh8, dst, lane);
      copy_tile<DHP>(kb + hd.d * 2, ldb, left, dh8, dst + G::TB, lane);
    } else {
      pc.issue(kb, kb + hd.d * 2, ldb, ldb, left, dh8, dst, wave, lane);
    }
  };
  for (int i = 0; i < NST - 1 && i < n_ring; ++i) issue(i);
  float L2 = a.lse[(long)p * a.T + qc];
  bf16x8 fq[G::KK], fdo[G::KK];
  float D = 0.f;
  {
    const unsigned char* dob = reinterpret_cast<const unsigned char*>(a.dout) + hd.wide_off + (long)q0 * ldw;
    const unsigned char* ob = reinterpret_cast<const unsigned char*>(a.o) + hd.wide_off + (long)q0 * ldw;
#pragma unroll
    for (int kk = 0; kk < G::KK; ++kk) {
      fq[kk] = own_cols_mem(hd.q + (long)q0 * ldb, ldb, T - q0, kk, dh8, lane);
      fdo[kk] = own_cols_mem(dob, ldw, T - q0, kk, dh8, lane);
      D += dot8(fdo[kk], own_cols_mem(ob, ldw, T - q0, kk, dh8, lane));
    }
    D += __shfl_xor(D, 32, 64);
    if ((SHARED ? wave == 0 : live) && hh == 0 && qi < T) a.dsum[(long)p * a.T + qi] = D;
#pragma unroll
    for (int kk = 0; kk < G::KK; ++kk) { landed(fq[kk]); landed(fdo[kk]); }
    landed(L2);
  }
  float16v dq[G::MB];
  zero_acc(dq);
  auto step = [&](int i, auto masked_c) __attribute__((always_inline)) {
    constexpr bool MASKED = decltype(masked_c)::value;
    const int k0 = 32 * tile_of(i);
    const unsigned char* tk = ring[i % NST][0];
    const unsigned char* tv = ring[i % NST][1];
    float16v s, dp;
#pragma unroll
    for (int r = 0; r < 16; ++r) { s[r] = 0.f; dp[r] = -D; }      // dp comes out as dP - D
    // All operand reads of a phase go out before its first product (the compiler's counted waits then let the
    // products start as their operands arrive), and those of the third product while the scores become dS: a read
    // issued right before its product would expose the LDS latency a dozen times per step.
    // (128 columns: in two halves, the registers do not hold all of them at once)
    constexpr int PART = G::KK < 4 ? G::KK : 4;
#pragma unroll
    for (int k1 = 0; k1 < G::KK; k1 += PART) {
      bf16x8 fk[PART], fv[PART];
#pragma unroll
      for (int kk = 0; kk < PART; ++kk) { fk[kk] = frag_cols_lds<DHP>(tk, k1 + kk, lane); fv[kk] = frag_cols_lds<DHP>(tv, k1 + kk, lane); }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int kk = 0; kk < PART; ++kk) {
        s = mfma(fk[kk], fq[k1 + kk], s);
        dp = mfma(fv[kk], fdo[k1 + kk], dp);
      }
      if (k1 + PART < G::KK) __builtin_amdgcn_sched_barrier(0);
    }
    bf16x8 kr[G::MB][2];
#pragma unroll
    for (int mb = 0; mb < G::MB; ++mb)
#pragma unroll
      for (int t = 0; t < 2; ++t)
        if (G::MB < 4) kr[mb][t] = frag_rows_lds<DHP>(tk, mb, t, lane);
    __builtin_amdgcn_sched_barrier(0);
    float ds[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      float pr = fast_exp2(fmaf(s[r], c, -L2));
      if (MASKED) {
        const int kj = k0 + tile_row_of(r, hh);
        if (!(CAUSAL ? kj <= qi : kj < T)) pr = 0.f;
      }
      ds[r] = pr * dp[r];
    }
    const Scores<EXACT> dq_s(ds);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int mb = 0; mb < G::MB; ++mb)
        dq[mb] = dq_s.times(G::MB < 4 ? kr[mb][t] : frag_rows_lds<DHP>(tk, mb, t, lane), t, dq[mb]);
  };
  // pair i complete and visible to those that read it, the buffer of pair i - 1 free and refilled
  auto advance = [&](int i) __attribute__((always_inline)) {
    if (SHARED) {
      if (i + NST - 2 < n_ring) copies_in_flight_read<2 * G::COPIES * (NST - 2)>();
      else copies_in_flight_read<0>();
    } else {
      if (i + NST - 2 < n_ring) copies_in_flight<G::PW * (NST - 2)>();
      else copies_in_flight<0>();
      workgroup_handover();
    }
    if (i + NST - 1 < n_ring) issue(i + NST - 1);
  };
  // whole tiles, then the masked one (SHARED: of the wavefront that has it), then (causal) the tiles the workgroup streams for its
  // later rows only
  const int n_own = SHARED ? n_ring : live ? own_nkt : 0;
  const bool masked_own = (CAUSAL || ragged) && (!SHARED || (nkt - 1) % AT_WAVES == wave);
  const int n_plain = masked_own ? n_own - 1 : n_own;
  int i = 0;
  for (; i < n_plain; ++i) { advance(i); step(i, std::false_type()); }
  if (i < n_own) { advance(i); step(i, std::true_type()); ++i; }
  for (; i < n_ring; ++i) advance(i);
  if (SHARED) {
    __syncthreads();                                               // everyone has left the rings
    const float ones[AT_WAVES] = {1.f, 1.f, 1.f, 1.f};
    meet_sums(dq, reinterpret_cast<float*>(smem), wave, lane, ones);
  }
  if (SHARED ? wave == 0 : live) {
    store_tile(reinterpret_cast<bf16_t*>(reinterpret_cast<unsigned char*>(a.dqkv) + (hd.q - reinterpret_cast<const unsigned char*>(a.qkv))) +
                   (long)q0 * hd.ld, hd.ld, T - q0, dq, a.scale, dh, staging[wave], lane);
    if (EXACT) redo_rows(not_finite(dq, 0.f), T - q0, [&](int r) { redo_q(a, hd, p, q0 + r, __shfl(D, r, 64), lane); });
  }
}

// dk, dv of four tiles of 32 keys (SHARED: of one; after the dq kernel: reads D).  128-wide heads hold 128 accumulators and 32 operand
// registers per lane, and the parts of two sets of scores: one workgroup per compute unit with all 512 registers; narrower
// ones fit three, or two where the scores are in three parts of 64 columns (in three, 40 registers spill).
template <int DHP, bool PAD, bool CAUSAL, bool SHARED>
__global__ __launch_bounds__(64 * AT_WAVES, SHARED || DHP == 128 ? 1 : DHP == 64 && PAD ? 2 : 3) void attn_bwd_kv_mfma_kernel(AttnArgs a) {
  constexpr int NST = ring_stages<DHP, SHARED>();
  typedef Geo<DHP> G;
  constexpr bool EXACT = exact_scores<DHP, PAD>();
  __shared__ __attribute__((aligned(1024))) unsigned char smem[rings<SHARED>() * NST][2][G::TB];   // [stage][q | do]
  __shared__ __attribute__((aligned(1024))) unsigned char own_v[SHARED ? 1 : AT_WAVES][G::TB];     // [wave]: the v rows of its own keys
  __shared__ __attribute__((aligned(256))) float stats[AT_WAVES][NST][64];          // [wave][stage][L2 | D] (a copy per wavefront)
  const int lane = threadIdx.x & 63, hh = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int T = (int)a.T, nt = (T + 31) >> 5;
  const BlockOf bo = block_of(a, SHARED ? nt : (nt + AT_WAVES - 1) / AT_WAVES);
  if (!bo.exists) return;
  const int blk = bo.slot;                                         // causal: early keys see the most queries
  const int kt = SHARED ? blk : AT_WAVES * blk + wave;
  const bool live = kt < nt;
  const unsigned p = bo.p;
  const Head hd = head_of(a, p);
  const unsigned ldb = (unsigned)(hd.ld * 2), ldw = (unsigned)(hd.d * 2);
  const int dh = PAD ? a.dh : DHP, dh8 = dh >> 3;
  const unsigned char* dob = reinterpret_cast<const unsigned char*>(a.dout) + hd.wide_off;
  unsigned char (*const ring)[2][G::TB] = smem + (SHARED ? wave * NST : 0);
  unsigned char* const own = own_v[SHARED ? 0 : wave];
  const unsigned lds0 = (unsigned)__builtin_amdgcn_readfirstlane((int)lds_address(ring)), lds_s = lds_address(stats[wave]);
  const bool ragged = (T & 31) != 0;
  const int k0 = live ? 32 * kt : 0, kj = 32 * kt + (lane & 31);
  const float c = a.scale * LOG2E;
  const float ninv_c = -1.0f / c;
  // lanes 0..31 fetch the row statistic of query l of each tile, lanes 32..63 its D
  const float* stat_src = (hh == 0 ? a.lse : a.dsum) + (long)p * a.T;
  const int q_first = CAUSAL ? SHARED ? kt : AT_WAVES * blk : 0;                 // query tiles the workgroup streams: q_first .. nt - 1
  const int own_first = CAUSAL ? kt : 0;                           // ... and the first one this wavefront's keys are seen by
  const PairCopy<DHP> pc(ldb, ldw, dh8, wave, lane);
  // the i-th pair of the ring: query tile q_first + i, this wavefront's share of its copies, or (SHARED) the wavefront's i-th
  // query tile, whole; and the statistics
  const int n_ring = SHARED ? every_fourth(nt - q_first, wave) : nt - q_first;
  auto tile_of = [&](int i) __attribute__((always_inline)) { return q_first + (SHARED ? wave + AT_WAVES * i : i); };
  auto issue = [&](int i) __attribute__((always_inline)) {
    const int qt = tile_of(i), q0 = 32 * qt, b = i % NST;
    const int left = ragged && qt == nt - 1 ? T - q0 : 32;
    const unsigned char* qb = hd.q + (long)q0 * ldb;
    const unsigned char* db = dob + (long)q0 * ldw;
    const unsigned dst = lds0 + (unsigned)b * (2u * G::TB);
    if (SHARED) {
      copy_tile<DHP>(qb, ldb, left, dh8, dst, lane);
      copy_tile<DHP>(db, ldw, left, dh8, dst + G::TB, lane);
    } else {
      pc.issue(qb, db, ldb, ldw, left, dh8, dst, wave, lane);
    }
    const int r = (lane & 31) < left ? (lane & 31) : left - 1;
    copy4_to_lds(stat_src + q0 + r, lds_s + (unsigned)b * 256u);
  };
  // The wavefront's own v tile stays in LDS for the whole loop (copied before the ring's first tiles, so it has landed
  // when the first of those has), its own k tile in registers: LDS and registers then both leave room for three
  // workgroups on a compute unit (heads of up to 64 columns).
  // (SHARED: one v tile for the four, copied by the first of them; they meet once it has landed)
  if (!SHARED || wave == 0) {
    copy_tile<DHP>(hd.v + (long)k0 * ldb, ldb, T - k0, dh8, lds_address(own), lane);
    if (PAD) {          // the v tile is an operand that is contracted along its columns: zeros past the head's width
      copies_in_flight<0>();
      asm volatile("" ::: "memory");
      for (int i = lane; i < 32 * (G::CPR - dh8); i += 64) {
        const int r = i / (G::CPR - dh8), ch = dh8 + i % (G::CPR - dh8);
        *reinterpret_cast<uint4*>(own + r * G::RB + ((ch ^ G::swz(r)) << 4)) = make_uint4(0u, 0u, 0u, 0u);
      }
      __builtin_amdgcn_wave_barrier();
    }
  }
  for (int i = 0; i < NST - 1 && i < n_ring; ++i) issue(i);
  bf16x8 fk[G::KK];
#pragma unroll
  for (int kk = 0; kk < G::KK; ++kk) fk[kk] = own_cols_mem(hd.k + (long)k0 * ldb, ldb, T - k0, kk, dh8, lane);
#pragma unroll
  for (int kk = 0; kk < G::KK; ++kk) landed(fk[kk]);
  if (SHARED) {
    copies_in_flight_read<0>();
    workgroup_handover();
  }
  float16v dk[G::MB], dv[G::MB];
  zero_acc(dk);
  zero_acc(dv);
  // one tile of 32 queries; MASKED: the tile on the diagonal (causal) or the one that runs past the last query
  auto step = [&](int i, auto masked_c) __attribute__((always_inline)) {
    constexpr bool MASKED = decltype(masked_c)::value;
    const int q0 = 32 * tile_of(i), b = i % NST;
    const unsigned char* tq = ring[b][0];
    const unsigned char* td = ring[b][1];
    const float* st = stats[wave][b];
    float16v s, dp;
#pragma unroll
    for (int g = 0; g < 4; ++g) {       // the statistics of the lane's 16 queries: rows 8 g + 4 hh .. + 3
      const float4 d4 = *reinterpret_cast<const float4*>(st + 32 + 8 * g + 4 * hh);
      // the products start from -L2 / c and -D: they come out as (s c - L2) / c and dP - D (EXACT: s, without the roundings of
      // the sum at the height of L2 / c)
      float4 a4 = make_float4(0.f, 0.f, 0.f, 0.f);
      if (!EXACT) a4 = *reinterpret_cast<const float4*>(st + 8 * g + 4 * hh);
      s[4 * g] = a4.x * ninv_c; s[4 * g + 1] = a4.y * ninv_c; s[4 * g + 2] = a4.z * ninv_c; s[4 * g + 3] = a4.w * ninv_c;
      dp[4 * g] = -d4.x; dp[4 * g + 1] = -d4.y; dp[4 * g + 2] = -d4.z; dp[4 * g + 3] = -d4.w;
    }
#pragma unroll
    for (int kk = 0; kk < G::KK; ++kk) {
      s = mfma(frag_cols_lds<DHP>(tq, kk, lane), fk[kk], s);
      dp = mfma(frag_cols_lds<DHP>(td, kk, lane), frag_cols_lds<DHP>(own, kk, lane), dp);
    }
    __builtin_amdgcn_sched_barrier(0);   // (keeps the second products' operand reads below: fewer live registers)
    float pr[16], ds[16];
    float4 l4 = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      if (EXACT && r % 4 == 0) l4 = *reinterpret_cast<const float4*>(st + tile_row_of(r, hh));
      const float L2r = r % 4 == 0 ? l4.x : r % 4 == 1 ? l4.y : r % 4 == 2 ? l4.z : l4.w;
      pr[r] = fast_exp2(EXACT ? fmaf(s[r], c, -L2r) : s[r] * c);
      if (MASKED) {
        const int qi = q0 + tile_row_of(r, hh);
        if (!(qi < T && (!CAUSAL || kj <= qi))) pr[r] = 0.f;
      }
      ds[r] = pr[r] * dp[r];
    }
    const Scores<EXACT> ps(pr), ss(ds);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int mb = 0; mb < G::MB; ++mb)
#pragma unroll
      for (int t = 0; t < 2; ++t) dv[mb] = ps.times(frag_rows_lds<DHP>(td, mb, t, lane), t, dv[mb]);
#pragma unroll
    for (int mb = 0; mb < G::MB; ++mb)
#pragma unroll
      for (int t = 0; t < 2; ++t) dk[mb] = ss.times(frag_rows_lds<DHP>(tq, mb, t, lane), t, dk[mb]);
  };
  auto advance = [&](int i) __attribute__((always_inline)) {
    if (SHARED) {
      if (i + NST - 2 < n_ring) copies_in_flight_read<(2 * G::COPIES + 1) * (NST - 2)>();
      else copies_in_flight_read<0>();
    } else {
      if (i + NST - 2 < n_ring) copies_in_flight<(G::PW + 1) * (NST - 2)>();
      else copies_in_flight<0>();
      workgroup_handover();
    }
    if (i + NST - 1 < n_ring) issue(i + NST - 1);
  };
  // (causal) the tiles streamed for the workgroup's earlier keys only, the tile on the diagonal, whole tiles, a ragged last one
  int i = 0;
  const int skip = SHARED ? 0 : live ? own_first - q_first : n_ring;
  for (; i < skip; ++i) advance(i);
  if (CAUSAL && (!SHARED || wave == 0) && i < n_ring) { advance(i); step(i, std::true_type()); ++i; }
  const bool ragged_own = ragged && (!SHARED || (nt - 1 - q_first) % AT_WAVES == wave);
  const int plain_end = ragged_own ? n_ring - 1 : n_ring;
  for (; i < plain_end; ++i) { advance(i); step(i, std::false_type()); }
  if (i < n_ring) { advance(i); step(i, std::true_type()); }
  if (SHARED) {
    __syncthreads();                                               // everyone has left the rings
    const float ones[AT_WAVES] = {1.f, 1.f, 1.f, 1.f};
    meet_sums(dk, reinterpret_cast<float*>(smem), wave, lane, ones);
    __syncthreads();
    meet_sums(dv, reinterpret_cast<float*>(smem), wave, lane, ones);
  }
  if (SHARED ? wave == 0 : live) {                                 // (the own v tile has served)
    bf16_t* first = reinterpret_cast<bf16_t*>(reinterpret_cast<unsigned char*>(a.dqkv) + (hd.k - reinterpret_cast<const unsigned char*>(a.qkv))) +
                    (long)k0 * hd.ld;
    store_tile(first, hd.ld, T - k0, dk, a.scale, dh, own, lane);
    store_tile(first + hd.d, hd.ld, T - k0, dv, 1.f, dh, own, lane);
    if (EXACT)
      redo_rows(not_finite(dv, not_finite(dk, 0.f)), T - k0,
                [&](int r) { redo_kv(a, hd, p, k0 + r, [&](int i) { return a.dsum[(long)p * a.T + i]; }, lane); });
  }
}

// Backward of a whole (sequence, head) problem of at most 128 TPW positions in ONE workgroup of four wavefronts, TPW tiles of
// 32 positions each (wavefront w: tiles w and, with two, 7 - w).  First the k and v tiles of the problem are in LDS and
// every wavefront takes its positions as queries (q, do and the row sums of do (.) o straight from memory): dq over the key
// tiles they see.  Then the q and do fragments, still in registers, replace k and v in LDS, the wavefront's own k and v
// rows having been read out, and the positions are taken as keys: dk, dv over the query tiles that see them.  Under a
// causal mask that is w + 1 + 8 - w steps either way: every wavefront has the same number.  Nothing is streamed, each
// tensor is read from memory once, and the arithmetic is that of the two-kernel form, in the same order per output
// element.  What bounds it is memory (80 flop per byte at 256 positions): the problem's 74 KB of LDS (64 columns) let two workgroups
// share a compute unit, so that one's loads run under the other's products.  All four tensors in LDS (130 KB, one
// workgroup of eight wavefronts) took 531 us for 12 layers of 512 problems of 256, this form 472,
// and 406 with the results leaving through LDS (store_tile).
template <int DHP, bool PAD, bool CAUSAL, int TPW>
__global__ __launch_bounds__(256, DHP == 128 ? 1 : 2) void attn_bwd_short_mfma_kernel(AttnArgs a) {
  typedef Geo<DHP> G;
  constexpr bool EXACT = exact_scores<DHP, PAD>();
  constexpr int NT = 4 * TPW;
  __shared__ __attribute__((aligned(1024))) unsigned char tiles[2][NT][G::TB];  // [k | v], then [q | do]
  __shared__ __attribute__((aligned(256))) float stats[NT][64];                 // per tile: L2 of its 32 queries, then D
  __shared__ __attribute__((aligned(256))) unsigned char staging[4][2048];      // [wave]: results on their way out
  const int lane = threadIdx.x & 63, hh = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int T = (int)a.T, nt = (T + 31) >> 5;
  const bool ragged = (T & 31) != 0;
  const unsigned p = blockIdx.x;
  const Head hd = head_of(a, p);
  const unsigned ldb = (unsigned)(hd.ld * 2), ldw = (unsigned)(hd.d * 2);
  const int dh = PAD ? a.dh : DHP, dh8 = dh >> 3;
  const unsigned char* dob = reinterpret_cast<const unsigned char*>(a.dout) + hd.wide_off;
  const unsigned char* ob = reinterpret_cast<const unsigned char*>(a.o) + hd.wide_off;
  const float c = a.scale * LOG2E;
  // 1. the wavefront's k and v tiles (rows past the end repeat the last one), its q and do rows and their statistics
  int tile[TPW];
#pragma unroll
  for (int i = 0; i < TPW; ++i) {
    tile[i] = i ? NT - 1 - wave : wave;
    if (tile[i] < nt) {
      const int r0 = 32 * tile[i];
      copy_tile<DHP>(hd.k + (long)r0 * ldb, ldb, T - r0, dh8, lds_address(tiles[0][tile[i]]), lane);
      copy_tile<DHP>(hd.v + (long)r0 * ldb, ldb, T - r0, dh8, lds_address(tiles[1][tile[i]]), lane);
    }
  }
  bf16x8 fq[TPW][G::KK], fdo[TPW][G::KK];
  float L2[TPW], D[TPW];
#pragma unroll
  for (int i = 0; i < TPW; ++i) {
    const int r0 = tile[i] < nt ? 32 * tile[i] : 0;        // (a spare tile repeats tile 0's loads and keeps nothing)
    const int ri = 32 * tile[i] + (lane & 31);
    L2[i] = a.lse[(long)p * a.T + (ri < T ? ri : T - 1)];
    D[i] = 0.f;
#pragma unroll
    for (int kk = 0; kk < G::KK; ++kk) {
      fq[i][kk] = own_cols_mem(hd.q + (long)r0 * ldb, ldb, T - r0, kk, dh8, lane);
      fdo[i][kk] = own_cols_mem(dob + (long)r0 * ldw, ldw, T - r0, kk, dh8, lane);
      D[i] += dot8(fdo[i][kk], own_cols_mem(ob + (long)r0 * ldw, ldw, T - r0, kk, dh8, lane));
    }
    D[i] += __shfl_xor(D[i], 32, 64);
    if (hh == 0) { stats[tile[i]][lane] = L2[i]; stats[tile[i]][32 + lane] = D[i]; }
  }
  copies_in_flight<0>();
  __builtin_amdgcn_s_waitcnt(0xC07F);                      // (lgkmcnt(0): the statistics are written)
  workgroup_handover();
  // 2. the positions as queries: dq
#pragma unroll
  for (int i = 0; i < TPW; ++i) {
    if (tile[i] >= nt) continue;
    const int ri = 32 * tile[i] + (lane & 31);             // this lane's position
    float16v dq[G::MB];
    zero_acc(dq);
    auto step = [&](int kt, auto masked_c) __attribute__((always_inline)) {
      constexpr bool MASKED = decltype(masked_c)::value;
      const unsigned char* tk = tiles[0][kt];
      const unsigned char* tv = tiles[1][kt];
      float16v s, dp;
#pragma unroll
      for (int r = 0; r < 16; ++r) { s[r] = 0.f; dp[r] = -D[i]; }      // dp comes out as dP - D
      bf16x8 fk[G::KK], fv[G::KK];
#pragma unroll
      for (int kk = 0; kk < G::KK; ++kk) { fk[kk] = frag_cols_lds<DHP>(tk, kk, lane); fv[kk] = frag_cols_lds<DHP>(tv, kk, lane); }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int kk = 0; kk < G::KK; ++kk) {
        s = mfma(fk[kk], fq[i][kk], s);
        dp = mfma(fv[kk], fdo[i][kk], dp);
      }
      bf16x8 kr[G::MB][2];
#pragma unroll
      for (int mb = 0; mb < G::MB; ++mb)
#pragma unroll
        for (int u = 0; u < 2; ++u) kr[mb][u] = frag_rows_lds<DHP>(tk, mb, u, lane);
      __builtin_amdgcn_sched_barrier(0);
      float ds[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        float pr = fast_exp2(fmaf(s[r], c, -L2[i]));
        if (MASKED) {
          const int kj = 32 * kt + tile_row_of(r, hh);
          if (!(CAUSAL ? kj <= ri : kj < T)) pr = 0.f;
        }
        ds[r] = pr * dp[r];
      }
      const Scores<EXACT> ss(ds);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int mb = 0; mb < G::MB; ++mb) dq[mb] = ss.times(kr[mb][u], u, dq[mb]);
    };
    const int n_own = CAUSAL ? tile[i] + 1 : nt;
    const int n_plain = CAUSAL ? n_own - 1 : (ragged ? n_own - 1 : n_own);
    int kt = 0;
    for (; kt < n_plain; ++kt) step(kt, std::false_type());
    if (kt < n_own) step(kt, std::true_type());
    store_tile(reinterpret_cast<bf16_t*>(reinterpret_cast<unsigned char*>(a.dqkv) + (hd.q - reinterpret_cast<const unsigned char*>(a.qkv))) +
                   (long)(32 * tile[i]) * hd.ld, hd.ld, T - 32 * tile[i], dq, a.scale, dh, staging[wave], lane);
    if (EXACT)
      redo_rows(not_finite(dq, 0.f), T - 32 * tile[i],
                [&](int r) { redo_q(a, hd, p, 32 * tile[i] + r, __shfl(D[i], r, 64), lane); });
  }
  // 3. own k and v rows out of LDS, q and do rows into it
  bf16x8 fk[TPW][G::KK], fv[TPW][G::KK];
#pragma unroll
  for (int i = 0; i < TPW; ++i)
#pragma unroll
    for (int kk = 0; kk < G::KK; ++kk) {                   // (a spare tile's slots hold nothing and are not used)
      fk[i][kk] = own_cols_lds<DHP>(tiles[0][tile[i]], kk, dh8, lane);
      fv[i][kk] = own_cols_lds<DHP>(tiles[1][tile[i]], kk, dh8, lane);
    }
  __builtin_amdgcn_s_waitcnt(0xC07F);
  workgroup_handover();
#pragma unroll
  for (int i = 0; i < TPW; ++i)
#pragma unroll
    for (int kk = 0; kk < G::KK; ++kk) {
      put_cols_lds<DHP>(tiles[0][tile[i]], kk, lane, fq[i][kk]);
      put_cols_lds<DHP>(tiles[1][tile[i]], kk, lane, fdo[i][kk]);
    }
  __builtin_amdgcn_s_waitcnt(0xC07F);
  workgroup_handover();
  // 4. the positions as keys: dk, dv
#pragma unroll
  for (int i = 0; i < TPW; ++i) {
    if (tile[i] >= nt) continue;
    const int ri = 32 * tile[i] + (lane & 31);
    float16v dk[G::MB], dv[G::MB];
    zero_acc(dk);
    zero_acc(dv);
    const float ninv_c = -1.0f / c;
    auto step = [&](int qt, auto masked_c) __attribute__((always_inline)) {
      constexpr bool MASKED = decltype(masked_c)::value;
      const unsigned char* tq = tiles[0][qt];
      const unsigned char* td = tiles[1][qt];
      const float* st = stats[qt];
      float16v s, dp;
#pragma unroll
      for (int g = 0; g < 4; ++g) {       // the statistics of the lane's 16 queries: rows 8 g + 4 hh .. + 3
        const float4 d4 = *reinterpret_cast<const float4*>(st + 32 + 8 * g + 4 * hh);
        // the products start from -L2 / c and -D: they come out as (s c - L2) / c and dP - D (EXACT: s)
        float4 a4 = make_float4(0.f, 0.f, 0.f, 0.f);
        if (!EXACT) a4 = *reinterpret_cast<const float4*>(st + 8 * g + 4 * hh);
        s[4 * g] = a4.x * ninv_c; s[4 * g + 1] = a4.y * ninv_c; s[4 * g + 2] = a4.z * ninv_c; s[4 * g + 3] = a4.w * ninv_c;
        dp[4 * g] = -d4.x; dp[4 * g + 1] = -d4.y; dp[4 * g + 2] = -d4.z; dp[4 * g + 3] = -d4.w;
      }
      bf16x8 fqs[G::KK], fds[G::KK];
#pragma unroll
      for (int kk = 0; kk < G::KK; ++kk) { fqs[kk] = frag_cols_lds<DHP>(tq, kk, lane); fds[kk] = frag_cols_lds<DHP>(td, kk, lane); }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int kk = 0; kk < G::KK; ++kk) {
        s = mfma(fqs[kk], fk[i][kk], s);
        dp = mfma(fds[kk], fv[i][kk], dp);
      }
      bf16x8 tr[G::MB][2], ur[G::MB][2];
#pragma unroll
      for (int mb = 0; mb < G::MB; ++mb)
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          tr[mb][u] = frag_rows_lds<DHP>(td, mb, u, lane);
          if (!EXACT) ur[mb][u] = frag_rows_lds<DHP>(tq, mb, u, lane);
        }
      __builtin_amdgcn_sched_barrier(0);
      float pr[16], ds[16];
      float4 l4 = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        if (EXACT && r % 4 == 0) l4 = *reinterpret_cast<const float4*>(st + tile_row_of(r, hh));
        const float L2r = r % 4 == 0 ? l4.x : r % 4 == 1 ? l4.y : r % 4 == 2 ? l4.z : l4.w;
        pr[r] = fast_exp2(EXACT ? fmaf(s[r], c, -L2r) : s[r] * c);
        if (MASKED) {
          const int qi = 32 * qt + tile_row_of(r, hh);
          if (!(qi < T && (!CAUSAL || ri <= qi))) pr[r] = 0.f;
        }
        ds[r] = pr[r] * dp[r];
      }
      const Scores<EXACT> ps(pr);
      if (!EXACT) {
        const Scores<EXACT> ss(ds);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int mb = 0; mb < G::MB; ++mb) { dv[mb] = ps.times(tr[mb][u], u, dv[mb]); dk[mb] = ss.times(ur[mb][u], u, dk[mb]); }
      } else {                           // (one after the other: fewer live registers)
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int mb = 0; mb < G::MB; ++mb)
#pragma unroll
          for (int u = 0; u < 2; ++u) ur[mb][u] = frag_rows_lds<DHP>(tq, mb, u, lane);
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int mb = 0; mb < G::MB; ++mb) dv[mb] = ps.times(tr[mb][u], u, dv[mb]);
        __builtin_amdgcn_sched_barrier(0);
        const Scores<EXACT> ss(ds);
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int mb = 0; mb < G::MB; ++mb) dk[mb] = ss.times(ur[mb][u], u, dk[mb]);
      }
    };
    int qt = CAUSAL ? tile[i] : 0;
    if (CAUSAL) { step(qt, std::true_type()); ++qt; }
    const int plain_end = ragged ? nt - 1 : nt;
    for (; qt < plain_end; ++qt) step(qt, std::false_type());
    if (qt < nt) step(qt, std::true_type());
    bf16_t* first = reinterpret_cast<bf16_t*>(reinterpret_cast<unsigned char*>(a.dqkv) + (hd.k - reinterpret_cast<const unsigned char*>(a.qkv))) +
                    (long)(32 * tile[i]) * hd.ld;
    store_tile(first, hd.ld, T - 32 * tile[i], dk, a.scale, dh, staging[wave], lane);
    store_tile(first + hd.d, hd.ld, T - 32 * tile[i], dv, 1.f, dh, staging[wave], lane);
    if (EXACT)
      redo_rows(not_finite(dv, not_finite(dk, 0.f)), T - 32 * tile[i],
                [&](int r) { redo_kv(a, hd, p, 32 * tile[i] + r, [&](int n) { return stats[n >> 5][32 + (n & 31)]; }, lane); });
  }
}

inline bool use_mfma(int dtype, const AttnArgs& a) { return dtype == 1 && a.dh <= 128; }

// The form with shared tiles: one workgroup per compute unit at most (of 104 to 138 KB of LDS), or, where two fit (32 columns) or a
// mask makes half of them short, two; from four tiles a sequence on.  us, forward / dq / dk, dv (or both of them in one kernel, up to
// 256 positions), heads x columns, sequences of positions, the form before -> this one: 2 x 32, 1 of 1024 25 / 22 / 33 -> 11 / 11 / 15;
// 2 x 32, 8 of 1024 27 / 25 / 35 -> 17 / 16 / 20; 4 x 64, 1 of 1024 24 / 20 / 29 -> 13 / 13 / 16; 2 x 128, 2 of 1024, causal, 41 / 43 / 68
// -> 19 / 21 / 27; 8 x 128, 4 of 435, causal, 20 / 23 / 36 -> 17 / 20 / 25; 8 x 64, 4 of 512, causal, 15 / 14 / 18 -> 12 / 14 / 15; 4 x 64,
// 8 of 256, causal, 11 / 19 -> 7 / 15; 8 x 32, 4 of 256 9 / 26 -> 7 / 14.  Beyond: 8 x 64, 2 of 600 16 / 15 / 19 -> 16 / 17 / 21, 4 x 64, 4 of
// 1024 25 / 21 / 29 -> 24 / 22 / 30, 8 of 1024 26 / 24 / 32 -> 43 / 42 / 58; T = 128: 6.3 / 9.5 -> 5.5 / 12, T = 64: 5.0 -> 5.5.
inline bool shares_tiles(const AttnArgs& a, bool two) {
  const long nt = (a.T + 31) / 32;
  return nt >= 4 && a.seqs * a.heads * nt <= (two ? 512 : 256);
}
template <int DHP, bool PAD, bool CAUSAL>
hipError_t launch_fwd(const AttnArgs& a, hipStream_t s) {
  AttnArgs m = a;
  if (shares_tiles(a, DHP == 32 || CAUSAL)) {
    hipLaunchKernelGGL((attn_fwd_mfma_kernel<DHP, PAD, CAUSAL, true>), dim3((unsigned)attn_grid(a, true)), dim3(64 * AT_WAVES), 0, s, m);
    return hipGetLastError();
  }
  m.by_problem = attn_grid(a) >= BY_PROBLEM_FROM;
  hipLaunchKernelGGL((attn_fwd_mfma_kernel<DHP, PAD, CAUSAL, false>), dim3((unsigned)attn_grid(a)), dim3(64 * AT_WAVES), 0, s, m);
  return hipGetLastError();
}
// sequences whose tiles two workgroups' LDS holds: a whole problem per workgroup
template <int DHP> constexpr long short_T() { return DHP == 128 ? 128 : 256; }
template <int DHP, bool PAD, bool CAUSAL>
hipError_t launch_bwd(const AttnArgs& a, hipStream_t s) {
  const bool is_short = a.T <= short_T<DHP>();
  const bool shared = (!is_short || a.T > 128) && shares_tiles(a, DHP == 32 || (CAUSAL && !is_short));
  if (is_short && !shared) {
    const long P = a.seqs * a.heads;
    if (P > 0x7fffffffL) return hipErrorInvalidValue;
    const dim3 grid((unsigned)P);
    if (a.T <= 128) {
      hipLaunchKernelGGL((attn_bwd_short_mfma_kernel<DHP, PAD, CAUSAL, 1>), grid, dim3(256), 0, s, a);
    } else {
      if constexpr (DHP < 128) hipLaunchKernelGGL((attn_bwd_short_mfma_kernel<DHP, PAD, CAUSAL, 2>), grid, dim3(256), 0, s, a);
    }
    return hipGetLastError();
  }
  const dim3 block(64 * AT_WAVES);
  if (shared) {
    const dim3 grid((unsigned)attn_grid(a, true));
    hipLaunchKernelGGL((attn_bwd_q_mfma_kernel<DHP, PAD, CAUSAL, true>), grid, block, 0, s, a);
    hipLaunchKernelGGL((attn_bwd_kv_mfma_kernel<DHP, PAD, CAUSAL, true>), grid, block, 0, s, a);
    return hipGetLastError();
  }
  const dim3 grid((unsigned)attn_grid(a));
  // dq is bound by its tile stream and gains from one XCD per problem; dk/dv is bound by its arithmetic and by the
  // tail, and keeps the longest-first order (by_problem = 0 as the caller leaves it)
  AttnArgs m = a;
  m.by_problem = attn_grid(a) >= BY_PROBLEM_FROM;
  hipLaunchKernelGGL((attn_bwd_q_mfma_kernel<DHP, PAD, CAUSAL, false>), grid, block, 0, s, m);
  hipLaunchKernelGGL((attn_bwd_kv_mfma_kernel<DHP, PAD, CAUSAL, false>), grid, block, 0, s, a);
  return hipGetLastError();
}

template <int DHP>
hipError_t pick_fwd(const AttnArgs& a, hipStream_t s) {
  if (a.dh == DHP) return a.causal ? launch_fwd<DHP, false, true>(a, s) : launch_fwd<DHP, false, false>(a, s);
  return a.causal ? launch_fwd<DHP, true, true>(a, s) : launch_fwd<DHP, true, false>(a, s);
}
template <int DHP>
hipError_t pick_bwd(const AttnArgs& a, hipStream_t s) {
  if (a.dh == DHP) return a.causal ? launch_bwd<DHP, false, true>(a, s) : launch_bwd<DHP, false, false>(a, s);
  return a.causal ? launch_bwd<DHP, true, true>(a, s) : launch_bwd<DHP, true, false>(a, s);
}

}  // namespace

// the plain kernels hold a row (two rows) of T floats in LDS; the limit is the same for every width but 64
bool attn_supported(int dtype, long T, int dh) {
  if (dtype == 1 && dh == 64) return T <= (1L << 20);
  return T <= 8192;
}

hipError_t launch_attn_fwd(int dtype, const AttnArgs& a, hipStream_t s) {
  const long P = a.seqs * a.heads;
  if (use_mfma(dtype, a)) {
    if (attn_grid(a) > 0x7fffffffL) return hipErrorInvalidValue;
    if (a.dh <= 32) return pick_fwd<32>(a, s);
    if (a.dh <= 64) return pick_fwd<64>(a, s);
    return pick_fwd<128>(a, s);
  }
  const dim3 grid((unsigned)P, (unsigned)a.T), block(64);
  const size_t lds = (size_t)a.T * 4;
  if (dtype == 0) hipLaunchKernelGGL(attn_fwd_plain_kernel<float>, grid, block, lds, s, a);
  else hipLaunchKernelGGL(attn_fwd_plain_kernel<bf16_t>, grid, block, lds, s, a);
  return hipGetLastError();
}

hipError_t launch_attn_bwd(int dtype, const AttnArgs& a, hipStream_t s) {
  const long P = a.seqs * a.heads;
  if (use_mfma(dtype, a)) {
    if (attn_grid(a) > 0x7fffffffL) return hipErrorInvalidValue;
    if (a.dh <= 32) return pick_bwd<32>(a, s);
    if (a.dh <= 64) return pick_bwd<64>(a, s);
    return pick_bwd<128>(a, s);
  }
  const dim3 grid((unsigned)P, (unsigned)a.T), block(64);
  if (dtype == 0) {
    hipLaunchKernelGGL(attn_bwd_q_plain_kernel<float>, grid, block, (size_t)a.T * 4, s, a);
    hipLaunchKernelGGL(attn_bwd_kv_plain_kernel<float>, grid, block, (size_t)a.T * 8, s, a);
  } else {
    hipLaunchKernelGGL(attn_bwd_q_plain_kernel<bf16_t>, grid, block, (size_t)a.T * 4, s, a);
    hipLaunchKernelGGL(attn_bwd_kv_plain_kernel<bf16_t>, grid, block, (size_t)a.T * 8, s, a);
  }
  return hipGetLastError();
}

}  // namespace hbp
