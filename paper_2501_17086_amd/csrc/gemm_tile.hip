// bf16 GEMM on the matrix cores for the shapes the 256 x 256 kernel does not serve well: sizes that are no multiple of
// its tile, few output tiles, and every epilogue it does not have.
//
//   workgroup   256 threads (2 x 2 wavefronts), one output tile of 128 x 128 or 64 x 64; two or three workgroups share a
//               compute unit (64 or 48 KB of LDS each), so that one's epilogue and fill run under the others' products.
//               (Launches that leave compute units without a tile: gemm_small_kernel below, 64 x 32 or 32 x 32.)
//   K pipeline  slices of 32 or 64 of both operands go global -> LDS directly through a ring of three or four stages of
//               16 KB (128-wide tiles in slices of 64: 32 KB), two or three slices ahead; one counted wait and one barrier
//               per slice.
//   edges       a lane's source row (or its chunk of 8 rows) is clamped to the matrix once per tile, so the main loop is
//               the same for every tile; what such lanes produce is never stored.  Only a last, partial slice of
//               the contraction is special: its chunks past the end are copied from a zero-filled device array.
//   layouts     as in gemm_mfma.hip: KC (contraction contiguous, 16-byte LDS reads) and RC (rows contiguous,
//               ds_read_b64_tr_b16), the 64 banks spread by an XOR of the 16-byte chunk index on both sides.
//   epilogue    32 rows of a wavefront's block at a time through LDS as fp32, so that every global access (aux, old
//               state, results) covers consecutive 16-byte pieces of a row; all modes, each access guarded.
#include "gemm_device.h"

namespace hbp {

namespace {

constexpr int NTHR = 256;

// One operand tile of T rows x BK of the contraction in LDS, copied by NW wavefronts.
template <int T, int BK, bool KC, int NW = 4>
struct Tile {
  static constexpr int BYTES = T * BK * 2;
  static constexpr int COPIES = BYTES / 1024 / NW;               // per wavefront and slice, 1 KB each
  static constexpr int CPR = KC ? BK / 8 : T / 8;                // 16-byte chunks per LDS row
  // the XOR on the chunk index of LDS row r (KC: a matrix row; RC: a contraction index)
  static __device__ __forceinline__ int swz(int r) {
    if (KC) return BK == 32 ? (r >> 2) & 3 : (r >> 1) & 7;
    return T == 128 ? 4 * (r & 3) : T == 64 ? 4 * ((r >> 1) & 1) : 0;   // (32: four rows are the 64 banks)
  }
  // LDS row and logical chunk of this lane's 16 bytes of copy i
  static __device__ __forceinline__ int lane_row(int i, int wave, int lane) { return (wave + NW * i) * (64 / CPR) + lane / CPR; }
  static __device__ __forceinline__ int lane_chunk(int i, int wave, int lane) {
    return (lane % CPR) ^ swz(lane_row(i, wave, lane));
  }
  // byte offset from the tile's first element at the slice's first contraction index; rows_left > 0 rows are there
  static __device__ __forceinline__ unsigned source(long ld, long rows_left, int i, int wave, int lane) {
    const int r = lane_row(i, wave, lane), c = lane_chunk(i, wave, lane);
    if (KC) return (unsigned)((r < rows_left ? r : rows_left - 1) * ld + 8 * c) * 2u;
    return (unsigned)(r * ld + (8 * c < rows_left ? 8 * c : rows_left - 8)) * 2u;
  }
  // is this lane's chunk of a slice that has k_left < BK contraction indices inside?
  static __device__ __forceinline__ bool in_tail(long k_left, int i, int wave, int lane) {
    return (KC ? 8 * lane_chunk(i, wave, lane) : lane_row(i, wave, lane)) < k_left;
  }
  // 32 rows x 16 k fragment: lane l holds row row0 + l % 32, k = kk + 8 (l / 32) .. + 7
  static __device__ __forceinline__ bf16x8 frag(const unsigned char* tile, int row0, int kk, int lane) {
    if (KC) {
      const int r = row0 + (lane & 31);
      const int c = (kk >> 3) + (lane >> 5);
      return __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(tile + r * (2 * BK) + ((c ^ swz(r)) << 4)));
    }
    typedef __attribute__((address_space(3))) short4v* lds_p;
    const int s = lane & 15;
    const int e = row0 + 16 * ((lane >> 4) & 1) + 4 * (s & 3);
    const int k = kk + 8 * (lane >> 5) + (s >> 2);               // (swz(k + 4) == swz(k))
    const unsigned char* p = tile + k * (2 * T) + (((e >> 3) ^ swz(k)) << 4) + (e & 7) * 2;
    const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_p)(p));
    const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_p)(p + 8 * T));
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  }
};

__device__ __forceinline__ bool fuses_aux(const GemmArgs& g) {
  return g.split_k == 1 && (g.mode == EPI_MUL_AUX || g.mode == EPI_MUL_1MZ2 || g.mode == EPI_RESID || g.mode == EPI_ADD_AUX);
}
// 8 consecutive sums of a row, at element off of C: what the launch fuses, and the store.  ra: the fused operand there; lm: the
// columns' coefficients (EPI_RESID without coefficients per element).
template <bool ACT>
__device__ __forceinline__ void finish8(const GemmArgs& g, long batch, int split, long off, bool use_aux, float (&v)[8],
                                        const Raw8<bf16_t>& ra, const float (&lm)[8]) {
  if (g.split_k > 1) {
    store8(reinterpret_cast<float*>(g.C) + ((long)split * g.batch + batch) * g.c_sb + off, v);
    return;
  }
  if (g.addf) {
    float f[8];
    load8(g.addf + batch * g.addf_sb + off, f);
#pragma unroll
    for (int x = 0; x < 8; ++x) v[x] += f[x];
  }
  if (ACT) {
    if (g.mode == EPI_ACT_GELU) {
      float dz[8];
#pragma unroll
      for (int x = 0; x < 8; ++x) gelu_both(v[x], v[x], dz[x]);
      store8(reinterpret_cast<bf16_t*>(g.out2) + batch * g.out2_sb + off, dz);
    } else {
#pragma unroll
      for (int x = 0; x < 8; ++x) v[x] = tanhf(v[x]);
    }
  } else if (use_aux) {
    float f[8];
    ra.unpack(f);
    if (g.mode == EPI_MUL_AUX) {
#pragma unroll
      for (int x = 0; x < 8; ++x) v[x] *= f[x];
    } else if (g.mode == EPI_MUL_1MZ2) {
#pragma unroll
      for (int x = 0; x < 8; ++x) v[x] *= (1.f - f[x] * f[x]);
    } else if (g.mode == EPI_ADD_AUX) {
#pragma unroll
      for (int x = 0; x < 8; ++x) v[x] += f[x];
    } else {
      float l8[8];
      if (g.lambda_mn) load8(reinterpret_cast<const bf16_t*>(g.lambda_mn) + batch * g.aux_sb + off, l8);
#pragma unroll
      for (int x = 0; x < 8; ++x) v[x] = fmaf(g.lambda_mn ? l8[x] : lm[x], f[x], v[x]);
    }
  }
  if (g.c_is_f32) store8(reinterpret_cast<float*>(g.C) + batch * g.c_sb + off, v);
  else store8(reinterpret_cast<bf16_t*>(g.C) + batch * g.c_sb + off, v);
}

// T x T output tile per workgroup, a ring of NST stages, WGS workgroups per compute unit.  ACT: the forward's activations (kept
// out of the other kernels' registers).  t: the tile's number in the product's list.
template <int T, int BK, int NST, bool A_KC, bool B_KC, bool ACT>
__device__ __forceinline__ void gemm_tile_body(const GemmArgs& g, int tiles_m, int tiles_n, int t) {
  typedef Tile<T, BK, A_KC> TA;
  typedef Tile<T, BK, B_KC> TB;
  constexpr int STAGE = TA::BYTES + TB::BYTES;
  constexpr int PER = TA::COPIES + TB::COPIES;             // copies per wavefront and slice
  constexpr int W = T / 2, NB = W / 32;                    // a wavefront's block: W x W, NB x NB MFMA blocks
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm0 = (wave >> 1) * W, wn0 = (wave & 1) * W;
  const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;

  const unsigned tiles_mn = (unsigned)tiles_m * tiles_n;
  const unsigned zb = (unsigned)t / tiles_mn, rem = (unsigned)t - zb * tiles_mn;
  const unsigned gr = rem / (8u * tiles_n), in_gr = rem - gr * 8u * tiles_n;
  const unsigned left = tiles_m - gr * 8u, gm = left < 8u ? left : 8u;
  const long m0 = (long)(gr * 8u + in_gr % gm) * T, n0 = (long)(in_gr / gm) * T;
  const long batch = zb / (unsigned)g.split_k;
  const int split = (int)(zb % (unsigned)g.split_k);
  const long kchunk = ((g.K + g.split_k - 1) / g.split_k + 31) / 32 * 32;   // (32 whatever BK: the shares do not depend on the tile)
  const long k_begin = (long)split * kchunk;
  const long k_end = k_begin + kchunk < g.K ? k_begin + kchunk : g.K;
  const int KT = k_end > k_begin ? (int)((k_end - k_begin + BK - 1) / BK) : 0;

  const long lda = A_KC ? g.a_sm : g.a_sk, ldb = B_KC ? g.b_sn : g.b_sk;
  const bf16_t* pa = reinterpret_cast<const bf16_t*>(g.A) + batch * g.a_sb + (A_KC ? m0 * lda + k_begin : m0 + k_begin * lda);
  const bf16_t* pb = reinterpret_cast<const bf16_t*>(g.B) + batch * g.b_sb + (B_KC ? n0 * ldb + k_begin : n0 + k_begin * ldb);
  const long step_a = A_KC ? BK : BK * lda, step_b = B_KC ? BK : BK * ldb;
  unsigned offa[TA::COPIES], offb[TB::COPIES];
#pragma unroll
  for (int i = 0; i < TA::COPIES; ++i) offa[i] = TA::source(lda, g.M - m0, i, wave, lane);
#pragma unroll
  for (int i = 0; i < TB::COPIES; ++i) offb[i] = TB::source(ldb, g.N - n0, i, wave, lane);

  auto issue = [&](int s) __attribute__((always_inline)) {
    const unsigned dst = lds0 + (unsigned)(s % NST) * STAGE + (unsigned)wave * 1024u;
    const long k_left = k_end - k_begin - (long)s * BK;
    if (k_left >= BK) {
#pragma unroll
      for (int i = 0; i < TA::COPIES; ++i) dma16_s(offa[i], pa, dst + 4096u * i);
#pragma unroll
      for (int i = 0; i < TB::COPIES; ++i) dma16_s(offb[i], pb, dst + TA::BYTES + 4096u * i);
    } else {
#pragma unroll
      for (int i = 0; i < TA::COPIES; ++i)
        dma16(TA::in_tail(k_left, i, wave, lane) ? reinterpret_cast<const void*>(reinterpret_cast<const char*>(pa) + offa[i])
                                                 : reinterpret_cast<const void*>(g_zero_chunks + lane), dst + 4096u * i);
#pragma unroll
      for (int i = 0; i < TB::COPIES; ++i)
        dma16(TB::in_tail(k_left, i, wave, lane) ? reinterpret_cast<const void*>(reinterpret_cast<const char*>(pb) + offb[i])
                                                 : reinterpret_cast<const void*>(g_zero_chunks + lane),
              dst + TA::BYTES + 4096u * i);
    }
    pa += step_a;
    pb += step_b;
  };

  // acc[i][j]: lane l, element r  <->  row wm0 + 32 i + l % 32, column wn0 + 32 j + 8 (r / 4) + 4 (l / 32) + r % 4
  float16v acc[NB][NB];
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

#pragma unroll 1
  for (int s = 0; s < NST - 1 && s < KT; ++s) issue(s);
#pragma unroll 1
  for (int s = 0; s < KT; ++s) {
    // this wavefront's share of slice s has landed once only the copies of the slices after it are outstanding
    if (NST > 3 && s + 2 < KT) wait_vm<2 * PER>();
    else if (s + 1 < KT) wait_vm<PER>();
    else wait_vm<0>();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();            // slice s is complete; everyone has read slice s - 1
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
    if (s + NST - 1 < KT) issue(s + NST - 1);
    const unsigned char* st = smem + (s % NST) * STAGE;
    bf16x8 fa[NB][BK / 16], fb[NB][BK / 16];
#pragma unroll
    for (int h = 0; h < BK / 16; ++h) {
#pragma unroll
      for (int j = 0; j < NB; ++j) fb[j][h] = TB::frag(st + TA::BYTES, wn0 + 32 * j, 16 * h, lane);
#pragma unroll
      for (int i = 0; i < NB; ++i) fa[i][h] = TA::frag(st, wm0 + 32 * i, 16 * h, lane);
    }
#pragma unroll
    for (int h = 0; h < BK / 16; ++h)
#pragma unroll
      for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[j][h], fa[i][h], acc[i][j], 0, 0, 0);
  }

  // ---- epilogue ----
  constexpr int LD = W + 4;                                // floats per staged row (16-byte aligned, banks spread)
  constexpr int LPR = W / 8, RPP = 64 / LPR, PASSES = 32 / RPP;
  static_assert(4 * 32 * LD * 4 <= NST * STAGE, "the staging area reuses the ring");
  __syncthreads();                                         // the last slice has been read by everyone
  float* stg = reinterpret_cast<float*>(smem) + wave * 32 * LD;
  const bf16_t* aux = g.aux ? reinterpret_cast<const bf16_t*>(g.aux) + batch * g.aux_sb : nullptr;
  const float* lam = g.lambda ? g.lambda + batch * g.lambda_sb : nullptr;
  const bool use_aux = fuses_aux(g);
  const long col = n0 + wn0 + 8 * (lane % LPR);
  const long col_in = col < g.N ? col : g.N - 8;           // (loads are clamped, stores guarded)
  float lm[8];
#pragma unroll
  for (int x = 0; x < 8; ++x) lm[x] = 1.f;
  if (!ACT && use_aux && lam && !g.lambda_mn) load8(lam + col_in, lm);
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    const long row0 = m0 + wm0 + 32 * i + lane / LPR;
    Raw8<bf16_t> ra[PASSES];
    if (!ACT && use_aux) {
#pragma unroll
      for (int ps = 0; ps < PASSES; ++ps) {
        const long row = row0 + ps * RPP < g.M ? row0 + ps * RPP : g.M - 1;
        ra[ps].load(aux + row * g.ldc + col_in);
      }
    }
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        *reinterpret_cast<float4*>(stg + (lane & 31) * LD + 32 * j + 8 * q + 4 * (lane >> 5)) =
            make_float4(acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]);
    __builtin_amdgcn_wave_barrier();                       // (a wavefront's LDS operations execute in order)
#pragma unroll
    for (int ps = 0; ps < PASSES; ++ps) {
      const long row = row0 + ps * RPP;
      float v[8];
      load8(stg + (lane / LPR + ps * RPP) * LD + 8 * (lane % LPR), v);
      if (row >= g.M || col >= g.N) continue;
      finish8<ACT>(g, batch, split, row * g.ldc + col, use_aux, v, ra[ps], lm);
    }
    __builtin_amdgcn_wave_barrier();                       // the next rows' writes stay behind these reads
  }
}

// ids are dealt to the 8 XCDs in turn: each takes a contiguous eighth of the tile list, in blocks of 8 tile rows
__device__ __forceinline__ int tile_of_id(int per_xcd) { return (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3); }
template <int T, int BK, int NST, int WGS, bool A_KC, bool B_KC, bool ACT>
__global__ __launch_bounds__(NTHR, WGS) void gemm_tile_kernel(GemmArgs g, int tiles_m, int tiles_n, int total, int per_xcd) {
  const int t = tile_of_id(per_xcd);
  if (t < total) gemm_tile_body<T, BK, NST, A_KC, B_KC, ACT>(g, tiles_m, tiles_n, t);
}
// several products' tiles in one list
template <int T, int BK, int NST, int WGS, bool A_KC, bool B_KC>
__global__ __launch_bounds__(NTHR, WGS) void gemm_tile_group_kernel(GemmGroup q) {
  const int t = tile_of_id(q.per_xcd);
  if (t >= q.total) return;
  const int i = q.of(t);
  gemm_tile_body<T, BK, NST, A_KC, B_KC, false>(q.g[i], q.tiles_m[i], q.tiles_n[i], t - q.start[i]);
}

// Launches of few tiles: a workgroup of four wavefronts owns TM x 32 of C and the wavefronts share the contraction out, each
// taking every fourth slice of 64 through an LDS ring of its own (no barrier in the loop); the four sums meet in LDS.
// What bounds such a launch is the time a compute unit takes to stream its tile's operands, about 64 KB of requests in flight over
// their latency.  Here 96 KB are asked for ahead (the 64 x 64 kernel: 48), over more compute units: 1200 x 256 x 1024 8.3 -> 6.2
// us, 54 GB/s per compute unit.  The fused operand is asked for before the first slice.
template <int TM, int STG, bool A_KC, bool B_KC, bool ACT>
__device__ __forceinline__ void gemm_small_body(const GemmArgs& g, int tiles_m, int tiles_n, int t) {
  constexpr int TN = 32, BK = 64, NB = TM / 32;
  typedef Tile<TM, BK, A_KC, 1> TA;
  typedef Tile<TN, BK, B_KC, 1> TB;
  constexpr int STAGE = TA::BYTES + TB::BYTES;
  constexpr int PER = TA::COPIES + TB::COPIES;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  unsigned char* const ring = smem + wave * (STG * STAGE);
  const unsigned lds0 = (unsigned)__builtin_amdgcn_readfirstlane(
      (int)(unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)ring);

  const unsigned tiles_mn = (unsigned)tiles_m * tiles_n;
  const unsigned zb = (unsigned)t / tiles_mn, rem = (unsigned)t - zb * tiles_mn;
  const unsigned gr = rem / (8u * tiles_n), in_gr = rem - gr * 8u * tiles_n;
  const unsigned left = tiles_m - gr * 8u, gm = left < 8u ? left : 8u;
  const long m0 = (long)(gr * 8u + in_gr % gm) * TM, n0 = (long)(in_gr / gm) * TN;
  const long batch = zb / (unsigned)g.split_k;
  const int split = (int)(zb % (unsigned)g.split_k);
  const long kchunk = ((g.K + g.split_k - 1) / g.split_k + 31) / 32 * 32;
  const long k_begin = (long)split * kchunk;
  const long k_end = k_begin + kchunk < g.K ? k_begin + kchunk : g.K;
  const int KT = k_end > k_begin ? (int)((k_end - k_begin + BK - 1) / BK) : 0;
  const int mine = KT > wave ? (KT - wave + 3) / 4 : 0;                      // slices wave, wave + 4, ..

  // this thread's piece of the result, 8 columns of a row (TM 32: of the first 128 threads)
  const int prow = tid >> 2, pcol = 8 * (tid & 3);
  const bool writes = prow < TM && m0 + prow < g.M && n0 + pcol < g.N;
  const bool use_aux = fuses_aux(g);
  const long off = (m0 + prow) * g.ldc + n0 + pcol;
  Raw8<bf16_t> ra;
  ra.v = make_uint4(0, 0, 0, 0);
  float lm[8];
#pragma unroll
  for (int x = 0; x < 8; ++x) lm[x] = 1.f;
  if (!ACT && use_aux && writes) {
    ra.load(reinterpret_cast<const bf16_t*>(g.aux) + batch * g.aux_sb + off);
    if (g.lambda && !g.lambda_mn) load8(g.lambda + batch * g.lambda_sb + n0 + pcol, lm);
  }

  const long lda = A_KC ? g.a_sm : g.a_sk, ldb = B_KC ? g.b_sn : g.b_sk;
  const long k_mine = k_begin + (long)wave * BK;
  const bf16_t* pa = reinterpret_cast<const bf16_t*>(g.A) + batch * g.a_sb + (A_KC ? m0 * lda + k_mine : m0 + k_mine * lda);
  const bf16_t* pb = reinterpret_cast<const bf16_t*>(g.B) + batch * g.b_sb + (B_KC ? n0 * ldb + k_mine : n0 + k_mine * ldb);
  const long step_a = 4 * (A_KC ? BK : BK * lda), step_b = 4 * (B_KC ? BK : BK * ldb);
  unsigned offa[TA::COPIES], offb[TB::COPIES];
#pragma unroll
  for (int i = 0; i < TA::COPIES; ++i) offa[i] = TA::source(lda, g.M - m0, i, 0, lane);
#pragma unroll
  for (int i = 0; i < TB::COPIES; ++i) offb[i] = TB::source(ldb, g.N - n0, i, 0, lane);
  auto issue = [&](int s) __attribute__((always_inline)) {
    const unsigned dst = lds0 + (unsigned)(s % STG) * STAGE;
    const long k_left = k_end - k_mine - (long)s * (4 * BK);
    if (k_left >= BK) {
#pragma unroll
      for (int i = 0; i < TA::COPIES; ++i) dma16_s(offa[i], pa, dst + 1024u * i);
#pragma unroll
      for (int i = 0; i < TB::COPIES; ++i) dma16_s(offb[i], pb, dst + TA::BYTES + 1024u * i);
    } else {
#pragma unroll
      for (int i = 0; i < TA::COPIES; ++i)
        dma16(TA::in_tail(k_left, i, 0, lane) ? reinterpret_cast<const void*>(reinterpret_cast<const char*>(pa) + offa[i])
                                              : reinterpret_cast<const void*>(g_zero_chunks + lane), dst + 1024u * i);
#pragma unroll
      for (int i = 0; i < TB::COPIES; ++i)
        dma16(TB::in_tail(k_left, i, 0, lane) ? reinterpret_cast<const void*>(reinterpret_cast<const char*>(pb) + offb[i])
                                              : reinterpret_cast<const void*>(g_zero_chunks + lane),
              dst + TA::BYTES + 1024u * i);
    }
    pa += step_a;
    pb += step_b;
  };

  float16v acc[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[i][r] = 0.f;
#pragma unroll 1
  for (int s = 0; s < STG - 1 && s < mine; ++s) issue(s);
#pragma unroll 1
  for (int s = 0; s < mine; ++s) {
    // slice s has landed once only the copies of the slices after it are outstanding; and the reads of slice s - 1, whose
    // stage the next copies go to, have returned
    if (STG > 3 && s + 2 < mine) wait_vm_lds<2 * PER>();
    else if (s + 1 < mine) wait_vm_lds<PER>();
    else wait_vm_lds<0>();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    if (s + STG - 1 < mine) issue(s + STG - 1);
    const unsigned char* st = ring + (s % STG) * STAGE;
    bf16x8 fa[NB][4], fb[4];
#pragma unroll
    for (int h = 0; h < 4; ++h) {
      fb[h] = TB::frag(st + TA::BYTES, 0, 16 * h, lane);
#pragma unroll
      for (int i = 0; i < NB; ++i) fa[i][h] = TA::frag(st, 32 * i, 16 * h, lane);
    }
#pragma unroll
    for (int h = 0; h < 4; ++h)
#pragma unroll
      for (int i = 0; i < NB; ++i) acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[h], fa[i][h], acc[i], 0, 0, 0);
  }

  constexpr int LD = TN + 4;
  static_assert(TM * LD * 4 <= STG * STAGE, "a wavefront's sums reuse its ring");
  wait_vm_lds<0>();                                        // its last slice has been read
  asm volatile("" ::: "memory");
  float* own = reinterpret_cast<float*>(ring);
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int q = 0; q < 4; ++q)
      *reinterpret_cast<float4*>(own + (32 * i + (lane & 31)) * LD + 8 * q + 4 * (lane >> 5)) =
          make_float4(acc[i][4 * q], acc[i][4 * q + 1], acc[i][4 * q + 2], acc[i][4 * q + 3]);
  __syncthreads();
  if (!writes) return;
  float v[8];
  const float* sums = reinterpret_cast<const float*>(smem) + prow * LD + pcol;
  load8(sums, v);
#pragma unroll
  for (int w = 1; w < 4; ++w) {
    float f[8];
    load8(sums + w * (STG * STAGE / 4), f);
#pragma unroll
    for (int x = 0; x < 8; ++x) v[x] += f[x];
  }
  finish8<ACT>(g, batch, split, off, use_aux, v, ra, lm);
}

template <int TM, int STG, bool A_KC, bool B_KC, bool ACT>
__global__ __launch_bounds__(NTHR, 1) void gemm_small_kernel(GemmArgs g, int tiles_m, int tiles_n, int total, int per_xcd) {
  const int t = tile_of_id(per_xcd);
  if (t < total) gemm_small_body<TM, STG, A_KC, B_KC, ACT>(g, tiles_m, tiles_n, t);
}
template <int TM, int STG, bool A_KC, bool B_KC>
__global__ __launch_bounds__(NTHR, 1) void gemm_small_group_kernel(GemmGroup q) {
  const int t = tile_of_id(q.per_xcd);
  if (t >= q.total) return;
  const int i = q.of(t);
  gemm_small_body<TM, STG, A_KC, B_KC, false>(q.g[i], q.tiles_m[i], q.tiles_n[i], t - q.start[i]);
}

template <int T, int BK, int NST, int WGS, bool A_KC, bool B_KC, bool ACT>
hipError_t launch_one(const GemmArgs& g, hipStream_t s) {
  auto kern = gemm_tile_kernel<T, BK, NST, WGS, A_KC, B_KC, ACT>;
  constexpr int lds = NST * 2 * T * BK * 2;
  if (lds > 65536) {
    static std::atomic<bool> attr_set[MAX_DEVICES];
    const hipError_t e = raise_lds_limit(reinterpret_cast<const void*>(kern), lds, attr_set);
    if (e != hipSuccess) return e;
  }
  const long tiles_m = (g.M + T - 1) / T, tiles_n = (g.N + T - 1) / T;
  const long total = tiles_m * tiles_n * g.batch * g.split_k;
  if (total > (1L << 28)) return hipErrorInvalidValue;
  const long per_xcd = (total + 7) / 8;
  hipLaunchKernelGGL(kern, dim3((unsigned)(8 * per_xcd)), dim3(NTHR), lds, s, g, (int)tiles_m, (int)tiles_n, (int)total,
                     (int)per_xcd);
  return hipGetLastError();
}
template <int T, int BK, int NST, int WGS>
hipError_t launch_pairing(const GemmArgs& g, hipStream_t s) {
  const bool a_kc = g.a_sk == 1, b_kc = g.b_sk == 1;
  if (a_kc && b_kc)
    return g.mode == EPI_ACT_GELU || g.mode == EPI_ACT_TANH ? launch_one<T, BK, NST, WGS, true, true, true>(g, s)
                                                            : launch_one<T, BK, NST, WGS, true, true, false>(g, s);
  if (a_kc) return launch_one<T, BK, NST, WGS, true, false, false>(g, s);
  if constexpr (WGS == 3) return hipErrorInvalidValue;     // (both operands with contiguous rows: two workgroups, below)
  else return launch_one<T, BK, NST, WGS, false, false, false>(g, s);
}

template <int TM, int STG, bool A_KC, bool B_KC, bool ACT>
hipError_t launch_small_one(const GemmArgs& g, hipStream_t s) {
  static std::atomic<bool> attr_set[MAX_DEVICES];
  auto kern = gemm_small_kernel<TM, STG, A_KC, B_KC, ACT>;
  constexpr int lds = 4 * STG * (TM + 32) * 64 * 2;
  const hipError_t e = raise_lds_limit(reinterpret_cast<const void*>(kern), lds, attr_set);
  if (e != hipSuccess) return e;
  const long tiles_m = (g.M + TM - 1) / TM, tiles_n = (g.N + 31) / 32;
  const long total = tiles_m * tiles_n * g.batch * g.split_k;
  if (total > (1L << 28)) return hipErrorInvalidValue;
  const long per_xcd = (total + 7) / 8;
  hipLaunchKernelGGL(kern, dim3((unsigned)(8 * per_xcd)), dim3(NTHR), lds, s, g, (int)tiles_m, (int)tiles_n, (int)total,
                     (int)per_xcd);
  return hipGetLastError();
}
template <int TM, int STG>
hipError_t launch_small(const GemmArgs& g, hipStream_t s) {
  const bool a_kc = g.a_sk == 1, b_kc = g.b_sk == 1;
  if (a_kc && b_kc)
    return g.mode == EPI_ACT_GELU || g.mode == EPI_ACT_TANH ? launch_small_one<TM, STG, true, true, true>(g, s)
                                                            : launch_small_one<TM, STG, true, true, false>(g, s);
  return a_kc ? launch_small_one<TM, STG, true, false, false>(g, s) : launch_small_one<TM, STG, false, false, false>(g, s);
}

template <typename K>
hipError_t launch_group(K kern, int lds, std::atomic<bool> (&attr_set)[MAX_DEVICES], const GemmGroup& q, hipStream_t s) {
  if (lds > 65536) {
    const hipError_t e = raise_lds_limit(reinterpret_cast<const void*>(kern), lds, attr_set);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(kern, dim3((unsigned)(8 * q.per_xcd)), dim3(NTHR), lds, s, q);
  return hipGetLastError();
}
template <int T, int BK, int NST, int WGS>
hipError_t launch_tile_group(const GemmGroup& q, hipStream_t s) {
  static std::atomic<bool> attr_set[2][MAX_DEVICES];
  constexpr int lds = NST * 2 * T * BK * 2;
  if (q.g[0].a_sk == 1) return launch_group(gemm_tile_group_kernel<T, BK, NST, WGS, true, false>, lds, attr_set[0], q, s);
  if constexpr (WGS == 3) return hipErrorInvalidValue;
  else return launch_group(gemm_tile_group_kernel<T, BK, NST, WGS, false, false>, lds, attr_set[1], q, s);
}
template <int TM, int STG>
hipError_t launch_small_group(const GemmGroup& q, hipStream_t s) {
  static std::atomic<bool> attr_set[2][MAX_DEVICES];
  constexpr int lds = 4 * STG * (TM + 32) * 64 * 2;
  return q.g[0].a_sk == 1 ? launch_group(gemm_small_group_kernel<TM, STG, true, false>, lds, attr_set[0], q, s)
                          : launch_group(gemm_small_group_kernel<TM, STG, false, false>, lds, attr_set[1], q, s);
}

}  // namespace

// (B with contiguous rows; the lines are those of launch_gemm_tile below)
hipError_t launch_gemm_tile_group(const GemmArgs* g, int n, int tm, int tn, hipStream_t s) {
  GemmGroup q;
  if (!make_group(q, g, n, tm, tn)) return hipErrorInvalidValue;
  if (tn == 32) return tm == 32 ? launch_small_group<32, 4>(q, s) : launch_small_group<64, 3>(q, s);
  if (tm == 64) return launch_tile_group<64, 64, 4, 2>(q, s);
  if (q.total <= 256) return launch_tile_group<128, 64, 4, 1>(q, s);
  return q.total >= 512 && g[0].a_sk == 1 ? launch_tile_group<128, 32, 3, 3>(q, s) : launch_tile_group<128, 32, 4, 2>(q, s);
}
hipError_t launch_gemm_tile(const GemmArgs& g, int tm, int tn, hipStream_t s) {
  if (tn == 32) return tm == 32 ? launch_small<32, 4>(g, s) : launch_small<64, 3>(g, s);
  if (tm == 64) return launch_pairing<64, 64, 4, 2>(g, s);
  const long tiles = (g.M + 127) / 128 * ((g.N + 127) / 128) * g.batch * g.split_k;
  // One tile per compute unit at most: slices of 64, whole 128-byte lines of a K-contiguous operand, 96 KB asked for ahead.  From
  // 512 on, the first operand K-contiguous: three workgroups per compute unit on rings of three stages, whose last round is
  // shorter and whose epilogues run under two others' products.  Measured, us, two workgroups and four stages of 32 / the other:
  // 192 tiles (3000 x 1000 x 2000) 27.7 / 24.5, 256 (8192 x 512 x 2048) 27.6 / 26.5, (4096 x 1024 x 4096) 44.2 / 43.0;
  // 1000 (16000 x 1024 x 256 with GELU) 34.8 / 31.8, 1034 (12000 x 1304 x 328) 34.4 / 32.8, 512 (32768 x 256 x 1024) 36.7 / 36.0.
  // Beyond those lines: 384 tiles (4096 x 1536 x 1536) 28.2 / 28.6 with three, 35.6 with slices of 64; both operands with
  // contiguous rows, 341 tiles, 21.1 / 24.1 with three.
  if (tiles <= 256) return launch_pairing<128, 64, 4, 1>(g, s);
  return tiles >= 512 && g.a_sk == 1 ? launch_pairing<128, 32, 3, 3>(g, s) : launch_pairing<128, 32, 4, 2>(g, s);
}

}  // namespace hbp
