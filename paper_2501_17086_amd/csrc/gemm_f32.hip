// fp32 GEMM on the matrix cores (v_mfma_f32_32x32x2_f32: fp32 products and sums, as fma on the vector units).
//
// The fp32 stacks are small: what bounds them is the latency of a launch's one chain, load -> multiply -> store, not a
// rate.  So there is no LDS staging and no barrier in the loop: operands go from memory (the caches) straight into
// the MFMA layout, a chunk of 32 of the contraction ahead in registers.  The contraction index is a dummy, so a lane half
// takes four consecutive k of every eight and a K-contiguous operand is read 16 bytes per lane; a row-contiguous one
// is read 128 bytes per half wavefront and k.
//   32-wide tiles  four wavefronts share one 32 x 32 block and split the contraction in quarters, added through LDS: four
//                  times the workgroups and a quarter of the chain
//   64-wide tiles  four wavefronts own a 32 x 32 block each: half the operand bytes per flop, for launches that fill the chip
// Rows past the matrix repeat the last one and are not stored; k past the end are zeros in both operands.
// Measured against the LDS-tiled fma kernel (gemm_generic.hip, which keeps what is not 16-byte aligned), us:
// 128 x 64 x 256, 8 blocks 28.9 -> 5.0 (32 wide); 64 x 256 x 128, 8 blocks 18.0 -> 5.2; 512 x 128 x 512, 8 blocks 73 -> 12;
// 1024 x 256 x 1024, 12 blocks 182 -> 93 (64 wide, 70 TFLOP/s).  Relative error against 64 bits 1.5e-7 .. 2.9e-7 with 32-wide
// tiles (the quarters are sums of their own) and 2.9e-7 .. 5.7e-7 with 64-wide ones, where the fma kernel has 2.9e-7 .. 5.7e-7.
#include "hbp_common.h"

namespace hbp {

namespace {

typedef float float16v __attribute__((ext_vector_type(16)));

constexpr int CH = 32;      // contraction indices per chunk: 16 per lane half

// one operand's 16 values per lane of the chunk at k0
template <bool KC, bool TAIL>
__device__ __forceinline__ void load_chunk(float (&v)[CH / 2], const float* p, long ld, long k0, long k_end, int h) {
#pragma unroll
  for (int u = 0; u < CH / 8; ++u) {
    const long k = k0 + 8 * u + 4 * h;
    if (KC) {               // (k_end is a multiple of 4 here: a group of four is inside or outside as a whole)
      const bool in = !TAIL || k < k_end;
      const float4 t = *reinterpret_cast<const float4*>(p + (in ? k : k_end - 4));
      v[4 * u] = in ? t.x : 0.f; v[4 * u + 1] = in ? t.y : 0.f; v[4 * u + 2] = in ? t.z : 0.f; v[4 * u + 3] = in ? t.w : 0.f;
    } else {
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const bool in = !TAIL || k + s < k_end;
        const float t = p[(in ? k + s : k_end - 1) * ld];
        v[4 * u + s] = in ? t : 0.f;
      }
    }
  }
}
__device__ __forceinline__ void multiply(float16v& acc, const float (&a)[CH / 2], const float (&b)[CH / 2]) {
#pragma unroll
  for (int i = 0; i < CH / 2; ++i)
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(b[i], a[i], acc, 0, 0, 0);   // lane l: output row l % 32
}

__device__ __forceinline__ float gelu_f(float a) { return 0.5f * a * (1.0f + erff(a * 0.70710678118654752440f)); }
__device__ __forceinline__ float gelu_grad_f(float a) {
  return 0.5f * (1.0f + erff(a * 0.70710678118654752440f)) + a * __expf(-0.5f * a * a) * 0.39894228040143267794f;
}
__device__ __forceinline__ void load4(const float* p, float (&o)[4]) {
  const float4 t = *reinterpret_cast<const float4*>(p);
  o[0] = t.x; o[1] = t.y; o[2] = t.z; o[3] = t.w;
}
__device__ __forceinline__ void store4(float* p, const float (&v)[4]) {
  *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]);
}

// four consecutive columns of a row of the result
__device__ __forceinline__ void finish(const GemmArgs& g, long batch, int split, long row, long col, float (&v)[4]) {
  if (row >= g.M || col >= g.N) return;
  const long off = row * g.ldc + col;
  float* C = reinterpret_cast<float*>(g.C);
  if (g.split_k > 1) { store4(C + ((long)split * g.batch + batch) * g.c_sb + off, v); return; }
  if (g.addf) {
    float t[4];
    load4(g.addf + batch * g.addf_sb + off, t);
#pragma unroll
    for (int x = 0; x < 4; ++x) v[x] += t[x];
  }
  float t[4] = {0.f, 0.f, 0.f, 0.f};
  if (g.mode == EPI_MUL_AUX || g.mode == EPI_MUL_1MZ2 || g.mode == EPI_RESID || g.mode == EPI_ADD_AUX)
    load4(reinterpret_cast<const float*>(g.aux) + batch * g.aux_sb + off, t);
  switch (g.mode) {
    case EPI_MUL_AUX:
#pragma unroll
      for (int x = 0; x < 4; ++x) v[x] *= t[x];
      break;
    case EPI_MUL_1MZ2:
#pragma unroll
      for (int x = 0; x < 4; ++x) v[x] *= (1.f - t[x] * t[x]);
      break;
    case EPI_ACT_GELU: {
      float d[4];
#pragma unroll
      for (int x = 0; x < 4; ++x) { d[x] = gelu_grad_f(v[x]); v[x] = gelu_f(v[x]); }
      store4(reinterpret_cast<float*>(g.out2) + batch * g.out2_sb + off, d);
      break;
    }
    case EPI_ACT_TANH:
#pragma unroll
      for (int x = 0; x < 4; ++x) v[x] = tanhf(v[x]);
      break;
    case EPI_RESID: {
      float l4[4] = {1.f, 1.f, 1.f, 1.f};
      if (g.lambda_mn) load4(reinterpret_cast<const float*>(g.lambda_mn) + batch * g.aux_sb + off, l4);
      else if (g.lambda) load4(g.lambda + batch * g.lambda_sb + col, l4);
#pragma unroll
      for (int x = 0; x < 4; ++x) v[x] = fmaf(l4[x], t[x], v[x]);
      break;
    }
    case EPI_ADD_AUX:
#pragma unroll
      for (int x = 0; x < 4; ++x) v[x] += t[x];
      break;
    default: break;
  }
  store4(C + batch * g.c_sb + off, v);
}

template <int T, bool A_KC, bool B_KC>
__global__ __launch_bounds__(256) void gemm_f32_kernel(GemmArgs g) {
  constexpr bool SPLIT = T == 32;
  __shared__ __attribute__((aligned(16))) float red[SPLIT ? 4 : 1][32][36];
  const int tid = threadIdx.x, lane = tid & 63, r = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const long batch = blockIdx.z / g.split_k;
  const int split = (int)(blockIdx.z % g.split_k);
  const long m0 = (long)blockIdx.y * T + (SPLIT ? 0 : 32 * (wave >> 1)), n0 = (long)blockIdx.x * T + (SPLIT ? 0 : 32 * (wave & 1));
  const long m = m0 + r < g.M ? m0 + r : g.M - 1, n = n0 + r < g.N ? n0 + r : g.N - 1;
  const long lda = A_KC ? g.a_sm : g.a_sk, ldb = B_KC ? g.b_sn : g.b_sk;
  const float* pa = reinterpret_cast<const float*>(g.A) + batch * g.a_sb + m * g.a_sm;
  const float* pb = reinterpret_cast<const float*>(g.B) + batch * g.b_sb + n * g.b_sn;
  const long kchunk = ((g.K + g.split_k - 1) / g.split_k + 15) / 16 * 16;
  long k = (long)split * kchunk, k_end = k + kchunk < g.K ? k + kchunk : g.K;
  if (SPLIT) {              // this wavefront's quarter
    const long q = ((k_end > k ? k_end - k : 0) + 31) / 32 * 8;
    k += wave * q;
    k_end = k + q < k_end ? k + q : k_end;
  }
  float16v acc;
#pragma unroll
  for (int i = 0; i < 16; ++i) acc[i] = 0.f;
  float a0[CH / 2], b0[CH / 2], a1[CH / 2], b1[CH / 2];
  auto load = [&](float (&a)[CH / 2], float (&b)[CH / 2], long k0) __attribute__((always_inline)) {
    if (k0 + CH <= k_end) {
      load_chunk<A_KC, false>(a, pa, lda, k0, k_end, h);
      load_chunk<B_KC, false>(b, pb, ldb, k0, k_end, h);
    } else {
      load_chunk<A_KC, true>(a, pa, lda, k0, k_end, h);
      load_chunk<B_KC, true>(b, pb, ldb, k0, k_end, h);
    }
  };
  if (k < k_end) {
    load(a0, b0, k);
    while (true) {
      if (k + CH < k_end) load(a1, b1, k + CH);
      multiply(acc, a0, b0);
      k += CH;
      if (k >= k_end) break;
      if (k + CH < k_end) load(a0, b0, k + CH);
      multiply(acc, a1, b1);
      k += CH;
      if (k >= k_end) break;
    }
  }
  if (SPLIT) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
      *reinterpret_cast<float4*>(&red[SPLIT ? wave : 0][r][8 * q + 4 * h]) =
          make_float4(acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]);
    __syncthreads();
    const int row = tid >> 3, c0 = (tid & 7) * 4;
    float v[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      const float4 t = *reinterpret_cast<const float4*>(&red[SPLIT ? p : 0][row][c0]);
      v[0] += t.x; v[1] += t.y; v[2] += t.z; v[3] += t.w;
    }
    finish(g, batch, split, m0 + row, n0 + c0, v);
  } else {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      float v[4] = {acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]};
      finish(g, batch, split, m0 + r, n0 + 8 * q + 4 * h, v);
    }
  }
}

template <int T, bool A_KC, bool B_KC>
hipError_t launch_one(const GemmArgs& g, hipStream_t s) {
  const dim3 grid((unsigned)((g.N + T - 1) / T), (unsigned)((g.M + T - 1) / T), (unsigned)(g.batch * g.split_k));
  hipLaunchKernelGGL((gemm_f32_kernel<T, A_KC, B_KC>), grid, dim3(256), 0, s, g);
  return hipGetLastError();
}
template <int T>
hipError_t launch_pairing(const GemmArgs& g, hipStream_t s) {
  if (g.a_sk == 1) return g.b_sk == 1 ? launch_one<T, true, true>(g, s) : launch_one<T, true, false>(g, s);
  return g.b_sk == 1 ? launch_one<T, false, true>(g, s) : launch_one<T, false, false>(g, s);
}
inline bool ok16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

}  // namespace

bool gemm_f32_ok(const GemmArgs& g) {
  const bool a_kc = g.a_sk == 1, b_kc = g.b_sk == 1;
  if (!(a_kc || g.a_sm == 1) || !(b_kc || g.b_sn == 1)) return false;
  // 16-byte pieces of K-contiguous operands, of the result and of what the epilogue reads
  if (a_kc && (g.K % 4 || g.a_sm % 4 || g.a_sb % 4 || !ok16(g.A))) return false;
  if (b_kc && (g.K % 4 || g.b_sn % 4 || g.b_sb % 4 || !ok16(g.B))) return false;
  if (g.N % 4 || g.ldc % 4 || g.c_sb % 4 || g.aux_sb % 4 || g.out2_sb % 4 || g.addf_sb % 4 || g.lambda_sb % 4) return false;
  if (!ok16(g.C) || !ok16(g.aux) || !ok16(g.out2) || !ok16(g.addf) || !ok16(g.lambda) || !ok16(g.lambda_mn)) return false;
  return (g.M + 31) / 32 <= 65535 && g.batch * g.split_k <= 65535;
}
// 64-wide tiles once there are two per compute unit.  Measured, 32 / 64 wide: 128 tiles of 64 (512 x 128 x 512, batch 8)
// 11.9 / 17.6 us, 384 (1000 x 200 x 808, batch 6) 49.1 / 57.0, 512 (512 x 512 x 128, batch 8) 18.5 / 14.3, 768 (1024 x
// 256 x 1024, batch 12) 99.8 / 92.5, 3072 (1024 x 1024 x 256, batch 12) 133 / 104.
hipError_t launch_gemm_f32(const GemmArgs& g, hipStream_t s) {
  const long tiles = (g.M + 63) / 64 * ((g.N + 63) / 64) * g.batch * g.split_k;
  return tiles >= 512 ? launch_pairing<64>(g, s) : launch_pairing<32>(g, s);
}

}  // namespace hbp
