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
// Rows past the matrix repeat the last one and are not stored; k past the end are zeros in both operands.  What is fused into the
// result is asked for behind the first operands.
// Measured, us (before: addresses in 64 bits and values selected lane by lane, the fused operand read at the end): 128 x 256 x 64, 8
// blocks, with act' 5.2 -> 3.5; 128 x 64 x 256 5.1 -> 4.7; 338 x 384 x 96, 10 blocks, with act' 15.8 -> 8.4; 384 x 96 x 338, parameter gradients
// of 10 blocks, 13.7 -> 8.4; 1024 x 256 x 1024, 12 blocks, 96 -> 71 (64 wide, 91 TFLOP/s), parameter gradients 96 -> 61.  One block, both
// operands K-contiguous (the forward's pairing: two chunks asked for before the fused operand; after the first chunk, as in the others, it
// delays the second): 338 x 384 x 96 4.7 -> 3.9, 338 x 96 x 128 3.5 -> 3.4, x 256 5.3 -> 5.0, x 384 6.05 -> 6.23, x 512 7.3 -> 7.15, 300 x 200 x
// 800 10.4 -> 9.3, 1000 x 256 x 1024 11.3 -> 11.2.  Relative error against 64 bits 1.5e-7 .. 2.9e-7 with 32-wide tiles (the quarters are
// sums of their own) and 2.9e-7 .. 5.7e-7 with 64-wide ones.
#include "hbp_common.h"

namespace hbp {

namespace {

typedef float float16v __attribute__((ext_vector_type(16)));

constexpr int CH = 32;      // contraction indices per chunk: 16 per lane half

// One operand: a lane's place in a chunk is a 32-bit byte offset that stays the same, the chunk's is in the scalar base, and
// a lane past the contraction's end gets an offset outside the buffer, where loads give zero.  (Addresses in 64 bits per lane and
// values selected one by one were most of a short contraction's time: a wavefront issues a vector instruction every four cycles.)
typedef float float4v __attribute__((ext_vector_type(4)));
constexpr unsigned OUTSIDE = 0x80000000u;
template <bool KC>
struct Operand {
  const char* base;         // of the next chunk
  unsigned off;             // this lane's row and half in it
  int ld4;                  // bytes between two k (row-contiguous)
  // row0: the block's first row, `rows` of them; k: the first contraction index
  __device__ __forceinline__ Operand(const void* p, long ld, long row0, long rows, long k, int r, int h) {
    base = reinterpret_cast<const char*>(p) + (KC ? row0 * ld + k : k * ld + row0) * 4;
    ld4 = (int)ld * 4;
    const int rc = r < rows ? r : (int)rows - 1;
    off = KC ? (unsigned)(rc * ld4 + 16 * h) : (unsigned)(4 * h * ld4 + 4 * rc);
  }
  // the lane's 16 values of the next chunk, `left` contraction indices of it there
  template <bool TAIL>
  __device__ __forceinline__ void load(float (&v)[CH / 2], int left, int h) {
    const __amdgpu_buffer_rsrc_t b = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(base), 0, 0x7fffffff, 0x00027000);
#pragma unroll
    for (int u = 0; u < CH / 8; ++u) {
      if (KC) {             // (`left` is a multiple of 4 here: a group of four is inside or outside as a whole)
        const unsigned o = !TAIL || 8 * u + 4 * h < left ? off : OUTSIDE;
        const float4v t = __builtin_bit_cast(float4v, __builtin_amdgcn_raw_buffer_load_b128(b, (int)o, 32 * u, 0));
#pragma unroll
        for (int s = 0; s < 4; ++s) v[4 * u + s] = t[s];
      } else {
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const unsigned o = !TAIL || 8 * u + 4 * h + s < left ? off : OUTSIDE;
          v[4 * u + s] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(b, (int)o, (8 * u + s) * ld4, 0));
        }
      }
    }
    base += KC ? CH * 4 : (long)CH * ld4;
  }
};
// a chunk's products, eight contraction indices at a time as long as there are any of the `left`  (A path of its own for whole chunks
// puts all of their loads before the first product: 5 to 15 % slower.)
__device__ __forceinline__ void multiply(float16v& acc, const float (&a)[CH / 2], const float (&b)[CH / 2], int left) {
#pragma unroll
  for (int u = 0; u < CH / 8; ++u) {
    if (8 * u >= left) break;
#pragma unroll
    for (int s = 0; s < 4; ++s)
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(b[4 * u + s], a[4 * u + s], acc, 0, 0, 0);   // lane l: output row l % 32
  }
}

__device__ __forceinline__ float gelu_f(float a) { return 0.5f * a * (1.0f + erff(a * 0.70710678118654752440f)); }
__device__ __forceinline__ float gelu_grad_f(float a) {
  return 0.5f * (1.0f + erff(a * 0.70710678118654752440f)) + a * __expf(-0.5f * a * a) * 0.39894228040143267794f;
}
__device__ __forceinline__ void store4(float* p, const float (&v)[4]) {
  *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]);
}

// four consecutive columns of a row of the result: what is fused into them is asked for (early: the operands' trip hides it) ...
struct Fused {
  float4v aux, lam, add;
  bool in;
  long off;
  __device__ __forceinline__ void ask(const GemmArgs& g, long batch, long row, long col) {
    in = row < g.M && col < g.N;
    off = row * g.ldc + col;
    aux = add = float4v{0.f, 0.f, 0.f, 0.f};
    lam = float4v{1.f, 1.f, 1.f, 1.f};
    if (!in || g.split_k > 1) return;
    if (g.addf) add = *reinterpret_cast<const float4v*>(g.addf + batch * g.addf_sb + off);
    if (g.mode == EPI_MUL_AUX || g.mode == EPI_MUL_1MZ2 || g.mode == EPI_RESID || g.mode == EPI_ADD_AUX)
      aux = *reinterpret_cast<const float4v*>(reinterpret_cast<const float*>(g.aux) + batch * g.aux_sb + off);
    if (g.mode == EPI_RESID && g.lambda_mn)
      lam = *reinterpret_cast<const float4v*>(reinterpret_cast<const float*>(g.lambda_mn) + batch * g.aux_sb + off);
    else if (g.mode == EPI_RESID && g.lambda) lam = *reinterpret_cast<const float4v*>(g.lambda + batch * g.lambda_sb + col);
  }
  // ... and applied
  __device__ __forceinline__ void finish(const GemmArgs& g, long batch, int split, float (&v)[4]) const {
    if (!in) return;
    float* C = reinterpret_cast<float*>(g.C);
    if (g.split_k > 1) { store4(C + ((long)split * g.batch + batch) * g.c_sb + off, v); return; }
#pragma unroll
    for (int x = 0; x < 4; ++x) v[x] += add[x];
    switch (g.mode) {
      case EPI_MUL_AUX:
#pragma unroll
        for (int x = 0; x < 4; ++x) v[x] *= aux[x];
        break;
      case EPI_MUL_1MZ2:
#pragma unroll
        for (int x = 0; x < 4; ++x) v[x] *= (1.f - aux[x] * aux[x]);
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
      case EPI_RESID:
#pragma unroll
        for (int x = 0; x < 4; ++x) v[x] = fmaf(lam[x], aux[x], v[x]);
        break;
      case EPI_ADD_AUX:
#pragma unroll
        for (int x = 0; x < 4; ++x) v[x] += aux[x];
        break;
      default: break;
    }
    store4(C + batch * g.c_sb + off, v);
  }
};

// one tile: column bx, row by, batch and share bz
template <int T, bool A_KC, bool B_KC>
__device__ __forceinline__ void gemm_f32_body(const GemmArgs& g, unsigned bx, unsigned by, unsigned bz) {
  constexpr bool SPLIT = T == 32;
  __shared__ __attribute__((aligned(16))) float red[SPLIT ? 4 : 1][32][36];
  const int tid = threadIdx.x, lane = tid & 63, r = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const long batch = bz / (unsigned)g.split_k;
  const int split = (int)(bz % (unsigned)g.split_k);
  const long m0 = (long)by * T + (SPLIT ? 0 : 32 * (wave >> 1)), n0 = (long)bx * T + (SPLIT ? 0 : 32 * (wave & 1));
  const long lda = A_KC ? g.a_sm : g.a_sk, ldb = B_KC ? g.b_sn : g.b_sk;
  const long kchunk = ((g.K + g.split_k - 1) / g.split_k + 15) / 16 * 16;
  long k = (long)split * kchunk, k_end = k + kchunk < g.K ? k + kchunk : g.K;
  if (SPLIT) {              // this wavefront's quarter
    const long q = ((k_end > k ? k_end - k : 0) + 31) / 32 * 8;
    k += wave * q;
    k_end = k + q < k_end ? k + q : k_end;
  }
  // (a wavefront's block may lie outside the matrix as a whole: it computes the last row or column again and stores nothing)
  const long ma = m0 < g.M ? m0 : g.M - 1, nb = n0 < g.N ? n0 : g.N - 1;
  int left = k_end > k ? (int)(k_end - k) : 0;             // contraction indices to load
  Operand<A_KC> A(reinterpret_cast<const float*>(g.A) + batch * g.a_sb, lda, ma, g.M - ma, left ? k : 0, r, h);
  Operand<B_KC> B(reinterpret_cast<const float*>(g.B) + batch * g.b_sb, ldb, nb, g.N - nb, left ? k : 0, r, h);
  float16v acc;
#pragma unroll
  for (int i = 0; i < 16; ++i) acc[i] = 0.f;
  float a0[CH / 2], b0[CH / 2], a1[CH / 2], b1[CH / 2];
  auto load = [&](float (&a)[CH / 2], float (&b)[CH / 2]) __attribute__((always_inline)) {
    if (left >= CH) {
      A.template load<false>(a, left, h);
      B.template load<false>(b, left, h);
    } else {
      A.template load<true>(a, left, h);
      B.template load<true>(b, left, h);
    }
    left -= CH;
  };
  int todo = left;          // ... and to multiply
  const int row = tid >> 3, c0 = (tid & 7) * 4;            // SPLIT: this thread's piece of the result
  Fused f[SPLIT ? 1 : 4];
  auto ask = [&]() __attribute__((always_inline)) {
    if (SPLIT) {
      f[0].ask(g, batch, m0 + row, n0 + c0);
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q) f[SPLIT ? 0 : q].ask(g, batch, m0 + r, n0 + 8 * q + 4 * h);
    }
  };
  if (left > 0) load(a0, b0);
  if constexpr (A_KC && B_KC) {          // two chunks on their way before the fused operand
    if (left > 0) load(a1, b1);
    ask();
    while (todo > 0) {
      multiply(acc, a0, b0, todo);
      if ((todo -= CH) <= 0) break;
      if (left > 0) load(a0, b0);
      multiply(acc, a1, b1, todo);
      if ((todo -= CH) <= 0) break;
      if (left > 0) load(a1, b1);
    }
  } else {
    ask();
    while (todo > 0) {
      if (left > 0) load(a1, b1);
      multiply(acc, a0, b0, todo);
      if ((todo -= CH) <= 0) break;
      if (left > 0) load(a0, b0);
      multiply(acc, a1, b1, todo);
      todo -= CH;
    }
  }
  if (SPLIT) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
      *reinterpret_cast<float4*>(&red[SPLIT ? wave : 0][r][8 * q + 4 * h]) =
          make_float4(acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]);
    __syncthreads();
    float v[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      const float4 t = *reinterpret_cast<const float4*>(&red[SPLIT ? p : 0][row][c0]);
      v[0] += t.x; v[1] += t.y; v[2] += t.z; v[3] += t.w;
    }
    f[0].finish(g, batch, split, v);
  } else {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      float v[4] = {acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]};
      f[SPLIT ? 0 : q].finish(g, batch, split, v);
    }
  }
}

template <int T, bool A_KC, bool B_KC>
__global__ __launch_bounds__(256) void gemm_f32_kernel(GemmArgs g) {
  gemm_f32_body<T, A_KC, B_KC>(g, blockIdx.x, blockIdx.y, blockIdx.z);
}
// several products' tiles in one list (both operands with contiguous rows)
template <int T>
__global__ __launch_bounds__(256) void gemm_f32_group_kernel(GemmGroup q) {
  const int t = (int)blockIdx.x, i = q.of(t);
  const unsigned r = (unsigned)(t - q.start[i]), tn = (unsigned)q.tiles_n[i], row = r / tn, tm = (unsigned)q.tiles_m[i], z = row / tm;
  gemm_f32_body<T, false, false>(q.g[i], r - row * tn, row - z * tm, z);
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
// 10.7 / 16.8 us, 384 (1000 x 200 x 808, batch 6) 39.2 / 39.6, 440 (700 x 256 x 1024, batch 10) 46.6 / 49.3, 512 (512 x 512 x 128,
// batch 8) 13.9 / 12.9, 768 (1024 x 256 x 1024, batch 12) 74.4 / 70.9, 3072 (1024 x 1024 x 256, batch 12) 99 / 92.
hipError_t launch_gemm_f32(const GemmArgs& g, hipStream_t s) {
  const long tiles = (g.M + 63) / 64 * ((g.N + 63) / 64) * g.batch * g.split_k;
  return tiles >= 512 ? launch_pairing<64>(g, s) : launch_pairing<32>(g, s);
}
// parameter gradients that fill the chip together at most (32-wide tiles by the line above)
bool gemm_f32_group_ok(const GemmArgs* g, int n) {
  if (n < 2 || n > GEMM_GROUP) return false;
  long tiles = 0;
  for (int i = 0; i < n; ++i) {
    if (!gemm_f32_ok(g[i]) || g[i].a_sm != 1 || g[i].b_sn != 1 || g[i].a_sk == 1 || g[i].b_sk == 1) return false;
    tiles += (g[i].M + 63) / 64 * ((g[i].N + 63) / 64) * g[i].batch * g[i].split_k;
  }
  return tiles < 512;
}
hipError_t launch_gemm_f32_group(const GemmArgs* g, int n, hipStream_t s) {
  GemmGroup q;
  if (!make_group(q, g, n, 32, 32)) return hipErrorInvalidValue;
  hipLaunchKernelGGL(gemm_f32_group_kernel<32>, dim3((unsigned)q.total), dim3(256), 0, s, q);
  return hipGetLastError();
}

}  // namespace hbp
