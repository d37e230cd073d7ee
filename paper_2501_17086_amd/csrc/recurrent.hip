// A whole chain along time in one launch: the forward pass of the recurrent kinds and exact backpropagation through
// time, step after step, with the weights resident on the chip.
//
// What bounds these chains is not arithmetic or bandwidth (a step of 32 x 1024 multiplies 0.1 GFLOP and moves a few
// hundred KB) but the hand-over between dependent steps: as launches of their own they cost 7 us each.  Here
//   - a workgroup of four wavefronts owns 32 channels and keeps their rows of every weight matrix in registers for the
//     whole chain (each wavefront a quarter of the contraction, as operands of v_mfma_f32_16x16x32_bf16);
//   - the batch is cut into groups of 16 RT rows that never exchange anything; the ceil(width / 32) workgroups of a
//     group exchange the vectors that the next product contracts over through memory, with device-scope accesses, in
//     the order of the matrix instruction's operand: a workgroup's 32 channels of 16 rows are 1 KB, and a reader takes
//     16 bytes per lane, consecutive over the wavefront;
//   - there are no flags and no barriers across workgroups: a slot is empty (a word that no result has) until its
//     owner writes it, and a reader re-reads its operands until that word is gone.  A hand-over is then one store and
//     one load.  A vector's slots are four deep, one per step in turn: once a workgroup has read the whole of a step's
//     first vector, every other one has left the step before, and it empties its own slots of that step.  They are
//     used again four steps later, and what a reader waits for in between was written after the owner had waited
//     for its own reads, which a wavefront's earlier stores (the emptying among them) precede;
//   - the four quarters of a product are added through LDS (one workgroup barrier per product), and the elementwise
//     part of the cell runs on the sums, two channels of a row per thread, the state staying in registers.
// Workgroups take their place in a group in the order they start (a device counter), and a group begins once all of its
// workgroups have started: from then on each of them keeps running, so that every wait inside the chain ends.  One group of a
// launch at most is incomplete at any time, and at most 64 workgroups are launched, a quarter of the compute units, so that
// this is soon the case.  Where it is not, because other kernels hold the compute units, or incomplete groups of many launches
// (nine or more) hold all of them against each other, a group that has waited for REC_ARRIVE_POLLS polls per step, about as
// long as the chain takes one workgroup, is left to its first workgroup alone, and the others end.  That one plays all of them in
// turn, with the same phases, sums and exchange, reading the weights from memory at every step: the same results bit for bit at
// 0.1 to 0.4 ms a step (width 1024: 60 to 90 times the time of the group).
//
// Measured (1024 steps, batch 32, width 1024): exact backpropagation of the RNN 14.5 -> 3.3 ms, forward of the GRU 20.9 ->
// 3.7 ms; 1.6 us per dependent product, of which 0.3 us are waiting for data that is not there yet: the rest is one
// trip to memory for the operand, 16 MFMAs, the sum through LDS and the cell.  Read as 8-byte pieces of the row-major
// states instead of packed operands the same hand-over took 3.8 us, and a group's workgroups on one XCD did not help.
#include "hbp_common.h"

namespace hbp {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float float4v __attribute__((ext_vector_type(4)));

constexpr unsigned REC_EMPTY = 0xFFFFFFFFu;    // two bf16 NaNs of a pattern that publish() never stores
constexpr int REC_SLOTS = 4;                   // steps a vector's slots are deep
constexpr int REC_SPIN_LIMIT = 1 << 24;        // polls inside the chain (bounded only so that a fault elsewhere cannot hang it)
constexpr int REC_ARRIVE_POLLS = 256;          // polls per step for the rest of a group to start
constexpr unsigned REC_ALONE = 1u << 31;       // in a group's word beside the number of workgroups that have started
constexpr int REC_COLS = 32;                   // channels per workgroup
constexpr int REC_MAX_WG = 64;
constexpr int REC_UNITS = 4;                   // exchanged vectors at most
constexpr int RED_LD = 36;                     // floats per row of a partial block in LDS

// 32 columns of a weight matrix, this wavefront's quarter of the contraction: step s covers 32 k
template <int KQ>
struct Weights {
  bf16x8 w[KQ][2];
  // Bt: row per output column, contraction contiguous; columns past ncols and k past K are zero
  __device__ __forceinline__ void load(const bf16_t* Bt, long ldb, int col0, int ncols, int K, int wave, int lane) {
#pragma unroll
    for (int s = 0; s < KQ; ++s)
#pragma unroll
      for (int ct = 0; ct < 2; ++ct) {
        const int col = col0 + 16 * ct + (lane & 15), k = (wave * KQ + s) * 32 + 8 * (lane >> 4);
        uint4 v = make_uint4(0u, 0u, 0u, 0u);
        if (col < ncols && k < K) v = *reinterpret_cast<const uint4*>(Bt + (long)col * ldb + k);
        w[s][ct] = __builtin_bit_cast(bf16x8, v);
      }
  }
};

// The exchanged vectors of a launch: unit u, step slot, group, 16-row tile, block of 32 channels -> 1 KB, in which row r
// and channels 8 q .. 8 q + 7 of the block are the 16 bytes of lane 16 q + r; behind them 1 KB of zeros.
struct Ring {
  char* base;
  int wpg, groups, rts, group;
  __device__ __forceinline__ unsigned at(int u, long step, int rt, int block) const {
    return (unsigned)((((u * REC_SLOTS + (int)(step & (REC_SLOTS - 1))) * groups + group) * rts + rt) * wpg + block) * 1024u;
  }
  __device__ __forceinline__ unsigned zeros() const { return (unsigned)(REC_UNITS * REC_SLOTS * groups * rts * wpg) * 1024u; }
};

// This wavefront's operands of 16 RT rows out of a vector: its quarter of the blocks.  Past the last one it reads zeros: the
// weights there are zeros too, but against a repeated block they would turn an infinity of its into NaN.
template <int KQ, int RT>
struct Operand {
  bf16x8 a[RT][KQ];
  // re-reads until no word is empty any more
  __device__ __forceinline__ void load(const Ring& ring, int u, long step, int wave, int lane, bool& dead) {
    typedef unsigned uint4v __attribute__((ext_vector_type(4)));
    const __amdgpu_buffer_rsrc_t rsrc =
        __builtin_amdgcn_make_buffer_rsrc(ring.base, 0, ring.zeros() + 1024, 0x00027000);
    for (int spins = 0;; ++spins) {
      uint4v q[RT][KQ];
      asm volatile("" ::: "memory");           // (every pass reads again)
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int s = 0; s < KQ; ++s) {
          const int kb = wave * KQ + s;
          // (a plain 16-byte load at device scope: sc1; every 4-byte word of it is either empty or whole)
          q[rt][s] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, lane * 16, (int)(kb < ring.wpg ? ring.at(u, step, rt, kb) : ring.zeros()), 16);
        }
      unsigned top = 0;
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int s = 0; s < KQ; ++s) {
          top = max(max(top, q[rt][s].x), q[rt][s].y);
          top = max(max(top, q[rt][s].z), q[rt][s].w);
          a[rt][s] = __builtin_bit_cast(bf16x8, q[rt][s]);
        }
      if (dead || !__any(top == REC_EMPTY)) return;
      if (spins >= REC_SPIN_LIMIT) dead = true;
    }
  }
};

// acc += this wavefront's quarter of the product
template <int KQ, int RT>
__device__ __forceinline__ void multiply(float4v (&acc)[RT][2], const Weights<KQ>& w, const Operand<KQ, RT>& o) {
#pragma unroll
  for (int s = 0; s < KQ; ++s)
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int ct = 0; ct < 2; ++ct)
        // weights first: lane l, element r <-> channel 16 ct + 4 (l / 16) + r, row l % 16
        acc[rt][ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w.w[s][ct], o.a[rt][s], acc[rt][ct], 0, 0, 0);
}
template <int RT>
__device__ __forceinline__ void clear(float4v (&acc)[RT][2]) {
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int ct = 0; ct < 2; ++ct) acc[rt][ct] = float4v{0.f, 0.f, 0.f, 0.f};
}

// Partial products of the four wavefronts, two sets used in turn (a set is rewritten two barriers after it was read).
template <int RT, int SLOTS>
struct Partials { float v[2][SLOTS][4][16 * RT][RED_LD]; };
template <int RT, int SLOTS>
__device__ __forceinline__ void put(Partials<RT, SLOTS>& p, int set, int slot, const float4v (&acc)[RT][2], int wave, int lane) {
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int ct = 0; ct < 2; ++ct)
      *reinterpret_cast<float4v*>(&p.v[set][slot][wave][16 * rt + (lane & 15)][16 * ct + 4 * (lane >> 4)]) = acc[rt][ct];
}
template <int RT, int SLOTS>
__device__ __forceinline__ float2 get(const Partials<RT, SLOTS>& p, int set, int slot, int row, int col) {
  float2 s = make_float2(0.f, 0.f);
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    const float2 t = *reinterpret_cast<const float2*>(&p.v[set][slot][w][row][col]);
    s.x += t.x; s.y += t.y;
  }
  return s;
}
// all partial products are written (loads from memory stay in flight across it)
__device__ __forceinline__ void meet() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0xC07F);
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// two channels of a row
__device__ __forceinline__ float2 un2(unsigned w) { return make_float2(__uint_as_float(w << 16), __uint_as_float(w & 0xFFFF0000u)); }
__device__ __forceinline__ unsigned ld2(const bf16_t* p) { return *reinterpret_cast<const unsigned*>(p); }
__device__ __forceinline__ float2 ldf2(const float* p) { return *reinterpret_cast<const float2*>(p); }
__device__ __forceinline__ unsigned pk(float2 v) { return pack_bf16x2(v.x, v.y); }
__device__ __forceinline__ void st2(bf16_t* p, unsigned w) { *reinterpret_cast<unsigned*>(p) = w; }
// for other workgroups: device scope, and never the empty word (a pair of NaNs of that pattern changes its first sign).
// Thread t writes word t of its workgroup's block.
__device__ __forceinline__ void publish(const Ring& ring, int u, long step, int rt, int member, unsigned w) {
  __hip_atomic_store(reinterpret_cast<unsigned*>(ring.base + ring.at(u, step, rt, member)) + threadIdx.x,
                     w == REC_EMPTY ? 0xFFFF7FFFu : w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <int RT>
__device__ __forceinline__ void empty(const Ring& ring, int u, long step, int member) {
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
    __hip_atomic_store(reinterpret_cast<unsigned*>(ring.base + ring.at(u, step, rt, member)) + threadIdx.x, REC_EMPTY,
                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename F>
__device__ __forceinline__ float2 map2(F f) { return make_float2(f(0), f(1)); }
__device__ __forceinline__ float at2(float2 v, int i) { return i ? v.y : v.x; }
__device__ __forceinline__ float sigmoid1(float a) { return 1.f / (1.f + expf(-a)); }

enum { K_RNN = 0, K_GATED = 1, K_LSTM = 2, K_GRU = 3 };

// This workgroup's group and member number, in the order of starting.  The counter of the launch, then a word per group: how many
// of it have started (`started`, thread 0: with this one), and whether it has been given up.  (One thread divides by wpg, in
// vector registers; the kernels do not divide by it again, for the compiler would take this quotient's reciprocal there, leave
// the result in a vector register and put every operand load whose address depends on it into a loop over the lanes: 11 % on
// the GRU.)
__device__ __forceinline__ void take_place(const RecArgs& a, int wpg, int& group, int& member, unsigned& started) {
  __shared__ int place[2];
  started = 0;
  if (threadIdx.x == 0) {
    const int n = atomicAdd(a.counter, 1), g = n / wpg;
    started = atomicAdd(reinterpret_cast<unsigned*>(a.counter) + 1 + g, 1u) + 1u;
    place[0] = g;
    place[1] = n - g * wpg;
  }
  __syncthreads();
  group = __builtin_amdgcn_readfirstlane(place[0]);
  member = __builtin_amdgcn_readfirstlane(place[1]);
}
// true once the whole group has started, false if its first member is to go on alone
__device__ __forceinline__ bool all_started(const RecArgs& a, int wpg, int group, unsigned started) {
  __shared__ int given_up;
  if (threadIdx.x == 0) {
    const int limit = a.wait != REC_WAIT ? 0 : a.L < REC_SPIN_LIMIT / REC_ARRIVE_POLLS ? (int)a.L * REC_ARRIVE_POLLS : REC_SPIN_LIMIT;
    unsigned* word = reinterpret_cast<unsigned*>(a.counter) + 1 + group;
    unsigned w = started;
    for (int polls = 0; !(w & REC_ALONE) && w != (unsigned)wpg; ++polls) {
      if (polls < limit) {
        __builtin_amdgcn_s_sleep(2);
        w = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      } else {                           // (fails only where another workgroup has started, or given up, in between)
        const unsigned was = atomicCAS(word, w, w | REC_ALONE);
        w = was == w ? w | REC_ALONE : was;
      }
    }
    given_up = (w & REC_ALONE) != 0;
  }
  __syncthreads();
  return __builtin_amdgcn_readfirstlane(given_up) == 0;
}

// Which channels and rows a thread has in the elementwise part: two channels (from c on) of RT rows.
template <int RT>
struct Place {
  int row[RT];            // (past the batch: its last row, nothing of it is stored)
  int c;
  bool on[RT], on_f[RT];  // inside the state, inside the inner state
  __device__ __forceinline__ void set(int group, int member, int N, int width, int width_f) {
    c = member * REC_COLS + 8 * (threadIdx.x >> 6) + 2 * (threadIdx.x & 3);
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      const int r = group * 16 * RT + 16 * rt + ((threadIdx.x >> 2) & 15);
      on[rt] = r < N && c < width;
      on_f[rt] = r < N && c < width_f;
      row[rt] = r < N ? r : N - 1;
    }
  }
};
// f(member): this workgroup's own, or (ALONE) all of the group's in turn
template <bool ALONE, typename F>
__device__ __forceinline__ void members(int own, int wpg, F f) {
  if (!ALONE) { f(own); return; }
#pragma unroll 1
  for (int m = 0; m < wpg; ++m) f(m);
}

// False, with nothing done, if the group has been given up.  ALONE: one workgroup plays every member of its group; what a member
// keeps in registers from phase to phase it reads again (the thread that wrote it reads it).
template <int KIND, int KQ, int RT, bool ALONE, int SLOTS>
__device__ __forceinline__ bool forward_chain(const RecArgs& a, const Ring& ring, int own, unsigned started, Partials<RT, SLOTS>& part) {
  constexpr int UNITS = KIND == K_LSTM ? 4 : KIND == K_GRU ? 3 : 2;
  constexpr bool TWO = KIND == K_RNN || KIND == K_GRU;       // two dependent products per step
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int N = (int)a.N, H = (int)a.H, F = (int)a.F, D = (int)a.D;
  Weights<KQ> w[ALONE ? 1 : UNITS];
  auto weights = [&](int u, int member) __attribute__((always_inline)) -> Weights<KQ>& {
    Weights<KQ>& t = w[ALONE ? 0 : u];
    const int col0 = member * REC_COLS;
    if (KIND == K_RNN && u == 1) t.load((const bf16_t*)a.W2, F, col0, D, F, wave, lane);
    else t.load((const bf16_t*)a.W1 + (KIND == K_RNN ? 0 : (long)u * H * H), H, col0, KIND == K_RNN ? F : H, H, wave, lane);
    return t;
  };
  if (!ALONE) {
#pragma unroll
    for (int u = 0; u < UNITS; ++u) weights(u, own);
    if (!all_started(a, ring.wpg, ring.group, started)) return false;     // (while the weights are on their way)
  }
  Operand<KQ, RT> in;
  // exchanged: unit 0 the (hidden) state, unit 1 the RNN's inner state or the GRU's r (.) x
  // this thread's share of the elementwise part: two channels of RT rows
  const int my_row = (tid >> 2) & 15, my_col = 8 * (tid >> 6) + 2 * (tid & 3);
  Place<RT> at;
  float2 xs[RT];                     // the state's (LSTM: the cell's) two channels, as stored
  const long sx = (long)N * D, sf = (long)N * F;
  bf16_t* x = (bf16_t*)a.x;
  bf16_t* z = (bf16_t*)a.z;
  bf16_t* lam = (bf16_t*)a.lambda_tok;
  auto place = [&](int member) __attribute__((always_inline)) {      // where the member's channels are, and its state at this step
    at.set(ring.group, member, N, KIND == K_RNN ? D : H, KIND == K_RNN ? F : H);
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) xs[rt] = at.on[rt] ? un2(ld2(x + (long)at.row[rt] * D + at.c)) : make_float2(0.f, 0.f);
  };
  members<ALONE>(own, ring.wpg, [&](int member) __attribute__((always_inline)) {
    place(member);
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
      publish(ring, 0, 0, rt, member, at.on[rt] ? ld2(x + (long)at.row[rt] * D + (KIND == K_LSTM ? H : 0) + at.c) : 0u);
  });
  bool dead = false;
  int set = 0;
#pragma unroll 1
  for (long l = 0; l < a.L; ++l, x += sx, z += sf) {
    float2 ux[RT][SLOTS], un[RT], lm[RT];
    // what does not depend on the step before is on its way while the operands are waited for
    auto read_step = [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
#pragma unroll
        for (int q = 0; q < SLOTS; ++q)
          ux[rt][q] = at.on_f[rt] ? ldf2(a.ux + l * sf + (long)at.row[rt] * F + (KIND == K_RNN ? 0 : q * H) + at.c) : make_float2(0.f, 0.f);
        if (KIND == K_GRU) un[rt] = at.on[rt] ? ldf2(a.ux + l * sf + (long)at.row[rt] * F + 2 * H + at.c) : make_float2(0.f, 0.f);
        if (KIND == K_RNN) {
          lm[rt] = make_float2(1.f, 1.f);
          if (a.lambda && at.on[rt]) lm[rt] = ldf2(a.lambda + l * D + at.c);
          else if (lam && at.on[rt]) lm[rt] = un2(ld2(lam + l * sx + (long)at.row[rt] * D + at.c));
        }
      }
    };
    members<ALONE>(own, ring.wpg, [&](int member) __attribute__((always_inline)) {
      if (ALONE) place(member);
      read_step();
      in.load(ring, 0, l, wave, lane, dead);
#pragma unroll
      for (int u = 0; u < SLOTS; ++u) {
        float4v acc[RT][2];
        clear(acc);
        multiply(acc, ALONE ? weights(u, member) : w[ALONE ? 0 : u], in);
        put(part, set, u, acc, wave, lane);
      }
      meet();
      if (l > 0) {       // every workgroup of the group has left step l - 1
        empty<RT>(ring, 0, l - 1, member);
        if (TWO) empty<RT>(ring, 1, l - 1, member);
      }
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        const int pr = 16 * rt + my_row, pc = my_col;
        float2 s[SLOTS];
#pragma unroll
        for (int q = 0; q < SLOTS; ++q) {
          s[q] = get(part, set, q, pr, pc);
          s[q].x += ux[rt][q].x; s[q].y += ux[rt][q].y;
        }
        const long xo = (long)at.row[rt] * D + at.c, fo = (long)at.row[rt] * F + at.c;
        if (KIND == K_RNN) {
          if (a.tanh_act) s[0] = map2([&](int i) { return tanhf(at2(s[0], i)); });
          const unsigned zw = pk(s[0]);
          publish(ring, 1, l, rt, member, at.on_f[rt] ? zw : 0u);
          if (at.on_f[rt]) st2(z + fo, zw);
        } else if (KIND == K_GATED) {
          const float2 u = map2([&](int i) { return sigmoid1(at2(s[0], i)); });
          const float2 cc = map2([&](int i) { return tanhf(at2(s[SLOTS > 1 ? 1 : 0], i)); });
          const float2 av = make_float2(1.f - u.x, 1.f - u.y);
          const unsigned o = pk(map2([&](int i) { return fmaf(at2(av, i), at2(xs[rt], i), at2(u, i) * at2(cc, i)); }));
          publish(ring, 0, l + 1, rt, member, at.on[rt] ? o : 0u);
          if (at.on[rt]) {
            st2(x + sx + xo, o);
            st2(z + fo, pk(u));
            st2(z + fo + H, pk(cc));
            st2(lam + l * sx + xo, pk(av));
          }
          xs[rt] = un2(o);
        } else if (KIND == K_LSTM) {
          constexpr int S1 = SLOTS > 1 ? 1 : 0, S2 = SLOTS > 2 ? 2 : 0, S3 = SLOTS > 3 ? 3 : 0;
          const float2 ig = map2([&](int i) { return sigmoid1(at2(s[0], i)); });
          const float2 fg = map2([&](int i) { return sigmoid1(at2(s[S1], i)); });
          const float2 og = map2([&](int i) { return sigmoid1(at2(s[S2], i)); });
          const float2 gg = map2([&](int i) { return tanhf(at2(s[S3], i)); });
          const float2 cn = map2([&](int i) { return fmaf(at2(fg, i), at2(xs[rt], i), at2(ig, i) * at2(gg, i)); });
          const float2 hn = map2([&](int i) { return at2(og, i) * tanhf(at2(cn, i)); });
          const unsigned cw = pk(cn), hw = pk(hn);
          publish(ring, 0, l + 1, rt, member, at.on[rt] ? hw : 0u);
          if (at.on[rt]) {
            st2(x + sx + xo + H, hw);
            st2(x + sx + xo, cw);
            st2(z + fo, pk(ig));
            st2(z + fo + H, pk(fg));
            st2(z + fo + 2 * H, pk(og));
            st2(z + fo + 3 * H, pk(gg));
            st2(lam + l * sx + xo, pk(fg));
            st2(lam + l * sx + xo + H, 0u);
          }
          xs[rt] = un2(cw);
        } else {
          const float2 r = map2([&](int i) { return sigmoid1(at2(s[SLOTS > 1 ? 1 : 0], i)); });
          const unsigned zw = pk(map2([&](int i) { return sigmoid1(at2(s[0], i)); }));
          publish(ring, 1, l, rt, member, at.on[rt] ? pk(make_float2(r.x * xs[rt].x, r.y * xs[rt].y)) : 0u);
          if (at.on[rt]) {
            st2(z + fo, zw);
            st2(z + fo + H, pk(r));
          }
          ux[rt][0] = un2(zw);         // (the second half of the step works on the stored gate)
        }
      }
      set ^= 1;
    });
    if (TWO) {
      members<ALONE>(own, ring.wpg, [&](int member) __attribute__((always_inline)) {
        if (ALONE) {
          place(member);
          read_step();
          if (KIND == K_GRU) {
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
              ux[rt][0] = at.on[rt] ? un2(ld2(z + (long)at.row[rt] * F + at.c)) : make_float2(0.f, 0.f);
          }
        }
        in.load(ring, 1, l, wave, lane, dead);
        float4v acc[RT][2];
        clear(acc);
        multiply(acc, ALONE ? weights(UNITS - 1, member) : w[ALONE ? 0 : UNITS - 1], in);
        put(part, set, 0, acc, wave, lane);
        meet();
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
          float2 s = get(part, set, 0, 16 * rt + my_row, my_col);
          const long xo = (long)at.row[rt] * D + at.c;
          if (KIND == K_RNN) {
            const unsigned o = pk(map2([&](int i) { return at2(s, i) + at2(lm[rt], i) * at2(xs[rt], i); }));
            publish(ring, 0, l + 1, rt, member, at.on[rt] ? o : 0u);
            if (at.on[rt]) st2(x + sx + xo, o);
            xs[rt] = un2(o);
          } else {
            const float2 zg = ux[rt][0];
            const float2 nn = map2([&](int i) { return tanhf(at2(s, i) + at2(un[rt], i)); });
            const float2 av = make_float2(1.f - zg.x, 1.f - zg.y);
            const unsigned o = pk(map2([&](int i) { return fmaf(at2(av, i), at2(xs[rt], i), at2(zg, i) * at2(nn, i)); }));
            publish(ring, 0, l + 1, rt, member, at.on[rt] ? o : 0u);
            if (at.on[rt]) {
              st2(x + sx + xo, o);
              st2(z + (long)at.row[rt] * F + 2 * H + at.c, pk(nn));
              st2(lam + l * sx + xo, pk(av));
            }
            xs[rt] = un2(o);
          }
        }
        set ^= 1;
      });
    }
  }
  return true;
}

template <int KIND, int KQ, int RT>
__global__ __launch_bounds__(256, 1) void rec_forward_kernel(RecArgs a, int wpg, int groups) {
  constexpr int SLOTS = KIND == K_LSTM ? 4 : KIND == K_RNN ? 1 : 2;
  __shared__ __attribute__((aligned(16))) Partials<RT, SLOTS> part;
  int group, member;
  unsigned started;
  take_place(a, wpg, group, member, started);
  const Ring ring = {reinterpret_cast<char*>(a.ring), wpg, groups, RT, group};
  if (!forward_chain<KIND, KQ, RT, false>(a, ring, member, started, part) && member == 0)
    forward_chain<KIND, KQ, RT, true>(a, ring, member, started, part);
}

// Exact backpropagation: g[l] = (da_l W1 + what goes past the product) (+ e_l) + lambda_l (.) g[l+1], l = L-1 .. 0; da as in
// gated_cell.hip.  Weights transposed: Wt1 = W1^T [H][F] (GRU: [W_z; W_r]^T [H][2H]), Wt2 = W2^T [F][D] (RNN) or W_n^T [H][H].
template <int KIND, int KQ, int RT, bool ALONE>
__device__ __forceinline__ bool backward_chain(const RecArgs& a, const Ring& ring, int own, unsigned started, Partials<RT, 1>& part) {
  constexpr int UNITS = KIND == K_LSTM ? 4 : KIND == K_GRU ? 3 : 2;
  constexpr bool TWO = KIND == K_RNN || KIND == K_GRU;       // two dependent products per step
  constexpr int U0 = TWO ? 1 : 0;                            // first unit of the (second) product with W1
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int N = (int)a.N, H = (int)a.H, F = (int)a.F, D = (int)a.D;
  Weights<KQ> w[ALONE ? 1 : UNITS];
  auto weights = [&](int u, int member) __attribute__((always_inline)) -> Weights<KQ>& {
    Weights<KQ>& t = w[ALONE ? 0 : u];
    const int col0 = member * REC_COLS;
    if (TWO && u == 0) t.load((const bf16_t*)a.Wt2, KIND == K_RNN ? D : H, col0, KIND == K_RNN ? F : H, KIND == K_RNN ? D : H, wave, lane);
    else t.load((const bf16_t*)a.Wt1 + (long)(u - U0) * H, KIND == K_GRU ? 2 * H : F, col0, KIND == K_RNN ? D : H, KIND == K_RNN ? F : H, wave, lane);
    return t;
  };
  if (!ALONE) {
#pragma unroll
    for (int u = 0; u < UNITS; ++u) weights(u, own);
    if (!all_started(a, ring.wpg, ring.group, started)) return false;     // (while the weights are on their way)
  }
  Operand<KQ, RT> in;
  // exchanged: the cells' da, a unit per gate; the RNN's da is unit 0 and its state gradient unit 1
  const int my_row = (tid >> 2) & 15, my_col = 8 * (tid >> 6) + 2 * (tid & 3);
  Place<RT> at;
  float2 gs[RT], gc[RT];             // the gradient's two channels as stored (LSTM: hidden and cell part)
  const long sx = (long)N * D, sf = (long)N * F;
  bf16_t* g = (bf16_t*)a.g + a.L * sx;
  const int ho = KIND == K_LSTM ? H : 0;
  auto place = [&](int member) __attribute__((always_inline)) {      // where the member's channels are, and its gradient (g points at it)
    at.set(ring.group, member, N, KIND == K_RNN ? D : H, KIND == K_RNN ? F : H);
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      gs[rt] = gc[rt] = make_float2(0.f, 0.f);
      if (at.on[rt]) gs[rt] = un2(ld2(g + (long)at.row[rt] * D + ho + at.c));
      if (KIND == K_LSTM && at.on[rt]) gc[rt] = un2(ld2(g + (long)at.row[rt] * D + at.c));
    }
  };
  members<ALONE>(own, ring.wpg, [&](int member) __attribute__((always_inline)) {
    place(member);
    if (KIND == K_RNN) {
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
        publish(ring, 1, a.L, rt, member, at.on[rt] ? ld2(g + (long)at.row[rt] * D + at.c) : 0u);
    }
  });
  bool dead = false;
  int set = 0;
  const bf16_t* x = (const bf16_t*)a.x + (a.L - 1) * sx;
  const bf16_t* z = (const bf16_t*)a.z + (a.L - 1) * sf;
  const bf16_t* lamt = (const bf16_t*)a.lambda_tok;
  const bf16_t* dphi = (const bf16_t*)a.dphi;
  const bf16_t* e = (const bf16_t*)a.e;
#pragma unroll 1
  for (long l = a.L - 1; l >= 0; --l, x -= sx, z -= sf, g -= sx) {
    unsigned lw[RT], lw2[RT], ew[RT], ew2[RT], zw[RT][4], xw[RT], xn[RT];
    float2 lmf[RT];
    float2 past[RT], pastc[RT];      // what reaches g[l] (hidden, cell) past the product with W1
    // what does not depend on the step after is on its way while the operands are waited for
    auto read_step = [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        const long xo = (long)at.row[rt] * D + at.c, fo = (long)at.row[rt] * F + at.c;
        lmf[rt] = make_float2(1.f, 1.f);
        lw[rt] = lw2[rt] = ew[rt] = ew2[rt] = xw[rt] = xn[rt] = 0u;
#pragma unroll
        for (int q = 0; q < 4; ++q) zw[rt][q] = 0u;
        if (at.on[rt]) {
          if (a.lambda) lmf[rt] = ldf2(a.lambda + l * D + at.c);
          else if (lamt) lw[rt] = ld2(lamt + l * sx + xo + ho);
          if (e) ew[rt] = ld2(e + l * sx + xo + ho);
          if (KIND == K_LSTM) {
            lw2[rt] = ld2(lamt + l * sx + xo);
            if (e) ew2[rt] = ld2(e + l * sx + xo);
            xn[rt] = ld2(x + sx + xo);
          }
          if (KIND != K_RNN) {
            xw[rt] = ld2(x + xo);
#pragma unroll
            for (int q = 0; q < (KIND == K_GATED ? 2 : KIND == K_GRU ? 3 : 4); ++q) zw[rt][q] = ld2(z + fo + q * H);
          }
        }
        if (KIND == K_RNN && at.on_f[rt]) {
          if (dphi) zw[rt][0] = ld2(dphi + l * sf + fo);
          else if (a.tanh_act) zw[rt][0] = ld2(z + fo);
        }
      }
    };
    // the LSTM's gradient at the cell state through the hidden part
    auto tanh_c = [&](int rt) __attribute__((always_inline)) {
      const float2 cn = un2(xn[rt]);
      return map2([&](int i) { return tanhf(at2(cn, i)); });
    };
    auto through_h = [&](int rt, float2 tc) __attribute__((always_inline)) {
      const float2 og = un2(zw[rt][2]);
      return map2([&](int i) { return at2(gs[rt], i) * at2(og, i) * (1.f - at2(tc, i) * at2(tc, i)); });
    };
    // what the cells' elementwise parts leave for the products
    auto publish_gates = [&](int member) __attribute__((always_inline)) {
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        const float2 G = gs[rt], xv = un2(xw[rt]);
        if (KIND == K_GATED) {
          const float2 u = un2(zw[rt][0]), cc = un2(zw[rt][1]);
          const float2 du = map2([&](int i) { return at2(G, i) * (at2(cc, i) - at2(xv, i)) * at2(u, i) * (1.f - at2(u, i)); });
          const float2 dc = map2([&](int i) { return at2(G, i) * at2(u, i) * (1.f - at2(cc, i) * at2(cc, i)); });
          publish(ring, 0, l, rt, member, at.on[rt] ? pk(du) : 0u);
          publish(ring, 1, l, rt, member, at.on[rt] ? pk(dc) : 0u);
        } else if (KIND == K_LSTM) {
          const float2 ig = un2(zw[rt][0]), fg = un2(zw[rt][1]), og = un2(zw[rt][2]), gg = un2(zw[rt][3]);
          const float2 tc = tanh_c(rt), th = through_h(rt, tc);
          pastc[rt] = make_float2(th.x * fg.x, th.y * fg.y);
          const float2 dct = make_float2(gc[rt].x + th.x, gc[rt].y + th.y);
          const float2 di = map2([&](int i) { return at2(dct, i) * at2(gg, i) * at2(ig, i) * (1.f - at2(ig, i)); });
          const float2 df = map2([&](int i) { return at2(dct, i) * at2(xv, i) * at2(fg, i) * (1.f - at2(fg, i)); });
          const float2 dO = map2([&](int i) { return at2(G, i) * at2(tc, i) * at2(og, i) * (1.f - at2(og, i)); });
          const float2 dg = map2([&](int i) { return at2(dct, i) * at2(ig, i) * (1.f - at2(gg, i) * at2(gg, i)); });
          publish(ring, 0, l, rt, member, at.on[rt] ? pk(di) : 0u);
          publish(ring, 1, l, rt, member, at.on[rt] ? pk(df) : 0u);
          publish(ring, 2, l, rt, member, at.on[rt] ? pk(dO) : 0u);
          publish(ring, 3, l, rt, member, at.on[rt] ? pk(dg) : 0u);
        } else if (KIND == K_GRU) {
          const float2 zg = un2(zw[rt][0]), nn = un2(zw[rt][2]);
          const float2 dn = map2([&](int i) { return at2(G, i) * at2(zg, i) * (1.f - at2(nn, i) * at2(nn, i)); });
          const float2 dz = map2([&](int i) { return at2(G, i) * (at2(nn, i) - at2(xv, i)) * at2(zg, i) * (1.f - at2(zg, i)); });
          publish(ring, 2, l, rt, member, at.on[rt] ? pk(dn) : 0u);
          publish(ring, 0, l, rt, member, at.on[rt] ? pk(dz) : 0u);
        }
      }
    };
    // RNN: g W2; GRU: what comes back through the candidate's product, dn W_n
    auto first_product = [&](int member) __attribute__((always_inline)) {
      in.load(ring, KIND == K_RNN ? 1 : 2, KIND == K_RNN ? l + 1 : l, wave, lane, dead);
      float4v acc[RT][2];
      clear(acc);
      multiply(acc, ALONE ? weights(0, member) : w[0], in);
      put(part, set, 0, acc, wave, lane);
      meet();
    };
    members<ALONE>(own, ring.wpg, [&](int member) __attribute__((always_inline)) {
      if (ALONE) place(member);
      read_step();
      publish_gates(member);
    });
    if (TWO) {
      members<ALONE>(own, ring.wpg, [&](int member) __attribute__((always_inline)) {
        if (ALONE) { place(member); read_step(); }
        first_product(member);
        if (l + 1 < a.L) {       // every workgroup of the group has left step l + 1
          empty<RT>(ring, 0, l + 1, member);
          empty<RT>(ring, 1, KIND == K_RNN ? l + 2 : l + 1, member);
          if (KIND == K_GRU) empty<RT>(ring, 2, l + 1, member);
        }
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
          const float2 s = get(part, set, 0, 16 * rt + my_row, my_col);
          if (KIND == K_RNN) {
            float2 v = s;
            const float2 t = un2(zw[rt][0]);
            if (dphi) v = make_float2(s.x * t.x, s.y * t.y);
            else if (a.tanh_act) v = make_float2(s.x * (1.f - t.x * t.x), s.y * (1.f - t.y * t.y));
            publish(ring, 0, l, rt, member, at.on_f[rt] ? pk(v) : 0u);
          } else {
            const float2 r = un2(zw[rt][1]), xv = un2(xw[rt]);
            const float2 dr = map2([&](int i) { return at2(s, i) * at2(xv, i) * at2(r, i) * (1.f - at2(r, i)); });
            publish(ring, 1, l, rt, member, at.on[rt] ? pk(dr) : 0u);
            past[rt] = make_float2(s.x * r.x, s.y * r.y);
          }
        }
        set ^= 1;
      });
    }
    members<ALONE>(own, ring.wpg, [&](int member) __attribute__((always_inline)) {
      if (ALONE) { place(member); read_step(); }
      if (KIND == K_GRU && ALONE) {      // (the sum that the member's registers hold otherwise)
        first_product(member);
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
          const float2 s = get(part, set, 0, 16 * rt + my_row, my_col), r = un2(zw[rt][1]);
          past[rt] = make_float2(s.x * r.x, s.y * r.y);
        }
        set ^= 1;
      }
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        if (KIND != K_GRU) past[rt] = make_float2(0.f, 0.f);
        if (KIND == K_LSTM && ALONE) {
          const float2 th = through_h(rt, tanh_c(rt)), fg = un2(zw[rt][1]);
          pastc[rt] = make_float2(th.x * fg.x, th.y * fg.y);
        }
      }
      float4v acc[RT][2];
      clear(acc);
#pragma unroll
      for (int u = U0; u < UNITS; ++u) {
        in.load(ring, u - U0, l, wave, lane, dead);
        multiply(acc, ALONE ? weights(u, member) : w[ALONE ? 0 : u], in);
      }
      put(part, set, 0, acc, wave, lane);
      meet();
      if (!TWO && l + 1 < a.L) {
#pragma unroll
        for (int u = 0; u < UNITS; ++u) empty<RT>(ring, u, l + 1, member);
      }
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        const float2 s = get(part, set, 0, 16 * rt + my_row, my_col);
        const float2 ev = un2(ew[rt]), lm = lamt ? un2(lw[rt]) : lmf[rt];
        const unsigned o = pk(map2([&](int i) { return (at2(s, i) + at2(past[rt], i) + at2(ev, i)) + at2(lm, i) * at2(gs[rt], i); }));
        const long xo = (long)at.row[rt] * D + at.c - sx;    // g points at g[l + 1]
        if (KIND == K_RNN) publish(ring, 1, l, rt, member, at.on[rt] ? o : 0u);
        if (at.on[rt]) st2(g + xo + ho, o);
        gs[rt] = un2(o);
        if (KIND == K_LSTM) {
          const float2 e2 = un2(ew2[rt]), l2 = un2(lw2[rt]);
          const unsigned oc = pk(map2([&](int i) { return (at2(pastc[rt], i) + at2(e2, i)) + at2(l2, i) * at2(gc[rt], i); }));
          if (at.on[rt]) st2(g + xo, oc);
          gc[rt] = un2(oc);
        }
      }
      set ^= 1;
    });
  }
  return true;
}

template <int KIND, int KQ, int RT>
__global__ __launch_bounds__(256, 1) void rec_backward_kernel(RecArgs a, int wpg, int groups) {
  __shared__ __attribute__((aligned(16))) Partials<RT, 1> part;
  int group, member;
  unsigned started;
  take_place(a, wpg, group, member, started);
  const Ring ring = {reinterpret_cast<char*>(a.ring), wpg, groups, RT, group};
  if (!backward_chain<KIND, KQ, RT, false>(a, ring, member, started, part) && member == 0)
    backward_chain<KIND, KQ, RT, true>(a, ring, member, started, part);
}

// the empty word into every slot (n 16-byte pieces), zeros into the block behind them, the counter at zero and the groups' words
__global__ __launch_bounds__(256) void rec_fill_kernel(uint4* p, long n, int* counter, unsigned word) {
  const long i = (long)blockIdx.x * 256 + threadIdx.x;
  const unsigned w = i < n ? REC_EMPTY : 0u;
  if (i < n + 64) p[i] = make_uint4(w, w, w, w);
  if (i == 0) *counter = 0;
  if (i < REC_MAX_WG) counter[1 + i] = (int)word;
}

inline long rec_width(const RecArgs& a) { return a.F > a.D && a.kind == K_RNN ? a.F : a.kind == K_RNN ? a.D : a.H; }
// rows per group / 16: one where that gives at most REC_MAX_WG workgroups, else two; 0: neither does
inline int rec_row_tiles(const RecArgs& a) {
  const long wpg = (rec_width(a) + REC_COLS - 1) / REC_COLS;
  for (int rt = 1; rt <= 2; ++rt)
    if ((a.N + 16 * rt - 1) / (16 * rt) * wpg <= REC_MAX_WG) return rt;
  return 0;
}
inline bool ok16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

template <int KIND, int KQ, int RT>
hipError_t launch_rec(const RecArgs& a, bool forward, hipStream_t s) {
  const long wpg = (rec_width(a) + REC_COLS - 1) / REC_COLS;
  const long wgs = (a.N + 16 * RT - 1) / (16 * RT) * wpg;
  const long n16 = REC_UNITS * REC_SLOTS * wgs * RT * 64;
  hipLaunchKernelGGL(rec_fill_kernel, dim3((unsigned)((n16 + 64 + 255) / 256)), dim3(256), 0, s, reinterpret_cast<uint4*>(a.ring), n16,
                     a.counter, a.wait == REC_ALONE_ANYHOW ? REC_ALONE : 0u);
  if (forward) hipLaunchKernelGGL((rec_forward_kernel<KIND, KQ, RT>), dim3((unsigned)wgs), dim3(256), 0, s, a, (int)wpg, (int)(wgs / wpg));
  else hipLaunchKernelGGL((rec_backward_kernel<KIND, KQ, RT>), dim3((unsigned)wgs), dim3(256), 0, s, a, (int)wpg, (int)(wgs / wpg));
  return hipGetLastError();
}
template <int KIND>
hipError_t launch_rec_kind(const RecArgs& a, bool forward, hipStream_t s) {
  const int rt = rec_row_tiles(a);
  const long K = KIND == K_RNN ? rec_width(a) : a.H;
  if (rt == 1) {
    if (K <= 256) return launch_rec<KIND, 2, 1>(a, forward, s);
    return K <= 512 ? launch_rec<KIND, 4, 1>(a, forward, s) : launch_rec<KIND, 8, 1>(a, forward, s);
  }
  if (K <= 256) return launch_rec<KIND, 2, 2>(a, forward, s);
  return K <= 512 ? launch_rec<KIND, 4, 2>(a, forward, s) : launch_rec<KIND, 8, 2>(a, forward, s);
}

}  // namespace

static_assert((1 + REC_MAX_WG) * sizeof(int) <= RECURRENT_COUNTER_BYTES, "a counter and a word per group");
size_t recurrent_ring_bytes() { return (size_t)REC_UNITS * REC_SLOTS * REC_MAX_WG * 2 * 1024 + 1024; }
// What fits: bf16, widths whose weights the registers hold (1024) and at most 64 workgroups (two row tiles each: 64 rows at
// width 1024, 128 at 512).  Everything else goes step by step (7 us per product against 1.6).
bool recurrent_ok(const RecArgs& a) {
  if (a.H % 8 || a.D % 8 || a.F % 8 || rec_width(a) > 1024 || rec_row_tiles(a) == 0) return false;
  if (a.N * a.F > (1L << 30) || a.N * a.D > (1L << 30)) return false;
  return ok16(a.x) && ok16(a.z) && ok16(a.W1) && ok16(a.W2) && ok16(a.Wt1) && ok16(a.Wt2) && ok16(a.g) &&
         ok16(a.ring) && ok16(a.ux) && ok16(a.lambda) && ok16(a.lambda_tok) && ok16(a.e) && ok16(a.dphi);
}
hipError_t launch_recurrent(const RecArgs& a, bool forward, hipStream_t s) {
  switch (a.kind) {
    case K_RNN: return launch_rec_kind<K_RNN>(a, forward, s);
    case K_GATED: return launch_rec_kind<K_GATED>(a, forward, s);
    case K_LSTM: return launch_rec_kind<K_LSTM>(a, forward, s);
    default: return launch_rec_kind<K_GRU>(a, forward, s);
  }
}

}  // namespace hbp
