// A whole chain along time in one launch: the forward pass of the recurrent kinds and exact backpropagation through
// time, step after step, with the weights resident on the chip.
//
// What bounds these chains is not arithmetic or bandwidth (a step of 32 x 1024 multiplies 0.1 GFLOP and moves a few
// hundred KB) but the hand-over between dependent steps: as launches of their own they cost 7 us each.  Here
//   - a workgroup of four wavefronts owns 32 channels and keeps their rows of every weight matrix in registers for the
//     whole chain (each wavefront a quarter of the contraction, as operands of v_mfma_f32_16x16x32_bf16);
//   - the batch is cut into groups of 8, 16 or 32 rows that never exchange anything; the ceil(width / 32) workgroups of a
//     group exchange the vectors that the next product contracts over, past the compute units' own caches, in
//     the order of the matrix instruction's operand: a workgroup's 32 channels of 16 rows are 1 KB, and a reader takes
//     16 bytes per lane, consecutive over the wavefront;
//   - a group's workgroups are on one XCD, and what they exchange stays in its L2: 0.29 us from a store to the load that sees it,
//     0.46 us between two XCDs.  Every launch brings as many workgroups to each of the eight XCDs (ids are dealt to them in
//     turn) as a group has; those of an XCD form teams, a team's first workgroup claims a group, and who has none ends;
//   - there are no flags and no barriers across workgroups: a slot is empty (a word that no result has) until its
//     owner writes it, and a reader re-reads its operands until that word is gone.  A hand-over is then one store and
//     one load.  A vector's slots are four deep, one per step in turn: once a workgroup has read the whole of a step's
//     first vector, every other one has left the step before, and it empties its own slots of that step, before it asks for the
//     next operands.  They are used again four steps later, and what a reader waits for in between was written after the owner
//     had waited for those operands, which a wavefront's earlier stores (the emptying among them) precede;
//   - the four quarters of a product are added through LDS (one workgroup barrier per product), and the elementwise
//     part of the cell runs on the sums, one or two channels of a row per thread, the state staying in registers.
// A group begins once all of its workgroups have started: from then on each of them keeps running, so that every wait inside the
// chain ends.  If a group has not got together on one XCD after a poll per step (other kernels hold its compute units), it is
// given up, and a second launch, which otherwise ends at once, takes what is left (short chains go to it whole): its workgroups, at
// most 64 in all, a quarter of the compute units, may be anywhere and exchange through memory.  They take their place in a group in
// the order they start (a device counter).  One group of that launch at most is incomplete at any time, so that this is soon the
// case.  Where it is not, because other kernels hold the compute units, or incomplete groups of many launches (nine or more) hold all
// of them against each other, a group that has waited for REC_ARRIVE_POLLS polls per step, about as long as the chain takes one
// workgroup, is left to its first workgroup alone, and the others end.  That one plays all of them in turn, reading the weights from
// memory at every step: 0.1 to 0.4 ms a step (width 1024: 60 to 90 times the time of the group).  The sums have the same order in
// every form: the same results bit for bit.
//
// The launch with groups on one XCD keeps up to 256 workgroups running, one per compute unit (64 rows of width 1024; 32 rows: 128).
// What other streams do meanwhile waits for it, other chains among it, and three or more of those that need a compute unit per
// workgroup may also keep each other's groups from getting together, which the second launch then does.  512 steps at width 1024, ms
// for 1, 2, 4 and 8 calls at once, all of them with 64 workgroups anywhere / as it is: 32 rows, forward of the RNN 1.50, 1.91, 3.72,
// 6.0 / 0.85, 1.18, 2.42, 3.7, of the GRU 1.77, 1.99, 2.29, 4.6 / 1.11, 1.21, 3.3, 6.6, of the LSTM 1.67, 1.83, 2.18, 4.3 / 1.42,
// 1.55, 3.6, 7.2; exact backpropagation of the RNN 1.63, 2.21, 4.22, 7.0 / 0.84, 1.12, 2.20, 3.5, of the GRU 1.95, 2.32, 2.55, 5.1 /
// 0.98, 1.16, 3.0, 5.0; 64 rows, forward of the RNN 2.17, 2.51, 2.77, 5.5 / 0.88, 1.37, 2.67, 7.7, of the GRU 2.69, 2.90, 3.33, 9.1 /
// 1.18, 2.27, 4.5, 9.2.  One or two calls gain in every kind; from three on the wide GRU and LSTM lose, by 1.75 times at most.  Where a fifth
// wavefront reads ahead (read_ahead) a second workgroup no longer fits beside the first, which keeps two calls apart and makes more of
// them wait: without / with it, gated cell 32 x 1024 0.82, 1.34, 2.2, 4.1 / 0.75, 0.83, 2.3, 4.5, exact backpropagation of 64 x 512 0.66,
// 0.91, 1.3, 2.9 / 0.59, 0.89, 1.0, 3.1, LSTM 64 x 512 1.21, 1.66, 2.0, 4.4 / 1.02, 1.09, 2.2, 4.4, exact backpropagation of the RNN 64 x 512
// 0.75, 0.91, 1.4, 2.6 / 0.68, 0.85, 1.1, 3.1 (to 3.7); the GRU at REC_GRU_AHEAD.
//
// Measured (1024 steps, batch 32, width 1024): exact backpropagation of the RNN 14.5 ms as launches of their own, 3.3 through
// memory, 1.7 on one XCD with groups of 8 rows; forward of the GRU 20.9, 3.6 and 2.4.  0.8 us per dependent product: about 0.4 from
// a store to the operands in registers, the rest 16 MFMAs, the sum through LDS and the cell.  Groups of 16 rows: 2.0 ms (a
// workgroup reads 32 KB per product then, 500 cycles); inputs of a step read when it begins: loads return in order, so the wait
// for the operands met a trip to memory, 10 % more; per-step addresses in 64 bits and branches around edges: 5 %.
#include "hbp_common.h"
#include <cstddef>

namespace hbp {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float float4v __attribute__((ext_vector_type(4)));

constexpr unsigned REC_EMPTY = 0xFFFFFFFFu;    // two bf16 NaNs of a pattern that publish() never stores
constexpr int REC_SLOTS = 4;                   // steps a vector's slots are deep
constexpr int REC_SPIN_LIMIT = 1 << 24;        // polls inside the chain (bounded only so that a fault elsewhere cannot hang it)
constexpr int REC_ARRIVE_POLLS = 256;          // polls per step for the rest of a group to start
constexpr unsigned REC_ALONE = 1u << 31;       // in a group's word beside the number of workgroups that have started
// times 64 cycles (1024 steps of the RNN and of the GRU: 3: 2.18 and 4.00 ms, 4: 2.06 and 4.01, 7: 2.22 and 4.00)
constexpr int REC_PAUSE = 4;
// the same where a forward pass with two products per step exchanges through memory (11 steps of 32 x 1024, 0 / 4 / 8 / 12: RNN 56.7,
// 47.8, 42.4, 42.8 us, GRU 57.2, 54.9, 51.2, 52.5)
constexpr int REC_PAUSE_FAR = 8;
// Steps from which groups on one XCD pay for their launch.  Groups anywhere / on one XCD, us, 8 steps of 32 x 1024: RNN 39.8 / 38.3,
// LSTM 35.4 / 36.8; 12 steps, forward: RNN 50.4 / 40.6, gated cell 41.0 / 39.2, LSTM 60.9 / 57.2, GRU 57.9 / 50.5; 1 x 64: 29.9 / 25.2,
// 23.8 / 24.2, 32.3 / 29.4, 32.4 / 29.6; backwards 54.0 / 46.2, 47.4 / 39.8, 65.8 / 55.5, 57.3 / 50.8.
constexpr int REC_LOCAL_FROM = 12;
constexpr int REC_COLS = 32;                   // channels per workgroup
constexpr int REC_MAX_WG = 64;
constexpr int REC_XCDS = 16;                   // XCDs that a launch may meet (the chip has eight)
constexpr int REC_TEAMS = 32;                  // teams of workgroups on one of them
constexpr int REC_LOCAL_GROUPS = 256;
constexpr int REC_LOCAL_POLLS = 1;             // polls per step for the rest of a team to start
constexpr int HW_XCC_ID = 20 | (3 << 11);      // hwreg(HW_REG_XCC_ID), its four bits
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

// Everything inside the chain goes through buffer accesses: a lane's place in a row is a 32-bit offset that stays the same, a
// step's place is in the (scalar) base, and a lane outside the batch or the width has an offset past the end, where loads give
// zero and stores do nothing: no branches and no address arithmetic per step.
typedef unsigned uint4v __attribute__((ext_vector_type(4)));
typedef unsigned uint2v __attribute__((ext_vector_type(2)));
constexpr unsigned REC_OUTSIDE = 0x80000000u;
// n bytes from p on
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer(const void* p, long n) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)n, 0x00027000);
}
// a step's n bytes of an array along time (n = 0: there is none)
struct Rows {
  char* base;
  long n;
  __device__ __forceinline__ __amdgpu_buffer_rsrc_t buf() const { return buffer(base, n); }
  __device__ __forceinline__ void next(bool go) { base += go ? n : 0; }
  __device__ __forceinline__ void before(bool go) { base -= go ? n : 0; }
};
// (an offset as it is in a register: not computed again, and not behind a branch, where it is used)
__device__ __forceinline__ unsigned kept(unsigned v) {
  asm volatile("" : "+v"(v));
  return v;
}

// Rows per group and how a workgroup's threads share them: RT tiles of 16 rows, or (RT = 0) half a tile.
//
// The exchanged vectors of a launch: unit u, step slot, group, 16-row tile, block of 32 channels -> 1 KB, in which row r
// and channels 8 q .. 8 q + 7 of the block are the 16 bytes of lane 16 q + r.  Half a tile: a pair of blocks is 1 KB, the even
// one's row r is lane 16 q + r and the odd one's lane 16 q + 8 + r: one load brings two blocks.
// LOCAL: the group is on one XCD, whose L2 is where its stores meet its loads; otherwise stores go to memory.
template <int RT> constexpr int rec_tiles() { return RT ? RT : 1; }
template <int RT> constexpr int rec_rows() { return RT ? 16 * RT : 8; }
template <int RT> constexpr int rec_channels() { return RT ? 2 : 1; }         // of a row that a thread has in the elementwise part
template <bool LOCAL, int RT>
struct Ring {
  __amdgpu_buffer_rsrc_t buf;
  int wpg, group;
  int slot, tile, mine;           // bytes of a step's slot of one unit, of a row tile; where the group's part of a slot is
  unsigned word;                  // where a thread's word of a block is
  __device__ __forceinline__ Ring(char* base, int wpg_, int groups, int group_)
      : wpg(wpg_), group(group_) {
    tile = RT ? wpg * 1024 : (wpg + 1) / 2 * 1024;
    mine = group * rec_tiles<RT>() * tile;
    slot = groups * rec_tiles<RT>() * tile;
    buf = buffer(base, (long)REC_UNITS * REC_SLOTS * slot);
    const int t = RT ? threadIdx.x : threadIdx.x >> 1;
    word = kept(RT ? t * 4 : threadIdx.x & 1 ? REC_OUTSIDE : (t >> 5) * 256 + (t & 31) * 4);
  }
  __device__ __forceinline__ int at(int u, long step, int rt, int block) const {
    return (u * REC_SLOTS + ((int)step & (REC_SLOTS - 1))) * slot + mine + rt * tile +
           (RT ? block * 1024 : (block >> 1) * 1024 + (block & 1) * 128);
  }
  __device__ __forceinline__ void put(int place, unsigned w) const {
    __builtin_amdgcn_raw_buffer_store_b32(w, buf, (int)word, place, LOCAL ? 0 : 16);
  }
};

// This wavefront's operands of the group's rows out of a vector: its quarter of the blocks.  Past the last one it has zeros: the
// weights there are zeros too, but against a repeated block they would turn an infinity of its into NaN.
template <int KQ, int RT>
struct Operand {
  static constexpr int TILES = rec_tiles<RT>(), LOADS = RT ? KQ : KQ / 2;
  uint4v q[TILES][LOADS];
  unsigned off[LOADS];
  template <bool LOCAL>
  __device__ __forceinline__ void set(const Ring<LOCAL, RT>& ring, int wave, int lane) {
#pragma unroll
    for (int s = 0; s < LOADS; ++s) {
      const int n = wave * LOADS + s, block = RT ? n : 2 * n + ((lane >> 3) & 1);
      off[s] = kept(block < ring.wpg ? n * 1024 + lane * 16 : REC_OUTSIDE);
    }
  }
  // The first time after a short pause: what the other workgroups publish at the same time as this one takes about that long to
  // be seen, and operands read too early are read twice.
  template <int PAUSE = REC_PAUSE, bool LOCAL>
  __device__ __forceinline__ void ask(const Ring<LOCAL, RT>& ring, int u, long step) {
    if (PAUSE) __builtin_amdgcn_s_sleep(PAUSE);
    asm volatile("" ::: "memory");             // (every pass reads again)
#pragma unroll
    for (int s = 0; s < LOADS; ++s)
#pragma unroll
      for (int rt = 0; rt < TILES; ++rt)
        // (a plain 16-byte load past the compute unit's own cache: sc1; every 4-byte word of it is either empty or whole)
        q[rt][s] = __builtin_amdgcn_raw_buffer_load_b128(ring.buf, (int)off[s], ring.at(u, step, rt, 0), 16);
  }
  // block s (half a tile: with its neighbour; what the weights of the one make of the other's rows is never looked at)
  __device__ __forceinline__ bf16x8 a(int rt, int s) const { return __builtin_bit_cast(bf16x8, q[rt][RT ? s : s / 2]); }
  __device__ __forceinline__ bool missing() const {
    unsigned top = 0;
#pragma unroll
    for (int s = 0; s < LOADS; ++s)
#pragma unroll
      for (int rt = 0; rt < TILES; ++rt) {
        top = max(max(top, q[rt][s].x), q[rt][s].y);
        top = max(max(top, q[rt][s].z), q[rt][s].w);
      }
    return __any(top == REC_EMPTY);
  }
  // until no word of what was asked for is empty any more, all of it is read again.  (Each block waited for by itself, and only
  // what was missing read again, or the products begun on every pass: 10 to 20 % slower.)  The first look stands by itself, so
  // that it does not wait for what was issued after the operands, as it would at the head of the loop.
  template <bool LOCAL>
  __device__ __forceinline__ void wait(const Ring<LOCAL, RT>& ring, int u, long step, bool& dead) {
    if (dead || !missing()) return;
    int spins = 0;
    do {
      if (++spins >= REC_SPIN_LIMIT) dead = true;
      ask<0>(ring, u, step);
    } while (missing() && !dead);
  }
};

// A wavefront's quarter of a product: the blocks of even and of odd number summed apart, in every form of the kernel
template <int RT>
struct Product {
  float4v v[2][RT ? RT : 1][2];
  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int i = 0; i < 4 * (RT ? RT : 1); ++i) v[i & 1][i >> 2][(i >> 1) & 1] = float4v{0.f, 0.f, 0.f, 0.f};
  }
};
// acc += block s (weights first: lane l, element r <-> channel 16 ct + 4 (l / 16) + r, row l % 16)
template <int KQ, int RT>
__device__ __forceinline__ void multiply(Product<RT>& acc, const Weights<KQ>& w, const Operand<KQ, RT>& o, int s) {
#pragma unroll
  for (int rt = 0; rt < (RT ? RT : 1); ++rt)
#pragma unroll
    for (int ct = 0; ct < 2; ++ct)
      acc.v[s & 1][rt][ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w.w[s][ct], o.a(rt, s), acc.v[s & 1][rt][ct], 0, 0, 0);
}
template <int KQ, int RT>
__device__ __forceinline__ void multiply_all(Product<RT>& acc, const Weights<KQ>& w, const Operand<KQ, RT>& o) {
#pragma unroll
  for (int s = 0; s < KQ; ++s) multiply(acc, w, o, s);
}

// Partial products of the four wavefronts, two sets used in turn (a set is rewritten two barriers after it was read).  Half a
// tile: its 8 rows' even blocks in rows 0 to 7, the odd ones in rows 8 to 15.
template <int RT, int SLOTS>
struct Partials { float v[2][SLOTS][4][16 * (RT ? RT : 1)][RED_LD]; };
template <int RT, int SLOTS>
__device__ __forceinline__ void put(Partials<RT, SLOTS>& p, int set, int slot, const Product<RT>& acc, int wave, int lane) {
#pragma unroll
  for (int rt = 0; rt < (RT ? RT : 1); ++rt)
#pragma unroll
    for (int ct = 0; ct < 2; ++ct) {
      float4v t;
#pragma unroll
      for (int i = 0; i < 4; ++i)
        t[i] = RT ? acc.v[0][rt][ct][i] + acc.v[1][rt][ct][i] : (lane & 8) ? acc.v[1][rt][ct][i] : acc.v[0][rt][ct][i];
      *reinterpret_cast<float4v*>(&p.v[set][slot][wave][16 * rt + (lane & 15)][16 * ct + 4 * (lane >> 4)]) = t;
    }
}
template <int RT, int SLOTS>
__device__ __forceinline__ float2 get(const Partials<RT, SLOTS>& p, int set, int slot, int row, int col) {
  float2 s = make_float2(0.f, 0.f);
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    if (RT) {
      const float2 t = *reinterpret_cast<const float2*>(&p.v[set][slot][w][row][col]);
      s.x += t.x; s.y += t.y;
    } else {
      s.x += p.v[set][slot][w][row][col] + p.v[set][slot][w][row + 8][col];
    }
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

// A thread's channels of a row, two (CH = 2), or one of the two that it shares a word with its neighbour for (in .x)
template <int CH>
__device__ __forceinline__ float2 un2(unsigned w) {
  const float2 v = make_float2(__uint_as_float(w << 16), __uint_as_float(w & 0xFFFF0000u));
  return CH == 2 ? v : make_float2(threadIdx.x & 1 ? v.y : v.x, 0.f);
}
template <int CH>
__device__ __forceinline__ unsigned pk(float2 v) {
  if (CH == 2) return pack_bf16x2(v.x, v.y);
  const float other = __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v.x), 0xB1, 0xF, 0xF, true));   // quad_perm [1,0,3,2]
  return threadIdx.x & 1 ? pack_bf16x2(other, v.x) : pack_bf16x2(v.x, other);
}
__device__ __forceinline__ unsigned bld2(__amdgpu_buffer_rsrc_t b, unsigned off, int more = 0) {
  return __builtin_amdgcn_raw_buffer_load_b32(b, (int)off, more, 0);
}
template <int CH>
__device__ __forceinline__ float2 bldf2(__amdgpu_buffer_rsrc_t b, unsigned off, int more = 0) {
  if (CH == 1) return make_float2(__builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(b, (int)off, more, 0)), 0.f);
  return __builtin_bit_cast(float2, (uint2v)__builtin_amdgcn_raw_buffer_load_b64(b, (int)off, more, 0));
}
__device__ __forceinline__ void bst2(unsigned w, __amdgpu_buffer_rsrc_t b, unsigned off, int more = 0) {
  __builtin_amdgcn_raw_buffer_store_b32(w, b, (int)off, more, 0);
}
// for other workgroups, at ring.at(...): never the empty word (a pair of NaNs of that pattern changes its first sign)
template <bool LOCAL, int RT>
__device__ __forceinline__ void publish(const Ring<LOCAL, RT>& ring, int place, unsigned w) {
  ring.put(place, w == REC_EMPTY ? 0xFFFF7FFFu : w);
}
template <bool LOCAL, int RT>
__device__ __forceinline__ void empty(const Ring<LOCAL, RT>& ring, int u, long step, int member) {
#pragma unroll
  for (int rt = 0; rt < rec_tiles<RT>(); ++rt) ring.put(ring.at(u, step, rt, member), REC_EMPTY);
}
template <int CH, typename F>
__device__ __forceinline__ float2 map2(F f) { return make_float2(f(0), CH == 2 ? f(1) : 0.f); }
__device__ __forceinline__ float at2(float2 v, int i) { return i ? v.y : v.x; }
__device__ __forceinline__ float sigmoid1(float a) { return 1.f / (1.f + expf(-a)); }

enum { K_RNN = 0, K_GATED = 1, K_LSTM = 2, K_GRU = 3 };

// The words that a launch's workgroups find their places with, all zero before it
struct PlaceWords {
  int ticket;                              // workgroups of the launch that may be anywhere, in the order of starting
  unsigned group[REC_MAX_WG];              // and per group how many of them have started, and whether it has been given up
  unsigned local[REC_LOCAL_GROUPS];        // the same of the launch with groups on one XCD each
  int claimed;                             // groups that have an XCD
  int on_xcd[REC_XCDS];                    // workgroups started on an XCD
  int team[REC_XCDS][REC_TEAMS];           // the group of the XCD's workgroups wpg t .. wpg t + wpg - 1, plus one
};
static_assert(sizeof(PlaceWords) <= RECURRENT_COUNTER_BYTES, "the words' place in the workspace");

// This workgroup's group and member number (group -1: none, it ends) and how many of the group have started (`started`, thread 0:
// with this one).  LOCAL: the workgroups of an XCD form teams in the order of starting; the first of a team claims the next
// group.  Otherwise groups are filled in the order of starting, those that the other launch has done being left out.  (One thread
// divides by wpg, in vector registers; the kernels do not divide by it again, for the compiler would take this quotient's
// reciprocal there, leave the result in a vector register and put every operand load whose address depends on it into a loop
// over the lanes: 11 % on the GRU.)
template <bool LOCAL>
__device__ __forceinline__ void take_place(const RecArgs& a, int wpg, int groups, int per, int locals, int& group, int& member,
                                           unsigned& started) {
  __shared__ int place[2];
  started = 0;
  if (threadIdx.x == 0) {
    PlaceWords* w = reinterpret_cast<PlaceWords*>(a.counter);
    int g = -1, m = 0;
    if (LOCAL) {
      const int xcd = (int)__builtin_amdgcn_s_getreg(HW_XCC_ID) & (REC_XCDS - 1);
      const int n = atomicAdd(&w->on_xcd[xcd], 1), t = n / wpg;
      m = n - t * wpg;
      if (t < REC_TEAMS) {
        int c;
        if (m == 0) {
          c = atomicAdd(&w->claimed, 1) + 1;
          __hip_atomic_store(&w->team[xcd][t], c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        } else {                           // (its first workgroup has started, and claims without waiting)
          while ((c = __hip_atomic_load(&w->team[xcd][t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) == 0) __builtin_amdgcn_s_sleep(1);
        }
        g = c <= groups ? c - 1 : -1;
      }
      if (g >= 0) started = atomicAdd(&w->local[g], 1u) + 1u;
    } else {
      const int n = atomicAdd(&w->ticket, 1);
      g = n / wpg;
      m = n - g * wpg;
      bool done = locals > 0;
      for (int i = g * per; i < g * per + per && i < locals; ++i)
        done = done && __hip_atomic_load(&w->local[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (unsigned)wpg;
      if (done) g = -1;
      else started = atomicAdd(&w->group[g], 1u) + 1u;
    }
    place[0] = g;
    place[1] = m;
  }
  __syncthreads();
  group = __builtin_amdgcn_readfirstlane(place[0]);
  member = __builtin_amdgcn_readfirstlane(place[1]);
}
// true once the whole group has started, false if it has been given up
template <bool LOCAL>
__device__ __forceinline__ bool all_started(const RecArgs& a, int wpg, int group, unsigned started) {
  __shared__ int given_up;
  if (threadIdx.x == 0) {
    const int polls_per_step = LOCAL && a.wait == REC_WAIT ? REC_LOCAL_POLLS : REC_ARRIVE_POLLS;
    const int limit = a.wait == REC_WAIT_NOT || a.wait == REC_ALONE_ANYHOW ? 0
                      : a.L < REC_SPIN_LIMIT / polls_per_step              ? (int)a.L * polls_per_step
                                                                           : REC_SPIN_LIMIT;
    PlaceWords* words = reinterpret_cast<PlaceWords*>(a.counter);
    unsigned* word = LOCAL ? &words->local[group] : &words->group[group];
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

// Which channels and rows a thread has in the elementwise part: two channels of a row per tile, or (half a tile) one.
template <int RT>
struct Place {
  static constexpr int TILES = rec_tiles<RT>(), CH = rec_channels<RT>();
  int row, col;                                       // in a tile, among the workgroup's channels
  bool on[TILES], on_f[TILES];                        // inside the state, inside the inner state
  unsigned x2[TILES], f2[TILES];                      // bytes to the pair of channels in bf16: in the state, in the inner state
  unsigned f4[TILES], c4[TILES];                      // to the thread's own in fp32: in the inner state, in a row of channels
  unsigned xs[TILES], fs[TILES];                      // as x2, f2, for the thread that stores the pair
  __device__ __forceinline__ Place() {
    const int t = threadIdx.x / (2 / CH);
    row = (t >> 2) & (RT ? 15 : 7);
    col = 8 * (t >> (RT ? 6 : 5)) + 2 * (t & 3) + (CH == 1 ? threadIdx.x & 1 : 0);
  }
  __device__ __forceinline__ void set(int group, int member, int N, int D, int F, int width, int width_f) {
    const int c = member * REC_COLS + col, pair = c & ~1;
    const bool stores = CH == 2 || !(threadIdx.x & 1);
#pragma unroll
    for (int rt = 0; rt < TILES; ++rt) {
      const int r = group * rec_rows<RT>() + 16 * rt + row;
      on[rt] = r < N && c < width;
      on_f[rt] = r < N && c < width_f;
      x2[rt] = kept(on[rt] ? (unsigned)(r * D + pair) * 2 : REC_OUTSIDE);
      f2[rt] = kept(on_f[rt] ? (unsigned)(r * F + pair) * 2 : REC_OUTSIDE);
      xs[rt] = CH == 2 ? x2[rt] : kept(stores ? x2[rt] : REC_OUTSIDE);
      fs[rt] = CH == 2 ? f2[rt] : kept(stores ? f2[rt] : REC_OUTSIDE);
      f4[rt] = kept(on_f[rt] ? (unsigned)(r * F + c) * 4 : REC_OUTSIDE);
      c4[rt] = kept(on[rt] ? (unsigned)c * 4 : REC_OUTSIDE);
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
// A phase publishes what it leaves for others first of all; its results, the emptying of slots and the question for the next
// phase's operands come after that, in the time that the others' words need to arrive.
template <int KIND, int KQ, int RT, bool ALONE, bool LOCAL, int SLOTS>
__device__ __forceinline__ bool forward_chain(const RecArgs& a, const Ring<LOCAL, RT>& ring, int own, unsigned started,
                                              Partials<RT, SLOTS>& part) {
  constexpr int UNITS = KIND == K_LSTM ? 4 : KIND == K_GRU ? 3 : 2;
  constexpr bool TWO = KIND == K_RNN || KIND == K_GRU;       // two dependent products per step
  // one product: a step's inputs are read two steps ahead, or (through memory, but for the LSTM with two row tiles) just before
  constexpr bool AHEAD = !TWO && (LOCAL || (KIND == K_LSTM && RT == 2));
  constexpr int PAUSE = LOCAL || !TWO ? REC_PAUSE : REC_PAUSE_FAR;
  constexpr int TILES = rec_tiles<RT>(), CH = rec_channels<RT>();
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
    if (!all_started<LOCAL>(a, ring.wpg, ring.group, started)) return false;     // (while the weights are on their way)
  }
  Operand<KQ, RT> in;
  in.set(ring, wave, lane);
  // exchanged: unit 0 the (hidden) state, unit 1 the RNN's inner state or the GRU's r (.) x
  Place<RT> at;
  float2 xs[TILES];                     // the state's (LSTM: the cell's) two channels, as stored
  const long sx = (long)N * D, sf = (long)N * F;
  const int h2 = 2 * H, h4 = 4 * H;  // a gate's distance in bytes
  Rows x = {(char*)a.x, 2 * sx}, z = {(char*)a.z, 2 * sf};         // of this step
  Rows lam = {(char*)a.lambda_tok, a.lambda_tok ? 2 * sx : 0};
  Rows ux = {(char*)a.ux, 4 * sf}, lc = {(char*)a.lambda, a.lambda ? 4L * D : 0}, lt = lam;      // of the step to be read
  auto place = [&](int member) __attribute__((always_inline)) {      // where the member's channels are, and its state at this step
    at.set(ring.group, member, N, D, F, KIND == K_RNN ? D : H, KIND == K_RNN ? F : H);
#pragma unroll
    for (int rt = 0; rt < TILES; ++rt) xs[rt] = un2<CH>(bld2(x.buf(), at.x2[rt]));
  };
  members<ALONE>(own, ring.wpg, [&](int member) __attribute__((always_inline)) {
    place(member);
#pragma unroll
    for (int rt = 0; rt < TILES; ++rt) publish(ring, ring.at(0, 0, rt, member), bld2(x.buf(), at.x2[rt], KIND == K_LSTM ? h2 : 0));
  });
  if (!ALONE && (AHEAD || TWO)) in.template ask<PAUSE>(ring, 0, 0);
  bool dead = false;
  int set = 0;
  // what a step takes besides the state before it
  struct Inputs { float2 ux[TILES][SLOTS], un[TILES], lm[TILES]; unsigned lw[TILES]; };
  auto read_step = [&](Inputs& v) __attribute__((always_inline)) {
    const __amdgpu_buffer_rsrc_t ub = ux.buf(), lb = lc.buf(), tb = lt.buf();
#pragma unroll
    for (int rt = 0; rt < TILES; ++rt) {
#pragma unroll
      for (int q = 0; q < SLOTS; ++q) v.ux[rt][q] = bldf2<CH>(ub, at.f4[rt], KIND == K_RNN ? 0 : q * h4);
      if (KIND == K_GRU) v.un[rt] = bldf2<CH>(ub, at.f4[rt], 2 * h4);
      if (KIND == K_RNN) {
        v.lm[rt] = bldf2<CH>(lb, at.c4[rt]);
        v.lw[rt] = bld2(tb, at.x2[rt]);
      }
    }
  };
  // the step to be read becomes the next one, or stays the last one
  auto advance = [&](bool more) __attribute__((always_inline)) { ux.next(more); lc.next(more); lt.next(more); };
  Inputs now, next;
  if (!ALONE) {
    read_step(now);
    advance(a.L > 1);
    if (AHEAD) { read_step(next); advance(a.L > 2); }
    if (!AHEAD && !TWO) in.template ask<PAUSE>(ring, 0, 0);
  }
#pragma unroll 1
  for (long l = 0; l < a.L; ++l) {
    const __amdgpu_buffer_rsrc_t zb = z.buf(), lb = lam.buf();
    x.next(true);
    const __amdgpu_buffer_rsrc_t xb = x.buf();       // of x[l + 1]
    members<ALONE>(own, ring.wpg, [&](int member) __attribute__((always_inline)) {
      if (ALONE) { x.base -= x.n; place(member); x.base += x.n; read_step(now); in.ask(ring, 0, l); }
      in.wait(ring, 0, l, dead);
      if (!ALONE && TWO) { read_step(next); advance(l + 2 < a.L); }
#pragma unroll
      for (int u = 0; u < SLOTS; ++u) {
        Product<RT> acc;
        acc.clear();
        multiply_all(acc, ALONE ? weights(u, member) : w[ALONE ? 0 : u], in);
        put(part, set, u, acc, wave, lane);
      }
      meet();
      // every workgroup of the group has left step l - 1 (before the first step: slots that are empty yet).  To memory, the stores
      // are on their way before the elementwise part: the operands asked for after them return after them.
      auto empty_all = [&]() __attribute__((always_inline)) {
        empty(ring, 0, l - 1, member);
        if (TWO) empty(ring, 1, l - 1, member);
      };
      if (!LOCAL) empty_all();
      unsigned zw[TILES], rw[TILES], ow[TILES], cw[TILES], gw[TILES], aw[TILES], hw[TILES];     // what the phase leaves, packed
#pragma unroll
      for (int rt = 0; rt < TILES; ++rt) {
        const int pr = 16 * rt + at.row, pc = at.col;
        float2 s[SLOTS];
#pragma unroll
        for (int q = 0; q < SLOTS; ++q) {
          s[q] = get(part, set, q, pr, pc);
          s[q].x += now.ux[rt][q].x; s[q].y += now.ux[rt][q].y;
        }
        constexpr int S1 = SLOTS > 1 ? 1 : 0, S2 = SLOTS > 2 ? 2 : 0, S3 = SLOTS > 3 ? 3 : 0;
        if (KIND == K_RNN) {
          if (a.tanh_act) s[0] = map2<CH>([&](int i) { return tanhf(at2(s[0], i)); });
          zw[rt] = pk<CH>(s[0]);
          publish(ring, ring.at(1, l, rt, member), at.on_f[rt] ? zw[rt] : 0u);
        } else if (KIND == K_GATED) {
          const float2 u = map2<CH>([&](int i) { return sigmoid1(at2(s[0], i)); });
          const float2 cc = map2<CH>([&](int i) { return tanhf(at2(s[S1], i)); });
          const float2 av = make_float2(1.f - u.x, 1.f - u.y);
          ow[rt] = pk<CH>(map2<CH>([&](int i) { return fmaf(at2(av, i), at2(xs[rt], i), at2(u, i) * at2(cc, i)); }));
          publish(ring, ring.at(0, l + 1, rt, member), at.on[rt] ? ow[rt] : 0u);
          zw[rt] = pk<CH>(u); cw[rt] = pk<CH>(cc); aw[rt] = pk<CH>(av);
          xs[rt] = un2<CH>(ow[rt]);
        } else if (KIND == K_LSTM) {
          const float2 ig = map2<CH>([&](int i) { return sigmoid1(at2(s[0], i)); });
          const float2 fg = map2<CH>([&](int i) { return sigmoid1(at2(s[S1], i)); });
          const float2 og = map2<CH>([&](int i) { return sigmoid1(at2(s[S2], i)); });
          const float2 gg = map2<CH>([&](int i) { return tanhf(at2(s[S3], i)); });
          const float2 cn = map2<CH>([&](int i) { return fmaf(at2(fg, i), at2(xs[rt], i), at2(ig, i) * at2(gg, i)); });
          const float2 hn = map2<CH>([&](int i) { return at2(og, i) * tanhf(at2(cn, i)); });
          hw[rt] = pk<CH>(hn);
          publish(ring, ring.at(0, l + 1, rt, member), at.on[rt] ? hw[rt] : 0u);
          cw[rt] = pk<CH>(cn); zw[rt] = pk<CH>(ig); rw[rt] = pk<CH>(fg); ow[rt] = pk<CH>(og); gw[rt] = pk<CH>(gg);
          xs[rt] = un2<CH>(cw[rt]);
        } else {
          const float2 r = map2<CH>([&](int i) { return sigmoid1(at2(s[S1], i)); });
          publish(ring, ring.at(1, l, rt, member), at.on[rt] ? pk<CH>(make_float2(r.x * xs[rt].x, r.y * xs[rt].y)) : 0u);
          rw[rt] = pk<CH>(r);
          now.ux[rt][0] = s[0];
        }
      }
      auto results = [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int rt = 0; rt < TILES; ++rt) {
        if (KIND == K_RNN) bst2(zw[rt], zb, at.fs[rt]);
        if (KIND == K_GATED) {
          bst2(ow[rt], xb, at.xs[rt]);
          bst2(zw[rt], zb, at.fs[rt]);
          bst2(cw[rt], zb, at.fs[rt], h2);
          bst2(aw[rt], lb, at.xs[rt]);
        }
        if (KIND == K_LSTM) {
          bst2(hw[rt], xb, at.xs[rt], h2);
          bst2(cw[rt], xb, at.xs[rt]);
          bst2(zw[rt], zb, at.fs[rt]);
          bst2(rw[rt], zb, at.fs[rt], h2);
          bst2(ow[rt], zb, at.fs[rt], 2 * h2);
          bst2(gw[rt], zb, at.fs[rt], 3 * h2);
          bst2(rw[rt], lb, at.xs[rt]);
          bst2(0u, lb, at.xs[rt], h2);
        }
        if (KIND == K_GRU) {       // (the second half of the step works on the stored gate)
          const float2 s = now.ux[rt][0];
          zw[rt] = pk<CH>(map2<CH>([&](int i) { return sigmoid1(at2(s, i)); }));
          now.ux[rt][0] = un2<CH>(zw[rt]);
          bst2(zw[rt], zb, at.fs[rt]);
          bst2(rw[rt], zb, at.fs[rt], h2);
        }
      }
      };
      constexpr bool RESULTS_FIRST = KIND == K_RNN || (!AHEAD && !TWO);
      if (RESULTS_FIRST) results();
      if (LOCAL) empty_all();
      if (!ALONE) {
        if (TWO) in.template ask<PAUSE>(ring, 1, l);
        else if (AHEAD) {
          in.ask(ring, 0, l + 1);
          now = next;
          read_step(next);
          advance(l + 3 < a.L);
        } else {                 // (through memory: the inputs' trip is part of the wait for the others' words)
          read_step(now);
          advance(l + 2 < a.L);
          in.template ask<PAUSE>(ring, 0, l + 1);
        }
      }
      if (!RESULTS_FIRST) results();
      set ^= 1;
    });
    if (TWO) {
      members<ALONE>(own, ring.wpg, [&](int member) __attribute__((always_inline)) {
        if (ALONE) {
          x.base -= x.n; place(member); x.base += x.n;
          read_step(now);
          if (KIND == K_GRU) {
#pragma unroll
            for (int rt = 0; rt < TILES; ++rt) now.ux[rt][0] = un2<CH>(bld2(zb, at.f2[rt]));
          }
          in.ask(ring, 1, l);
        }
        in.wait(ring, 1, l, dead);
        Product<RT> acc;
        acc.clear();
        multiply_all(acc, ALONE ? weights(UNITS - 1, member) : w[ALONE ? 0 : UNITS - 1], in);
        put(part, set, 0, acc, wave, lane);
        meet();
        unsigned ow[TILES], nw[TILES], aw[TILES];
#pragma unroll
        for (int rt = 0; rt < TILES; ++rt) {
          float2 s = get(part, set, 0, 16 * rt + at.row, at.col);
          if (KIND == K_RNN) {
            const float2 lm = a.lambda ? now.lm[rt] : a.lambda_tok ? un2<CH>(now.lw[rt]) : make_float2(1.f, 1.f);
            ow[rt] = pk<CH>(map2<CH>([&](int i) { return at2(s, i) + at2(lm, i) * at2(xs[rt], i); }));
          } else {
            const float2 zg = now.ux[rt][0];
            const float2 nn = map2<CH>([&](int i) { return tanhf(at2(s, i) + at2(now.un[rt], i)); });
            const float2 av = make_float2(1.f - zg.x, 1.f - zg.y);
            ow[rt] = pk<CH>(map2<CH>([&](int i) { return fmaf(at2(av, i), at2(xs[rt], i), at2(zg, i) * at2(nn, i)); }));
            nw[rt] = pk<CH>(nn); aw[rt] = pk<CH>(av);
          }
          publish(ring, ring.at(0, l + 1, rt, member), at.on[rt] ? ow[rt] : 0u);
          xs[rt] = un2<CH>(ow[rt]);
        }
#pragma unroll
        for (int rt = 0; rt < TILES; ++rt) {
          bst2(ow[rt], xb, at.xs[rt]);
          if (KIND == K_GRU) {
            bst2(nw[rt], zb, at.fs[rt], 2 * h2);
            bst2(aw[rt], lb, at.xs[rt]);
          }
        }
        if (!ALONE) in.template ask<PAUSE>(ring, 0, l + 1);
        if (!ALONE) now = next;
        set ^= 1;
      });
    }
    if (ALONE) advance(l + 1 < a.L);
    z.next(true);
    lam.next(true);
  }
  return true;
}

// A fifth wavefront that has no part in the chain: it asks for the inputs of the step READ_AHEAD further on, a word of every 64 bytes,
// so that they are in the XCD's L2 when the others read them.  Loads return in order, so a wavefront that reads its inputs from memory
// waits for them where it waits for the exchanged words behind them.  The words land in a corner of LDS that nobody reads (direct
// copies: no register waits for one).  It meets every barrier of the chain, which keeps it in step.
// Measured, us, without / with it: 1024 steps of 32 x 1024, gated cell, forward, 1729 / 1439; 500 of 64 x 512, forward, LSTM 1142 / 957,
// gated cell 660 / 592, exact backpropagation of the RNN 793 / 720; 400 of 20 x 200, forward, GRU 633 / 589, RNN 526 / 492; the GRU of more
// channels at REC_GRU_AHEAD.
// Not for the LSTM and the GRU above 512 channels, whose registers do not leave room (two of five wavefronts share a SIMD: 256 each), nor the
// RNN (1024 steps of 32 x 1024 1650 / 1700, exact 1940 / 2130), nor backwards for the LSTM (no change) and the GRU of up to 256 channels
// (400 of 20 x 200 642 / 674), nor for one or two rows of that width for the gated cell (500 steps 509 /
// 539, of four rows 528 / 506).
constexpr int READ_AHEAD = 4;
// A workgroup of five wavefronts has a compute unit for itself; of four, two share one.  The GRU of 257 to 512 channels gains the least
// from reading ahead, and does so only with up to this many workgroups, of which four calls at once still find a place.  512 steps, ms for
// 1, 2, 4 and 8 calls at once, without / with it: 64 x 512 (128 workgroups), forward 1.01, 1.67, 1.82, 3.6 / 0.95, 1.12, 2.3, 4.4, exact
// backpropagation 0.82, 1.18, 1.46, 2.8 / 0.78, 0.92, 1.8, 3.5; 48 x 384 (72), forward 0.95, 1.24, 1.58, 3.2 / 0.89, 1.00, 2.56, 3.7; 32 x
// 512 (64), forward 0.95, 1.57, 2.8, 3.2 / 0.88, 0.98, 1.9, 2.3 (3.1), exact 0.82, 0.93, 1.4, 2.8 / 0.77, 0.80, 0.98, 2.6.
constexpr int REC_GRU_AHEAD = 64;
template <int KIND, int KQ, bool FORWARD> constexpr bool reads_ahead() {
  return (KQ < 8 || KIND == K_GATED) && (FORWARD || KIND == K_RNN || KIND == K_GATED || (KIND == K_GRU && KQ == 4));
}
template <int KIND, int RT, bool FORWARD>
__device__ __forceinline__ void read_ahead(const RecArgs& a, int group, int member, unsigned* corner) {
  constexpr int ROWS = rec_rows<RT>();
  constexpr int GATES = KIND == K_RNN ? 1 : KIND == K_GATED ? 2 : KIND == K_LSTM ? 4 : 3;
  // places of 64 bytes per row of the batch: forward, the gates' inputs (fp32: two each) and the RNN's coefficients per token;
  // backward, the gates, the state (not the RNN), the loss gradient and the coefficients (LSTM: of both parts)
  constexpr int PART = KIND == K_LSTM ? 2 : 1;
  constexpr int ITEMS = FORWARD ? 2 * GATES + (KIND == K_RNN ? 1 : 0) : GATES + (KIND == K_RNN ? 0 : 1) + 2 * PART;
  constexpr int SLOTS = (ITEMS * ROWS + 63) / 64;
  const int lane = threadIdx.x & 63;
  const long N = a.N, H = a.H, D = a.D, F = a.F, c0 = (long)member * REC_COLS;
  const char* at[SLOTS];
  long stride[SLOTS];
#pragma unroll
  for (int s = 0; s < SLOTS; ++s) {
    const int i = (lane + 64 * s) / ROWS;
    const long r = (long)group * ROWS + (lane + 64 * s) % ROWS;
    const char* base = nullptr;                    // of an array of W values of `size` bytes per row, from value c on
    long W = D, c = c0, end = KIND == K_RNN ? D : H;
    int size = 2;
    if (FORWARD) {
      if (i < 2 * GATES) {
        base = (const char*)a.ux; W = F; size = 4; end = KIND == K_RNN ? F : H;
        c = c0 + 16 * (i & 1);
        if (c < end) c += (i >> 1) * H; else base = nullptr;
        end = F;
      } else if (i < ITEMS) {
        base = (const char*)a.lambda_tok;
      }
    } else if (i < GATES) {
      base = (const char*)(KIND == K_RNN && a.dphi ? a.dphi : a.z); W = F; end = KIND == K_RNN ? F : H;
      if (c < end) c += i * H; else base = nullptr;
      end = F;
    } else if (i < ITEMS) {
      const int j = i - GATES - (KIND == K_RNN ? 0 : 1);     // -1: the state
      base = (const char*)(j < 0 ? a.x : j < PART ? a.e : a.lambda_tok);
      if (c >= end) base = nullptr;
      if (KIND == K_LSTM && j >= 0 && j % PART) c += H;
      end = D;
    }
    stride[s] = N * W * size;
    at[s] = base && r < N && c < end ? base + (r * W + c) * size : nullptr;
  }
  const unsigned place = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned*)corner;
#pragma unroll 1
  for (long l = 0; l < a.L; ++l) {
    const long step = FORWARD ? l + READ_AHEAD : a.L - 1 - l - READ_AHEAD;
    if (step >= 0 && step < a.L) {
#pragma unroll
      for (int s = 0; s < SLOTS; ++s) {
        if (at[s])
          asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %0, off\n"
                       :: "v"(at[s] + step * stride[s]), "s"(place) : "memory");
      }
    }
    __builtin_amdgcn_s_barrier();
    if (KIND == K_RNN || KIND == K_GRU) __builtin_amdgcn_s_barrier();
  }
  __builtin_amdgcn_s_waitcnt(0x0F70);              // (the last of them have landed before the LDS is given back)
}

template <int KIND, int KQ, int RT, bool LOCAL, bool AHEAD>
__global__ __launch_bounds__(AHEAD ? 320 : 256, 1) void rec_forward_kernel(RecArgs a, int wpg, int groups, int per, int locals) {
  constexpr int SLOTS = KIND == K_LSTM ? 4 : KIND == K_RNN ? 1 : 2;
  __shared__ __attribute__((aligned(16))) Partials<RT, SLOTS> part;
  int group, member;
  unsigned started;
  take_place<LOCAL>(a, wpg, groups, per, locals, group, member, started);
  if (group < 0) return;
  if constexpr (AHEAD) {
    __shared__ unsigned corner[64];
    if (threadIdx.x >= 256) {
      if (all_started<LOCAL>(a, wpg, group, started)) read_ahead<KIND, RT, true>(a, group, member, corner);
      return;
    }
  }
  const Ring<LOCAL, RT> ring(reinterpret_cast<char*>(a.ring), wpg, groups, group);
  const bool done = forward_chain<KIND, KQ, RT, false>(a, ring, member, started, part);
  if (!LOCAL && !done && member == 0) forward_chain<KIND, KQ, RT, true>(a, ring, member, started, part);
}

// Exact backpropagation: g[l] = (da_l W1 + what goes past the product) (+ e_l) + lambda_l (.) g[l+1], l = L-1 .. 0; da as in
// gated_cell.hip.  Weights transposed: Wt1 = W1^T [H][F] (GRU: [W_z; W_r]^T [H][2H]), Wt2 = W2^T [F][D] (RNN) or W_n^T [H][H].
template <int KIND, int KQ, int RT, bool ALONE, bool LOCAL>
__device__ __forceinline__ bool backward_chain(const RecArgs& a, const Ring<LOCAL, RT>& ring, int own, unsigned started,
                                               Partials<RT, 1>& part) {
  constexpr int UNITS = KIND == K_LSTM ? 4 : KIND == K_GRU ? 3 : 2;
  constexpr bool TWO = KIND == K_RNN || KIND == K_GRU;       // two dependent products per step
  constexpr int U0 = TWO ? 1 : 0;                            // first unit of the (second) product with W1
  constexpr int TILES = rec_tiles<RT>(), CH = rec_channels<RT>();
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int N = (int)a.N, H = (int)a.H, F = (int)a.F, D = (int)a.D;
  Weights<KQ> w[ALONE ? 1 : UNITS];
  auto weights = [&](int u, int member) __attribute__((always_inline)) -> Weights<KQ>& {
    Weights<KQ>& t = w[ALONE ? 0 : u];
    const int col0 = member * REC_COLS;
    if (TWO && u == 0) t.load((const bf16_t*)a.Wt2, KIND == K_RNN ? D : H, col0, KIND == K_RNN ? F : H, KIND == K_RNN ? D : H, wave, lane);
    else t.load((const bf16_t*)a.Wt1 + (long)(u - U0) * H, KIND == K_GRU ? 2 * H : F, col0, KIND == K_RNN ? D : H,
                KIND == K_RNN ? F : H, wave, lane);
    return t;
  };
  if (!ALONE) {
#pragma unroll
    for (int u = 0; u < UNITS; ++u) weights(u, own);
    if (!all_started<LOCAL>(a, ring.wpg, ring.group, started)) return false;     // (while the weights are on their way)
  }
  Operand<KQ, RT> in, in2;
  in.set(ring, wave, lane);
  in2.set(ring, wave, lane);
  // exchanged: the cells' da, a unit per gate; the RNN's da is unit 0 and its state gradient unit 1
  Place<RT> at;
  float2 gs[TILES], gc[TILES];             // the gradient's two channels as stored (LSTM: hidden and cell part)
  const long sx = (long)N * D, sf = (long)N * F, last = a.L - 1;
  const int h2 = 2 * H, ho = KIND == K_LSTM ? h2 : 0;        // a gate's distance in bytes, and the hidden part's
  Rows g = {(char*)a.g + 2 * sx * a.L, 2 * sx};              // g[l + 1]
  // the inputs of the step to be read (x: states l and l + 1)
  Rows lc = {(char*)a.lambda + (a.lambda ? 4 * last * D : 0), a.lambda ? 4L * D : 0};
  Rows lt = {(char*)a.lambda_tok + (a.lambda_tok ? 2 * last * sx : 0), a.lambda_tok ? 2 * sx : 0};
  Rows e = {(char*)a.e + (a.e ? 2 * last * sx : 0), a.e ? 2 * sx : 0};
  Rows x = {(char*)a.x + 2 * last * sx, 2 * sx};
  Rows z = {(char*)(KIND == K_RNN && a.dphi ? a.dphi : a.z) + 2 * last * sf, 2 * sf};
  auto place = [&](int member) __attribute__((always_inline)) {      // where the member's channels are, and its gradient
    at.set(ring.group, member, N, D, F, KIND == K_RNN ? D : H, KIND == K_RNN ? F : H);
#pragma unroll
    for (int rt = 0; rt < TILES; ++rt) {
      gs[rt] = un2<CH>(bld2(g.buf(), at.x2[rt], ho));
      gc[rt] = KIND == K_LSTM ? un2<CH>(bld2(g.buf(), at.x2[rt])) : make_float2(0.f, 0.f);
    }
  };
  members<ALONE>(own, ring.wpg, [&](int member) __attribute__((always_inline)) {
    place(member);
    if (KIND == K_RNN) {
#pragma unroll
      for (int rt = 0; rt < TILES; ++rt) publish(ring, ring.at(1, a.L, rt, member), bld2(g.buf(), at.x2[rt]));
    }
  });
  if (!ALONE && KIND == K_RNN) in.ask(ring, 1, a.L);
  bool dead = false;
  int set = 0;
  // what a step takes besides the gradient above it
  struct Inputs {
    unsigned lw[TILES], lw2[TILES], ew[TILES], ew2[TILES], zw[TILES][4], xw[TILES], xn[TILES];
    float2 lmf[TILES];
  };
  auto read_step = [&](Inputs& v) __attribute__((always_inline)) {
    const __amdgpu_buffer_rsrc_t lb = lc.buf(), tb = lt.buf(), eb = e.buf(), xb = x.buf(), zb = z.buf();
    const __amdgpu_buffer_rsrc_t nb = buffer(x.base + x.n, x.n);
#pragma unroll
    for (int rt = 0; rt < TILES; ++rt) {
      if (KIND == K_RNN) v.lmf[rt] = bldf2<CH>(lb, at.c4[rt]);
      v.lw[rt] = bld2(tb, at.x2[rt], ho);
      v.ew[rt] = bld2(eb, at.x2[rt], ho);
      if (KIND == K_LSTM) {
        v.lw2[rt] = bld2(tb, at.x2[rt]);
        v.ew2[rt] = bld2(eb, at.x2[rt]);
        v.xn[rt] = bld2(nb, at.x2[rt]);
      }
      if (KIND != K_RNN) v.xw[rt] = bld2(xb, at.x2[rt]);
#pragma unroll
      for (int q = 0; q < (KIND == K_RNN ? 1 : KIND == K_GATED ? 2 : KIND == K_GRU ? 3 : 4); ++q) v.zw[rt][q] = bld2(zb, at.f2[rt], q * h2);
    }
  };
  // the step to be read becomes the one before, or stays the first
  auto advance = [&](bool more) __attribute__((always_inline)) {
    lc.before(more); lt.before(more); e.before(more); x.before(more); z.before(more);
  };
  Inputs now, next;
  if (!ALONE) { read_step(now); advance(last > 0); }
#pragma unroll 1
  for (long l = last; l >= 0; --l) {
    float2 past[TILES], pastc[TILES];      // what reaches g[l] (hidden, cell) past the product with W1
    // the LSTM's gradient at the cell state through the hidden part
    auto tanh_c = [&](int rt) __attribute__((always_inline)) {
      const float2 cn = un2<CH>(now.xn[rt]);
      return map2<CH>([&](int i) { return tanhf(at2(cn, i)); });
    };
    auto through_h = [&](int rt, float2 tc) __attribute__((always_inline)) {
      const float2 og = un2<CH>(now.zw[rt][2]);
      return map2<CH>([&](int i) { return at2(gs[rt], i) * at2(og, i) * (1.f - at2(tc, i) * at2(tc, i)); });
    };
    // what the cells' elementwise parts leave for the products
    auto publish_gates = [&](int member) __attribute__((always_inline)) {
#pragma unroll
      for (int rt = 0; rt < TILES; ++rt) {
        const float2 G = gs[rt], xv = un2<CH>(now.xw[rt]);
        if (KIND == K_GATED) {
          const float2 u = un2<CH>(now.zw[rt][0]), cc = un2<CH>(now.zw[rt][1]);
          const float2 du = map2<CH>([&](int i) { return at2(G, i) * (at2(cc, i) - at2(xv, i)) * at2(u, i) * (1.f - at2(u, i)); });
          const float2 dc = map2<CH>([&](int i) { return at2(G, i) * at2(u, i) * (1.f - at2(cc, i) * at2(cc, i)); });
          publish(ring, ring.at(0, l, rt, member), at.on[rt] ? pk<CH>(du) : 0u);
          publish(ring, ring.at(1, l, rt, member), at.on[rt] ? pk<CH>(dc) : 0u);
        } else if (KIND == K_LSTM) {
          const float2 ig = un2<CH>(now.zw[rt][0]), fg = un2<CH>(now.zw[rt][1]), og = un2<CH>(now.zw[rt][2]), gg = un2<CH>(now.zw[rt][3]);
          const float2 tc = tanh_c(rt), th = through_h(rt, tc);
          pastc[rt] = make_float2(th.x * fg.x, th.y * fg.y);
          const float2 dct = make_float2(gc[rt].x + th.x, gc[rt].y + th.y);
          const float2 di = map2<CH>([&](int i) { return at2(dct, i) * at2(gg, i) * at2(ig, i) * (1.f - at2(ig, i)); });
          const float2 df = map2<CH>([&](int i) { return at2(dct, i) * at2(xv, i) * at2(fg, i) * (1.f - at2(fg, i)); });
          const float2 dO = map2<CH>([&](int i) { return at2(G, i) * at2(tc, i) * at2(og, i) * (1.f - at2(og, i)); });
          const float2 dg = map2<CH>([&](int i) { return at2(dct, i) * at2(ig, i) * (1.f - at2(gg, i) * at2(gg, i)); });
          publish(ring, ring.at(0, l, rt, member), at.on[rt] ? pk<CH>(di) : 0u);
          publish(ring, ring.at(1, l, rt, member), at.on[rt] ? pk<CH>(df) : 0u);
          publish(ring, ring.at(2, l, rt, member), at.on[rt] ? pk<CH>(dO) : 0u);
          publish(ring, ring.at(3, l, rt, member), at.on[rt] ? pk<CH>(dg) : 0u);
        } else if (KIND == K_GRU) {
          const float2 zg = un2<CH>(now.zw[rt][0]), nn = un2<CH>(now.zw[rt][2]);
          const float2 dn = map2<CH>([&](int i) { return at2(G, i) * at2(zg, i) * (1.f - at2(nn, i) * at2(nn, i)); });
          const float2 dz = map2<CH>([&](int i) { return at2(G, i) * (at2(nn, i) - at2(xv, i)) * at2(zg, i) * (1.f - at2(zg, i)); });
          publish(ring, ring.at(2, l, rt, member), at.on[rt] ? pk<CH>(dn) : 0u);
          publish(ring, ring.at(0, l, rt, member), at.on[rt] ? pk<CH>(dz) : 0u);
        }
      }
    };
    // RNN: g W2; GRU: what comes back through the candidate's product, dn W_n
    auto first_product = [&](int member) __attribute__((always_inline)) {
      constexpr int U = KIND == K_RNN ? 1 : 2;
      const long at_l = KIND == K_RNN ? l + 1 : l;
      if (ALONE) in.ask(ring, U, at_l);
      in.wait(ring, U, at_l, dead);
      if (!ALONE) { read_step(next); advance(l > 1); }
      Product<RT> acc;
      acc.clear();
      multiply_all(acc, ALONE ? weights(0, member) : w[0], in);
      put(part, set, 0, acc, wave, lane);
      meet();
    };
    // the operands of the product with W1: the first two units are asked for together, each later one as soon as its registers are
    // free (the LSTM with two row tiles has registers for one unit: 24 would be spilled)
    constexpr int HELD = UNITS - U0 == 1 || (KIND == K_LSTM && RT == 2) ? 1 : 2;
    auto ask_second = [&]() __attribute__((always_inline)) {
      in.ask(ring, 0, l);
      if (HELD == 2) in2.ask(ring, 1, l);
    };
    if (KIND != K_RNN) {
      members<ALONE>(own, ring.wpg, [&](int member) __attribute__((always_inline)) {
        if (ALONE) { place(member); read_step(now); }
        publish_gates(member);
        if (!ALONE) {
          if (TWO) in.ask(ring, 2, l);
          else ask_second();
        }
      });
    }
    if (TWO) {
      members<ALONE>(own, ring.wpg, [&](int member) __attribute__((always_inline)) {
        if (ALONE) { place(member); read_step(now); }
        first_product(member);
#pragma unroll
        for (int rt = 0; rt < TILES; ++rt) {
          const float2 s = get(part, set, 0, 16 * rt + at.row, at.col);
          if (KIND == K_RNN) {
            const float2 t = un2<CH>(now.zw[rt][0]);
            const float2 v = map2<CH>([&](int i) {
              return at2(s, i) * (a.dphi ? at2(t, i) : a.tanh_act ? 1.f - at2(t, i) * at2(t, i) : 1.f);
            });
            publish(ring, ring.at(0, l, rt, member), at.on_f[rt] ? pk<CH>(v) : 0u);
          } else {
            const float2 r = un2<CH>(now.zw[rt][1]), xv = un2<CH>(now.xw[rt]);
            const float2 dr = map2<CH>([&](int i) { return at2(s, i) * at2(xv, i) * at2(r, i) * (1.f - at2(r, i)); });
            publish(ring, ring.at(1, l, rt, member), at.on[rt] ? pk<CH>(dr) : 0u);
            past[rt] = make_float2(s.x * r.x, s.y * r.y);
          }
        }
        // every workgroup of the group has left step l + 1 (at the last step: slots that are empty yet)
        empty(ring, 0, l + 1, member);
        empty(ring, 1, KIND == K_RNN ? l + 2 : l + 1, member);
        if (KIND == K_GRU) empty(ring, 2, l + 1, member);
        if (!ALONE) {
          ask_second();
        }
        set ^= 1;
      });
    }
    members<ALONE>(own, ring.wpg, [&](int member) __attribute__((always_inline)) {
      if (ALONE) { place(member); read_step(now); }
      if (KIND == K_GRU && ALONE) {      // (the sum that the member's registers hold otherwise)
        first_product(member);
#pragma unroll
        for (int rt = 0; rt < TILES; ++rt) {
          const float2 s = get(part, set, 0, 16 * rt + at.row, at.col), r = un2<CH>(now.zw[rt][1]);
          past[rt] = make_float2(s.x * r.x, s.y * r.y);
        }
        set ^= 1;
      }
#pragma unroll
      for (int rt = 0; rt < TILES; ++rt) {
        if (KIND != K_GRU) past[rt] = make_float2(0.f, 0.f);
        if (KIND == K_LSTM && ALONE) {
          const float2 th = through_h(rt, tanh_c(rt)), fg = un2<CH>(now.zw[rt][1]);
          pastc[rt] = make_float2(th.x * fg.x, th.y * fg.y);
        }
      }
      if (ALONE) ask_second();
      Product<RT> acc;
      acc.clear();
#pragma unroll
      for (int u = 0; u < UNITS - U0; ++u) {
        Operand<KQ, RT>& o = HELD == 2 && (u & 1) ? in2 : in;
        o.wait(ring, u, l, dead);
        // (one product per step: behind the first operands, so that reading those again does not wait for memory; 1024 steps of
        // 32 x 1024 on one XCD 4 to 5 % faster for the gated cell and 2.8 % for the LSTM, 8 to 11 steps through memory the same)
        if (!ALONE && !TWO && u == 0) { read_step(next); advance(l > 1); }
        multiply_all(acc, ALONE ? weights(u + U0, member) : w[ALONE ? 0 : u + U0], o);
        if (u + HELD < UNITS - U0) o.ask(ring, u + HELD, l);
      }
      put(part, set, 0, acc, wave, lane);
      meet();
      unsigned o[TILES], oc[TILES];
#pragma unroll
      for (int rt = 0; rt < TILES; ++rt) {
        const float2 s = get(part, set, 0, 16 * rt + at.row, at.col);
        const float2 ev = un2<CH>(now.ew[rt]);
        const float2 lm = a.lambda_tok ? un2<CH>(now.lw[rt]) : KIND == K_RNN && a.lambda ? now.lmf[rt] : make_float2(1.f, 1.f);
        o[rt] = pk<CH>(map2<CH>([&](int i) { return (at2(s, i) + at2(past[rt], i) + at2(ev, i)) + at2(lm, i) * at2(gs[rt], i); }));
        if (KIND == K_RNN) publish(ring, ring.at(1, l, rt, member), at.on[rt] ? o[rt] : 0u);
        gs[rt] = un2<CH>(o[rt]);
        if (KIND == K_LSTM) {
          const float2 e2 = un2<CH>(now.ew2[rt]), l2 = un2<CH>(now.lw2[rt]);
          oc[rt] = pk<CH>(map2<CH>([&](int i) { return (at2(pastc[rt], i) + at2(e2, i)) + at2(l2, i) * at2(gc[rt], i); }));
          gc[rt] = un2<CH>(oc[rt]);
        }
      }
      if (!TWO) {
#pragma unroll
        for (int u = 0; u < UNITS; ++u) empty(ring, u, l + 1, member);
      }
      const __amdgpu_buffer_rsrc_t gb = buffer(g.base - g.n, g.n);       // g[l]
#pragma unroll
      for (int rt = 0; rt < TILES; ++rt) {
        bst2(o[rt], gb, at.xs[rt], ho);
        if (KIND == K_LSTM) bst2(oc[rt], gb, at.xs[rt]);
      }
      if (!ALONE && KIND == K_RNN) in.ask(ring, 1, l);
      if (!ALONE) now = next;
      set ^= 1;
    });
    if (ALONE) advance(l > 0);
    g.before(true);
  }
  return true;
}

template <int KIND, int KQ, int RT, bool LOCAL, bool AHEAD>
__global__ __launch_bounds__(AHEAD ? 320 : 256, 1) void rec_backward_kernel(RecArgs a, int wpg, int groups, int per, int locals) {
  __shared__ __attribute__((aligned(16))) Partials<RT, 1> part;
  int group, member;
  unsigned started;
  take_place<LOCAL>(a, wpg, groups, per, locals, group, member, started);
  if (group < 0) return;
  if constexpr (AHEAD) {
    __shared__ unsigned corner[64];
    if (threadIdx.x >= 256) {
      if (all_started<LOCAL>(a, wpg, group, started)) read_ahead<KIND, RT, false>(a, group, member, corner);
      return;
    }
  }
  const Ring<LOCAL, RT> ring(reinterpret_cast<char*>(a.ring), wpg, groups, group);
  const bool done = backward_chain<KIND, KQ, RT, false>(a, ring, member, started, part);
  if (!LOCAL && !done && member == 0) backward_chain<KIND, KQ, RT, true>(a, ring, member, started, part);
}

// the empty word into every slot (n 16-byte pieces); the words of the places at zero, but for those of the groups (`word`) and of
// the groups on one XCD whose number modulo 16 has its bit set in `gone`
__global__ __launch_bounds__(256) void rec_fill_kernel(uint4* p, long n, PlaceWords* places, unsigned word, unsigned gone) {
  const long i = (long)blockIdx.x * 256 + threadIdx.x;
  if (i < n) p[i] = make_uint4(REC_EMPTY, REC_EMPTY, REC_EMPTY, REC_EMPTY);
  if (blockIdx.x == 0) {
    constexpr int LOCAL0 = offsetof(PlaceWords, local) / 4;
    for (int j = threadIdx.x; j < (int)(sizeof(PlaceWords) / 4); j += 256)
      reinterpret_cast<unsigned*>(places)[j] =
          j >= 1 && j < 1 + REC_MAX_WG                                                              ? word
          : j >= LOCAL0 && j < LOCAL0 + REC_LOCAL_GROUPS && ((gone >> ((j - LOCAL0) & 15)) & 1u) ? REC_ALONE
                                                                                                   : 0u;
  }
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
// The groups on one XCD each: of 8 rows where every XCD of the eight then has a compute unit for each workgroup, else of 16.
// Half the rows are half the bytes that a workgroup reads in every phase (32 KB at width 1024 and 16 rows, 500 cycles at a
// compute unit's 64 bytes), for the same number of matrix instructions.  Widths to 512, where those bytes weigh less: only as long as
// that leaves half of the chip to others.  Measured, 512 steps of 128 x 512, ms, all of the chip in groups of 8 / half of it in groups
// of 16, one call | two at once | four: RNN forward 0.82 / 0.83 | 1.30 / 1.24 | 2.35 / 2.39, GRU 1.10 / 1.19 | 1.64 / 1.62 | 6.1 / 2.3,
// LSTM 1.32 / 1.52 | 4.3 / 2.0 | 6.4 / 5.1, exact backpropagation of the GRU 1.00 / 0.99 | 1.22 / 1.28 | 4.7 / 1.4; 64 x 1024: GRU
// 1.18 / 1.53 | 2.3 / 1.6 | 4.5 / 4.7, exact 1.13 / 1.21 | 2.2 / 1.3 | 4.1 / 4.0, LSTM 1.54 / 1.82 | 2.9 / 1.9 | 5.2 / 5.2.
inline bool rec_half(const RecArgs& a, long wpg) {
  const long n = (a.N + 7) / 8, xcds = wpg > 16 ? 8 : 4;
  return (n + xcds - 1) / xcds * wpg <= 32 && n * ((wpg + 1) / 2) <= REC_MAX_WG * 2;       // (and the vectors fit their memory)
}

// RT: row tiles of the groups anywhere, RTL: of those on one XCD
template <int KIND, int KQ, int RT, int RTL>
hipError_t launch_rec(const RecArgs& a, bool forward, hipStream_t s) {
  const long wpg = (rec_width(a) + REC_COLS - 1) / REC_COLS;
  const int groups = (int)((a.N + rec_rows<RT>() - 1) / rec_rows<RT>()), locals = (int)((a.N + rec_rows<RTL>() - 1) / rec_rows<RTL>());
  const long ring = (long)REC_UNITS * REC_SLOTS * groups * RT * wpg * 1024;
  const long ring_local = (long)REC_UNITS * REC_SLOTS * locals * (RTL ? wpg : (wpg + 1) / 2) * 1024;
  const bool on_xcd = (a.wait & 255) == REC_ON_XCD, local = on_xcd || (a.wait == REC_WAIT && a.L >= REC_LOCAL_FROM);
  const long n16 = (ring + (local ? ring_local : 0)) / 16;
  hipLaunchKernelGGL(rec_fill_kernel, dim3((unsigned)((n16 + 255) / 256)), dim3(256), 0, s, reinterpret_cast<uint4*>(a.ring), n16,
                     reinterpret_cast<PlaceWords*>(a.counter), a.wait == REC_ALONE_ANYHOW ? REC_ALONE : 0u,
                     on_xcd ? (unsigned)a.wait >> 8 : 0u);
  // enough workgroups that every XCD of the eight has a group's number of them for each group it can be asked to take
  const dim3 everywhere((unsigned)(8 * wpg * ((locals + 7) / 8))), anywhere((unsigned)(groups * wpg));
  RecArgs l = a;
  l.ring = reinterpret_cast<char*>(a.ring) + ring;
  const int per = rec_rows<RT>() / rec_rows<RTL>();
  auto on_xcds = [&](auto kern, bool ahead) { hipLaunchKernelGGL(kern, everywhere, dim3(ahead ? 320 : 256), 0, s, l, (int)wpg, locals, 1, 0); };
  constexpr bool FW = reads_ahead<KIND, KQ, true>(), BW = reads_ahead<KIND, KQ, false>();
  constexpr bool GRU4 = KIND == K_GRU && KQ == 4, GATED2 = KIND == K_GATED && KQ == 2;
  const bool crowded = GRU4 && locals * wpg > REC_GRU_AHEAD;
  if (forward) {
    if (local && crowded) on_xcds(rec_forward_kernel<KIND, KQ, RTL, true, FW && !GRU4>, false);
    else if (local) on_xcds(rec_forward_kernel<KIND, KQ, RTL, true, FW>, FW);
    hipLaunchKernelGGL((rec_forward_kernel<KIND, KQ, RT, false, false>), anywhere, dim3(256), 0, s, a, (int)wpg, groups, per, local ? locals : 0);
  } else {
    if (local && (crowded || (GATED2 && a.N <= 2))) on_xcds(rec_backward_kernel<KIND, KQ, RTL, true, BW && !GRU4 && !GATED2>, false);
    else if (local) on_xcds(rec_backward_kernel<KIND, KQ, RTL, true, BW>, BW);
    hipLaunchKernelGGL((rec_backward_kernel<KIND, KQ, RT, false, false>), anywhere, dim3(256), 0, s, a, (int)wpg, groups, per, local ? locals : 0);
  }
  return hipGetLastError();
}
template <int KIND, int KQ>
hipError_t launch_rec_rows(const RecArgs& a, bool forward, hipStream_t s) {
  const bool half = rec_half(a, (rec_width(a) + REC_COLS - 1) / REC_COLS);
  if (rec_row_tiles(a) == 1) return half ? launch_rec<KIND, KQ, 1, 0>(a, forward, s) : launch_rec<KIND, KQ, 1, 1>(a, forward, s);
  return half ? launch_rec<KIND, KQ, 2, 0>(a, forward, s) : launch_rec<KIND, KQ, 2, 1>(a, forward, s);
}
template <int KIND>
hipError_t launch_rec_kind(const RecArgs& a, bool forward, hipStream_t s) {
  const long K = KIND == K_RNN ? rec_width(a) : a.H;
  if (K <= 256) return launch_rec_rows<KIND, 2>(a, forward, s);
  if (K <= 512) return launch_rec_rows<KIND, 4>(a, forward, s);
  return launch_rec_rows<KIND, 8>(a, forward, s);
}

}  // namespace

// the groups anywhere (at most REC_MAX_WG workgroups of two tiles), and those on one XCD each: at most 8 x 32 workgroups of half
// a tile, or twice REC_MAX_WG of a tile
size_t recurrent_ring_bytes() { return (size_t)REC_UNITS * REC_SLOTS * REC_MAX_WG * 2 * 1024 * 2; }
// What fits: bf16, widths whose weights the registers hold (1024) and at most 64 workgroups (two row tiles each: 64 rows at
// width 1024, 128 at 512).  Everything else goes step by step (7 us per product against 0.8 to 1.6).
bool recurrent_ok(const RecArgs& a) {
  if (a.H % 8 || a.D % 8 || a.F % 8 || rec_width(a) > 1024 || rec_row_tiles(a) == 0) return false;
  if (a.N * a.F > (1L << 30) || a.N * a.D > (1L << 30)) return false;
  return ok16(a.x) && ok16(a.z) && ok16(a.W1) && ok16(a.W2) && ok16(a.Wt1) && ok16(a.Wt2) && ok16(a.g) &&
         ok16(a.ring) && ok16(a.ux) && ok16(a.lambda) && ok16(a.lambda_tok) && ok16(a.e) && ok16(a.dphi);
}
void recurrent_on_xcd(const RecArgs& a, int* groups, int* members, size_t* offset) {
  const long wpg = (rec_width(a) + REC_COLS - 1) / REC_COLS;
  *groups = (int)(rec_half(a, wpg) ? (a.N + 7) / 8 : (a.N + 15) / 16);
  *members = (int)wpg;
  *offset = offsetof(PlaceWords, local);
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
