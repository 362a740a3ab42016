// Both substitution passes of a solve as ONE launch (paper, Section "Introduction": LU and Cholesky are named as the
// factorisations behind solving systems of linear equations).  The block step of solve.hip,
//   X_i = Z_i - M_i [X_{i-2}; X_{i-1}],   Z_i = W_i S_i,   S_i = B_i - sum_{j<i-2} L_ij X_j
// over row blocks of 256, mirrored in the backward pass, is split into workgroups of 16 rows and 16 NB right-hand sides
// that wait in place for what they read:
//   sum workgroups       accumulate  sum_j L_ij X_j  over the blocks j as they appear and publish their piece of S_i;
//   solution workgroups  hold their rows of W_i and M_i in registers before anything they wait for is there, multiply
//                        S_i, X_{i-2}, X_{i-1} in the order in which these appear, and publish their piece of X_i.
// The four waves of a workgroup (one per SIMD) split k and add their partial blocks through LDS in a fixed order, so the
// result depends neither on timing nor on the launch.
//
// What bounds it is the hop X_{i-1} -> X_i, 2 n / 256 of them in sequence: a store to the device's point of coherence, a
// load from it, 16 dependent MFMAs a wave, a rendezvous in LDS.  Measured 3.2 - 4 us a hop with few right-hand sides, where a
// launch per hop takes 6.6 - 8: prepared LU solves, fp64, n = 4000 with 1 right-hand side 211 -> 102 us, with 64 255 -> 186,
// n = 8192 571 -> 271 and 746 -> 566.  (One counter that deals the pieces out, instead of the claims below: 150, 243, 367, 743; two
// thousand atomics on one address.)
//
// Hand-over.  A piece of X or S is its own signal: the areas the passes publish in are filled with a bit pattern that is never
// published (kEmpty, a NaN; a result with these bits is stored as another NaN), every element is stored and loaded as an
// atomic of device scope, and a reader loads its operand again until no element is empty.  No counter and no fence is
// needed, and nothing is assumed about the order of two stores.  The sum workgroups, many readers of one block, first look at a
// flag that each piece of X also sets, and then load through their L2; an element that is still empty there is loaded from the
// point of coherence.  A solution workgroup looks at flags, too, until the block two positions back can be there.
//
// Order.  A piece waits only for pieces with a smaller index, and a workgroup begins with the piece of its own index.  An XCD
// starts its share of the workgroups in order, but knows nothing of the others': two such launches on two streams can fill each an
// XCD with workgroups that wait for one that the other launch keeps from starting.  So a piece belongs to the workgroup that has
// claimed it, and one that has waited for kFlowSearchTicks gives its piece back, takes the first piece up to its own that nobody
// has, and so on until there is none.  The first piece that is not done is then always at work or taken next, whichever workgroups
// of a launch are there, and every launch ends.  What is published is checked against the claim, so a workgroup that starts late
// and finds its piece taken has only wasted its time.
// A launch that does not come on for kFlowWaitTicks all the same (none is known that would not) gives up: every wait ends, and the
// last workgroup of a column tile to finish substitutes row by row for it (flow_recover): B is not written before the forward pass
// of the tile is complete, and Y never after, so nothing it needs is lost.  It takes 0.27 s at n = 4096 with 1 right-hand side, 0.53 s
// with 64, and grows with n^2.
#pragma once
#include <type_traits>
#include "dla_common.hpp"

namespace dla {

constexpr int kFlowThreads = 256;
constexpr int kFlowBlock = 256;               // rows of a block of the substitution
constexpr int kFlowTiles = kFlowBlock / 16;   // workgroups along a block's rows
constexpr int kFlowLook = 2;                  // blocks that M covers
constexpr long long kFlowSearchTicks = 200000;  // 2 ms of the 100 MHz wall clock, several times the longest solve up to n = 8192
constexpr long long kFlowWaitTicks = 100000000; // 1 s

constexpr int kFlowCoherent = 16;             // sc1: a load from the device's point of coherence

template <typename T>
struct FlowBits;
template <>
struct FlowBits<double> {
  using type = unsigned long long;
  static constexpr type kEmpty = 0x7FF9D1A5C3B2E607ull;
};
template <>
struct FlowBits<float> {
  using type = unsigned int;
  static constexpr type kEmpty = 0x7FD1A5C3u;
};

constexpr int64_t kFlowMaxLd = 1000000;       // 256 rows of the factor lie within 2 GiB

template <typename T>
struct FlowArgs {
  const T* F;      // the factor
  T* B;            // right-hand sides, overwritten by X
  const T* nf;     // negated inverses of the diagonal blocks, forward pass: 256 x 256 each
  const T* nb;     // and backward pass (Cholesky: the same, read transposed)
  const T* mf;     // M of the forward pass: 256 x 512 each
  const T* mb;     // M of the backward pass (Cholesky: its transpose, 512 x 256)
  T* Y;            // solution of the forward pass
  T* X;            // solution of the backward pass
  T* S;            // what the blocks start from, forward pass; the backward pass's lies behind it
  int* flags;      // [pass][position][column tile][16]: the piece of X_i is there
  int* done;       // [column tile]: pieces that are through;  behind them: a wait has given up
  int* claims;     // [piece]: a workgroup has it
  long long wait_ticks, search_ticks;
  int absent;      // -1, or (diagnostic) of the workgroups with this index modulo 8 only those of the last block solved are there
  int64_t lda, ldb, ldy;
  int n, nrhs, blocks, tiles_n, expected;  // expected: pieces per column tile
};

// Position p of a pass (p-th block solved) has a sum from p = kFlowLook + 1 on.
__host__ __device__ inline int flow_groups(int blocks) { return blocks + (blocks > kFlowLook + 1 ? blocks - kFlowLook - 1 : 0); }
__host__ __device__ inline int flow_pieces(int blocks, int tiles_n) { return 2 * flow_groups(blocks) * kFlowTiles * tiles_n; }
// Piece number id: pass, position, sum or solution, 16 rows, 16 NB columns.  The column tiles of the same rows are eight pieces
// apart, so that one XCD's L2 serves their left operand.
struct FlowPiece {
  bool back, sum;
  int p, rt, ct;
  __host__ __device__ int block(int blocks) const { return back ? blocks - 1 - p : p; }
};
__host__ __device__ inline FlowPiece flow_piece(int id, int blocks, int tiles_n) {
  const int per_group = kFlowTiles * tiles_n, groups = flow_groups(blocks), sums = groups - blocks;
  FlowPiece f;
  f.back = id >= groups * per_group;
  if (f.back) id -= groups * per_group;
  // X_0, X_1, then  S_3 X_2, S_4 X_3, ...: a sum as early as its last block allows; at the end the solutions without a sum
  const int group = id / per_group, local = id % per_group;
  f.p = group;
  f.sum = false;
  if (group >= kFlowLook) {
    const int pair = (group - kFlowLook) / 2;
    if (pair < sums) {
      f.sum = (group - kFlowLook) % 2 == 0;
      f.p = pair + (f.sum ? kFlowLook + 1 : kFlowLook);
    } else {
      f.p = group - sums;
    }
  }
  f.rt = (local / (kNumXcd * tiles_n)) * kNumXcd + local % kNumXcd;
  f.ct = (local / kNumXcd) % tiles_n;
  return f;
}
// Whether there is such a piece (the last block of the matrix may have fewer rows).
__host__ __device__ inline bool flow_piece_is(const FlowPiece& f, int n, int blocks) { return f.block(blocks) * kFlowBlock + f.rt * 16 < n; }
inline int flow_expected(int n, int blocks) {
  const int full = blocks > kFlowLook + 1 ? blocks - kFlowLook - 1 : 0;  // blocks with a sum
  return 2 * ((n + 15) / 16) + full * kFlowTiles + (full ? (n + 15) / 16 - (kFlowLook + 1) * kFlowTiles : 0);
}
inline int64_t flow_ints(int64_t blocks, int tiles_n) { return 2 * blocks * tiles_n * kFlowTiles + tiles_n + 1 + flow_pieces((int)blocks, tiles_n); }

// What a launch finds: two areas of count elements each empty, no flag set, no piece claimed or done.  By the launch in front of it
// (the pre-pass's first, or one of its own), kFlowThreads to a workgroup.
template <typename T>
struct FlowInit {
  T* area;
  T* sums;        // or null
  int64_t count;  // 0: nothing to do
  int* ints;
  int nints;
};
constexpr int kFlowInitPerThread = 8;
template <typename T>
inline int flow_init_workgroups(const FlowInit<T>& a) {
  const int64_t most = a.count > a.nints ? a.count : a.nints;
  return (int)((most + kFlowThreads * kFlowInitPerThread - 1) / (kFlowThreads * kFlowInitPerThread));
}
template <typename T>
__device__ __forceinline__ void flow_init(const FlowInit<T>& a, int wg) {
#pragma unroll
  for (int e = 0; e < kFlowInitPerThread; ++e) {
    const int64_t i = ((int64_t)wg * kFlowInitPerThread + e) * kFlowThreads + threadIdx.x;
    if (i < a.count) {
      a.area[i] = __builtin_bit_cast(T, FlowBits<T>::kEmpty);
      if (a.sums) a.sums[i] = __builtin_bit_cast(T, FlowBits<T>::kEmpty);
    }
    if (i < a.nints) a.ints[i] = 0;
  }
}
template <typename T>
__global__ void __launch_bounds__(kFlowThreads) flow_init_kernel(const FlowInit<T> a) {
  flow_init(a, (int)blockIdx.x);
}

template <int SCOPE = __HIP_MEMORY_SCOPE_AGENT, typename T>
__device__ __forceinline__ T flow_load(const T* p) {
  using U = typename FlowBits<T>::type;
  return __builtin_bit_cast(T, __hip_atomic_load(reinterpret_cast<const U*>(p), __ATOMIC_RELAXED, SCOPE));
}
template <typename T>
__device__ __forceinline__ bool flow_there(T x) {
  return __builtin_bit_cast(typename FlowBits<T>::type, x) != FlowBits<T>::kEmpty;
}
// over the wave, as a value that the compiler knows to be uniform: no branch on it is a divergent one
__device__ __forceinline__ bool flow_all(bool x) { return __builtin_amdgcn_ballot_w64(!x) == 0; }
template <typename T>
__device__ __forceinline__ void flow_store(T* p, T x) {
  using U = typename FlowBits<T>::type;
  U u = __builtin_bit_cast(U, x);
  if (u == FlowBits<T>::kEmpty) u ^= 1;
  __hip_atomic_store(reinterpret_cast<U*>(p), u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Where a workgroup's wait hands what it has found from one wave to the others, with one barrier between the two: the next wait
// takes the other slot, however many positions were found, so that a slot is written again only behind the barrier of the wait
// between, in front of which every wave has read it.
struct FlowSlots {
  int waits = 0;
  __host__ __device__ int next() { return waits++ & 1; }
};

template <typename T, int NB>
struct FlowTile {  // (32-bit byte offsets throughout: kFlowMaxLd)
  static constexpr int STEPS = kFlowBlock / 16;  // k-steps of a wave per block
  using acc_t = typename Mfma<T>::acc_t;
  using vec2_t = typename Mfma<T>::vec2_t;

  int lane, wave, l15, kq;
  int col[NB];        // this lane's columns, clamped
  int* gave_up;       // the launch's flag
  long long limit;    // of a wait
  bool last_try;      // behind it the launch gives up
  int late = 0;       // a wait of this wave has ended without what it waited for: 1 to look for work, 2 the launch has given up

  // k of step s: pairs dealt round-robin to the waves and lane groups, as the left operand's pairs are one load
  static __device__ __forceinline__ int k_step(int s) { return 32 * (s >> 1) + (s & 1); }
  __device__ __forceinline__ int k_of(int s) const { return kq + k_step(s); }

  // a wait that is not over yet: true to go on waiting
  __device__ __forceinline__ bool again(int spins, long long t0) {
    if (spins % 32 == 31 || limit == 0) {
      if (!flow_all(__hip_atomic_load(gave_up, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0)) {
        late = 2;
      } else if (wall_clock64() - t0 > limit) {
        late = last_try ? 2 : 1;
        if (last_try) __hip_atomic_store(gave_up, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    }
    return late == 0;
  }

  static __device__ __forceinline__ T load_one(__amdgpu_buffer_rsrc_t rs, int vo, int so) {
    if constexpr (sizeof(T) == 8) return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(rs, vo, so, 0));
    else return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(rs, vo, so, 0));
  }
  // 16 rows of a left operand, row `row` for this lane: element (row, k) at base[row * ld + k], TRANS: base[k * ld + row].
  // Beyond kc: zero, by the resource's extent or an offset outside of it.
  template <bool TRANS>
  __device__ __forceinline__ void load_left(T (&a)[STEPS], const T* base, int ld, int row, int kc) const {
    constexpr int E = (int)sizeof(T);
    constexpr int kOob = 0x7FFFFFF0;  // the extent is below
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(base), 0, TRANS ? kc * ld * E : ((kFlowBlock - 1) * ld + kFlowBlock) * E, 0x00020000);
    if constexpr (TRANS) {
#pragma unroll
      for (int s = 0; s < STEPS; ++s) a[s] = load_one(rs, (kq * ld + row) * E, k_step(s) * ld * E);
    } else if (kc == kFlowBlock) {  // uniform
#pragma unroll
      for (int s = 0; s < STEPS; s += 2) {
        if constexpr (E == 8) {
          const double2_t v = __builtin_bit_cast(double2_t, __builtin_amdgcn_raw_buffer_load_b128(rs, (row * ld + kq) * E, k_step(s) * E, 0));
          a[s] = v[0];
          a[s + 1] = v[1];
        } else {
          const float2_t v = __builtin_bit_cast(float2_t, __builtin_amdgcn_raw_buffer_load_b64(rs, (row * ld + kq) * E, k_step(s) * E, 0));
          a[s] = v[0];
          a[s + 1] = v[1];
        }
      }
    } else {
#pragma unroll
      for (int s = 0; s < STEPS; ++s) a[s] = load_one(rs, k_of(s) < kc ? (row * ld + k_of(s)) * E : kOob, 0);
    }
  }

  // kc rows of an area (ld: its leading dimension); true if no element is empty.  Buffer loads: the extent makes what lies
  // beyond kc zero, and one lane offset serves all steps (with flat addresses the variants of this load took 110 more
  // registers between them).  AUX: cache policy, 0 or kFlowCoherent.
  template <int AUX>
  __device__ __forceinline__ bool load_area(T (&b)[NB][STEPS], const T* base, int ld, int kc) const {
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(base), 0, kc * ld * (int)sizeof(T), 0x00020000);
    asm volatile("" ::: "memory");  // each call loads anew
#pragma unroll
    for (int s = 0; s < STEPS; ++s)
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        const int vo = (kq * ld + col[j]) * (int)sizeof(T), so = k_step(s) * ld * (int)sizeof(T);
        if constexpr (sizeof(T) == 8) b[j][s] = __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(rs, vo, so, AUX));
        else b[j][s] = __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(rs, vo, so, AUX));
      }
    bool there = true;
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int s = 0; s < STEPS; ++s) there = there & flow_there(b[j][s]);
    return flow_all(there);
  }
  // again and again until no element is empty
  __device__ __forceinline__ void load_published(T (&b)[NB][STEPS], const T* base, int ld, int kc) {
    const long long t0 = wall_clock64();
    for (int spins = 0;; ++spins)
      if (load_area<kFlowCoherent>(b, base, ld, kc) || !again(spins, t0)) break;
  }
  // kc rows of the right-hand sides
  __device__ __forceinline__ void load_rhs(T (&b)[NB][STEPS], const T* base, int64_t ld, int kc) const {
#pragma unroll
    for (int s = 0; s < STEPS; ++s) {
      const int k = k_of(s);
      const T* const q = base + (k < kc ? k : kc - 1) * ld;
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        b[j][s] = q[col[j]];
        if (k >= kc) b[j][s] = T(0);
      }
    }
  }

  // the workgroup waits for the first `count` of 16 flags: one wave looks at them, every `pause` (64 cycles each)
  template <int PAUSE>
  __device__ __forceinline__ void wait_flags(const int* flags, int count) {
    if (wave == 0) {
      const int* const p = flags + (l15 < count ? l15 : count - 1);
      const long long t0 = wall_clock64();
      for (int spins = 0; late == 0; ++spins) {
        if (flow_all(__hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) || !again(spins, t0)) break;
        __builtin_amdgcn_s_sleep(PAUSE);
      }
    }
    lds_barrier();
  }

  // as wait_flags for the pieces of position 0; tells how many positions from there on are complete (of the `left` that there
  // are, `stride` flags apart, all whole but perhaps the first): looks at up to 4 if `behind`, which it is for the next time
  // if it has not had to wait
  template <int PAUSE>
  __device__ __forceinline__ int wait_positions(const int* flags, int stride, int count, int left, bool& behind, int* shared) {
    if (wave == 0) {
      const int pos = behind ? lane >> 4 : 0;
      const bool off = pos >= left || (pos == 0 && l15 >= count);
      const int* const p = flags + (off ? 0 : pos * stride + l15);
      const long long t0 = wall_clock64();
      unsigned long long missing = 0;
      int spins = 0;
      for (; late == 0; ++spins) {
        missing = __builtin_amdgcn_ballot_w64(__hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0);
        if ((missing & 0xFFFF) == 0 || !again(spins, t0)) break;
        __builtin_amdgcn_s_sleep(PAUSE);
      }
      int whole = !behind ? 1 : missing == 0 ? 4 : (int)(__builtin_ctzll(missing) >> 4);
      whole = whole < left ? (whole < 1 ? 1 : whole) : left;
      if (lane == 0) *shared = 2 * whole + (spins == 0 ? 1 : 0);
    }
    lds_barrier();
    const int found = __builtin_amdgcn_readfirstlane(*shared);
    behind = (found & 1) != 0;
    return found >> 1;
  }

  __device__ __forceinline__ void multiply(acc_t (&acc)[NB], const T (&a)[STEPS], const T (&b)[NB][STEPS]) const {
#pragma unroll
    for (int s = 0; s < STEPS; ++s)
#pragma unroll
      for (int j = 0; j < NB; ++j) acc[j] = Mfma<T>::mma(a[s], b[j][s], acc[j]);
  }
};

// The column tile's systems row by row, by one workgroup, from the factor itself: what is left to do when a wait of the
// launch has given up.  Every other workgroup of the tile is through.
template <typename T, int KIND>
__device__ __attribute__((noinline)) void flow_recover(const T* F, int64_t lda, T* B, int64_t ldb, T* Y, T* X, int64_t ldy, int n, int nrhs,
                                                       int c0, int width, T* red) {
  const int tid = (int)threadIdx.x, x = tid & 15, part = tid >> 4;
  auto get = [&](const T* p) { return flow_load(p); };
  for (int j = 0; j < width; ++j) {
    const int c = c0 + j * 16 + x;
    const bool on = c < nrhs;
    const int cc = on ? c : nrhs - 1;
    int missing = 0;
    for (int r = part; r < n; r += 16)
      if (!flow_there(get(Y + (int64_t)r * ldy + cc))) missing = 1;
    const bool forward = __syncthreads_or(missing) != 0;  // (complete: B may hold part of X, but Y is all that is needed)
    for (int pass = forward ? 0 : 1; pass < 2; ++pass) {
      T* const V = pass ? X : Y;
      for (int q = 0; q < n; ++q) {
        const int r = pass ? n - 1 - q : q;
        T s = T(0);
        for (int k = part; k < q; k += 16) {
          const int kk = pass ? n - 1 - k : k;
          const T f = KIND == 1 && pass ? F[(int64_t)kk * lda + r] : F[(int64_t)r * lda + kk];
          s += f * get(V + (int64_t)kk * ldy + cc);
        }
        red[tid] = s;
        __syncthreads();
        if (part == 0 && on) {
          for (int w = 1; w < 16; ++w) s += red[w * 16 + x];
          T v = (pass ? get(Y + (int64_t)r * ldy + c) : B[(int64_t)r * ldb + c]) - s;
          if (KIND == 1 || pass) v /= F[(int64_t)r * lda + r];
          flow_store(V + (int64_t)r * ldy + c, v);
          if (pass) B[(int64_t)r * ldb + c] = v;
        }
        __syncthreads();
      }
    }
  }
}

// Takes the first piece up to `own` that nobody has (one wave); -1: there is none.
static __device__ __attribute__((noinline)) int flow_search(int* claims, int own, int n, int blocks, int tiles_n) {
  const int lane = (int)threadIdx.x & 63;
  for (int base = 0; base <= own; base += 64) {
    const int id = base + lane;
    bool open = false;
    if (id <= own && flow_piece_is(flow_piece(id, blocks, tiles_n), n, blocks))
      open = __hip_atomic_load(claims + id, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0;
    for (unsigned long long mask = __builtin_amdgcn_ballot_w64(open); mask != 0; mask &= mask - 1) {
      const int at = base + __builtin_ctzll(mask);
      int before = 1;
      if (lane == 0) before = __hip_atomic_exchange(claims + at, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (__builtin_amdgcn_readfirstlane(before) == 0) return at;
    }
  }
  return -1;
}

// Computes and publishes one piece, by the whole workgroup; TAKEN: the workgroup has it already, else it claims it on the way.
// last_try: a wait that is over makes the launch give up.  Returns 0; 1 where a wait has been too long: the piece is then back; 2 + ct
// where column tile ct is through and the launch has given up.
// KIND: 0 LU, 1 Cholesky (FactorKind)
template <typename T, int KIND, int NB, bool TAKEN>
__device__ __forceinline__ int flow_run(const FlowArgs<T>& g, const int piece, const bool last_try, T* const red) {
  using Tile = FlowTile<T, NB>;
  using acc_t = typename Tile::acc_t;
  constexpr int STEPS = Tile::STEPS;
  constexpr int64_t SB = kFlowBlock;
  constexpr bool CH = KIND == 1;
  __shared__ int shared_late[6];
  int tid = (int)threadIdx.x;
  if (TAKEN && NB == 2) asm volatile("" : "+v"(tid));  // (or what the workgroup's first piece has computed is kept for this one)
  Tile t;
  t.lane = tid & 63;
  t.wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  t.l15 = t.lane & 15;
  t.kq = t.wave * 8 + 2 * (t.lane >> 4);
  t.gave_up = g.done + g.tiles_n;
  t.limit = g.search_ticks;
  t.last_try = last_try;
  int claimed = 0;  // what the piece's claim was before (one thread); looked at when the piece is ready
  const FlowPiece f = flow_piece(piece, g.blocks, g.tiles_n);
  const bool back = f.back, sum_wg = f.sum;
  const int p = f.p, rt = f.rt, ct = f.ct;
  const int last = g.blocks - 1, i = f.block(g.blocks);
  auto rows_of = [&](int q) { return g.n - q * (int)SB < (int)SB ? g.n - q * (int)SB : (int)SB; };
  const int rows = rows_of(i), r0 = rt * 16, ldy = (int)g.ldy;
  if (r0 >= rows) return 0;  // uniform
  const int row = r0 + t.l15 < rows ? r0 + t.l15 : rows - 1;  // this lane's row of the left operands
#pragma unroll
  for (int j = 0; j < NB; ++j) t.col[j] = ct * 16 * NB + j * 16 + t.l15 < g.nrhs ? ct * 16 * NB + j * 16 + t.l15 : g.nrhs - 1;
  auto flags_of = [&](bool bk, int pos) { return g.flags + (((int64_t)(bk ? g.blocks : 0) + pos) * g.tiles_n + ct) * kFlowTiles; };
  T* const S = back ? g.S + (int64_t)g.n * g.ldy : g.S;
  auto pieces_of = [&](int q) { return (rows_of(q) + 15) / 16; };
  T* const V = back ? g.X : g.Y;   // where the pass publishes
  auto block_at = [&](T* area, int q) { return area + (int64_t)q * SB * g.ldy; };

  acc_t acc[NB];
#pragma unroll
  for (int j = 0; j < NB; ++j) acc[j] = acc_t{0, 0, 0, 0};
  T b[NB][STEPS], a0[STEPS], a1[STEPS];

  // The products, in the order in which their right operands appear.  Sum: the blocks solved at the positions 0, 1, ...;
  // solution: the block two positions back, S_i, the block before this.  The left operand of the next is on its way
  // while a right operand is waited for.
  const int from_s = p >= 2 ? 1 : 0;  // which of a solution's products is S_i's
  const int count = sum_wg ? p - kFlowLook : (p < kFlowLook ? p : kFlowLook) + 1;
  auto block_of = [&](int q) {  // the block whose rows the right operand of product q is
    if (sum_wg) return back ? last - q : q;
    const int d = q == from_s ? 0 : (q < from_s ? 2 : 1);
    return back ? i + d : i - d;
  };
  auto left = [&](T (&a)[STEPS], int q) __attribute__((always_inline)) {
    const int j = block_of(q);
    const T* base;
    int64_t ld;
    if (sum_wg) {
      ld = g.lda;
      base = CH && back ? g.F + (int64_t)j * SB * ld + (int64_t)i * SB : g.F + (int64_t)i * SB * ld + (int64_t)j * SB;
    } else if (q == from_s) {
      ld = SB;
      base = (back && !CH ? g.nb : g.nf) + (int64_t)i * SB * SB;
    } else {
      // M's columns, forward: [i-2, i-1], only i-1 where i = 1;  backward: [i+1, i+2]
      const int64_t at = back ? (int64_t)(j - i - 1) * SB : (i == 1 ? 0 : (int64_t)(j - i + 2) * SB);
      ld = CH && back ? SB : 2 * SB;
      base = (back ? g.mb : g.mf) + (int64_t)i * 2 * SB * SB + (CH && back ? at * SB : at);
    }
    if (CH && back) t.template load_left<true>(a, base, (int)ld, row, rows_of(j));
    else t.template load_left<false>(a, base, (int)ld, row, rows_of(j));
  };
  bool behind = true;
  int complete = 0;  // positions that a look at the flags has found complete
  FlowSlots slots;
  auto step = [&](const T (&a)[STEPS], int q) __attribute__((always_inline)) {
    const int j = block_of(q), kc = rows_of(j);
    const T* const x = block_at(sum_wg || q != from_s ? V : p > kFlowLook ? S : g.Y, j);
    bool there = false;
    if (sum_wg && q + 1 < count) {
      // not urgent: one wave looks at the flags, and the block comes through the L2, once for the XCD's workgroups (where a
      // line was brought with another block's rows, before these were there, the loads below follow)
      if (q >= complete) {
        const int stride = g.tiles_n * kFlowTiles;
        int* const found = &shared_late[slots.next()];
        if (count - q > 2) complete = q + t.template wait_positions<32>(flags_of(back, q), stride, pieces_of(j), count - 1 - q, behind, found);
        else complete = q + t.template wait_positions<8>(flags_of(back, q), stride, pieces_of(j), count - 1 - q, behind, found);
      }
      there = t.template load_area<0>(b, x, ldy, kc);
    } else if (!sum_wg && q == from_s && p <= kFlowLook && !back) {
      t.load_rhs(b, g.B + (int64_t)i * SB * g.ldb, g.ldb, kc);
      there = true;
    } else if (!sum_wg && q == 0) {
      // not before the block solved before is at hand does it look at the elements
      if (p > kFlowLook) t.template wait_flags<16>(flags_of(back, p - kFlowLook - 1), pieces_of(back ? i + kFlowLook + 1 : i - kFlowLook - 1));
      else if (back && last > 0) t.template wait_flags<16>(flags_of(false, last - 1), pieces_of(last - 1));
    }
    if (!there) t.load_published(b, x, ldy, kc);
    t.multiply(acc, a, b);
  };
  // A solution's product with S_i holds its largest terms, the diagonal of W_i: what comes behind it is added up by itself, from zero
  // (partial sums at the size of the result are rounded there, half of an ulp each)
  bool parted = false;
  auto part = [&](int q) __attribute__((always_inline)) {
    if (sum_wg || q != from_s || q + 1 >= count) return;  // uniform
    parted = true;
#pragma unroll
    for (int j = 0; j < NB; ++j) {
#pragma unroll
      for (int v = 0; v < 4; ++v) red[4 * NB * 256 + ((t.wave * NB + j) * 4 + v) * 64 + t.lane] = acc[j][v];
      acc[j] = acc_t{0, 0, 0, 0};
    }
  };
  left(a0, 0);
  for (int q = 0; q < count; q += 2) {
    if (q + 1 < count) left(a1, q + 1);
    // (between the left operands, which do not wait for it, and the first right operand, which takes as long)
    if (!TAKEN && q == 0 && tid == 0) claimed = __hip_atomic_exchange(g.claims + piece, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    step(a0, q);
    part(q);
    if (q + 1 >= count) break;
    if (q + 2 < count) left(a0, q + 2);
    step(a1, q + 1);
    part(q + 1);
  }

  // ---- the waves' partial blocks added up: element (row_of(wave, lane), l15) of each column block is this thread's
#pragma unroll
  for (int j = 0; j < NB; ++j)
#pragma unroll
    for (int v = 0; v < 4; ++v) red[((t.wave * NB + j) * 4 + v) * 64 + t.lane] = acc[j][v];
  if (t.lane == 0) shared_late[2 + t.wave] = t.late | (!TAKEN && claimed != 0 ? 4 : 0);
  lds_barrier();
  const int late = shared_late[2] | shared_late[3] | shared_late[4] | shared_late[5];
  if (!TAKEN && (late & 4) != 0) return 0;  // uniform: another workgroup has it
  const int er = r0 + Mfma<T>::row_of(t.wave, t.lane);
  const int64_t gr = (int64_t)i * SB + er;
  if (late == 0) {
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const int c = (ct * NB + j) * 16 + t.l15;
      T x[4];
#pragma unroll
      for (int w = 0; w < 4; ++w) x[w] = red[((w * NB + j) * 4 + t.wave) * 64 + t.lane];
      T sum = ((x[0] + x[1]) + x[2]) + x[3];
      if (parted) {
#pragma unroll
        for (int w = 0; w < 4; ++w) x[w] = red[4 * NB * 256 + ((w * NB + j) * 4 + t.wave) * 64 + t.lane];
        sum += ((x[0] + x[1]) + x[2]) + x[3];
      }
      if (er < rows && c < g.nrhs) {
        if (sum_wg) {
          // (the backward pass starts from Y, which is complete once a block of X is there)
          const T old = back ? flow_load(g.Y + gr * g.ldy + c) : g.B[gr * g.ldb + c];
          flow_store(S + gr * g.ldy + c, old - sum);
        } else {
          flow_store(V + gr * g.ldy + c, -sum);
          if (back) g.B[gr * g.ldb + c] = -sum;
        }
      }
    }
  }
  // the piece is at the point of coherence (these stores write through) before its flag and before the count
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (tid == 0) {
    int rest = late;  // 1; 2 or 3: the launch has given up
    if (late == 1) {
      __hip_atomic_store(g.claims + piece, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (the piece is back before the search)
    } else {
      if (late == 0 && !sum_wg) __hip_atomic_store(flags_of(back, p) + rt, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const int before = __hip_atomic_fetch_add(g.done + ct, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      rest = before == g.expected - 1 && __hip_atomic_load(t.gave_up, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0 ? 2 + ct : 0;
    }
    shared_late[0] = rest;
  }
  __syncthreads();
  return __builtin_amdgcn_readfirstlane(shared_late[0]);
}

template <typename T, int KIND, int NB>
__global__ void __launch_bounds__(kFlowThreads, NB == 1 ? 3 : 2) flow_kernel(const FlowArgs<T> g) {
  __shared__ T red[2 * 4 * NB * 256];
  __shared__ int next;
  const int own = (int)blockIdx.x;
  if (own % kNumXcd == g.absent && own < flow_pieces(g.blocks, g.tiles_n) - kFlowTiles * g.tiles_n) return;  // uniform
  int rest = flow_run<T, KIND, NB, false>(g, own, false, red);
  // ---- rare: for a column tile of a launch that has given up, the substitution; else other pieces (see Order above)
  long long waited = 0;  // in vain, since something came on
  if (rest == 0) return;  // uniform
  for (;;) {
    if (rest > 1) flow_recover<T, KIND>(g.F, g.lda, g.B, g.ldb, g.Y, g.X, g.ldy, g.n, g.nrhs, (rest - 2) * NB * 16, NB, red);
    waited = rest == 1 ? waited + g.search_ticks : 0;
    __syncthreads();
    if (threadIdx.x < 64) {
      const int found = flow_search(g.claims, own, g.n, g.blocks, g.tiles_n);
      if (threadIdx.x == 0) next = found;
    }
    __syncthreads();
    const int piece = __builtin_amdgcn_readfirstlane(next);
    if (piece < 0) return;  // uniform
    rest = flow_run<T, KIND, NB, true>(g, piece, waited + g.search_ticks >= g.wait_ticks, red);
  }
}

}  // namespace dla
