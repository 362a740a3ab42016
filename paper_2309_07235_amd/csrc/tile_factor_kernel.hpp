// A whole factorisation as one launch, in 64 x 64 tiles (paper, Section "Linear Algebra Benchmarks": A = L*U without
// pivoting, A = L*L^T; the tiling is this library's).  Workgroups wait in place for what they read:
//   workgroup 0 walks the diagonal: block s lies in its LDS, is factored there (diag_stages), then the two blocks beside the
//     next one, (s, s+1) and (s+1, s), are solved from copies and block (s+1, s+1) gets their product, so that from one
//     diagonal block to the next nothing leaves the workgroup;
//   the other workgroups take tiles, (i, j) with step s = min(i, j), one at a time: the tile is kept in accumulators, the products of
//     the tiles in front of it, (i, k) (k, j), are subtracted as these appear, and it is solved once block s is factored.  The tiles
//     beside the diagonal are also copied, unsolved, for workgroup 0, which is through with a block about when they are there.
// So a tile of the matrix is read and written once, there is one launch instead of six per block column, and the chain of
// the diagonal is free of hand-overs.  It is one launch also because its workgroups wait for each other both ways: two launches on
// two streams that share a hardware queue would run one after the other.
//
// A tile's workgroup has eight waves, four 32 x 32 parts of the tile times two halves of each product's depth; or they are two teams
// of four that each have a tile of their own (TileTeam), so that one's start, solve and publication hide behind the other's
// products, which is what large matrices with aligned tiles need and what costs the chain of smaller ones (launch_tiles_as).
//
// What bounds it is that chain while the matrix is small: LU 18, Cholesky 16 us per 64 columns, of which the four stages of the
// diagonal block are 11.5, the two solves 1.9 - 3.4, the product with the next block's first factor 2.3.  (A block of 128 in the
// pipeline, with its head update and two hand-overs between kernels, is 47.)  Beyond, the tiles' products.  us, the pipeline against
// this: LU fp64 n = 300 125 -> 98, n = 4000 1866 -> 1391 (31 TFLOP/s), n = 7000 6880 -> 5235 (44), Cholesky n = 1024 in blocks of 64
// 713 -> 269, n = 4000 1580 -> 1115.
// Half of 128 registers per lane for two workgroups of eight waves spills; a workgroup on the chain's compute unit costs the
// chain 2 - 4 us a step.
//
// Hand-over.  Published tiles are stored past the L2s (kTilePast), each workgroup waits for its stores and then sets a flag.
// A tile of the factor is read through the reader's L2 where no line of it can be there from before: lines are not shared
// between tiles (base and leading dimension multiples of 128 bytes) and only its owner has touched it, on the XCD that it
// publishes it from; otherwise, and for everything that is reused or written by workgroup 0, by loads past the L2.
//
// Order.  Tiles are taken from a counter by step, the three that workgroup 0 needs before it publishes block s first in step s
// (tile_of): (s+1, s), (s, s+1) and (s+1, s+1).  A workgroup waits only for workgroup 0 and for tiles taken before its own, so that
// three workgroups beside workgroup 0 that are there to the end are enough (Cholesky: two), however few the others let run.  Waits
// are bounded like those of the pipeline (chain_wait).
#pragma once
#include "head_kernel.hpp"

namespace dla {

constexpr int kTileNb = 64;
constexpr int kTileThreads = kDiagThreads;
constexpr int kTileSub = kTileNb / kIb;             // 4
constexpr int kTileLd = kTileNb + 1;
constexpr int kTileElems = kTileNb * kTileNb;
constexpr int kTileInvRing = 16;                    // steps whose inverted sub-blocks are kept
constexpr int kTileInv = 2 * kTileSub * 256;        // per step: of the lower factor, of the upper one (LU)
constexpr int kTilePast = 16;                       // sc1: past the L2
constexpr int64_t kTileMaxLd = 1000000;             // 64 rows lie within 2 GiB
constexpr int kTileMaxNt = 128;                     // tiles per side (what tile_factor_kernel's search for a step reaches)

template <typename T>
struct TileArgs {
  T* A;
  int64_t lda;
  int n, nt;        // order; tiles per side
  int k0;           // what lies in front of the matrix, factored already
  const int* broken; // or null: set where that went wrong
  int* info;
  T* inv;           // [kTileInvRing][2][4][256]: inverted sub-blocks, row-major
  T* pre;           // [2][3][64 x 64]: unsolved (s, s+1), (s+1, s) and (s+1, s+1), by parity of s + 1
  int* ints;        // TileFlags
  long long wait_ticks;  // below 0: a wait gives up at once
};
// Flags and counters: a wait gave up, tiles taken; then a flag per tile and what belongs to the blocks of the diagonal.
struct TileFlags {
  int nt;
  static constexpr int kGaveUp = 0, kTicket = 1, kFirst = 2;
  __host__ __device__ int low(int i, int k) const { return kFirst + i * nt + k; }                  // tile (i, k), i > k
  __host__ __device__ int up(int j, int k) const { return kFirst + nt * nt - 1 - (j * nt + k); }   // tile (k, j), k < j: from the other end
  __host__ __device__ int diag(int s) const { return kFirst + nt * nt + s; }                       // waves that have stored their part of block s, of 4
  __host__ __device__ int copied(int s, int what) const { return kFirst + nt * nt + nt + 4 * s + what; }  // pre of block s
  __host__ __device__ int read(int s) const { return kFirst + nt * nt + 5 * nt + s; }              // tiles that have read block s
  __host__ __device__ int count() const { return kFirst + nt * nt + 6 * nt; }
};
// LDS of workgroup 0: block, pivots, inverses, the slices of both solves.
constexpr int kTileSlices = (kTileNb + 1) * kTileLd + 2 * kTileNb + 2 * kTileSub * kBlk, kTileLds = kTileSlices + 8 * kTileSub * 4 * 64 + kBlk;
template <typename T>
inline size_t tile_workspace_bytes(int nt) {
  return (size_t)(kTileInvRing * kTileInv + 6 * kTileElems) * sizeof(T) + (size_t)TileFlags{nt}.count() * sizeof(int);
}

static __global__ void __launch_bounds__(256) tile_clear_kernel(int* p, int n) {
  const int i = (int)(blockIdx.x * 256 + threadIdx.x);
  if (i < n) p[i] = 0;
}

template <int AUX>
__device__ __forceinline__ double tile_load(__amdgpu_buffer_rsrc_t rs, int vo, int so, double*) {
  return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(rs, vo, so, AUX));
}
template <int AUX>
__device__ __forceinline__ float tile_load(__amdgpu_buffer_rsrc_t rs, int vo, int so, float*) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, vo, so, AUX));
}
template <typename T>
__device__ __forceinline__ void tile_store(T* p, T x) {  // past the L2
  using U = std::conditional_t<sizeof(T) == 8, unsigned long long, unsigned int>;
  __hip_atomic_store(reinterpret_cast<U*>(p), __builtin_bit_cast(U, x), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ T tile_get(const T* p) {  // past the L2
  using U = std::conditional_t<sizeof(T) == 8, unsigned long long, unsigned int>;
  return __builtin_bit_cast(T, __hip_atomic_load(reinterpret_cast<const U*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}

// the same through a resource: one lane offset, the rest in the instruction (64-bit addresses of 70 loads do not fit the registers)
template <typename T>
__device__ __forceinline__ T tile_get(__amdgpu_buffer_rsrc_t rs, int vo, int so) {
  return tile_load<kTilePast>(rs, vo, so, (T*)nullptr);
}
template <typename T>
__device__ __forceinline__ void tile_store(__amdgpu_buffer_rsrc_t rs, int vo, int so, T x) {
  if constexpr (sizeof(T) == 8) __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2_t, x), rs, vo, so, kTilePast);
  else __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned int, x), rs, vo, so, kTilePast);
}
// Nothing is loaded in front of what was waited for.
__device__ __forceinline__ void tile_order() { asm volatile("" ::: "memory"); }

// X = M^-1 P as head_solve, for 64 rows: sub-block (s, r), s > r, of M at D + s * bs + r * br, element (i, k) at i * rs + k * cs;
// inverted diagonal sub-block r at inv + r * kBlk, element (i, k) at i * irs + k * ics.
template <typename T>
__device__ __forceinline__ void tile_solve(const T* D, int bs, int br, int rs, int cs, const T* inv, int irs, int ics, int lane,
                                           typename Mfma<T>::acc_t (&acc)[kTileSub]) {
  using acc_t = typename Mfma<T>::acc_t;
  const int row = head_prow<T>(lane & 15), l4 = lane >> 4;
  const T* const d0 = D + row * rs + 4 * l4 * cs;
  const T* const i0 = inv + row * irs + 4 * l4 * ics;
  static_for<0, kTileSub>([&](auto rc) {
    constexpr int r = decltype(rc)::value;
    acc_t x = {0, 0, 0, 0};
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) x = Mfma<T>::mma(i0[r * kBlk + kk * ics], acc[r][kk], x);
    acc[r] = x;
    static_for<r + 1, kTileSub>([&](auto sc) {
      constexpr int s = decltype(sc)::value;
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) acc[s] = Mfma<T>::mma(-d0[s * bs + r * br + kk * cs], x[kk], acc[s]);
    });
  });
}

// A wave waits until ok() holds for all of its lanes.
template <typename F>
__device__ __forceinline__ void tile_spin(int* ints, long long limit, int pause, F&& ok) {
  const long long t0 = wall_clock64();
  for (int spins = 0;; ++spins) {
    if (__builtin_amdgcn_ballot_w64(!ok()) == 0) break;
    if (spins % 32 == 31 || limit < 0) {
      if (__builtin_amdgcn_ballot_w64(__hip_atomic_load(ints, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) != 0) break;
      if (wall_clock64() - t0 > limit) {
        __hip_atomic_store(ints, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        break;
      }
    }
    if (pause == 1) __builtin_amdgcn_s_sleep(2);
    if (pause == 2) __builtin_amdgcn_s_sleep(8);
  }
}
// The waves that work on one tile: all eight of a workgroup, or four, one of its two teams, which share the compute unit but wait
// for nothing of each other.  A team meets at a count in LDS (s_barrier is the workgroup's): each wave adds one and looks until all
// four of this meeting have.  The waves of a workgroup are all there, so every meeting ends.
template <int WAVES>
struct TileTeam {
  int wave;      // within the team
  int* arrived;  // four waves: the team's count, which starts at zero
  int meetings = 0;
  __device__ __forceinline__ void barrier() {
    if constexpr (WAVES == kTileThreads / 64) {
      lds_barrier();
    } else {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
      meetings += WAVES;
      if ((threadIdx.x & 63) == 0) __hip_atomic_fetch_add(arrived, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      while (__builtin_amdgcn_readfirstlane(__hip_atomic_load(arrived, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) < meetings) {}
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    }
  }
};
// A team waits, by its first wave.
template <int WAVES, typename F>
__device__ __forceinline__ void tile_wait(int* ints, long long limit, TileTeam<WAVES>& team, int pause, F&& ok) {
  if (team.wave == 0) tile_spin(ints, limit, pause, ok);
  team.barrier();
  tile_order();
}
__device__ __forceinline__ bool tile_flag(const int* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0; }
// every wave's stores are past the L2s, then the flag
template <int WAVES>
__device__ __forceinline__ void tile_publish(int* flag, TileTeam<WAVES>& team, int tid) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  team.barrier();
  if (tid == 0) __hip_atomic_store(flag, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ---- workgroup 0
// Waves 4 .. 7 store the strips beside the stages, see to it that the copies for the next block are there two stages ahead and
// have them in registers when the last panel is solved; they do both solves.  Waves 0 .. 3 publish the block meanwhile.
template <typename T, int KIND>
__device__ __forceinline__ void tile_chain(const TileArgs<T>& g, T* const smem) {
  using acc_t = typename Mfma<T>::acc_t;
  constexpr bool LU = KIND == KIND_LU;
  T* const S = smem;
  T* const sRd = S + (kTileNb + 1) * kTileLd;
  T* const iLo = sRd + 2 * kTileNb;          // inverted sub-blocks, row-major, rows of 17
  T* const iUp = iLo + kTileSub * kBlk;
  T* const slices = smem + kTileSlices;      // of both solves: x (LU), y
  T* const corner = slices + 8 * kTileSub * 4 * 64;  // 16 x 17
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const TileFlags fl{g.nt};

  // block 0: its rows to LDS, padded with the identity
  {
    const int lane = (int)threadIdx.x & 63, v = g.n < kTileNb ? g.n : kTileNb;
#pragma unroll
    for (int e = 0; e < kTileElems / kTileThreads; ++e) {
      const int r = wave + e * 8, c = lane;
      const T x = g.A[(int64_t)(r < v ? r : v - 1) * g.lda + (c < v ? c : v - 1)];
      S[r * kTileLd + c] = r < v && c < v ? x : (r == c ? T(1) : T(0));
    }
  }
  lds_barrier();
  if (wave == 0) {
    const int lane = (int)threadIdx.x & 63;
    DiagSub<T, KIND> sub;
#pragma unroll
    for (int j = 0; j < 16; ++j) sub.a[j] = S[(lane & 15) * kTileLd + j];
    sub.factor(lane);
    sub.template store<kTileNb>(S, sRd, lane, 0);
  }
  lds_barrier();
  int info = 0;
  for (int s = 0; s < g.nt; ++s) {
    // (the lane's place as a value of this iteration: its many multiples would otherwise be kept from one to the next, in scratch)
    int tid = (int)threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63, l15 = lane & 15, l4 = lane >> 4;
    const int64_t k0 = (int64_t)s * kTileNb;
    const int b = g.n - (int)k0 < kTileNb ? g.n - (int)k0 : kTileNb;
    const bool more = s + 1 < g.nt;
    T* const At = g.A + k0 * g.lda + k0;
    T* const inv = g.inv + (int64_t)(s % kTileInvRing) * kTileInv;
    constexpr int E = (int)sizeof(T);
    const __amdgpu_buffer_rsrc_t pre = __builtin_amdgcn_make_buffer_rsrc(g.pre + (int64_t)((s + 1) & 1) * 3 * kTileElems, 0, 3 * kTileElems * E, 0x00020000);
    const __amdgpu_buffer_rsrc_t ri = __builtin_amdgcn_make_buffer_rsrc(inv, 0, kTileInv * E, 0x00020000);
    const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(At, 0, ((b - 1) * (int)g.lda + b) * E, 0x00020000);  // (rows beyond: dropped)
    constexpr int kOob = 0x7FFFFFF0;
    const int ldE = (int)g.lda * E;
    const int slice0 = (wave & 3) * kIb;
    acc_t x[kTileSub], y[kTileSub];  // (waves 4 .. 7)
    // the 16 x 16 blocks of the next diagonal block that this wave updates: block 0 is wave 0's, which goes on to factor it;
    // wave 4, on the same SIMD, has none; the others have blocks m + 1, m + 7, m + 13 (Cholesky: of the lower triangle)
    constexpr int kBlocks = LU ? 15 : 9, kMine = LU ? 3 : 2;
    const int m = wave < 4 ? wave - 1 : wave - 2;
    auto mine = [&](int q) { return wave == 0 ? q == 0 : wave != 4 && m + 6 * q < kBlocks; };
    auto row_of = [&](int q) {
      const int e = wave == 0 ? 0 : m + 6 * q + 1;
      return LU ? e >> 2 : (e >= 6 ? 3 : e >= 3 ? 2 : e >= 1 ? 1 : 0);
    };
    auto col_of = [&](int q) {
      const int e = wave == 0 ? 0 : m + 6 * q + 1, r = row_of(q);
      return LU ? e & 3 : e - r * (r + 1) / 2;
    };
    acc_t c[kMine];
    auto next_block = [&] {
#pragma unroll
      for (int q = 0; q < kMine; ++q)
        if (mine(q)) {  // uniform
#pragma unroll
          for (int v = 0; v < 4; ++v) c[q][v] = tile_get<T>(pre, (Mfma<T>::row_of(0, lane) * kTileNb + l15) * E, (2 * kTileElems + (row_of(q) * kIb + Mfma<T>::row_of(v, 0)) * kTileNb + col_of(q) * kIb) * E);
        }
    };
    bool there = false;
    // rows [o, o + 16) from column o on and columns [o, o + 16) below them, by the four waves of which this one is number w
    auto strip = [&](int o, int w) __attribute__((always_inline)) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int r = o + w * 4 + q, c = o + lane;
        tile_store<T>(ra, c < b && r < b ? c * E : kOob, r * ldE, LU || c <= r ? S[r * kTileLd + (c < kTileNb ? c : kTileNb)] : T(0));
      }
#pragma unroll
      for (int q = 0; q < kTileSub - 1; ++q) {
        const int r = o + kIb + q * kIb + w * 4;  // (a row beyond the block is beyond its extent, or beyond b)
        tile_store<T>(ra, o + l15 < b && r + l4 < b ? (o + l15) * E + l4 * ldE : kOob, r * ldE, S[(r + l4 < kTileNb ? r + l4 : kTileNb) * kTileLd + o + l15]);
      }
    };
    auto beside = [&](int o) __attribute__((always_inline)) {
      strip(o, wave - 4);
      if (more && o == kIb) {  // an early look
        const bool ok = !LU && lane == 0 ? true : tile_flag(g.ints + fl.copied(s + 1, lane < 3 ? lane : 1));
        there = s + 1 < kTileInvRing && __builtin_amdgcn_ballot_w64(!ok) == 0;
      }
    };
    auto beside_last = [&](int o) __attribute__((always_inline)) {
      if (more) {
        if (!there) {  // the copies of the blocks beside the next diagonal block, and the place of its inverses in the ring
          const int gone = s + 1 - kTileInvRing;
          const int readers = gone >= 0 ? (LU ? 2 : 1) * (g.nt - 1 - gone) : 0;
          const int* const p = g.ints + (lane < 3 ? fl.copied(s + 1, lane) : fl.read(gone < 0 ? 0 : gone));
          const int want = lane < 3 ? (LU || lane > 0 ? 1 : 0) : (lane == 3 ? readers : 0);
          tile_spin(g.ints, g.wait_ticks, 0, [&] { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= want; });
        }
        tile_order();
        const int vo = (4 * l4 * kTileNb + slice0 + l15) * E;  // (the column panel's copy is transposed)
#pragma unroll
        for (int q = 0; q < kTileSub; ++q)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            if constexpr (LU) x[q][v] = tile_get<T>(pre, vo, (q * kIb + v) * kTileNb * E);
            y[q][v] = tile_get<T>(pre, vo, (kTileElems + (q * kIb + v) * kTileNb) * E);
          }
        next_block();
      }
      strip(o, wave - 4);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    };
    diag_stages<T, KIND, kTileNb>(S, sRd, kTileNb, tid, beside, beside_last, [&](auto upper_c, int q, int unit, const T (&v)[16]) {
      constexpr bool UPPER = decltype(upper_c)::value;
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        (UPPER ? iUp : iLo)[q * kBlk + (UPPER ? unit * 17 + j : j * 17 + unit)] = v[j];
        tile_store<T>(ri, (UPPER ? unit * 16 : unit) * E, ((UPPER ? kTileSub * 256 : 0) + q * 256 + (UPPER ? j : j * 16)) * E, v[j]);
      }
    });
    lds_barrier();
    if (wave == 0 && info == 0) {  // breakdown: the first pivot that is zero (LU) or not positive (Cholesky)
      const T d = LU ? S[lane * (kTileLd + 1)] : sRd[kTileNb + lane];
      const unsigned long long bad = __builtin_amdgcn_ballot_w64(lane < b && (LU ? d == T(0) : !(d > T(0))));
      if (bad) info = (int)k0 + __builtin_ctzll(bad) + 1;
    }
    if (wave < 4) {
      strip(3 * kIb, wave);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      if (lane == 0) __hip_atomic_fetch_add(g.ints + fl.diag(s), 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    } else if (more) {
      auto slice = [&](int at, const acc_t (&z)[kTileSub]) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < kTileSub; ++q)
#pragma unroll
          for (int v = 0; v < 4; ++v) slices[(at * 16 + q * 4 + v) * 64 + lane] = z[q][v];
      };
      if constexpr (LU) {
        tile_solve(S, kIb * kTileLd, kIb, kTileLd, 1, iLo, 17, 1, lane, x);
        slice(wave - 4, x);
        __builtin_amdgcn_sched_barrier(0);  // (or the fragments of both are loaded first, more than the registers hold)
        tile_solve(S, kIb, kIb * kTileLd, 1, kTileLd, iUp, 1, 17, lane, y);
      } else {
        tile_solve(S, kIb * kTileLd, kIb, kTileLd, 1, iLo, 17, 1, lane, y);
      }
      slice(wave, y);
    }
    if (!more) break;
    if (wave < 4) next_block();
    lds_barrier();
    // the product, with the first sub-block on its way to its factors as soon as it is there
    auto product = [&](int q) __attribute__((always_inline)) {
      const T* const sy = slices + (4 + row_of(q)) * 1024 + lane;
      const T* const sx = slices + ((LU ? 0 : 4) + col_of(q)) * 1024 + lane;
#pragma unroll
      for (int e = 0; e < 16; ++e) c[q] = Mfma<T>::mma(-sy[e * 64], sx[e * 64], c[q]);
    };
    if (wave == 0) {
      product(0);
#pragma unroll
      for (int v = 0; v < 4; ++v) corner[Mfma<T>::row_of(v, lane) * 17 + l15] = c[0][v];
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup", "local");
      DiagSub<T, KIND> sub;
#pragma unroll
      for (int j = 0; j < 16; ++j) sub.a[j] = corner[l15 * 17 + j];
      sub.factor(lane);
      sub.template store<kTileNb>(S, sRd, lane, 0);
    } else {
#pragma unroll
      for (int q = 0; q < kMine; ++q)
        if (mine(q)) {  // uniform
          product(q);
#pragma unroll
          for (int v = 0; v < 4; ++v) S[(row_of(q) * kIb + Mfma<T>::row_of(v, lane)) * kTileLd + col_of(q) * kIb + l15] = c[q][v];
        }
    }
    lds_barrier();
  }
  if (threadIdx.x == 0) {
    const int before = g.k0 > 0 ? *g.info : 0;
    const bool bad = __hip_atomic_load(g.ints + TileFlags::kGaveUp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0 || (g.broken && *g.broken != 0);
    *g.info = bad ? -1 : before != 0 ? before : info != 0 ? g.k0 + info : 0;
  }
}

// ---- the team of tile (i, j).  AUX: how other tiles are read (0 through the L2, kTilePast)
template <typename T, int KIND, int AUX, int WAVES>
__device__ __forceinline__ void tile_owner(const TileArgs<T>& g, T* const smem, TileTeam<WAVES>& team, const int i, const int j) {
  using acc_t = typename Mfma<T>::acc_t;
  constexpr bool LU = KIND == KIND_LU;
  constexpr int E = (int)sizeof(T), kOob = 0x7FFFFFF0, kFlags = 0x00020000;
  // (the lane's place as a value of this tile, as in tile_chain)
  int tid = (int)threadIdx.x % (WAVES * 64);
  asm volatile("" : "+v"(tid));
  const int lane = tid & 63, wave = team.wave;
  const int l15 = lane & 15, l4 = lane >> 4;
  const TileFlags fl{g.nt};
  const int s = i < j ? i : j, far = i < j ? j : i;
  const int ld = (int)g.lda;
  auto valid = [&](int t) { return g.n - t * kTileNb < kTileNb ? g.n - t * kTileNb : kTileNb; };
  auto tile_at = [&](int r, int c) { return g.A + (int64_t)r * kTileNb * g.lda + (int64_t)c * kTileNb; };
  // a tile's resource: rows beyond the matrix are beyond its extent
  auto res_of = [&](int r, int c) { return __builtin_amdgcn_make_buffer_rsrc(tile_at(r, c), 0, ((valid(r) - 1) * ld + kTileNb) * E, kFlags); };
  const int rows = valid(i), cols = valid(j);
  // this wave's 32 x 32 of the tile; with eight waves also half of each product's k, where waves 4 .. 7 start from zero and are
  // added at the end
  constexpr int NT = WAVES * 64;
  const int r0 = (wave >> 1 & 1) * 2 * kIb, c0 = (wave & 1) * 2 * kIb, khalf = WAVES == 8 ? wave >> 2 : 0;
  acc_t acc[2][2];
  {
    const __amdgpu_buffer_rsrc_t rs = res_of(i, j);
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int r = r0 + p * kIb + Mfma<T>::row_of(v, lane), c = c0 + q * kIb + l15;
          T x = tile_load<0>(rs, khalf == 0 && c < cols && r < rows ? (r * ld + c) * E : kOob, 0, (T*)nullptr);
          if (i == j && r == c && r >= rows && khalf == 0) x = T(1);
          acc[p][q][v] = x;
        }
  }
  if (!LU && i > j) {  // the tile above the diagonal
    T* const Z = tile_at(j, i);
#pragma unroll
    for (int e = 0; e < kTileElems / NT; ++e) {
      const int r = wave + e * WAVES;
      if (r < cols && lane < rows) Z[(int64_t)r * g.lda + lane] = T(0);
    }
  }

  // ---- the products in front of it.  k of a fragment's step e: 32 half + 8 (e / 2) + 2 l4 + e % 2
  const int depth = i == j ? s - 1 : s;  // (block (s, s) gets its last product on the diagonal's chain)
  T a[2][2][8], b[2][2][8];
  int avo[2], bvo[2];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int r = r0 + q * kIb + l15, c = c0 + q * kIb + l15, kk = 32 * khalf + 2 * l4;
    avo[q] = r < rows ? (r * ld + kk) * E : kOob;
    bvo[q] = c < cols ? (LU ? kk * ld + c : c * ld + kk) * E : kOob;
  }
  auto fetch = [&](auto xc, int k, int half) __attribute__((always_inline)) {  // (half: of a wave that has both)
    constexpr int X = decltype(xc)::value;
    const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(tile_at(i, k), 0, (kTileNb - 1) * ld * E + kTileNb * E, kFlags);
    const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc(LU ? tile_at(k, j) : tile_at(j, k), 0, (kTileNb - 1) * ld * E + kTileNb * E, kFlags);
    auto pair = [&](__amdgpu_buffer_rsrc_t r, int vo, int so, T& x, T& y) __attribute__((always_inline)) {
      if constexpr (E == 8) {
        const double2_t w = __builtin_bit_cast(double2_t, __builtin_amdgcn_raw_buffer_load_b128(r, vo, so, AUX));
        x = w[0];
        y = w[1];
      } else {
        const float2_t w = __builtin_bit_cast(float2_t, __builtin_amdgcn_raw_buffer_load_b64(r, vo, so, AUX));
        x = w[0];
        y = w[1];
      }
    };
#pragma unroll
    for (int e = 0; e < 8; e += 2)
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        pair(ra, avo[q], (32 * half + 4 * e) * E, a[X][q][e], a[X][q][e + 1]);
        if constexpr (LU) {
          b[X][q][e] = tile_load<AUX>(rb, bvo[q], (32 * half + 4 * e) * ld * E, (T*)nullptr);
          b[X][q][e + 1] = tile_load<AUX>(rb, bvo[q], (32 * half + 4 * e + 1) * ld * E, (T*)nullptr);
        } else {
          pair(rb, bvo[q], (32 * half + 4 * e) * E, b[X][q][e], b[X][q][e + 1]);
        }
      }
  };
  auto multiply = [&](auto xc) __attribute__((always_inline)) {
    constexpr int X = decltype(xc)::value;
#pragma unroll
    for (int e = 0; e < 8; ++e)
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        const T l = -a[X][p][e];
#pragma unroll
        for (int q = 0; q < 2; ++q) acc[p][q] = Mfma<T>::mma(l, b[X][q][e], acc[p][q]);
      }
  };
  using h0 = std::integral_constant<int, 0>;
  using h1 = std::integral_constant<int, 1>;
  int* const shared = reinterpret_cast<int*>(smem);
  const int* const fa = g.ints + fl.low(i, 0);                   // (row block i) tiles (i, k)
  const int* const fb = g.ints + (LU ? fl.up(j, 0) : fl.low(j, 0));
  for (int k = 0; k < depth;) {
    // how many of the next 32 pairs of tiles are there: lanes 0 .. 31 the left ones, 32 .. 63 the right ones
    int ready = 0;
    if (wave == 0) {
      const int q = lane & 31;
      const int at = k + (k + q < depth ? q : 0);
      const int* const p = LU && lane >= 32 ? fb - at : (lane < 32 ? fa : fb) + at;
      const long long t0 = wall_clock64();
      for (int spins = 0;; ++spins) {
        const unsigned long long miss = __builtin_amdgcn_ballot_w64(!tile_flag(p));
        const unsigned both = (unsigned)miss | (unsigned)(miss >> 32);
        ready = both ? __builtin_ctz(both) : 32;
        if (ready) break;
        if (spins % 32 == 31 || g.wait_ticks < 0) {
          if (__builtin_amdgcn_ballot_w64(tile_flag(g.ints)) != 0) ready = 1;
          if (wall_clock64() - t0 > g.wait_ticks) {
            __hip_atomic_store(g.ints, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            ready = 1;
          }
          if (ready) break;
        }
        if (depth - k > 2) __builtin_amdgcn_s_sleep(8);
      }
      if (lane == 0) shared[0] = ready;
    }
    team.barrier();
    ready = __builtin_amdgcn_readfirstlane(shared[0]);
    tile_order();
    if (ready > depth - k) ready = depth - k;
    const int end = k + ready;
    fetch(h0{}, k, 0);
    if constexpr (WAVES == 8) {
      for (; k < end; k += 2) {
        if (k + 1 < end) fetch(h1{}, k + 1, 0);
        multiply(h0{});
        if (k + 1 >= end) {
          ++k;
          break;
        }
        if (k + 2 < end) fetch(h0{}, k + 2, 0);
        multiply(h1{});
      }
    } else {
      for (; k < end; ++k) {
        fetch(h1{}, k, 1);
        multiply(h0{});
        if (k + 1 < end) fetch(h0{}, k + 1, 0);
        multiply(h1{});
      }
    }
    team.barrier();  // (shared[0] is read)
  }

  // ---- the tile to LDS, the halves of k added up
  T* const P = smem;
  T* const D = P + kTileNb * kTileLd;
  T* const sInv = D + kTileNb * kTileLd;
  auto each = [&](auto&& f) __attribute__((always_inline)) {
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[p][q][v] = f(r0 + p * kIb + Mfma<T>::row_of(v, lane), c0 + q * kIb + l15, (T)acc[p][q][v]);
  };
  if constexpr (WAVES == 8) {
    if (khalf != 0) each([&](int r, int c, T x) { return P[r * kTileLd + c] = x; });
    team.barrier();
    if (khalf == 0) each([&](int r, int c, T x) { return P[r * kTileLd + c] += x; });
  } else {
    each([&](int r, int c, T x) { return P[r * kTileLd + c] = x; });
  }
  // ---- unsolved, for the diagonal's chain (the column panel's transposed)
  if (far == s + 1 || i == j) {
    const int at = far == s + 1 ? s + 1 : s, what = i == j ? 2 : (i < j ? 0 : 1);
    T* const out = g.pre + ((int64_t)(at & 1) * 3 + what) * kTileElems;
    if (khalf == 0) each([&](int r, int c, T x) {
      tile_store(out + (what == 1 ? c * kTileNb + r : r * kTileNb + c), x);
      return x;
    });
    tile_publish(g.ints + fl.copied(at, what), team, tid);
  }
  if (i == j) return;

  // ---- solved with block s
  tile_wait(g.ints, g.wait_ticks, team, 1, [&] { return __hip_atomic_load(g.ints + fl.diag(s), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= 4; });
  {
    const T* const src = tile_at(s, s);
    const T* const inv = g.inv + (int64_t)(s % kTileInvRing) * kTileInv + (LU && i > j ? kTileSub * 256 : 0);
    constexpr int W = kTileSub * 256 / NT;
    T d[kTileElems / NT], w[W];
#pragma unroll
    for (int e = 0; e < kTileElems / NT; ++e) d[e] = tile_get(src + (int64_t)(wave + e * WAVES) * g.lda + lane);
#pragma unroll
    for (int e = 0; e < W; ++e) w[e] = tile_get(inv + tid + e * NT);
#pragma unroll
    for (int e = 0; e < kTileElems / NT; ++e) D[(wave + e * WAVES) * kTileLd + lane] = d[e];
#pragma unroll
    for (int e = 0; e < W; ++e) {
      const int at = tid + e * NT, r = at >> 4 & 15, c = at & 15;
      sInv[(at >> 8) * kBlk + r * 17 + c] = w[e];
    }
  }
  team.barrier();
  if (tid == 0) __hip_atomic_fetch_add(g.ints + fl.read(s), 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (wave < 4) {
    const bool x_job = LU && i < j;
    const int t = wave * kIb + l15;  // this lane's column (row panel) or row
    acc_t x[kTileSub];
#pragma unroll
    for (int q = 0; q < kTileSub; ++q)
#pragma unroll
      for (int v = 0; v < 4; ++v) x[q][v] = x_job ? P[(q * kIb + 4 * l4 + v) * kTileLd + t] : P[t * kTileLd + q * kIb + 4 * l4 + v];
    if (LU && !x_job) tile_solve(D, kIb, kIb * kTileLd, 1, kTileLd, sInv, 1, 17, lane, x);
    else tile_solve(D, kIb * kTileLd, kIb, kTileLd, 1, sInv, 17, 1, lane, x);
    T* const out = tile_at(i, j);
    if (t < (x_job ? cols : rows)) {
#pragma unroll
      for (int q = 0; q < kTileSub; ++q)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int k = q * kIb + 4 * l4 + v;
          tile_store(x_job ? out + (int64_t)k * g.lda + t : out + (int64_t)t * g.lda + k, x[q][v]);
        }
    }
  }
  tile_publish(g.ints + (i > j ? fl.low(i, j) : fl.up(j, i)), team, tid);
}

// The order in which tiles are taken.  Step s: (s+1, s), (s, s+1) (LU), (s+1, s+1), then the others of block column and row s.  Block
// (0, 0) is not among them, it starts on the diagonal's chain.  Tiles in front of those of step s, and tile number id:
template <int KIND>
__host__ __device__ inline int tile_before(int nt, int s) { return KIND == KIND_LU ? 2 * s * nt - s * s : s * nt - s * (s - 1) / 2; }
template <int KIND>
__host__ __device__ inline int tile_count(int nt) { return tile_before<KIND>(nt, nt - 1); }
template <int KIND>
__host__ __device__ inline void tile_of(int nt, int id, int* i, int* j) {
  int s = 0;
  for (int step = 64; step > 0; step >>= 1)  // the last s with tile_before(s) <= id
    while (s + step < nt - 1 && tile_before<KIND>(nt, s + step) <= id) s += step;
  const int q = id - tile_before<KIND>(nt, s);
  *i = *j = s;
  if (KIND == KIND_LU) {
    if (q == 2) *i = *j = s + 1;
    else if (q < 2) (q == 0 ? *i : *j) = s + 1;
    else ((q & 1) ? *i : *j) = s + 2 + (q - 3) / 2;
  } else {
    *i = q < 2 ? s + 1 : s + q;
    if (q == 1) *j = s + 1;
  }
}

// Tiles from the counter until there are none left.
template <typename T, int KIND, int AUX, int WAVES>
__device__ __forceinline__ void tile_owners(const TileArgs<T>& g, T* const smem, int* const ticket, TileTeam<WAVES> team) {
  const int tid = (int)threadIdx.x % (WAVES * 64), tiles = tile_count<KIND>(g.nt);
  for (;;) {
    team.barrier();
    if (tid == 0) *ticket = __hip_atomic_fetch_add(g.ints + TileFlags::kTicket, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    team.barrier();
    const int id = __builtin_amdgcn_readfirstlane(*ticket);
    if (id >= tiles) return;  // uniform
    int i, j;
    tile_of<KIND>(g.nt, id, &i, &j);
    if constexpr (WAVES == 4) {  // beside the diagonal: before the other team
      if (i - j <= 2 && j - i <= 2) __builtin_amdgcn_s_setprio(3);
      else __builtin_amdgcn_s_setprio(0);
    }
    tile_owner<T, KIND, AUX, WAVES>(g, smem, team, i, j);
  }
}

// The whole factorisation in one launch; TEAMS: how many tiles a workgroup has at a time.
constexpr int kTileTeamElems = 2 * kTileNb * kTileLd + kTileSub * kBlk;
template <typename T, int TEAMS>
constexpr int tile_lds_bytes() {
  constexpr int elems = TEAMS * kTileTeamElems > kTileLds ? TEAMS * kTileTeamElems : kTileLds, bytes = elems * (int)sizeof(T);
  return bytes > 84 * 1024 ? bytes : 84 * 1024;  // (more than half of a compute unit's: one workgroup each)
}
template <typename T, int KIND, int AUX, int TEAMS>
__global__ void __launch_bounds__(kTileThreads, 2) tile_factor_kernel(const TileArgs<T> g) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  __shared__ int ticket[TEAMS], arrived[TEAMS];
  T* const smem = reinterpret_cast<T*>(smem_raw);
  constexpr int WAVES = kTileThreads / 64 / TEAMS;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), t = TEAMS == 1 ? 0 : wave / WAVES;
  if (threadIdx.x < TEAMS) arrived[threadIdx.x] = 0;
  __syncthreads();
  if (blockIdx.x == 0) tile_chain<T, KIND>(g, smem);
  else tile_owners<T, KIND, AUX, WAVES>(g, smem + t * kTileTeamElems, ticket + t, TileTeam<WAVES>{wave % WAVES, arrived + t});
}

}  // namespace dla
