// Plain bulk generation: leapfrog kernels (GGL, RANECU, DRAND48, RANNYU), lane-per-stream kernels
// (XOR128, RANMAR; and, for four-way interleaved output, RANLUX) and MT19937.
#include <array>

#include "device.h"

namespace prng {
namespace {

// ============================================================ lane kernels
// PACK: streams interleaved four by four (element v of stream s at
// ((s / 4) row_elems + elem_off + v) 16 + (s % 4) 4 bytes); 4-byte dtypes only.
template <class G, int DT, bool PACK = false>
__global__ __launch_bounds__(256) void k_lane_generate(uint32_t* __restrict__ state, uint64_t n, uint32_t draws,
                                                       uint32_t p, void* __restrict__ out, uint64_t row_elems,
                                                       uint64_t elem_off) {
  constexpr uint32_t T = G::T;
  __shared__ __attribute__((aligned(16))) uint32_t stage_all[4][stage_words<T>()];
  const int lane = threadIdx.x & 63;
  uint32_t* stage = stage_all[threadIdx.x >> 6];
  const uint64_t si = (uint64_t)blockIdx.x * 256u + threadIdx.x;
  G g;
  if constexpr (requires { g.p; }) g.p = p;
  uint32_t vbeg = 0;
  const bool live = si < n;
  if (live)
    g.load(state, n, si, vbeg);
  else
    g.zero();
  const uint32_t vend = live ? vbeg + draws : vbeg;
  constexpr uint64_t es = DT == F64 ? 8 : 4;
  // element of position v at q + 4 v, or q + 16 v when PACK (element 0 is position vbeg)
  uint64_t q = 0;
  if (live) {
    if constexpr (PACK)
      q = reinterpret_cast<uint64_t>(out) + ((si >> 2) * row_elems + elem_off) * 16ull + (si & 3u) * 4ull - 16ull * vbeg;
    else
      q = reinterpret_cast<uint64_t>(out) + (si * row_elems + elem_off) * es - 4ull * vbeg;
  }
  lane_loop<G, DT, PACK>(g, stage, lane, vbeg, vbeg, vend, q, !PACK, row_elems * es);
  if (live) g.store(state, n, si, vbeg, vend);
}

// XOR128 plain generation with every stream cut into K segments of S
// positions: block b works on segment j = b / nb of the 256 streams
// (b mod nb) of that range, nb = ceil(n / 256).  Every segment starts from
// the snapshot `snap` taken before the launch, segment j > 0 jumped j S
// positions ahead; the last segment writes the final state.  XOR128's draws
// carry no position structure, so segments run in the stream's own
// coordinates; S is even, so fp64 pairs never straddle a boundary.  64-draw
// chunks put two workgroups on a CU; long launches of many streams, bound by
// their stores, take 128-draw chunks.
template <int DT, int TT>
__global__ __launch_bounds__(256) void k_xor128_split(uint32_t* __restrict__ state, const uint32_t* __restrict__ snap,
                                                      uint64_t n, uint32_t draws, uint32_t S, uint32_t K,
                                                      const uint32_t* __restrict__ pow2, void* __restrict__ out,
                                                      uint64_t row_elems, uint64_t elem_off) {
  using G = Xor128<TT>;
  constexpr uint32_t T = G::T;
  __shared__ __attribute__((aligned(16))) uint32_t stage_all[4][stage_words<T>()];
  const int lane = threadIdx.x & 63;
  uint32_t* stage = stage_all[threadIdx.x >> 6];
  const uint32_t nb = (uint32_t)((n + 255) / 256);
  const uint32_t j = blockIdx.x / nb;
  const uint64_t si = (uint64_t)(blockIdx.x - j * nb) * 256u + threadIdx.x;
  const bool live = si < n;
  G g;
  const uint32_t beg = j * S, end = j + 1u == K ? draws : min((j + 1u) * S, draws);
  if (live) {
    if (j == 0) {
      uint32_t v0;
      g.load(snap, n, si, v0);
    } else {
      g.load_jumped_pow2(snap, n, si, beg, pow2);
    }
  } else {
    g.zero();
  }
  constexpr uint64_t es = DT == F64 ? 8 : 4;
  const uint64_t q = live ? reinterpret_cast<uint64_t>(out) + (si * row_elems + elem_off) * es : 0;
  lane_loop<G, DT>(g, stage, lane, beg, beg, live ? end : beg, q, true, row_elems * es);
  if (live && j + 1u == K) g.store(state, n, si, beg, end);
}

// One stream at a time per workgroup: its four wavefronts twist and store
// each block together, so that the chip writes few rows at a time, each in
// bursts.  A workgroup takes streams 2b and 2b + 1 and fetches the second
// one's table into registers before it generates the first, so that only
// the first table's load is waited for.
template <int DT>
__global__ __launch_bounds__(256) void k_mt_generate(uint32_t* __restrict__ state, uint64_t n, uint32_t draws,
                                                     void* __restrict__ out, uint64_t row_elems, uint64_t elem_off) {
  __shared__ __attribute__((aligned(16))) uint32_t mt[624];
  __shared__ __attribute__((aligned(16))) uint32_t stage[628];
  const int tid = (int)threadIdx.x;
  const uint64_t s0 = 2ull * blockIdx.x;
  if (s0 >= n) return;  // the whole workgroup
  const bool two = s0 + 1 < n;
  constexpr uint64_t es = DT == F64 ? 8 : 4;
  uint32_t* const sp0 = state + s0 * kMtStride;
  uint32_t* const sp1 = sp0 + kMtStride;
  uint32_t nxt[3] = {0u, 0u, 0u}, nxt_pos = 0u;
  if (two) {
#pragma unroll
    for (int q = 0; q < 3; ++q)
      if (tid + 256 * q < 624) nxt[q] = sp1[tid + 256 * q];
    nxt_pos = sp1[624];
  }
  mt_body<DT>(mt, stage, tid, sp0, uni(sp0[624]), 0u, draws,
              reinterpret_cast<uint64_t>(out) + (s0 * row_elems + elem_off) * es, sp0);
  if (!two) return;
#pragma unroll
  for (int q = 0; q < 3; ++q)
    if (tid + 256 * q < 624) mt[tid + 256 * q] = nxt[q];
  __syncthreads();
  mt_body<DT>(mt, stage, tid, nullptr, uni(nxt_pos), 0u, draws,
              reinterpret_cast<uint64_t>(out) + ((s0 + 1) * row_elems + elem_off) * es, sp1);
}

// Emitter of mt_twist_emit for 4-byte rows: word i of the block at `at` + 4 i.
template <int DT>
struct MtRowEmit {
  uint64_t at;
  __device__ __forceinline__ void operator()(int i, uint32_t w) const {
    const uint32_t u = mt_temper(w);
    put<uint32_t>(at + 4ull * (uint32_t)i, DT == U32 ? u : __float_as_uint(mt_f32<DT>(u)));
  }
};

template <int DT>
__device__ __forceinline__ void mt_row_wave(uint32_t* mt, int lane, uint32_t& pos, uint32_t draws, uint64_t row) {
  uint32_t done = 0;
  while (done < draws) {
    if (pos >= 624u) {
      mt_twist(mt, lane);
      pos = 0;
    }
    const MtRowEmit<DT> emit{row + 4ull * done};
    if (pos == 0u && draws - done > 624u) {
      // a whole block with draws after it: stored during the twist that makes the next block
      mt_twist_emit(mt, lane, emit);
      done += 624u;
      continue;
    }
    const uint32_t m = min(624u - pos, draws - done);
    for (uint32_t j = (uint32_t)lane; j < m; j += 64u) emit((int)j, mt[pos + j]);
    pos += m;
    done += m;
  }
}

// One stream per wavefront, its words stored straight from the twist that
// consumes them (256 bytes of the row per store): no barriers, and 17 VALU
// instructions per 64 draws where k_mt_generate, whose phases and stores fill
// 227 and 156 of 256 lanes, takes 25.  f32: 10007 x 1537 31 -> 23 us, 16384 x
// 4096 74 -> 62 us, 65536 x 300 85 -> 68 us, 256 x 4096 12.2 -> 8.6 us.
template <int DT>
__global__ __launch_bounds__(256) void k_mt_wave(uint32_t* __restrict__ state, uint64_t n, uint32_t draws,
                                                 void* __restrict__ out, uint64_t row_elems, uint64_t elem_off) {
  static_assert(DT != F64, "an fp64 element takes the words of two lanes");
  __shared__ uint32_t mt_all[4][624];
  const int lane = threadIdx.x & 63;
  const uint64_t s = (uint64_t)blockIdx.x * 4u + (threadIdx.x >> 6);
  if (s >= n) return;  // whole wavefront; no block-wide barrier is used
  uint32_t* mt = mt_all[threadIdx.x >> 6];
  uint32_t* sp = state + s * kMtStride;
  for (int i = lane; i < 624; i += 64) mt[i] = sp[i];
  uint32_t pos = uni(sp[624]);
  wave_sync();
  const uint64_t row = reinterpret_cast<uint64_t>(out) + (s * row_elems + elem_off) * 4ull;
  mt_row_wave<DT>(mt, lane, pos, draws, row);
  wave_sync();
  for (int i = lane; i < 624; i += 64) sp[i] = mt[i];
  if (lane == 0) sp[624] = pos;
}

// ============================================================ leapfrog kernels
// Multiplicative and affine generators (GGL, RANECU, DRAND48, RANNYU): one
// wavefront per stream; lane l produces positions 4 l .. 4 l + 3 of every
// block of 256, so that each store instruction writes 256 consecutive
// elements of the row (1 KB for u32/f32, four per lane) with no LDS
// transpose, and the stream's row is written front to back.  Within its four
// positions a lane steps the recurrence; to its next four it leaps by a^253
// from the last (the affine map of 253 steps for the 48-bit LCGs), so every
// position still costs one multiplication.

constexpr uint32_t kLeapQuad = 4, kLeapBlock = 64 * kLeapQuad;

// a^(4 l + 1) mod m for the 64 lanes: each lane's first position in one multiplication
template <uint64_t A, uint64_t Mod>
struct LaneStart {
  static constexpr std::array<uint32_t, 64> table() {
    std::array<uint32_t, 64> t{};
    for (uint32_t l = 0; l < 64; ++l) t[l] = (uint32_t)cpowmod(A, kLeapQuad * l + 1, Mod);
    return t;
  }
  static constexpr std::array<uint32_t, 64> kPow = table();
};

// GGL: the output of position v is X_{v+1} = a^{v+1} X_0.
struct LeapGgl {
  using Steps = Ggl<>;  // the same recurrence, with the map of q steps
  static constexpr int BITS = 31;
  static constexpr bool kNtOut = false;
  static constexpr uint32_t A = 16807u, AL = (uint32_t)cpowmod(A, kLeapBlock - 3, 2147483647u);
  uint32_t x;  // X of the lane's first position in the current block
  __device__ void load(const uint32_t* st, uint64_t, uint64_t si) { x = st[si]; }
  // lane l: X_{4l+1}, the state of its first position
  __device__ void start(int lane) { x = mulmod_2p31<1u>(x, LaneStart<A, 2147483647u>::kPow[lane]); }
  // draws of the lane's four positions; leaves x at the last one
  __device__ __forceinline__ void quad(uint32_t* u) {
    u[0] = x;
#pragma unroll
    for (int j = 1; j < 4; ++j) {
      x = mul_mod_2p31<A, 1u>(x);
      u[j] = x;
    }
  }
  __device__ __forceinline__ void leap() { x = mulmod_2p31<1u>(x, AL); }
  // state after the position at offset j of the quad (x at the quad's first position)
  __device__ void store_at(uint32_t j, uint32_t* st, uint64_t, uint64_t si) const {
    uint32_t y = x;
    for (uint32_t i = 0; i < j; ++i) y = mul_mod_2p31<A, 1u>(y);
    st[si] = y;
  }
  static __device__ float paper_f32(uint32_t u) { return Ggl<>::paper_f32(u); }
  // the map of q steps, w times over
  __device__ void advance_q(uint64_t j0, uint64_t, uint32_t w) {
    for (uint32_t i = 0; i < w; ++i) x = mulmod_2p31<1u>(x, (uint32_t)j0);
  }
};

// RANECU: both MLCGs leap; the draw combines the two states.
struct LeapRanecu {
  using Steps = Ranecu<>;  // the same recurrence, with the map of q steps
  static constexpr int BITS = 31;
  static constexpr bool kNtOut = true;  // two MLCG steps per draw between the stores
  static constexpr uint32_t A1 = 40014u, A2 = 40692u;
  static constexpr uint32_t B1 = (uint32_t)cpowmod(A1, kLeapBlock - 3, 2147483563u),
                            B2 = (uint32_t)cpowmod(A2, kLeapBlock - 3, 2147483399u);
  uint32_t s1, s2;
  __device__ void load(const uint32_t* st, uint64_t sn, uint64_t si) {
    s1 = st[si];
    s2 = st[sn + si];
  }
  __device__ void start(int lane) {
    s1 = mulmod_2p31<85u>(s1, LaneStart<A1, 2147483563u>::kPow[lane]);
    s2 = mulmod_2p31<249u>(s2, LaneStart<A2, 2147483399u>::kPow[lane]);
  }
  static __device__ __forceinline__ uint32_t combine(uint32_t a, uint32_t b) {
    int32_t z = (int32_t)a - (int32_t)b;
    z += (z <= 0) ? 2147483562 : 0;
    return (uint32_t)z;
  }
  __device__ __forceinline__ void quad(uint32_t* u) {
    u[0] = combine(s1, s2);
#pragma unroll
    for (int j = 1; j < 4; ++j) {
      s1 = mul_mod_2p31<A1, 85u>(s1);
      s2 = mul_mod_2p31<A2, 249u>(s2);
      u[j] = combine(s1, s2);
    }
  }
  __device__ __forceinline__ void leap() {
    s1 = mulmod_2p31<85u>(s1, B1);
    s2 = mulmod_2p31<249u>(s2, B2);
  }
  __device__ void store_at(uint32_t j, uint32_t* st, uint64_t sn, uint64_t si) const {
    uint32_t a = s1, b = s2;
    for (uint32_t i = 0; i < j; ++i) {
      a = mul_mod_2p31<A1, 85u>(a);
      b = mul_mod_2p31<A2, 249u>(b);
    }
    st[si] = a;
    st[sn + si] = b;
  }
  static __device__ float paper_f32(uint32_t u) { return Ranecu<>::paper_f32(u); }
  __device__ void advance_q(uint64_t j0, uint64_t j1, uint32_t w) {
    for (uint32_t i = 0; i < w; ++i) {
      s1 = mulmod_2p31<85u>(s1, (uint32_t)j0);
      s2 = mulmod_2p31<249u>(s2, (uint32_t)j1);
    }
  }
};

// DRAND48 / RANNYU: the draw is X >> 16 of the 48-bit state.
template <uint64_t A, uint64_t C>
struct LeapLcg48 {
  using Steps = Lcg48<128, A, C>;  // the same recurrence, with the map of q steps
  static constexpr int BITS = 32;
  static constexpr bool kNtOut = false;
  static constexpr uint64_t M = (1ull << 48) - 1;
  static constexpr Affine48 PL = caffine_pow(A, C, kLeapBlock - 3);
  uint64_t x;
  __device__ void load(const uint32_t* st, uint64_t sn, uint64_t si) {
    x = (uint64_t)st[si] | ((uint64_t)st[sn + si] << 32);
  }
  static constexpr std::array<Affine48, 64> starts() {
    std::array<Affine48, 64> t{};
    for (uint32_t l = 0; l < 64; ++l) t[l] = caffine_pow(A, C, kLeapQuad * l + 1);
    return t;
  }
  static constexpr std::array<Affine48, 64> kStart = starts();
  // lane l: X_{4l+1}, the state of its first position
  __device__ void start(int lane) {
    const Affine48 f = kStart[lane];
    x = (f.a * x + f.c) & M;
  }
  __device__ __forceinline__ void quad(uint32_t* u) {
    u[0] = (uint32_t)(x >> 16);
#pragma unroll
    for (int j = 1; j < 4; ++j) {
      x = (A * x + C) & M;
      u[j] = (uint32_t)(x >> 16);
    }
  }
  __device__ __forceinline__ void leap() { x = (PL.a * x + PL.c) & M; }
  __device__ void store_at(uint32_t j, uint32_t* st, uint64_t sn, uint64_t si) const {
    uint64_t y = x;
    for (uint32_t i = 0; i < j; ++i) y = (A * y + C) & M;
    st[si] = (uint32_t)y;
    st[sn + si] = (uint32_t)(y >> 32);
  }
  __device__ void advance_q(uint64_t j0, uint64_t j1, uint32_t w) {
    for (uint32_t i = 0; i < w; ++i) x = (j0 * x + j1) & M;
  }
};

// n streams from `state` on, whose rows lie sn words apart
template <class L, int DT, bool QUADS>
__global__ __launch_bounds__(256) void k_leap_generate(uint32_t* __restrict__ state, uint64_t sn, uint64_t n,
                                                       uint32_t draws, void* __restrict__ out, uint64_t row_elems,
                                                       uint64_t elem_off) {
  const int lane = threadIdx.x & 63;
  const uint64_t s = (uint64_t)blockIdx.x * 4u + (threadIdx.x >> 6);
  if (s >= n || draws == 0) return;  // whole wavefront
  L g;
  g.load(state, sn, s);
  g.start(lane);  // X of position 4 l
  constexpr uint64_t es = DT == F64 ? 8 : 4;
  // position v's element at byte row + 4 v (an fp64 element per pair of draws)
  const uint64_t row = reinterpret_cast<uint64_t>(out) + (s * row_elems + elem_off) * es;
  // blocks k with 256 (k + 2) <= draws: every lane fills its four positions and leaps
  const uint32_t full = draws / kLeapBlock;
  uint32_t k = 0;
  uint32_t u[4];
#pragma unroll 2
  for (; k + 1u < full; ++k) {
    g.quad(u);
    quad_emit<L, DT, QUADS>(row, k * kLeapBlock + kLeapQuad * (uint32_t)lane, u, draws);
    g.leap();
  }
  // the last one or two blocks: a lane leaps only if it has a later position;
  // the lane of the last position stores the state after it
  const uint32_t last = draws - 1u;
  for (; k * kLeapBlock < draws; ++k) {
    const uint32_t v = k * kLeapBlock + kLeapQuad * (uint32_t)lane;
    if (v < draws) {
      L h = g;  // quad() moves the state to the quad's last position
      h.quad(u);
      quad_emit<L, DT, QUADS>(row, v, u, draws);
      if (v + kLeapBlock < draws) {
        h.leap();
        g = h;
      } else if (last - v < kLeapQuad) {
        g.store_at(last - v, state, sn, s);
      }
    }
  }
}

// Plain generation by quarters of rows: the four wavefronts of a workgroup
// share its four streams, wavefront w generating positions [w Q, (w + 1) Q)
// (Q a multiple of 256) of each row in turn, from the stream's state advanced
// w Q positions (the map of Q steps, j0/j1, applied w times).  At any moment a
// workgroup's stores fall in four contiguous stretches of adjacent rows; this
// store order measured 4-5% faster than one wavefront per row.  Every
// wavefront reads the four states before the barrier; the wavefront of a
// row's last position writes its new state after it.
template <class L, int DT, bool QUADS>
__global__ __launch_bounds__(256) void k_leap_quarters(uint32_t* __restrict__ state, uint64_t sn, uint64_t n,
                                                       uint32_t draws, uint32_t Q, uint64_t j0, uint64_t j1,
                                                       void* __restrict__ out, uint64_t row_elems, uint64_t elem_off) {
  const int lane = threadIdx.x & 63;
  const uint32_t w = uni(threadIdx.x >> 6);
  const uint64_t s0 = (uint64_t)blockIdx.x * 4u;
  L g[4];
#pragma unroll
  for (int r = 0; r < 4; ++r)
    if (s0 + r < n) g[r].load(state, sn, s0 + r);
  __syncthreads();
  const uint32_t beg = w * Q, end = min(beg + Q, draws);
  if (beg >= end) return;  // whole wavefront, after the barrier
  constexpr uint64_t es = DT == F64 ? 8 : 4;
  const uint32_t last = draws - 1u;
  for (int r = 0; r < 4; ++r) {
    const uint64_t s = s0 + r;
    if (s >= n) break;
    L h = g[r];
    h.advance_q(j0, j1, w);  // X of position w Q
    h.start(lane);           // X of position w Q + 4 l
    const uint64_t row = reinterpret_cast<uint64_t>(out) + (s * row_elems + elem_off) * es;
    uint32_t u[4];
    uint32_t v = beg + kLeapQuad * (uint32_t)lane;
    // blocks whose next block is still inside the quarter: fill, then leap
    for (; v + kLeapBlock + (kLeapBlock - kLeapQuad * (uint32_t)lane) <= end; v += kLeapBlock) {
      h.quad(u);
      quad_emit<L, DT, QUADS>(row, v, u, end);
      h.leap();
    }
    // the remaining one or two blocks: leap only towards a later position
    for (; v - kLeapQuad * (uint32_t)lane < end; v += kLeapBlock) {
      if (v < end) {
        L q = h;
        q.quad(u);
        quad_emit<L, DT, QUADS>(row, v, u, end);
        if (v + kLeapBlock < end) {
          q.leap();
          h = q;
        } else if (end == draws && last - v < kLeapQuad) {
          h.store_at(last - v, state, sn, s);
        }
      }
    }
  }
}

template <class L, bool QUADS>
hipError_t launch_leap_rows(int dtype, uint32_t* st, uint64_t sn, uint64_t n, uint64_t draws, void* out,
                            uint64_t row_elems, uint64_t off, hipStream_t s) {
  const dim3 grid((unsigned)((n + 3) / 4)), block(256);
  const uint32_t d = (uint32_t)draws;
  // rows of at least four blocks per wavefront go by quarters
  if (draws >= 16 * kLeapBlock) {
    const uint64_t Q = ((draws + 3) / 4 + kLeapBlock - 1) / kLeapBlock * kLeapBlock;
    const uint32_t q = (uint32_t)Q;
    uint64_t j0 = 0, j1 = 0;
    L::Steps::q_map(Q, j0, j1);
    switch (dtype) {
      case U32:
        hipLaunchKernelGGL((k_leap_quarters<L, U32, QUADS>), grid, block, 0, s, st, sn, n, d, q, j0, j1, out, row_elems,
                           off);
        break;
      case F32:
        hipLaunchKernelGGL((k_leap_quarters<L, F32, QUADS>), grid, block, 0, s, st, sn, n, d, q, j0, j1, out, row_elems,
                           off);
        break;
      case F64:
        hipLaunchKernelGGL((k_leap_quarters<L, F64, QUADS>), grid, block, 0, s, st, sn, n, d, q, j0, j1, out, row_elems,
                           off);
        break;
      case F32P:
        if constexpr (requires { L::paper_f32(0u); }) {
          hipLaunchKernelGGL((k_leap_quarters<L, F32P, QUADS>), grid, block, 0, s, st, sn, n, d, q, j0, j1, out,
                             row_elems, off);
          break;
        }
        return hipErrorInvalidValue;
      default:
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
  }
  switch (dtype) {
    case U32:
      hipLaunchKernelGGL((k_leap_generate<L, U32, QUADS>), grid, block, 0, s, st, sn, n, d, out, row_elems, off);
      break;
    case F32:
      hipLaunchKernelGGL((k_leap_generate<L, F32, QUADS>), grid, block, 0, s, st, sn, n, d, out, row_elems, off);
      break;
    case F64:
      hipLaunchKernelGGL((k_leap_generate<L, F64, QUADS>), grid, block, 0, s, st, sn, n, d, out, row_elems, off);
      break;
    case F32P:
      if constexpr (requires { L::paper_f32(0u); }) {
        hipLaunchKernelGGL((k_leap_generate<L, F32P, QUADS>), grid, block, 0, s, st, sn, n, d, out, row_elems, off);
        break;
      }
      return hipErrorInvalidValue;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// every row 16-byte aligned, or rows at any alignment
template <class L>
hipError_t launch_leap(int dtype, uint32_t* st, uint64_t n, uint64_t draws, void* out, uint64_t row_elems,
                       uint64_t off, hipStream_t s) {
  const uint64_t es = elem_bytes(dtype);
  const bool quads = ((reinterpret_cast<uint64_t>(out) + off * es) | (n > 1 ? row_elems * es : 0)) % 16 == 0;
  return for_stream_ranges(n, kWaveStreams, [&](uint64_t s0, uint64_t m) {
    void* const o = static_cast<char*>(out) + s0 * row_elems * es;
    return quads ? launch_leap_rows<L, true>(dtype, st + s0, n, m, draws, o, row_elems, off, s)
                 : launch_leap_rows<L, false>(dtype, st + s0, n, m, draws, o, row_elems, off, s);
  });
}

// Interleaved rows of the multiplicative and affine generators: W wavefronts
// on the four streams of a row, lane t of them at positions t, t + 64 W, ...,
// leaping by the map of 64 W steps, so that a store instruction writes 1 KB of
// the row and no LDS is needed.  Lane t's first position is the state advanced
// t + 1 steps: maps.a[0] is the map of one step, and one application per set
// bit of t follows.  Bound by the stores (GGL 16384 x 4096 f32, one lane per
// stream through an LDS transpose on 256 wavefronts: 117 us before, 51 us now).
template <class G, int DT, int W>
__global__ __launch_bounds__(W == 16 ? 1024 : 256) void k_leap_pack4(uint32_t* __restrict__ state, uint64_t n,
                                                                     uint32_t draws, SplitMaps maps, uint64_t leap_a,
                                                                     uint64_t leap_c, void* __restrict__ out,
                                                                     uint64_t row_elems, uint64_t elem_off) {
  constexpr int kBits = W == 1 ? 6 : W == 4 ? 8 : 10;
  const uint64_t row = W == 1 ? (uint64_t)blockIdx.x * 4u + (threadIdx.x >> 6) : (uint64_t)blockIdx.x;
  const uint32_t t = W == 1 ? threadIdx.x & 63u : threadIdx.x;
  const bool live = 4u * row < n;  // n is a multiple of four
  G g[4];
  if (live) {
    uint32_t unused;
#pragma unroll
    for (int k = 0; k < 4; ++k) g[k].load(state, n, 4u * row + k, unused);
  }
  if constexpr (W > 1) __syncthreads();  // every wavefront has read the states
  if (!live || t >= draws) return;
#pragma unroll
  for (int k = 0; k < 4; ++k) g[k].advance(maps.a[0], maps.c[0]);
  for (int b = 0; b < kBits; ++b) {
    if ((t >> b) & 1u) {
#pragma unroll
      for (int k = 0; k < 4; ++k) g[k].advance(maps.a[b], maps.c[b]);
    }
  }
  uint64_t at = reinterpret_cast<uint64_t>(out) + (row * row_elems + elem_off + t) * 16ull;
  for (uint32_t v = t;; v += 64u * W) {
    uint32_t o[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) o[k] = DT == U32 ? g[k].draw() : __float_as_uint(cvt32<G, DT>(g[k].draw()));
    put<v4u>(at, v4u{o[0], o[1], o[2], o[3]});
    if (draws - v <= 64u * W) {  // the lane's last position; the row's last one gives the new states
      if (v == draws - 1u) {
#pragma unroll
        for (int k = 0; k < 4; ++k) g[k].store(state, n, 4u * row + k, 0u, 0u);
      }
      return;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) g[k].advance(leap_a, leap_c);
    at += 1024ull * W;
  }
}

template <class G, int W>
hipError_t launch_leap_pack_w(int dtype, uint32_t* st, uint64_t n, uint64_t draws, void* out, uint64_t row_elems,
                              uint64_t off, hipStream_t s) {
  const uint64_t rows = n / 4;
  const dim3 grid((unsigned)(W == 1 ? (rows + 3) / 4 : rows)), block(W == 16 ? 1024 : 256);
  const uint32_t d = (uint32_t)draws;
  SplitMaps maps{};
  for (int k = 0; k < kMaxSplitBits; ++k) G::q_map(1ull << k, maps.a[k], maps.c[k]);
  uint64_t la = 0, lc = 0;
  G::q_map(64ull * W, la, lc);
  switch (dtype) {
    case U32:
      hipLaunchKernelGGL((k_leap_pack4<G, U32, W>), grid, block, 0, s, st, n, d, maps, la, lc, out, row_elems, off);
      break;
    case F32:
      hipLaunchKernelGGL((k_leap_pack4<G, F32, W>), grid, block, 0, s, st, n, d, maps, la, lc, out, row_elems, off);
      break;
    case F32P:
      if constexpr (requires { G::paper_f32(0u); }) {
        hipLaunchKernelGGL((k_leap_pack4<G, F32P, W>), grid, block, 0, s, st, n, d, maps, la, lc, out, row_elems,
                           off);
        break;
      }
      return hipErrorInvalidValue;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <class G>
hipError_t launch_lane_pack(int dtype, uint32_t p, uint32_t* st, uint64_t n, uint64_t draws, void* out,
                            uint64_t row_elems, uint64_t off, hipStream_t s) {
  const dim3 grid((unsigned)((n + 255) / 256)), block(256);
  const uint32_t d = (uint32_t)draws;
  switch (dtype) {
    case U32:
      hipLaunchKernelGGL((k_lane_generate<G, U32, true>), grid, block, 0, s, st, n, d, p, out, row_elems, off);
      break;
    case F32:
      hipLaunchKernelGGL((k_lane_generate<G, F32, true>), grid, block, 0, s, st, n, d, p, out, row_elems, off);
      break;
    case F32P:
      if constexpr (requires { G::paper_f32(0u); }) {
        hipLaunchKernelGGL((k_lane_generate<G, F32P, true>), grid, block, 0, s, st, n, d, p, out, row_elems, off);
        break;
      }
      return hipErrorInvalidValue;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// wavefronts per row of four streams: about 4096 in all, none without a position
template <class G>
hipError_t launch_leap_pack(int dtype, uint32_t* st, uint64_t n, uint64_t draws, void* out, uint64_t row_elems,
                            uint64_t off, hipStream_t s) {
  if (n > kWaveStreams || leap_packed_per_lane(std::is_same_v<G, Ranecu<>>, n, draws))
    return launch_lane_pack<G>(dtype, 0u, st, n, draws, out, row_elems, off, s);
  const uint64_t want = std::min((4096 + n / 4 - 1) / (n / 4), (draws + 63) / 64);
  if (want >= 16) return launch_leap_pack_w<G, 16>(dtype, st, n, draws, out, row_elems, off, s);
  if (want >= 4) return launch_leap_pack_w<G, 4>(dtype, st, n, draws, out, row_elems, off, s);
  return launch_leap_pack_w<G, 1>(dtype, st, n, draws, out, row_elems, off, s);
}

template <class G>
hipError_t launch_lane_gen(int dtype, uint32_t p, uint32_t* st, uint64_t n, uint64_t draws, void* out,
                           uint64_t row_elems, uint64_t off, hipStream_t s) {
  const dim3 grid((unsigned)((n + 255) / 256)), block(256);
  const uint32_t d = (uint32_t)draws;
  switch (dtype) {
    case U32:
      hipLaunchKernelGGL((k_lane_generate<G, U32>), grid, block, 0, s, st, n, d, p, out, row_elems, off);
      break;
    case F32:
      hipLaunchKernelGGL((k_lane_generate<G, F32>), grid, block, 0, s, st, n, d, p, out, row_elems, off);
      break;
    case F64:
      hipLaunchKernelGGL((k_lane_generate<G, F64>), grid, block, 0, s, st, n, d, p, out, row_elems, off);
      break;
    case F32P:
      if constexpr (requires { G::paper_f32(0u); }) {
        hipLaunchKernelGGL((k_lane_generate<G, F32P>), grid, block, 0, s, st, n, d, p, out, row_elems, off);
        break;
      }
      return hipErrorInvalidValue;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// one stream per wavefront (4-byte dtypes) or per workgroup
hipError_t launch_mt_rows(bool wave, int dtype, uint32_t* st, uint64_t n, uint64_t draws, void* out,
                          uint64_t row_elems, uint64_t off, hipStream_t s) {
  const dim3 gw((unsigned)((n + 3) / 4)), grid((unsigned)((n + 1) / 2)), block(256);
  const uint32_t d = (uint32_t)draws;
  if (wave) {
    if (dtype == U32)
      hipLaunchKernelGGL((k_mt_wave<U32>), gw, block, 0, s, st, n, d, out, row_elems, off);
    else if (dtype == F32)
      hipLaunchKernelGGL((k_mt_wave<F32>), gw, block, 0, s, st, n, d, out, row_elems, off);
    else if (dtype == F32P)
      hipLaunchKernelGGL((k_mt_wave<F32P>), gw, block, 0, s, st, n, d, out, row_elems, off);
    else
      return hipErrorInvalidValue;
    return hipGetLastError();
  }
  switch (dtype) {
    case U32:
      hipLaunchKernelGGL((k_mt_generate<U32>), grid, block, 0, s, st, n, d, out, row_elems, off);
      break;
    case F32:
      hipLaunchKernelGGL((k_mt_generate<F32>), grid, block, 0, s, st, n, d, out, row_elems, off);
      break;
    case F64:
      hipLaunchKernelGGL((k_mt_generate<F64>), grid, block, 0, s, st, n, d, out, row_elems, off);
      break;
    case F32P:
      hipLaunchKernelGGL((k_mt_generate<F32P>), grid, block, 0, s, st, n, d, out, row_elems, off);
      break;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_generate(int kind, uint32_t p, uint32_t* st, uint64_t n, uint64_t draws, int dtype, void* out,
                           uint64_t row_elems, uint64_t off, hipStream_t s) {
  switch (kind) {
    case GGL:
      return launch_leap<LeapGgl>(dtype, st, n, draws, out, row_elems, off, s);
    case XOR128:
      return launch_lane_gen<Xor128<>>(dtype, p, st, n, draws, out, row_elems, off, s);
    case RANECU:
      return launch_leap<LeapRanecu>(dtype, st, n, draws, out, row_elems, off, s);
    case RANMAR:
      if (ranmar_row_per_lane(n, draws))
        return launch_lane_gen<Ranmar<>>(dtype, p, st, n, draws, out, row_elems, off, s);
      return launch_ranmar(dtype, st, n, draws, out, row_elems, off, s);
    case DRAND48:
      return launch_leap<LeapLcg48<25214903917ull, 11u>>(dtype, st, n, draws, out, row_elems, off, s);
    case RANNYU:
      return launch_leap<LeapLcg48<31167285ull, 0u>>(dtype, st, n, draws, out, row_elems, off, s);
    case RANLUX:  // prng_generate runs RANLUX through launch_lux_plain
      return hipErrorInvalidValue;
    case MT19937: {
      const bool wave = dtype != F64 && mt_row_per_wave(n, draws);
      return for_stream_ranges(n, kWaveStreams / 2, [&](uint64_t s0, uint64_t m) {
        return launch_mt_rows(wave, dtype, st + s0 * kMtStride, m, draws,
                              static_cast<char*>(out) + s0 * row_elems * elem_bytes(dtype), row_elems, off, s);
      });
    }
  }
  return hipErrorInvalidValue;
}

namespace {
template <int TT>
hipError_t launch_xor128_chunks(uint32_t* st, const uint32_t* snap, uint64_t n, uint64_t draws, int dtype, uint32_t S,
                                uint32_t K, const uint32_t* pow2, void* out, uint64_t row_elems, uint64_t off,
                                hipStream_t s) {
  const dim3 grid((unsigned)((n + 255) / 256 * K)), block(256);
  const uint32_t d = (uint32_t)draws;
  switch (dtype) {
    case U32:
      hipLaunchKernelGGL((k_xor128_split<U32, TT>), grid, block, 0, s, st, snap, n, d, S, K, pow2, out, row_elems,
                         off);
      break;
    case F32:
      hipLaunchKernelGGL((k_xor128_split<F32, TT>), grid, block, 0, s, st, snap, n, d, S, K, pow2, out, row_elems,
                         off);
      break;
    case F64:
      hipLaunchKernelGGL((k_xor128_split<F64, TT>), grid, block, 0, s, st, snap, n, d, S, K, pow2, out, row_elems,
                         off);
      break;
    case F32P:
      hipLaunchKernelGGL((k_xor128_split<F32P, TT>), grid, block, 0, s, st, snap, n, d, S, K, pow2, out, row_elems,
                         off);
      break;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}
}  // namespace

hipError_t launch_xor128_split(uint32_t* st, const uint32_t* snap, uint64_t n, uint64_t draws, int dtype, uint32_t S,
                               uint32_t K, const uint32_t* pow2, void* out, uint64_t row_elems, uint64_t off,
                               hipStream_t s) {
  if (xor128_long_segments(n, draws))
    return launch_xor128_chunks<128>(st, snap, n, draws, dtype, S, K, pow2, out, row_elems, off, s);
  return launch_xor128_chunks<64>(st, snap, n, draws, dtype, S, K, pow2, out, row_elems, off, s);
}

hipError_t launch_generate_packed(int kind, uint32_t p, uint32_t* st, uint64_t n, uint64_t draws, int dtype,
                                  void* out, uint64_t row_elems, uint64_t off, hipStream_t s) {
  switch (kind) {
    case GGL:
      return launch_leap_pack<Ggl<>>(dtype, st, n, draws, out, row_elems, off, s);
    case XOR128:
      return launch_lane_pack<Xor128<>>(dtype, p, st, n, draws, out, row_elems, off, s);
    case RANECU:
      return launch_leap_pack<Ranecu<>>(dtype, st, n, draws, out, row_elems, off, s);
    case RANMAR:
      if (ranmar_packed_per_lane(n, draws))
        return launch_lane_pack<Ranmar<>>(dtype, p, st, n, draws, out, row_elems, off, s);
      return launch_ranmar_packed(dtype, st, n, draws, out, row_elems, off, s);
    case RANLUX:
      return launch_lane_pack<Ranlux<96>>(dtype, p, st, n, draws, out, row_elems, off, s);
    case DRAND48:
      return launch_leap_pack<Drand48<>>(dtype, st, n, draws, out, row_elems, off, s);
    case RANNYU:
      return launch_leap_pack<Rannyu<>>(dtype, st, n, draws, out, row_elems, off, s);
  }
  return hipErrorInvalidValue;
}


}  // namespace prng
