// In-kernel consumers: exact mantissa sums and 64-bin histograms per stream.
#include <bit>

#include "device.h"

namespace prng {
namespace {

template <class G>
__global__ __launch_bounds__(256) void k_lane_fused(uint32_t* __restrict__ state, uint64_t n, uint32_t draws,
                                                    uint32_t p, uint64_t* __restrict__ sum,
                                                    uint32_t* __restrict__ hist, int accumulate) {
  __shared__ uint32_t hist_all[4][64 * kPitch];
  const int lane = threadIdx.x & 63;
  uint32_t* hcol = hist_all[threadIdx.x >> 6] + lane;
#pragma unroll
  for (int b = 0; b < 64; ++b) hcol[b * kPitch] = 0;
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
  constexpr uint32_t T = G::T;
  const bool has = vend > vbeg;
  const uint32_t maxb = wave_max(has ? vbeg : 0u);
  const uint32_t minE = wave_min(has ? vend : 0xFFFFFFFFu);
  const uint32_t maxE = wave_max(has ? vend : 0u);
  const uint32_t nchunks = (maxE + T - 1) / T;
  uint64_t total = 0;
  FusedSink<G::BITS> sink{0u, hcol};
  for (uint32_t c = 0; c < nchunks; ++c) {
    const uint32_t lo = c * T;
    sink.acc = 0;
    if (lo >= maxb && lo + T <= minE)
      g.template chunk<false>(lo, vbeg, vend, sink);
    else
      g.template chunk<true>(lo, vbeg, vend, sink);
    total += sink.acc;
  }
  wave_sync();
  if (live) {
    g.store(state, n, si, vbeg, vend);
    sum[si] = (accumulate ? sum[si] : 0ull) + total;
    uint32_t* hp = hist + si * 64u;
#pragma unroll
    for (int b = 0; b < 64; ++b) hp[b] = (accumulate ? hp[b] : 0u) + hcol[b * kPitch];
  }
}

// In-kernel consumer with every stream cut into 64 W segments of S draws, one
// per lane of the W wavefronts that share the stream (W = 1: four streams per
// workgroup; otherwise a stream per workgroup).  Lane j starts from the
// stream's state advanced j S draws: one application per set bit of j of the
// map of S 2^k steps (a multiplier, an affine map, or for XOR128 the object's
// matrix T^(S 2^k), S a power of two), so no jump data is prepared.  Sums and
// counts are whole numbers, so they add up to those of one pass whatever the
// cut.
//
// One lane per stream (k_lane_fused) runs ceil(n / 64) wavefronts, 64 of them
// at 4096 streams, one dependent step after the other; here every SIMD has
// work from about 1024 / W streams on, and the bound is VALU issue.  RANECU takes
// 20 instructions per draw, 72 cycles of a SIMD for a wavefront's (2.4 for an
// addition or a mask, 4.2 for the others), which is 2.0 ms for 2^32 draws at 2.35
// GHz.  4096 streams x 2^20 draws of RANECU: 46.0 ms with one lane per stream,
// 2.0 ms so (2.1e12 draws/s); 2^30 draws of GGL 0.27 ms.
//
// The histogram has 32 columns of 64 bins: the LDS takes a wavefront in halves
// of 32 lanes, so lanes l and l + 32 share a column without a bank conflict,
// and at 8.4 KB per wavefront four wavefronts run per SIMD (64 columns: two).
constexpr int kSplitT = 16;     // draws per unrolled chunk
template <class G, int W>
__global__ __launch_bounds__(W == 16 ? 1024 : 256) void k_split_fused(uint32_t* __restrict__ state, uint64_t n,
                                                                      uint32_t draws, uint32_t S, SplitMaps maps,
                                                                      uint64_t* __restrict__ sum,
                                                                      uint32_t* __restrict__ hist, int accumulate) {
  constexpr int NH = W == 1 ? 4 : 1;  // histograms per workgroup
  constexpr int kBits = W == 1 ? 6 : W == 4 ? 8 : 10;
  __shared__ uint32_t hist_all[NH][64 * kHistPitch];
  __shared__ uint64_t part[W];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint64_t si = W == 1 ? (uint64_t)blockIdx.x * 4u + wave : (uint64_t)blockIdx.x;
  const bool live = si < n;
  uint32_t* h = hist_all[W == 1 ? wave : 0];
  const uint32_t j = W == 1 ? (uint32_t)lane : threadIdx.x;
  for (uint32_t i = j; i < 64 * kHistPitch; i += 64 * W) h[i] = 0;
  G g;
  g.zero();
  uint32_t cnt = 0;
  if (live) {
    uint32_t unused;
    g.load(state, n, si, unused);
    cnt = j * S < draws ? min(S, draws - j * S) : 0u;  // j S < 2^30 + 2^20
    for (int k = 0; k < kBits; ++k) {
      if constexpr (requires { g.advance_by(maps.mat); }) {
        if (((j >> k) & 1u) && cnt) g.advance_by(maps.mat + 512 * k);
      } else {
        if ((j >> k) & 1u) g.advance(maps.a[k], maps.c[k]);
      }
    }
  }
  if constexpr (W > 1) __syncthreads();  // the histogram is clear, every wavefront has read the state
  wave_sync();
  FusedSink<G::BITS, kHistPitch, W == 1 ? __HIP_MEMORY_SCOPE_WAVEFRONT : __HIP_MEMORY_SCOPE_WORKGROUP> sink{
      0u, h + (lane & 31)};
  uint64_t total = 0;
  uint32_t i = 0;
  for (; i + kSplitT <= cnt; i += kSplitT) {
    sink.acc = 0;
    g.template chunk<false>(0u, 0u, 0u, sink);
    total += sink.acc;
  }
  if (i < cnt) {
    sink.acc = 0;
    g.template chunk<true>(0u, 0u, cnt - i, sink);
    total += sink.acc;
  }
  if (cnt && j * S + cnt == draws) g.store(state, n, si, 0u, 0u);
  for (int o = 32; o > 0; o >>= 1) total += (uint64_t)__shfl_xor((unsigned long long)total, o);
  if constexpr (W > 1) {
    if (lane == 0) part[wave] = total;
    __syncthreads();
    if (wave != 0) return;
    total = 0;
#pragma unroll
    for (int w = 0; w < W; ++w) total += part[w];
  }
  wave_sync();
  if (!live) return;
  uint32_t hb = 0;
#pragma unroll
  for (int l = 0; l < 32; ++l) hb += h[lane * kHistPitch + l];
  if (lane == 0) sum[si] = (accumulate ? sum[si] : 0ull) + total;
  hist[si * 64u + lane] = (accumulate ? hist[si * 64u + lane] : 0u) + hb;
}

// Emitter of mt_twist_emit for the fused consumer: the draw's top 24 bits
// (the f32 value times 2^24) into the lane's sum and the wave's histogram.
// The histogram has kMtCols columns of 64 bins (lane l counts in column
// l mod kMtCols; one pad word per bin): with a single one, 32 lanes of random
// bins cost five extra LDS cycles per draw of a wavefront, a third of the LDS
// time, which bounds the kernel beside VALU issue.
constexpr int kMtCols = 8, kMtHistPitch = kMtCols + 1;
struct MtFusedEmit {
  uint32_t* h;  // the lane's column
  uint32_t part;
  __device__ __forceinline__ void operator()(int, uint32_t w) {
    const uint32_t k = mt_temper(w) >> 8;
    part += k;
    __hip_atomic_fetch_add(&h[(k >> 18) * kMtHistPitch], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
  }
};

__global__ __launch_bounds__(256) void k_mt_fused(uint32_t* __restrict__ state, uint64_t n, uint32_t draws,
                                                  uint64_t* __restrict__ sum, uint32_t* __restrict__ hist,
                                                  int accumulate) {
  __shared__ uint32_t mt_all[4][624];
  __shared__ uint32_t h_all[4][64 * kMtHistPitch];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const uint64_t s = (uint64_t)blockIdx.x * 4u + w;
  if (s >= n) return;
  uint32_t* mt = mt_all[w];
  uint32_t* const h = h_all[w];
  uint32_t* const col = h + (lane & (kMtCols - 1));
  uint32_t* sp = state + s * kMtStride;
  for (int i = lane; i < 624; i += 64) mt[i] = sp[i];
  for (int i = lane; i < 64 * kMtHistPitch; i += 64) h[i] = 0;
  uint32_t pos = uni(sp[624]);
  wave_sync();
  uint32_t done = 0;
  uint64_t acc = 0;
  while (done < draws) {
    if (pos >= 624u) {
      mt_twist(mt, lane);
      pos = 0;
    }
    if (pos == 0u && draws - done > 624u) {
      // a whole block with draws after it: consumed during the twist that
      // makes the next block
      MtFusedEmit emit{col, 0u};
      mt_twist_emit(mt, lane, emit);
      acc += emit.part;
      done += 624u;
      continue;
    }
    const uint32_t m = min(624u - pos, draws - done);
    uint32_t part = 0;
    for (uint32_t j = lane; j < m; j += 64) {
      const uint32_t k = mt_temper(mt[pos + j]) >> 8;
      part += k;
      __hip_atomic_fetch_add(&col[(k >> 18) * kMtHistPitch], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
    }
    acc += part;
    pos += m;
    done += m;
  }
  wave_sync();
  for (int o = 32; o > 0; o >>= 1) acc += (uint64_t)__shfl_xor((unsigned long long)acc, o);
  for (int i = lane; i < 624; i += 64) sp[i] = mt[i];
  if (lane == 0) {
    sp[624] = pos;
    sum[s] = (accumulate ? sum[s] : 0ull) + acc;
  }
  uint32_t hb = 0;
#pragma unroll
  for (int c = 0; c < kMtCols; ++c) hb += h[lane * kMtHistPitch + c];
  hist[s * 64u + lane] = (accumulate ? hist[s * 64u + lane] : 0u) + hb;
}

template <class G>
hipError_t launch_lane_fused(uint32_t p, uint32_t* st, uint64_t n, uint64_t draws, uint64_t* sum, uint32_t* hist,
                             bool acc, hipStream_t s) {
  const dim3 grid((unsigned)((n + 255) / 256)), block(256);
  hipLaunchKernelGGL((k_lane_fused<G>), grid, block, 0, s, st, n, (uint32_t)draws, p, sum, hist, acc ? 1 : 0);
  return hipGetLastError();
}

// G: the kind's 16-draw generator; L: its one-lane-per-stream generator
template <class G, class L>
hipError_t launch_split_fused(double draw_us, uint32_t* st, uint64_t n, uint64_t draws, uint64_t* sum, uint32_t* hist,
                              bool acc, hipStream_t s) {
  constexpr bool kXor = requires(G g) { g.advance_by(st); };
  const int W = consumer_width(draw_us, kXor, n, draws);
  if (W == 0) return launch_lane_fused<L>(0u, st, n, draws, sum, hist, acc, s);
  uint64_t S = (draws + 64ull * W - 1) / (64ull * W);
  SplitMaps maps{};
  if constexpr (kXor) {
    S = std::bit_ceil(S);
    maps.mat = object_tables(XOR128, st, n) + 512 * std::countr_zero(S);  // log2(S) + 9 < 32: S 64 W < 2^31
  } else {
    for (int k = 0; k < kMaxSplitBits; ++k) G::q_map(S << k, maps.a[k], maps.c[k]);
  }
  const dim3 grid((unsigned)(W == 1 ? (n + 3) / 4 : n));
  const uint32_t d = (uint32_t)draws, seg = (uint32_t)S;
  if (W == 1)
    hipLaunchKernelGGL((k_split_fused<G, 1>), grid, dim3(256), 0, s, st, n, d, seg, maps, sum, hist, acc ? 1 : 0);
  else if (W == 4)
    hipLaunchKernelGGL((k_split_fused<G, 4>), grid, dim3(256), 0, s, st, n, d, seg, maps, sum, hist, acc ? 1 : 0);
  else
    hipLaunchKernelGGL((k_split_fused<G, 16>), grid, dim3(1024), 0, s, st, n, d, seg, maps, sum, hist, acc ? 1 : 0);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_fused(int kind, uint32_t p, uint32_t* st, uint64_t n, uint64_t draws, uint64_t* sum,
                        uint32_t* hist, bool acc, hipStream_t s) {
  switch (kind) {
    case GGL:
      return launch_split_fused<Ggl<kSplitT>, Ggl<>>(kGglDrawUs, st, n, draws, sum, hist, acc, s);
    case XOR128:
      return launch_split_fused<Xor128<kSplitT>, Xor128<>>(kXor128DrawUs, st, n, draws, sum, hist, acc, s);
    case RANECU:
      return launch_split_fused<Ranecu<kSplitT>, Ranecu<>>(kRanecuDrawUs, st, n, draws, sum, hist, acc, s);
    case RANMAR:
      if (n > kWaveStreams || ranmar_consumer_per_lane(n, draws))
        return launch_lane_fused<Ranmar<>>(p, st, n, draws, sum, hist, acc, s);
      return launch_ranmar_fused(st, n, draws, sum, hist, acc, s);
    case RANLUX:
      return launch_lane_fused<Ranlux<>>(p, st, n, draws, sum, hist, acc, s);
    case DRAND48:
      return launch_split_fused<Drand48<kSplitT>, Drand48<>>(kDrand48DrawUs, st, n, draws, sum, hist, acc, s);
    case RANNYU:
      return launch_split_fused<Rannyu<kSplitT>, Rannyu<>>(kRannyuDrawUs, st, n, draws, sum, hist, acc, s);
    case MT19937:
      return for_stream_ranges(n, kWaveStreams, [&](uint64_t s0, uint64_t m) {
        hipLaunchKernelGGL(k_mt_fused, dim3((unsigned)((m + 3) / 4)), dim3(256), 0, s, st + s0 * kMtStride, m,
                           (uint32_t)draws, sum + s0, hist + 64 * s0, acc ? 1 : 0);
        return hipGetLastError();
      });
  }
  return hipErrorInvalidValue;
}


}  // namespace prng
