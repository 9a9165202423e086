// RANMAR with one stream per wavefront: plain rows, interleaved rows and the
// in-kernel consumer.
#include "device.h"

namespace prng {
namespace {

// States of a workgroup's 4 R consecutive streams, moved through LDS as 4 R
// adjacent words of each of the 98 state rows.
template <int R>
struct StateTile {
  static constexpr int kPitch = 99;  // odd: the 4 R words of one state row fall in different banks
  uint32_t w[4 * R][kPitch];
  __device__ void load(const uint32_t* __restrict__ st, uint64_t n, uint64_t s0, int tid) {
    for (int i = tid; i < 98 * 4 * R; i += 256)
      if (s0 + i % (4 * R) < n) w[i % (4 * R)][i / (4 * R)] = st[(uint64_t)(i / (4 * R)) * n + s0 + i % (4 * R)];
  }
  __device__ void store(uint32_t* __restrict__ st, uint64_t n, uint64_t s0, int tid) const {
    for (int i = tid; i < 98 * 4 * R; i += 256)
      if (s0 + i % (4 * R) < n) st[(uint64_t)(i / (4 * R)) * n + s0 + i % (4 * R)] = w[i % (4 * R)][i / (4 * R)];
  }
};

// R streams per wavefront, one after the other (R = 1: states read and written
// directly).  Bound by LDS latency at few streams (four dependent steps per
// 256 positions) and by the row stores at many.  f32, one lane per stream
// before: 256 streams x 4096 151 -> 7.0 us, 4096 x 1000 54.9 -> 8.2 us,
// 16384 x 4096 154.6 -> 48.4 us (5.8 TB/s).  R = 2 over R = 1 at 65536 x 300:
// 28.3 and 61.6 us (R = 4: 28.7, but 11.6 instead of 8.2 us at 4096 x 1000).
template <int DT, int R>
__global__ __launch_bounds__(256) void k_ranmar_rows(uint32_t* __restrict__ state, uint64_t n, uint32_t draws,
                                                     uint32_t c_end, void* __restrict__ out, uint64_t row_elems,
                                                     uint64_t elem_off) {
  __shared__ __attribute__((aligned(16))) uint32_t ring_all[4][RanmarWave::kRing];
  __shared__ StateTile<R == 1 ? 0 : R> tile;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  RanmarWave w(ring_all[wave], lane);
  constexpr uint64_t es = DT == F64 ? 8 : 4;
  const uint64_t s0 = (uint64_t)xcd_block<8 / R>() * (4u * R);
  if constexpr (R == 1) {
    const uint64_t s = s0 + wave;
    if (s >= n) return;  // whole wavefront; no block-wide barrier is used
    const uint32_t c0 = w.load(state, n, s);
    ranmar_row<DT>(w, c0, draws, reinterpret_cast<uint64_t>(out) + (s * row_elems + elem_off) * es);
    w.store(state, n, s, draws, RanmarWave::c_back(c0, c_end));
  } else {
    tile.load(state, n, s0, (int)threadIdx.x);
    __syncthreads();
    for (int r = wave * R; r < wave * R + R && s0 + r < n; ++r) {
      const uint32_t c0 = w.load(tile.w[r], 1, 0);
      ranmar_row<DT>(w, c0, draws, reinterpret_cast<uint64_t>(out) + ((s0 + r) * row_elems + elem_off) * es);
      w.store(tile.w[r], 1, 0, draws, RanmarWave::c_back(c0, c_end));
      wave_sync();
    }
    __syncthreads();
    tile.store(state, n, s0, (int)threadIdx.x);
  }
}

// Four wavefronts on the four streams of an interleaved row: each generates
// 256 positions of its stream, then stores a quarter of them for all four, so
// that a lane writes one 16-byte element.
template <int DT>
__global__ __launch_bounds__(256) void k_ranmar_pack4(uint32_t* __restrict__ state, uint64_t n, uint32_t draws,
                                                      uint32_t c_end, void* __restrict__ out, uint64_t row_elems,
                                                      uint64_t elem_off) {
  __shared__ __attribute__((aligned(16))) uint32_t ring_all[4][RanmarWave::kRing];
  __shared__ uint32_t c_all[4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint64_t s = (uint64_t)xcd_block<8>() * 4u + wave;  // n is a multiple of four
  RanmarWave w(ring_all[wave], lane);
  const uint32_t c0 = w.load(state, n, s);
  if (lane == 0) c_all[wave] = c0;
  __syncthreads();
  uint32_t v = 64u * (uint32_t)wave + (uint32_t)lane;
  uint32_t c[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) c[k] = RanmarWave::c_at(c_all[k], v);
  const uint64_t row = reinterpret_cast<uint64_t>(out) + ((s >> 2) * row_elems + elem_off) * 16ull;
  auto emit = [&](int h) {
    uint32_t o[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint32_t u = (ring_all[k][256 * h + 64 * wave + lane] - c[k]) & RanmarWave::MASK;
      o[k] = DT == U32 ? u : __float_as_uint(quad_f32<RanmarOut, DT>(u));
      c[k] = RanmarWave::c_back(c[k], RanmarWave::c_off(256));
    }
    if (v < draws) put<v4u>(row + 16ull * v, v4u{o[0], o[1], o[2], o[3]});
    v += 256u;
  };
  // one barrier per half: a half is overwritten only after the barrier that
  // follows the other half, which every wavefront reaches after storing it
  for (uint32_t pos = 0; pos < draws; pos += 512u) {
    w.half<0>();
    __syncthreads();
    emit(0);
    if (pos + 256u >= draws) break;
    w.half<1>();
    __syncthreads();
    emit(1);
  }
  w.store(state, n, s, draws, RanmarWave::c_back(c0, c_end));
}

// The in-kernel consumer: a step's draws are taken as they are made.  One lane
// per stream before: 256 streams x 2^18 8.0 ms, now 0.24 ms (latency of a
// step); 4096 x 2^18 8.0 ms, now 0.54 ms (VALU and LDS).
__global__ __launch_bounds__(256) void k_ranmar_fused(uint32_t* __restrict__ state, uint64_t n, uint32_t draws,
                                                      uint32_t c_end, uint64_t* __restrict__ sum,
                                                      uint32_t* __restrict__ hist, int accumulate) {
  __shared__ __attribute__((aligned(16))) uint32_t ring_all[4][RanmarWave::kRing];
  __shared__ uint32_t hist_all[4][64 * kHistPitch];
  const int lane = threadIdx.x & 63;
  const uint64_t s = (uint64_t)xcd_block<8>() * 4u + (threadIdx.x >> 6);
  if (s >= n) return;  // whole wavefront; no block-wide barrier is used
  uint32_t* h = hist_all[threadIdx.x >> 6];
  for (int i = lane; i < 64 * kHistPitch; i += 64) h[i] = 0;
  RanmarWave w(ring_all[threadIdx.x >> 6], lane);
  const uint32_t c0 = w.load(state, n, s);
  uint32_t c = RanmarWave::c_at(c0, (uint32_t)lane);
  FusedSink<24, kHistPitch> sink{0u, h + (lane & 31)};
  uint64_t total = 0;
  auto take = [&](uint32_t y) {
    sink(0, (y - c) & RanmarWave::MASK);
    c = RanmarWave::c_back(c, RanmarWave::c_off(64));
  };
  uint32_t pos = 0;
  for (; pos + 512u <= draws; pos += 512u) {
    sink.acc = 0;
    take(w.step<0>());
    take(w.step<1>());
    take(w.step<2>());
    take(w.step<3>());
    take(w.step<4>());
    take(w.step<5>());
    take(w.step<6>());
    take(w.step<7>());
    total += sink.acc;
  }
  sink.acc = 0;
  auto rest = [&](auto piece) {
    constexpr int S = decltype(piece)::value;
    const uint32_t at = pos + 64u * S;
    if (at >= draws) return;
    const uint32_t y = w.step<S>();
    if (at + (uint32_t)lane < draws) sink(0, (y - c) & RanmarWave::MASK);
    c = RanmarWave::c_back(c, RanmarWave::c_off(64));
  };
  rest(std::integral_constant<int, 0>{});
  rest(std::integral_constant<int, 1>{});
  rest(std::integral_constant<int, 2>{});
  rest(std::integral_constant<int, 3>{});
  rest(std::integral_constant<int, 4>{});
  rest(std::integral_constant<int, 5>{});
  rest(std::integral_constant<int, 6>{});
  rest(std::integral_constant<int, 7>{});
  total += sink.acc;
  wave_sync();
  for (int o = 32; o > 0; o >>= 1) total += (uint64_t)__shfl_xor((unsigned long long)total, o);
  uint32_t hb = 0;
#pragma unroll
  for (int l = 0; l < 32; ++l) hb += h[lane * kHistPitch + l];
  if (lane == 0) sum[s] = (accumulate ? sum[s] : 0ull) + total;
  hist[s * 64u + lane] = (accumulate ? hist[s * 64u + lane] : 0u) + hb;
  w.store(state, n, s, draws, RanmarWave::c_back(c0, c_end));
}

}  // namespace

namespace {
template <int R>
hipError_t launch_rows(int dtype, uint32_t* st, uint64_t n, uint64_t draws, void* out, uint64_t row_elems,
                       uint64_t off, hipStream_t s) {
  const dim3 grid((unsigned)((n + 4 * R - 1) / (4 * R))), block(256);
  const uint32_t d = (uint32_t)draws, ce = RanmarWave::c_off(draws);
  switch (dtype) {
    case U32:
      hipLaunchKernelGGL((k_ranmar_rows<U32, R>), grid, block, 0, s, st, n, d, ce, out, row_elems, off);
      break;
    case F32:
      hipLaunchKernelGGL((k_ranmar_rows<F32, R>), grid, block, 0, s, st, n, d, ce, out, row_elems, off);
      break;
    case F64:
      hipLaunchKernelGGL((k_ranmar_rows<F64, R>), grid, block, 0, s, st, n, d, ce, out, row_elems, off);
      break;
    case F32P:
      hipLaunchKernelGGL((k_ranmar_rows<F32P, R>), grid, block, 0, s, st, n, d, ce, out, row_elems, off);
      break;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}
}  // namespace

hipError_t launch_ranmar(int dtype, uint32_t* st, uint64_t n, uint64_t draws, void* out, uint64_t row_elems,
                         uint64_t off, hipStream_t s) {
  // below 4096 streams one stream per wavefront spreads further
  if (n >= 4096) return launch_rows<2>(dtype, st, n, draws, out, row_elems, off, s);
  return launch_rows<1>(dtype, st, n, draws, out, row_elems, off, s);
}

hipError_t launch_ranmar_packed(int dtype, uint32_t* st, uint64_t n, uint64_t draws, void* out, uint64_t row_elems,
                                uint64_t off, hipStream_t s) {
  const dim3 grid((unsigned)(n / 4)), block(256);
  const uint32_t d = (uint32_t)draws, ce = RanmarWave::c_off(draws);
  switch (dtype) {
    case U32:
      hipLaunchKernelGGL((k_ranmar_pack4<U32>), grid, block, 0, s, st, n, d, ce, out, row_elems, off);
      break;
    case F32:
      hipLaunchKernelGGL((k_ranmar_pack4<F32>), grid, block, 0, s, st, n, d, ce, out, row_elems, off);
      break;
    case F32P:
      hipLaunchKernelGGL((k_ranmar_pack4<F32P>), grid, block, 0, s, st, n, d, ce, out, row_elems, off);
      break;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_ranmar_fused(uint32_t* st, uint64_t n, uint64_t draws, uint64_t* sum, uint32_t* hist, bool acc,
                               hipStream_t s) {
  const dim3 grid((unsigned)((n + 3) / 4)), block(256);
  hipLaunchKernelGGL(k_ranmar_fused, grid, block, 0, s, st, n, (uint32_t)draws, RanmarWave::c_off(draws), sum, hist,
                     acc ? 1 : 0);
  return hipGetLastError();
}

}  // namespace prng
