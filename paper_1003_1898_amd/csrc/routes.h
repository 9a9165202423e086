// Which kernel a call takes and how its streams are cut: rules on stream and
// draw counts, on the host.
#pragma once
#include <algorithm>
#include <bit>
#include <cstdint>

namespace prng {

// Output up to about this many bytes stays in the 256 MB last-level cache,
// whatever order its rows are stored in; more of it is bound by that order.
constexpr uint64_t kCachedBytes = 320'000'000;

// A launch holds less than 2^32 threads: beyond this many streams a stream gets
// a lane instead of a wavefront, or the streams several launches.
constexpr uint64_t kWaveStreams = 1ull << 25;

// launch(first, count) over the streams 0 .. n - 1, at most `most` (a multiple
// of four) at a time, up to the first failure; the last launch's result.
template <class F>
auto for_stream_ranges(uint64_t n, uint64_t most, F launch) {
  uint64_t s0 = 0;
  auto e = launch(s0, std::min(n, most));
  for (s0 = most; s0 < n && e == decltype(e){}; s0 += most) e = launch(s0, std::min(n - s0, most));
  return e;
}

// A stream's draws cut into K segments of S (the last one shorter); K = 1: uncut.
struct Cut {
  uint64_t S, K;
};

// ---------------------------------------------------------------- RANLUX rows
constexpr uint32_t kLuxSplitMax = 64;  // segments of a stream at most

// Whether segments from 96 draws on, about one wavefront per SIMD, beat the
// fewest that lux_cut takes anyway.  The copy of the states and a jump take
// about as long as 200 draws of p = 24, 130 of p = 97 and 100 of p = 389 (a
// draw's time is near p + 114 in some unit); against that stand the draws past
// the first 96, and a second segment below 48 draws hides its jump behind the
// first.  Few and many segments, f32, at 4096 streams: p = 24 x 256 19 and 24
// us, x 384 27 and 25 (from a block's start 19 and 22), x 576 26 and 22; p = 97 x
// 224 23 and 21, x 256 23 and 26, x 384 33 and 28; p = 389 x 192 36 and 36, x 224
// 38 and 29.  More streams leave less to gain: p = 24 20011 x 384 28 and 31 us, x
// 768 41 and 37; p = 97 20011 x 256 25 and 29, x 384 34 and 33, 40000 x 512 43 and
// 46, x 3000 189 and 214; p = 24 40000 x 2048 95 and 112; p = 389 40000 x 300 51
// and 48.  f64 calls gain more: where an odd count has left the streams at odd
// positions, a draw takes up to four times as long (p = 24 20011 x 4000 389 and
// 227 us, p = 97 40000 x 3000 592 and 345).
inline bool lux_short_segments(uint64_t waves, uint64_t d, uint32_t p, bool f64) {
  if (d <= 192) return false;
  if (waves > 256 && p < 60 && d >= 3072 && !f64) return false;  // cut already: 24000 x 3072 92 and 108 us
  if (waves > 512 && p < (f64 ? 60u : 150u)) return false;
  const uint64_t gain = (d - 96) * (p + 114ull) * (d <= 240 ? 2 : 1);
  return gain >= (waves <= 256 ? 39000u : waves <= 512 ? 57000u : 100000u);
}

// The borrow chain runs one step at a time per lane, and the kernel needs two
// wavefronts per SIMD to overlap it with the stores: about 2048 wavefronts where
// a segment keeps 1536 draws.  Shorter segments, where they pay, are for calls
// that own their snapshot area (not `shared`).  S is a multiple of 96.
inline Cut lux_cut(uint64_t n, uint64_t d, uint32_t p, bool f64, bool shared) {
  const uint64_t waves = (n + 63) / 64;
  uint64_t K = std::min<uint64_t>({kLuxSplitMax, (2048 + waves - 1) / waves, std::max<uint64_t>(1, d / 1536)});
  if (!shared && lux_short_segments(waves, d, p, f64))
    K = std::max(K, std::min<uint64_t>({kLuxSplitMax, (1024 + waves - 1) / waves, std::max<uint64_t>(1, d / 96)}));
  if (K == 1) return {d, 1};
  const uint64_t S = ((d + K - 1) / K + 95) / 96 * 96;
  return {S, (d + S - 1) / S};  // (K - 1) S < d: no segment is empty
}

// ---------------------------------------------------------------- XOR128 rows
// From this many streams on, one lane per stream keeps the SIMDs busy by itself.
constexpr uint64_t kXorLanes = 32768;

// Few long segments, staged in 128-draw chunks (one workgroup per CU), for many
// streams and for output beyond the cache; otherwise many short segments in
// 64-draw chunks (two workgroups per CU).  f32, long and short: 20032 x 4096
// (328 MB) 80 and 100 us, 12032 x 8192 (394 MB) 85 and 123 us, 24000 x 16384
// 305 and 331 us; 20032 x 3072 (246 MB) 92 and 48 us, 12032 x 6000 (289 MB) 108
// and 73 us.  Below 8192 streams long segments leave SIMDs idle (4096 x 32768
// 149 and 154 us, 1024 x 32768 134 and 44 us).
inline bool xor128_long_segments(uint64_t n, uint64_t d) {
  return n >= kXorLanes || (n >= 8192 && 4 * n * d > kCachedBytes);
}

// d draws of n streams.  Segments start from jumped states.
// Long segments: at least 2048 draws, or two where fewer streams leave SIMDs idle
// (20032 x 3072 68 us in two, 92 uncut; 28000 x 3072 100 and 94), about 4096
// wavefronts in all.
// Short ones: about 2048 wavefronts in segments of a power of two from 128 draws
// on: a jump costs a matrix product (2 us) per set bit of its distance, and the
// power of two leaves only those of the segment's number.  f64 4096 x 2000 127
// us uncut, 34 us in 32 segments.  The copy of the states and a jump cost about
// as much as 200 draws, less where the uncut call would end inside a 128-draw
// chunk.  Uncut and in segments of 128, f32: 4096 x 192 11.5 and 11.0 us, x 224
// 12.0 and 16.1, x 256 10.1 and 13.0, x 300 15.1 and 14.4, x 384 14.1 and 13.2, x
// 512 18.1 and 16.4; 20011 x 256 12.1 and 15.0, x 320 17.1 and 15.2, x 512 19.8 and
// 20.6, x 640 23.4 and 21.2.
// `shared`: the snapshot area is every call's of the GPU, and short calls leave it alone.
inline Cut xor128_cut(uint64_t n, uint64_t d, bool shared) {
  const uint64_t waves = (n + 63) / 64;
  uint64_t S = d;
  if (xor128_long_segments(n, d)) {
    const uint64_t least = n < 26000 && d >= 3072 && !shared ? 2 : 1;
    const uint64_t K = std::min<uint64_t>({8, (4096 + waves - 1) / waves, std::max<uint64_t>(least, d / 2048)});
    S = ((d + K - 1) / K + 127) / 128 * 128;
  } else if (shared ? d >= 4096 : d > (n < 16384 ? 256u : 512u) || (d > 300 && d % 128 != 0) || d == 192) {
    const uint64_t want = 2048 / waves;
    S = std::max<uint64_t>(128, std::bit_ceil((d + want - 1) / want));
  }
  return {S, (d + S - 1) / S};  // (K - 1) S < d: no segment is empty
}

// --------------------------------------------------------------- MT19937 rows
// 4-byte rows by one wavefront per stream, cached, or by a workgroup, past the
// cache.  The workgroup's take more instructions but write fewer rows at a time,
// which pays once states and rows no longer fit the 256 MB last-level cache
// together.  f32, wavefront and workgroup: 65536 x 400 (270 MB) 71 and 83 us,
// x 500 (296 MB) 108 and 88, x 4096 359 and 249; 40000 x 1000 (260 MB) 58 and 68,
// x 1500 (340 MB) 112 and 86; 20011 x 3072 (296 MB) 59 and 67, x 4096 98 and 86;
// 15040 x 12576 176 and 159.  Rows that start at uneven places cost the workgroup
// some of that (27360 x 2125, 301 MB, 62 and 88 us; 28083 x 8075 261 and 279).
// States beyond the cache by themselves leave nothing to lose (131072 x 800 247
// and 280, x 2000 406 and 382; 96000 x 64 112 and 96).
constexpr uint64_t kMtStateBytes = 2512;
inline bool mt_row_per_wave(uint64_t n, uint64_t draws) {
  const bool even = draws % 4 == 0;
  if (n <= 14000) return true;
  if (n >= 110000) return draws <= 1500;
  if (draws >= (even ? 8192u : 6500u)) return !even && n < 32768;
  if (n <= 18000) return true;
  const uint64_t bytes = n * (kMtStateBytes + 4 * draws);
  if (n <= 22528) return bytes <= 300'000'000u;
  if (n > 80000) return bytes <= 264'500'000u;
  return bytes <= (even || n > 40000 ? 280'000'000u : 305'000'000u);
}

// --------------------------------------------------------------------- RANMAR
// One lane per stream keeps at least three quarters of the 1024 SIMDs busy (one
// wavefront each; its window takes most of the registers).
inline bool lanes_fill(uint64_t n) {
  const uint64_t waves = (n + 63) / 64, rounds = (waves + 1023) / 1024;
  return 4 * waves >= 3 * 1024 * rounds;
}

// Rows by one lane per stream or by one wavefront.  A lane's time does not fall
// with the stream count; it stores its rows in longer runs, which shows in long
// launches, and a call of one whole 128-draw chunk has no ragged rows.  f32, lane
// and wavefront: 65536 x 4096 176 and 255 us, 44000 x 4096 157 and 172, 40000 x
// 4096 154 and 157, 40000 x 128 12 and 16, 28000 x 128 12 and 12; 40000 x 1000 55
// and 32, 16384 x 4096 155 and 48, 4096 x 1000 50 and 8.
inline bool ranmar_row_per_lane(uint64_t n, uint64_t draws) {
  return lanes_fill(n) || (n >= 28672 && draws == 128) || (n >= 43008 && n < 49152 && draws >= 4096);
}

// Interleaved rows by one lane per stream or by four wavefronts on a row's four
// streams, from the times of both in us.  A lane's chunks of 128 draws go out
// whole only where every wavefront is full; ragged ends cost it 14 us.  Lane and
// wavefronts: 40000 x 1 19 and 27 us, x 128 12 and 30, x 256 18 and 31, x 512 27
// and 34, x 1000 61 and 40; 24000 x 256 16 and 21, x 512 25 and 23; 16384 x 100 27
// and 15; 81920 x 384 44 and 67; 48000 x 2048 83 and 95.
inline bool ranmar_packed_per_lane(uint64_t n, uint64_t draws) {
  if (lanes_fill(n)) return true;
  if (n >= 45056 && n < 49152 && n % 64 == 0 && draws % 128 == 0 && draws >= 2048) return true;
  const double rounds = (double)((n + 65535) / 65536), d = (double)draws, chunks = (double)((draws + 127) / 128);
  const double whole = 7.0 + 4.9 * chunks + (draws % 128 ? 14.0 : 0.0) + (n % 64 ? 0.014 * d : 0.0);
  const double lane = rounds * (draws < 128 ? 18.0 + 0.07 * d : whole);
  return lane < 4.0 + (double)n * (62e-5 + 3e-7 * d);
}

// Consumer by one lane per stream or by one wavefront, which pays for its window
// and histogram with every stream.  Lane and wavefront: 20011 x 16 23 and 28 us,
// x 256 24 and 30, x 512 33 and 31; 32768 x 512 34 and 45, x 1000 56 and 52; 16384 x
// 16 22 and 21; 40000 x 16 33 to 50 and 45 (a lane's times depend on where the
// histograms lie in memory), 81920 x 16 99 and 88.
inline bool ranmar_consumer_per_lane(uint64_t n, uint64_t draws) {
  return n >= 17000 && n <= 36000 && draws <= (n >= 24000 ? 512u : 256u);
}

// ------------------------------------------ interleaved rows of the leap kinds
// GGL, RANECU, DRAND48 and RANNYU leap along a row of four streams, after up to
// ten products per stream that bring a lane to its place: RANECU, whose states
// are two, keeps one lane per stream where few whole 128-draw chunks of full
// wavefronts are cheaper (times in us), the others for one chunk.  Lane and leap:
// RANECU 65536 x 128 12 and 22, x 256 20 and 27, x 512 33 and 38, x 1024 70 and 60,
// 40000 x 256 18 and 19, x 384 24 and 23; GGL 65536 x 128 10 and 12, x 256 15 and
// 14, 32768 x 128 8 and 8, 44000 x 128 (a wavefront not full) 10 and 9.
// A few draws pay for those products as much: RANECU 65536 x 24 14 and 16, x 48 17
// and 19, 131072 x 24 26 and 29, 54848 x 35 14 and 16; 65536 x 8 12 and 13, x 64 21
// and 20, 44032 x 32 14 and 12, 98304 x 32 26 and 23.
inline bool leap_packed_per_lane(bool ranecu, uint64_t n, uint64_t draws) {
  if (ranecu && draws >= 12 && draws <= 60) {
    const uint64_t r = (n + 65535) / 65536;
    return r * 65536 - n <= 16384 &&
           (double)r * (10.1 + 0.075 * (double)draws) < 3.9 + (double)n * (11.2e-5 + 2.66e-6 * (double)draws);
  }
  if (draws % 128) return false;
  if (!ranecu) return draws == 128 && (n % 64 ? n >= 56000 && n <= 65536 : n >= 38000);
  if (n % 64) return false;
  const double rounds = (double)((n + 65535) / 65536), d = (double)draws;
  return draws <= 768 && rounds * (4.7 + 0.051 * d) < 1.5 + (double)n * (30e-5 + 6.5e-7 * d);
}

// ----------------------------------------------------------------- the consumer
// A draw of one lane per stream, its dependent steps hidden by at most two
// wavefronts per SIMD, in us (over ten thousand draws).
constexpr double kGglDrawUs = 0.0235, kXor128DrawUs = 0.0245, kRanecuDrawUs = 0.0435, kDrand48DrawUs = 0.0222,
                 kRannyuDrawUs = 0.0195;

// Wavefronts per stream of the cut consumer (1, 4 or 16), or 0 for one lane per
// stream: the least of the times in us, fitted to 795 calls of 64 to 262144
// streams (the choice loses 0.6% to the best one on average).  A wavefront pays
// for its histogram and, per draw, issue where the chip is full (2048 wavefronts)
// or latency where it is not; a jump of XOR128 costs 2.2 us per bit of the segment's
// number.  A lane pays for storing 64 bins by itself.  Lane and W = 1: GGL 20011 x
// 256 18 and 20 us, x 1000 40 and 26; 28000 x 512 25 and 29; 65536 x 16 72 and 58 (from
// about 36000 streams on a lane's times depend on where the histograms lie: 50000 x
// 1184 46 to 76 and 56);
// XOR128 64 x 512 17 and 22, 4096 x 1000 39 and 33, 20011 x 4096 114 and 146.
inline int consumer_width(double draw, bool matrix, uint64_t n, uint64_t draws) {
  const double N = (double)n, d = (double)draws;
  double best = (n <= 51200 ? 0.72e-3 : 0.95e-3) * N + draw * d;
  if (n <= 36000) best = std::max(13.0 + N / 7000.0, 8.0 + N / 5000.0 + draw * d);
  if (n <= 64) best = (matrix ? 4.0 : 7.0) + draw * d;
  int width = 0;
  const struct { int W, bits; double group; } kinds[] = {{1, 6, 1.4}, {4, 8, 2.0}, {16, 10, 14.0}};
  for (const auto& k : kinds) {
    if (n > kWaveStreams / k.W) break;
    uint64_t S = (draws + 64ull * k.W - 1) / (64ull * k.W);
    double latency = 0.3 * k.bits * draw, issue = 12.0 * draw;  // of the jump
    double step = 0.67 * draw;                                  // a draw's latency
    if (matrix) {
      S = std::bit_ceil(S);
      const uint64_t last = draws ? (draws - 1) / S : 0;  // the last segment's number
      latency = issue = 2.2 * (double)std::min<int>(k.bits, std::bit_width(last));
      step = 1.3 * draw;
    }
    const double rounds = (double)((n * k.W + 1023) / 1024) / (2.0 * k.W);  // of the fullest SIMD, two wavefronts each
    const double t = 4.0 + std::max(2.0 + latency + step * (double)S,
                                    rounds * (k.group + k.W * (issue + 1.25 * draw * (double)S)));
    if (t < best) {
      best = t;
      width = k.W;
    }
  }
  return width;
}

}  // namespace prng
