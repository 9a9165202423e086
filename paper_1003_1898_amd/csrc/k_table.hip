// Stream table: persistent lane and MT19937 kernels, MT19937 jump windows, snapshots, counters.
#include "device.h"

namespace prng {
namespace {

__global__ __launch_bounds__(256) void k_table_lane(const TableTask* __restrict__ tasks, uint32_t ntasks,
                                                    const TableRow* __restrict__ rows,
                                                    const uint32_t* __restrict__ tails, uint32_t* counter,
                                                    const uint32_t* __restrict__ aux) {
  // RANLUX's three-byte stage of 96-draw chunks takes a little more than the
  // 64-draw word stage
  constexpr int SW = std::max(stage_words<kTableT>(), (StageSplit24<kLuxTableT>::kBytes + 3) / 4);
  __shared__ __attribute__((aligned(16))) uint32_t stage_all[4][SW];
  const int lane = threadIdx.x & 63;
  uint32_t* stage = stage_all[threadIdx.x >> 6];
  for (uint32_t t = next_task(counter, lane); t < ntasks; t = next_task(counter, lane)) {
    const TableTask task = tasks[t];
    const uint32_t kind = uni(task.kind), dt = uni(task.dtype), p = uni(task.p);
#define PRNG_TASK(K, G, SPLIT)                                                              \
  case K * 4 + U32: lane_task<G, U32, SPLIT>(stage, lane, rows, tails, task, p, aux); break; \
  case K * 4 + F32: lane_task<G, F32, SPLIT>(stage, lane, rows, tails, task, p, aux); break; \
  case K * 4 + F64: lane_task<G, F64, SPLIT>(stage, lane, rows, tails, task, p, aux); break;
    switch (kind * 4 + dt) {
      PRNG_TASK(GGL, Ggl<kTableT>, false)
      PRNG_TASK(XOR128, Xor128<kTableT>, false)
      PRNG_TASK(RANECU, Ranecu<kTableT>, false)
      PRNG_TASK(DRAND48, Drand48<kTableT>, false)
      PRNG_TASK(RANNYU, Rannyu<kTableT>, false)
      PRNG_TASK(RANLUX, Ranlux<kLuxTableT>, true)
      default:
        break;
    }
#undef PRNG_TASK
    wave_sync();
  }
}

// RANMAR tasks, a segment per wavefront: wavefront v takes segment v mod 64 of
// task v / 64 and generates it as the plain kernel does.  The jump costs about as
// much as 500 draws (97 reads and products for 97 window values); one lane per
// segment, as the other kinds run, it costs 20k operations per lane and the window
// and its chunk take a SIMD's registers for a single wavefront.  The grid holds a
// wavefront per segment (up to 2^25 of them), which the dispatcher spreads: a task
// counter on which every wavefront drew its next segment took 15 ns a segment on
// the whole chip (40000 rows of 64 draws 587 us).
__global__ __launch_bounds__(256) void k_table_ranmar(const TableTask* __restrict__ tasks, uint32_t ntasks,
                                                      const TableRow* __restrict__ rows,
                                                      const uint32_t* __restrict__ tails) {
  __shared__ __attribute__((aligned(16))) uint32_t ring_all[4][RanmarWave::kRing];
  const int lane = threadIdx.x & 63;
  RanmarWave w(ring_all[threadIdx.x >> 6], lane);
  // a task's sixteen workgroups, whose streams share the state's lines, on one XCD
  for (uint64_t v = (uint64_t)xcd_block<16>() * 4u + uni(threadIdx.x >> 6); v < 64ull * ntasks; v += 4ull * gridDim.x) {
    const TableTask& task = tasks[v / 64u];
    const uint32_t i = (uint32_t)(v % 64u);
    if (i >= uni(task.nseg)) continue;
    const uint64_t g = task.g0 + i;
    uint32_t r, j;
    if (task.tail) {
      r = uni(tails[g]);
      j = rows[r].nseg - 1u;
    } else {
      r = uni(segment_row(rows, task, g));
      j = (uint32_t)(g - rows[r].first);
    }
    const TableRow& rw = *uni_ptr(rows + r);
    const uint32_t S = rw.seg_len, beg = j * S, last = j + 1u == rw.nseg ? 1u : 0u;
    const uint32_t draws = (last ? rw.draws : beg + S) - beg;  // S is even: fp64 pairs stay whole
    const uint32_t c0 = j == 0 ? w.load(rw.state, rw.sn, rw.si)
                               : w.load_jumped(rw.state, rw.sn, rw.si, uni_ptr(rw.jump + (j - 1u) * rw.jstride));
    const uint64_t row = reinterpret_cast<uint64_t>(rw.out) + 4ull * beg;
    const uint32_t dt = uni(task.dtype);
    if (dt == U32)
      ranmar_row<U32>(w, c0, draws, row);
    else if (dt == F32)
      ranmar_row<F32>(w, c0, draws, row);
    else
      ranmar_row<F64>(w, c0, draws, row);
    if (last)
      w.store(rw.wstate, rw.wsn, rw.wsi, draws,
              RanmarWave::c_back(c0, (uint32_t)((uint64_t)draws * RanmarWave::D % RanmarWave::M)));
    wave_sync();
  }
}

// One task = one MT19937 row or segment of a row.  A row starts at position
// k0 (the stream's block position, 0..624; position 624 m + w is word w of
// the m-th block after the current one).  Segment j > 0 of a row cut at
// seg_len S (a multiple of 624) starts at position j S, from the window of
// the block before it that k_table_mt_jump built; with fp64 output a boundary
// that would split a pair of draws moves one draw later.  One task per
// workgroup, its four wavefronts sharing the stream (a segment's chain runs
// about four times as wide as on one wavefront).
__global__ __launch_bounds__(256) void k_table_mt(const TableTask* __restrict__ tasks, uint32_t ntasks,
                                                  const TableRow* __restrict__ rows, uint32_t* counter) {
  __shared__ __attribute__((aligned(16))) uint32_t mt[624];
  __shared__ __attribute__((aligned(16))) uint32_t stage[628];
  __shared__ uint32_t task_slot;
  const int tid = (int)threadIdx.x;
  // the next task index, uniform over the workgroup
  auto fetch = [&]() -> uint32_t {
    __syncthreads();  // every thread has read the previous index
    if (tid == 0) task_slot = atomicAdd(counter, 1u);
    __syncthreads();
    return task_slot;
  };
  for (uint32_t t = fetch(); t < ntasks; t = fetch()) {
    const TableRow& rw = rows[tasks[t].row0];
    const uint32_t dt = uni(tasks[t].dtype);
    const uint32_t draws = uni(rw.draws), S = uni(rw.seg_len);
    const uint32_t j = uni((uint32_t)tasks[t].g0), last = j + 1u == uni(rw.nseg) ? 1u : 0u;
    const uint32_t* snap = rw.state + rw.si * kMtStride;
    const uint32_t k0 = uni(snap[624]);
    uint32_t beg = k0, end = k0 + draws;
    if (S) {
      const uint32_t par = dt == F64 ? 1u : 0u;
      if (j) beg = j * S + (par & ((j * S - k0) & 1u));
      if (!last) end = (j + 1u) * S + (par & (((j + 1u) * S - k0) & 1u));
    }
    const uint32_t* src = j ? rw.jstate + (j - 1u) * kMtStride : snap;
    const uint32_t pos0 = j ? 624u : k0, skip = j ? beg - j * S : 0u;
    uint32_t* dst = last ? rw.wstate + rw.wsi * kMtStride : nullptr;
    const uint32_t per = dt == F64 ? 2u : 1u;
    const uint64_t outp = reinterpret_cast<uint64_t>(rw.out) + (uint64_t)((beg - k0) / per) * (4ull * per);
    if (dt == U32)
      mt_body<U32>(mt, stage, tid, src, pos0, skip, end - beg, outp, dst);
    else if (dt == F32)
      mt_body<F32>(mt, stage, tid, src, pos0, skip, end - beg, outp, dst);
    else
      mt_body<F64>(mt, stage, tid, src, pos0, skip, end - beg, outp, dst);
  }
}

// Jump-ahead of MT19937 segment starts, one block per segment.  From the
// row's starting window x_0 .. x_623 (the current block), the block extends
// the raw sequence x_n = x_{n-227} ^ twist(x_{n-624}, x_{n-623}) in LDS (227
// words at a time, each chunk reading only earlier chunks), then forms the
// window J words ahead as word k = XOR of x_{i+k} over the set coefficients
// i of x^J mod the characteristic polynomial (the segment's jump data lists
// their exponents).  The low 31 bits of word 0 are not part of the state and
// come out arbitrary; the next twist reads only its top bit.
//
// The LDS bounds it: word by word, about 10^4 coefficients read 624 words each
// (142 us a block).  Coefficients are therefore taken six at a time: the groups
// i = 6 b of one pattern w of set bits are summed first, S_w[m] = XOR of
// x_{6b+m}, into B_t = XOR of S_w over the patterns with bit t, and word k is
// the XOR of B_t[k + t], t = 0 .. 5: some 3800 reads (a group each, padded per
// pattern) of 630 words.
constexpr int kMtSeqWords = 624 + 19936;
constexpr int kJumpThreads = 1024;  // four teams of 256 split each pattern's groups
constexpr int kJumpQ = 6, kJumpPatterns = 1 << kJumpQ;
constexpr int kJumpGroups = (19937 + kJumpQ - 1) / kJumpQ;
constexpr int kJumpSpan = 624 + kJumpQ - 1;      // words a group is read for
// zeros, for the padding groups (the last group reads a word past the sequence)
constexpr int kJumpZero = kMtSeqWords + 8;
constexpr int kJumpPitch = kJumpSpan + 3;
constexpr int kJumpRound = 16;                   // groups per round: four of each team
constexpr int kJumpList = (kJumpGroups + (kJumpPatterns - 1) * (kJumpRound - 1) + 7) / 8 * 8;
static_assert(kJumpZero + kJumpPitch < 65536, "list entries are 16 bits");
static_assert(4 * kJumpQ * kJumpPitch <= kJumpZero, "the teams' sums reuse the sequence");

__global__ __launch_bounds__(kJumpThreads) void k_table_mt_jump(const uint32_t* __restrict__ list, uint32_t n,
                                                                const TableRow* __restrict__ rows) {
  __shared__ uint32_t seq[kJumpZero + kJumpPitch];
  __shared__ uint32_t coef[624 + 1];  // bit i of the polynomial
  __shared__ __attribute__((aligned(16))) uint16_t groups[kJumpList];
  __shared__ uint32_t first[kJumpPatterns + 1], cursor[kJumpPatterns];
  const int tid = threadIdx.x;
  const int team = (int)uni((uint32_t)(tid >> 8)), t = tid & 255;  // a team is whole wavefronts
  // thread t of a team owns words t, t + 256 and t + 512 < 629, so that the 64
  // lanes of every LDS read take 64 consecutive words
  const bool hi = t + 512 < kJumpSpan;
  auto pattern = [&](int b) {
    const int e = kJumpQ * b;
    const uint64_t w = (uint64_t)coef[e >> 5] | ((uint64_t)coef[(e >> 5) + 1] << 32);
    return (uint32_t)(w >> (e & 31)) & (uint32_t)(kJumpPatterns - 1);
  };
  for (uint32_t r = blockIdx.x; r < n; r += gridDim.x) {
    const TableRow& rw = rows[list[2 * r]];
    const uint32_t j = list[2 * r + 1];  // >= 1
    const uint32_t* src = rw.state + rw.si * kMtStride;
    uint32_t* dst = rw.jstate + (j - 1u) * kMtStride;
    const uint32_t* jd = rw.jump + (j - 1u) * rw.jstride;
    const uint32_t nbits = min(uni(jd[0]), 19937u);
    for (int i = tid; i < 624; i += kJumpThreads) seq[i] = src[i];
    for (int i = tid; i < 625; i += kJumpThreads) coef[i] = 0u;
    for (int i = kMtSeqWords + tid; i < kJumpZero + kJumpPitch; i += kJumpThreads) seq[i] = 0u;
    for (int i = tid; i < kJumpList; i += kJumpThreads) groups[i] = (uint16_t)kJumpZero;
    if (tid < kJumpPatterns) cursor[tid] = 0u;
    __syncthreads();
    for (uint32_t q = tid; q < nbits; q += kJumpThreads) {
      const uint32_t e = min((jd[1 + (q >> 1)] >> (16u * (q & 1u))) & 0xFFFFu, 19936u);
      atomicOr(&coef[e >> 5], 1u << (e & 31));
    }
    for (int n0 = 624; n0 < kMtSeqWords; n0 += 227) {
      const int x = n0 + tid;
      if (tid < 227 && x < kMtSeqWords) {
        const uint32_t y = (seq[x - 624] & kMtUpper) | (seq[x - 623] & kMtLower);
        seq[x] = seq[x - 227] ^ (y >> 1) ^ ((y & 1u) ? kMtA : 0u);
      }
      __syncthreads();
    }
    // the groups sorted by pattern, every pattern's padded to whole rounds
    for (int b = tid; b < kJumpGroups; b += kJumpThreads) atomicAdd(&cursor[pattern(b)], 1u);
    __syncthreads();
    if (tid < kJumpPatterns) {  // wavefront 0
      const uint32_t c = tid == 0 ? 0u : (cursor[tid] + kJumpRound - 1u) / kJumpRound * kJumpRound;
      uint32_t at = c;
      for (int o = 1; o < 64; o <<= 1) {
        const uint32_t v = (uint32_t)__shfl_up((int)at, o);
        if (tid >= o) at += v;
      }
      first[tid + 1] = at;
      cursor[tid] = at - c;
      if (tid == 0) first[0] = 0u;
    }
    __syncthreads();
    for (int b = tid; b < kJumpGroups; b += kJumpThreads) {
      const uint32_t w = pattern(b);
      if (w) groups[atomicAdd(&cursor[w], 1u)] = (uint16_t)(kJumpQ * b);
    }
    __syncthreads();
    uint32_t B[kJumpQ][3] = {};
    for (uint32_t w = 1; w < (uint32_t)kJumpPatterns; ++w) {
      const uint32_t end = uni(first[w + 1]);
      uint32_t a0 = 0, a1 = 0, a2 = 0;
      for (uint32_t i = uni(first[w]) + 4u * (uint32_t)team; i < end; i += kJumpRound) {
        const v2u g = *reinterpret_cast<const v2u*>(groups + i);
        const uint32_t g0 = uni(g.x), g1 = uni(g.y);
        const uint32_t* p[4] = {seq + (g0 & 0xFFFFu) + t, seq + (g0 >> 16) + t, seq + (g1 & 0xFFFFu) + t,
                                seq + (g1 >> 16) + t};
        a0 ^= p[0][0] ^ p[1][0] ^ p[2][0] ^ p[3][0];
        a1 ^= p[0][256] ^ p[1][256] ^ p[2][256] ^ p[3][256];
        if (hi) a2 ^= p[0][512] ^ p[1][512] ^ p[2][512] ^ p[3][512];
      }
#pragma unroll
      for (int q = 0; q < kJumpQ; ++q) {
        const uint32_t m = 0u - ((w >> q) & 1u);
        B[q][0] ^= a0 & m;
        B[q][1] ^= a1 & m;
        B[q][2] ^= a2 & m;
      }
    }
    __syncthreads();  // the sequence is read
#pragma unroll
    for (int q = 0; q < kJumpQ; ++q) {
      uint32_t* s = seq + (team * kJumpQ + q) * kJumpPitch + t;
      s[0] = B[q][0];
      s[256] = B[q][1];
      if (hi) s[512] = B[q][2];
    }
    __syncthreads();
    if (tid < 624) {
      uint32_t v = 0;
#pragma unroll
      for (int q = 0; q < 4 * kJumpQ; ++q) v ^= seq[q * kJumpPitch + tid + q % kJumpQ];
      dst[tid] = v;
      if (tid == 0) dst[624] = 624u;
    }
    __syncthreads();  // everything is rebuilt for the next segment
  }
}

// Copies the starting states of split streams (one thread per word).
// Start of a run: clears the task counters (block 0) and copies the starting
// states of the cut streams (a kernel rather than a memset and a copy, so
// that both are one ordinary node when the run is captured into a graph).
__global__ void k_table_prepare(uint32_t* counters, int n_counters, const SnapRow* __restrict__ rows, uint32_t n,
                                uint32_t max_words) {
  if (blockIdx.x == 0 && (int)threadIdx.x < n_counters) counters[threadIdx.x] = 0u;
  const uint64_t total = (uint64_t)n * max_words;
  for (uint64_t t = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; t < total; t += (uint64_t)gridDim.x * blockDim.x) {
    const uint32_t r = (uint32_t)(t / max_words), w = (uint32_t)(t % max_words);
    const SnapRow& sr = rows[r];
    if (w >= sr.words) continue;
    if (sr.aos)
      sr.dst[sr.di * kMtStride + w] = sr.src[sr.si * kMtStride + w];
    else
      sr.dst[w * sr.dn + sr.di] = sr.src[w * sr.sn + sr.si];
  }
}


}  // namespace

hipError_t launch_table_lane(int cls, const TableTask* tasks, uint32_t ntasks, const TableRow* rows,
                             const uint32_t* tails, uint32_t* counter, const uint32_t* aux, int grid, hipStream_t s) {
  if (cls == 0)
    hipLaunchKernelGGL(k_table_lane, dim3(grid), dim3(256), 0, s, tasks, ntasks, rows, tails, counter, aux);
  else  // sixteen workgroups per task of 64 segments
    hipLaunchKernelGGL(k_table_ranmar, dim3(std::min<uint32_t>(ntasks, 1u << 19) * 16u), dim3(256), 0, s, tasks, ntasks,
                       rows, tails);
  return hipGetLastError();
}

hipError_t launch_table_prepare(uint32_t* counters, int n_counters, const SnapRow* rows, uint32_t n,
                                uint32_t max_words, hipStream_t s) {
  if (n_counters > 256) return hipErrorInvalidValue;
  const uint64_t threads = (uint64_t)n * max_words;
  const unsigned grid = (unsigned)std::max<uint64_t>(1, std::min<uint64_t>((threads + 255) / 256, 4096));
  hipLaunchKernelGGL(k_table_prepare, dim3(grid), dim3(256), 0, s, counters, n_counters, rows, n, max_words);
  return hipGetLastError();
}

hipError_t launch_table_mt_jump(const uint32_t* list, uint32_t n, const TableRow* rows, hipStream_t s) {
  if (n == 0) return hipSuccess;
  const unsigned grid = std::min<uint32_t>(n, 1024u);
  hipLaunchKernelGGL(k_table_mt_jump, dim3(grid), dim3(kJumpThreads), 0, s, list, n, rows);
  return hipGetLastError();
}

hipError_t launch_table_mt(const TableTask* tasks, uint32_t ntasks, const TableRow* rows, uint32_t* counter, int grid,
                           hipStream_t s) {
  hipLaunchKernelGGL(k_table_mt, dim3(grid), dim3(256), 0, s, tasks, ntasks, rows, counter);
  return hipGetLastError();
}


}  // namespace prng
