// Serving loop (include/prng.h, prng_server_*): generator states stay resident
// on the device; requests (stream, count, dtype) are admitted in arrival order
// as output memory in a fixed device pool frees up, packed into batches and
// generated by stream-table launches.  A batch holds requests of one class of
// generator kinds (the stream table's kernel classes: GGL, XOR128, RANECU,
// DRAND48, RANNYU, RANLUX; RANMAR; MT19937), and each batch slot has a HIP
// stream of its own: batches run side by side on the chip, those of one class
// too (a batch's persistent kernel fills the CUs that the one before it frees
// as its last tasks drain), so requests that arrive while others run are
// batched and overlap with them on the device (continuous batching).  No
// generator stream is in two batches at once, so batches need no order
// between them on the device.  A request's elements are the next `count` of its
// stream in per-stream arrival order, exactly as a plain generation would give
// them.
#include <hip/hip_runtime.h>
#include <sys/prctl.h>

#include <algorithm>
#include <atomic>
#include <chrono>
#include <condition_variable>
#include <cstring>
#include <list>
#include <map>
#include <memory>
#include <mutex>
#include <new>
#include <set>
#include <thread>
#include <tuple>
#include <vector>

#include "host.h"
#include "jump.h"
#include "server_book.h"

using namespace prng;

namespace {

constexpr uint64_t kServerMaxSegments = 32768;  // per request (bounds the resident jump tables)
constexpr uint64_t kServerSegAuto = 384;
constexpr int kServerClasses = kLaneClasses + 1;  // the lane classes, then MT19937

int server_class(int kind) { return kind == MT19937 ? kLaneClasses : lane_class(kind); }

struct Batch {
  int slot;
  int cls;
  prng_table* t = nullptr;
  std::unique_ptr<Plan> plan;  // host data of the upload, kept until the batch is done
  std::vector<uint64_t> tickets;
  size_t ws_off = 0, ws_bytes = 0;
};

// Jump data for the server's fixed segment length, resident in the pool.
class ServerJumps : public JumpSource {
 public:
  uint64_t L = 0;  // base segment length, a multiple of 384 (0: requests are never cut)
  std::map<std::pair<int, uint32_t>, const uint32_t*> base;  // (kind, p) -> device address of j = 1
  std::map<std::pair<int, uint32_t>, uint32_t> count;
  const uint32_t* aux_ = nullptr;
  // Per kind: the lane kinds of one batch share a persistent kernel, whose
  // time is its longest task's, so their lengths keep task times about even
  // (a RANLUX p = 223 draw costs about four of the others') while a jump stays
  // small next to the draws it saves.  GGL, RANECU, DRAND48 and RANNYU 2 L;
  // XOR128 4 L (its resident jump data is a 128 x 128 GF(2) matrix, 2 KB, per
  // segment of the longest request); RANLUX (576-bit products) L / 2, at
  // least 384 and a multiple of 384; RANMAR (97^2 multiply-adds, a class of
  // its own) 4 L; MT19937 (a window built from ~10^4 others over a whole CU)
  // 512 L, a multiple of 624.
  uint64_t seg_len(int kind) const override {
    if (!L) return 0;
    switch (kind) {
      case RANLUX:
        return std::max<uint64_t>((L / 2 + 383) / 384 * 384, 384);
      case XOR128:
        return 4 * L;
      case RANMAR:
        return 4 * L;
      case MT19937:
        return (std::max<uint64_t>(512 * L, 1248) + 623) / 624 * 624;
      default:
        return 2 * L;
    }
  }
  // (seg_len 0: requests are never cut)
  const uint32_t* lookup(int kind, uint32_t p, uint32_t j) const override {
    auto it = base.find({kind, kind == RANLUX ? p : 0u});
    if (it == base.end() || j == 0 || j > count.at({kind, kind == RANLUX ? p : 0u})) return nullptr;
    return it->second + (size_t)(j - 1) * jump_slot_words(kind);
  }
  const uint32_t* aux() const override { return aux_; }
};

}  // namespace

struct prng_server {
  std::vector<prng_gen*> gens;
  char* pool = nullptr;
  size_t pool_bytes = 0, fixed_bytes = 0;
  RequestBook book;  // requests, their states and the output arena
  ServerJumps jumps;
  int max_inflight = 4, max_batch = 1024;
  uint64_t max_draws = 0;
  int device = 0;
  std::vector<hipStream_t> streams;        // per slot
  std::vector<hipEvent_t> events, starts;  // per slot: batch end (and start, timed)
  std::vector<int> slot_busy;
  int class_busy[kServerClasses] = {};       // batches in flight per class
  std::mutex mu;
  std::condition_variable cv_work, cv_done;
  std::list<uint64_t> waiting;  // not yet admitted, arrival order
  std::vector<Batch> inflight;
  std::thread worker;
  bool stop = false;
  std::chrono::steady_clock::time_point epoch;
  uint64_t n_batches = 0;
  int64_t plan_ns = 0;    // host time spent planning and enqueuing batches
  double gpu_ms = 0.0;    // sum of batch durations on the device
  int err_code = 0;
  std::string err_msg;

  int64_t now_ns() const {
    return std::chrono::duration_cast<std::chrono::nanoseconds>(std::chrono::steady_clock::now() - epoch).count();
  }
  void run();
  bool complete_finished(int64_t now);
  bool admit(int64_t now);
};

bool prng_server::complete_finished(int64_t now) {
  bool any = false;
  for (size_t b = 0; b < inflight.size();) {
    Batch& bt = inflight[b];
    const hipError_t q = hipEventQuery(events[bt.slot]);
    if (q == hipErrorNotReady) {
      ++b;
      continue;
    }
    if (q != hipSuccess && err_code == 0) {
      err_code = PRNG_EHIP;
      err_msg = std::string("batch failed: ") + hipGetErrorString(q);
    }
    float ms = 0.f;
    if (q == hipSuccess && hipEventElapsedTime(&ms, starts[bt.slot], events[bt.slot]) == hipSuccess) gpu_ms += ms;
    book.finish(bt.tickets, q == hipSuccess, now);
    book.arena.release(bt.ws_off, bt.ws_bytes);
    delete bt.t;
    slot_busy[bt.slot] = 0;
    --class_busy[bt.cls];
    inflight.erase(inflight.begin() + (long)b);
    any = true;
  }
  if (any) cv_done.notify_all();
  return any;
}

bool prng_server::admit(int64_t now) {
  int slot = -1;
  for (int i = 0; i < max_inflight; ++i)
    if (!slot_busy[i]) {
      slot = i;
      break;
    }
  if (slot < 0 || waiting.empty()) return false;
  // The class of the batch: that of the earliest arrived request whose class
  // may take a slot.  A class may take any free slot but the ones that other
  // classes with arrived requests and no batch in flight still need, so that
  // a busy class queues its next batch behind the running one while no class
  // waits for a slot.
  int free_slots = 0;
  for (int i = 0; i < max_inflight; ++i) free_slots += slot_busy[i] ? 0 : 1;
  bool waits[kServerClasses] = {};
  int first_of[kServerClasses];
  int order = 0, seen = 0;
  for (int c = 0; c < kServerClasses; ++c) first_of[c] = -1;
  for (auto it = waiting.begin(); it != waiting.end() && seen < kServerClasses; ++it, ++order) {
    const Req& r = book.reqs[*it];
    if (r.t_arrive > now) break;
    const int c = server_class(gens[r.gen]->kind);
    if (first_of[c] < 0) {
      first_of[c] = order;
      waits[c] = true;
      ++seen;
    }
  }
  // candidates, earliest first
  int cand[kServerClasses], n_cand = 0;
  for (int c = 0; c < kServerClasses; ++c) {
    if (!waits[c]) continue;
    int needed = 0;  // slots other idle classes with arrived requests need
    for (int o = 0; o < kServerClasses; ++o)
      if (o != c && waits[o] && class_busy[o] == 0) ++needed;
    if (free_slots - 1 < needed && class_busy[c] > 0) continue;
    cand[n_cand++] = c;
  }
  std::sort(cand, cand + n_cand, [&](int a, int b) { return first_of[a] < first_of[b]; });
  std::vector<uint64_t> take;
  std::vector<std::list<uint64_t>::iterator> take_it;
  const size_t batch_cap = (pool_bytes - fixed_bytes) / (size_t)max_inflight;
  size_t batch_bytes = 0;
  int cls = -1;
  // the first candidate class that has a request it can take now (its other
  // requests may all wait behind requests of the same streams in flight)
  for (int ci = 0; ci < n_cand && take.empty(); ++ci) {
    cls = cand[ci];
    std::set<std::pair<uint32_t, uint64_t>> keys, blocked;
    for (auto it = waiting.begin(); it != waiting.end() && (int)take.size() < max_batch; ++it) {
      Req& r = book.reqs[*it];
      if (r.t_arrive > now) break;  // not arrived yet (arrival order)
      if (server_class(gens[r.gen]->kind) != cls) continue;  // another class's batch takes it
      const auto key = std::make_pair(r.gen, r.stream);
      // per-stream FIFO: a stream busy in flight, already in this batch, or with
      // an earlier request left waiting keeps its later requests waiting too
      if (book.busy.count(key) || keys.count(key) || blocked.count(key)) {
        blocked.insert(key);
        continue;
      }
      // a batch takes at most its share of the pool, so that several batches
      // overlap (and the next one is planned while the previous ones run)
      if (!take.empty() && batch_bytes + r.out_bytes > batch_cap) break;
      size_t off;
      if (!book.arena.alloc(r.out_bytes, &off)) break;  // memory budget: admit in order, never over-allocate
      batch_bytes += r.out_bytes;
      r.out_off = off;
      keys.insert(key);
      take.push_back(*it);
      take_it.push_back(it);
    }
  }
  if (take.empty()) return false;
  // plan the batch as a stream table
  std::vector<prng_table_row> rows(take.size());
  for (size_t i = 0; i < take.size(); ++i) {
    const Req& r = book.reqs[take[i]];
    rows[i] = prng_table_row{r.gen, (uint32_t)r.dtype, r.stream, r.count, pool + r.out_off};
  }
  std::unique_ptr<Plan> P;
  size_t ws = 0;
  int rc;
  for (;;) {
    P.reset(new Plan());
    rc = make_plan(gens.data(), (int)gens.size(), rows.data(), rows.size(), SegSpec{}, &jumps, *P);
    if (rc != PRNG_OK || book.arena.alloc(P->total, &ws)) break;
    // no room for the workspace next to the outputs: admit the first half
    if (take.size() == 1) {
      rc = 1;
      if (inflight.empty()) {
        rc = fail(PRNG_ENOMEM, "pool too small for request %llu and its workspace", (unsigned long long)take[0]);
      }
      break;
    }
    const size_t keep_n = take.size() / 2;
    for (size_t i = keep_n; i < take.size(); ++i) book.arena.release(book.reqs[take[i]].out_off, book.reqs[take[i]].out_bytes);
    take.resize(keep_n);
    take_it.resize(keep_n);
    rows.resize(keep_n);
  }
  if (rc != PRNG_OK) {
    for (uint64_t tk : take) book.arena.release(book.reqs[tk].out_off, book.reqs[tk].out_bytes);
    if (rc < 0 && err_code == 0) {
      err_code = rc;
      err_msg = last_error();
    }
    return false;
  }
  prng_table* t = nullptr;
  hipStream_t s = streams[slot];
  hipError_t e = hipEventRecord(starts[slot], s);
  if (e != hipSuccess) rc = hip_fail(e, "hipEventRecord");
  if (rc == PRNG_OK) rc = table_from_plan(*P, pool + ws, s, false, false, &t);
  if (rc == PRNG_OK) e = enqueue_run(t, s);
  if (rc == PRNG_OK && e == hipSuccess) e = hipEventRecord(events[slot], s);
  if (rc != PRNG_OK || e != hipSuccess) {
    if (err_code == 0) {
      err_code = rc != PRNG_OK ? rc : PRNG_EHIP;
      err_msg = rc != PRNG_OK ? last_error() : hipGetErrorString(e);
    }
    delete t;
    (void)hipStreamSynchronize(s);
    book.arena.release(ws, P->total);
    for (uint64_t tk : take) book.arena.release(book.reqs[tk].out_off, book.reqs[tk].out_bytes);
    return false;
  }
  // commit
  for (auto it : take_it) waiting.erase(it);
  for (uint64_t tk : take) {
    Req& r = book.reqs[tk];
    r.state = INFLIGHT;
    r.t_admit = now;
    book.busy.insert({r.gen, r.stream});
  }
  Batch b;
  b.slot = slot;
  b.cls = cls;
  b.t = t;
  b.plan = std::move(P);
  b.tickets = std::move(take);
  b.ws_off = ws;
  b.ws_bytes = b.plan->total;
  slot_busy[slot] = 1;
  ++class_busy[cls];
  inflight.push_back(std::move(b));
  ++n_batches;
  plan_ns += now_ns() - now;
  return true;
}

void prng_server::run() {
  (void)hipSetDevice(device);
  // The worker polls for finished batches every 20 us while batches are in
  // flight; with the default 50 us timer slack each wait would run to about
  // 70 us, and a slot would stay idle that long after its batch ends.
  (void)prctl(PR_SET_TIMERSLACK, 1000UL, 0UL, 0UL, 0UL);
  std::unique_lock<std::mutex> lk(mu);
  while (!stop) {
    const int64_t now = now_ns();
    bool progressed = complete_finished(now);
    if (err_code == 0) progressed |= admit(now);
    if (progressed) continue;
    // nothing to do right now: sleep until the next arrival, a submission, or
    // a short poll interval while batches are in flight
    int64_t wait_ns = inflight.empty() ? 2000000 : 20000;
    if (!waiting.empty()) {
      const int64_t next = book.reqs[waiting.front()].t_arrive - now;
      if (next > 0) wait_ns = std::min<int64_t>(wait_ns, next);
      else wait_ns = std::min<int64_t>(wait_ns, 20000);
    }
    cv_work.wait_for(lk, std::chrono::nanoseconds(std::max<int64_t>(wait_ns, 1000)));
  }
}

PRNG_API int prng_server_create(prng_server** out, prng_gen* const* gens, int n_gens, void* d_pool, size_t pool_bytes,
                                int max_inflight, int max_batch, uint32_t seg_len, uint64_t max_request_draws) {
  if (!out) return fail(PRNG_EINVAL, "s is NULL");
  *out = nullptr;
  if (!gens || n_gens <= 0) return fail(PRNG_EINVAL, "no generator objects");
  for (int i = 0; i < n_gens; ++i)
    if (!gens[i]) return fail(PRNG_EINVAL, "generator %d is NULL", i);
  if (!d_pool || (reinterpret_cast<uintptr_t>(d_pool) & 255)) return fail(PRNG_EINVAL, "pool NULL or not 256-byte aligned");
  if (max_inflight < 1 || max_inflight > 16) return fail(PRNG_EINVAL, "max_inflight must be in [1, 16]");
  if (max_batch < 1) return fail(PRNG_EINVAL, "max_batch must be >= 1");
  if (max_request_draws == 0 || max_request_draws > kMaxDrawsPerLaunch)
    return fail(PRNG_EINVAL, "max_request_draws must be in [1, 2^30]");
  try {
    std::unique_ptr<prng_server> S(new prng_server());
    S->gens.assign(gens, gens + n_gens);
    S->pool = static_cast<char*>(d_pool);
    S->pool_bytes = pool_bytes;
    S->max_inflight = max_inflight;
    S->max_batch = max_batch;
    S->max_draws = max_request_draws;
    HIP_TRY(hipGetDevice(&S->device));
    // resident jump tables at the front of the pool
    const uint64_t L = seg_len == PRNG_SEG_NEVER ? 0
                       : seg_len == PRNG_SEG_AUTO ? kServerSegAuto
                                                  : (std::max<uint64_t>(seg_len, 384) + 383) / 384 * 384;
    S->jumps.L = L;
    std::vector<uint32_t> host;
    std::map<std::pair<int, uint32_t>, size_t> offs;
    bool lux = false;
    for (prng_gen* g : S->gens) {
      if (L == 0) continue;
      const auto key = std::make_pair(g->kind, g->kind == RANLUX ? g->p : 0u);
      if (offs.count(key)) continue;
      const uint64_t Lk = S->jumps.seg_len(g->kind);
      const uint64_t K = (max_request_draws + Lk - 1) / Lk;  // segments of the longest request
      if (K > kServerMaxSegments)
        return fail(PRNG_EINVAL, "max_request_draws above %llu for this segment length",
                    (unsigned long long)(kServerMaxSegments * Lk));
      const uint32_t nj = (uint32_t)(K - 1);  // segments j = 1..K-1 start from jumped states
      const uint32_t stride = jump_slot_words(g->kind);
      offs[key] = host.size();
      S->jumps.count[key] = nj;
      host.resize(host.size() + (size_t)nj * stride, 0u);
      if (!fill_jumps(g->kind, g->p, Lk, nj, host.data() + offs[key]))
        return fail(PRNG_EINVAL, "no jump data for kind %d", g->kind);
      if (g->kind == RANLUX) lux = true;
    }
    size_t aux_off = host.size();
    if (lux) {
      host.resize(host.size() + kRanluxAuxWords);
      fill_ranlux_aux(host.data() + aux_off);
    }
    S->fixed_bytes = align256(host.size() * 4);
    if (S->fixed_bytes + (1u << 20) > pool_bytes) return fail(PRNG_EINVAL, "pool too small (%zu bytes)", pool_bytes);
    if (!host.empty()) HIP_TRY(hipMemcpy(S->pool, host.data(), host.size() * 4, hipMemcpyHostToDevice));
    const uint32_t* dev = reinterpret_cast<const uint32_t*>(S->pool);
    for (auto& kv : offs) S->jumps.base[kv.first] = dev + kv.second;
    S->jumps.aux_ = lux ? dev + aux_off : nullptr;
    S->book.arena.init(S->fixed_bytes, pool_bytes - S->fixed_bytes);
    S->events.resize(max_inflight);
    S->starts.resize(max_inflight);
    S->slot_busy.assign(max_inflight, 0);
    S->streams.assign(max_inflight, nullptr);
    for (int i = 0; i < max_inflight; ++i) {
      HIP_TRY(hipStreamCreateWithFlags(&S->streams[i], hipStreamNonBlocking));
      HIP_TRY(hipEventCreate(&S->events[i]));
      HIP_TRY(hipEventCreate(&S->starts[i]));
    }
    S->epoch = std::chrono::steady_clock::now();
    prng_server* raw = S.release();
    raw->worker = std::thread([raw] { raw->run(); });
    *out = raw;
  } catch (const std::bad_alloc&) {
    return fail(PRNG_ENOMEM, "out of host memory");
  } catch (const std::system_error&) {
    return fail(PRNG_ENOMEM, "could not start the server thread");
  }
  return PRNG_OK;
}

PRNG_API void prng_server_destroy(prng_server* s) {
  if (!s) return;
  {
    std::lock_guard<std::mutex> lk(s->mu);
    s->stop = true;
  }
  s->cv_work.notify_all();
  if (s->worker.joinable()) s->worker.join();
  for (hipStream_t st : s->streams)
    if (st) (void)hipStreamSynchronize(st);
  for (auto& b : s->inflight) delete b.t;
  for (hipEvent_t e : s->events) (void)hipEventDestroy(e);
  for (hipEvent_t e : s->starts) (void)hipEventDestroy(e);
  for (hipStream_t st : s->streams)
    if (st) (void)hipStreamDestroy(st);
  delete s;
}

PRNG_API int64_t prng_server_now_ns(const prng_server* s) { return s ? s->now_ns() : -1; }

PRNG_API int prng_server_submit_many(prng_server* s, uint64_t n, const uint32_t* gen, const uint64_t* stream,
                                     const uint64_t* count, const int* dtype, const int64_t* arrive_ns, int keep,
                                     uint64_t* tickets) {
  if (!s) return fail(PRNG_EINVAL, "s is NULL");
  if (n && (!gen || !stream || !count || !dtype || !tickets)) return fail(PRNG_EINVAL, "NULL array");
  std::lock_guard<std::mutex> lk(s->mu);
  if (s->err_code) return fail(s->err_code, "server stopped: %s", s->err_msg.c_str());
  const int64_t now = s->now_ns();
  int64_t last = s->waiting.empty() ? INT64_MIN : s->book.reqs[s->waiting.back()].t_arrive;
  for (uint64_t i = 0; i < n; ++i) {
    if (gen[i] >= s->gens.size()) return fail(PRNG_EINVAL, "request %llu: generator index out of range", (unsigned long long)i);
    if (stream[i] >= s->gens[gen[i]]->n) return fail(PRNG_EINVAL, "request %llu: stream out of range", (unsigned long long)i);
    if (dtype[i] < U32 || dtype[i] > F64) return fail(PRNG_EINVAL, "request %llu: unknown dtype", (unsigned long long)i);
    if (const char* why = check_request_size(count[i], dtype[i] == F64 ? 2 : 1, elem_bytes(dtype[i]), s->max_draws,
                                             s->pool_bytes - s->fixed_bytes))
      return fail(PRNG_EINVAL, "request %llu: %s", (unsigned long long)i, why);
    const int64_t t = (arrive_ns && arrive_ns[i] >= 0) ? arrive_ns[i] : now;
    if (t < last) return fail(PRNG_EINVAL, "request %llu: arrivals must be non-decreasing", (unsigned long long)i);
    last = t;
  }
  for (uint64_t i = 0; i < n; ++i) {
    Req r;
    r.gen = gen[i];
    r.stream = stream[i];
    r.count = count[i];
    r.dtype = dtype[i];
    r.keep = keep ? 1 : 0;
    r.t_arrive = (arrive_ns && arrive_ns[i] >= 0) ? arrive_ns[i] : now;
    r.out_bytes = count[i] * elem_bytes(dtype[i]);
    tickets[i] = s->book.reqs.size();
    s->book.reqs.push_back(r);
    s->waiting.push_back(tickets[i]);
  }
  s->cv_work.notify_all();
  return PRNG_OK;
}

PRNG_API int prng_server_submit(prng_server* s, uint32_t gen, uint64_t stream, uint64_t count, int dtype,
                                uint64_t* ticket) {
  const int64_t now = -1;
  return prng_server_submit_many(s, 1, &gen, &stream, &count, &dtype, &now, 1, ticket);
}

PRNG_API int prng_server_result(prng_server* s, uint64_t ticket, int timeout_ms, void** d_out, size_t* bytes) {
  if (!s) return fail(PRNG_EINVAL, "s is NULL");
  std::unique_lock<std::mutex> lk(s->mu);
  if (ticket >= s->book.reqs.size()) return fail(PRNG_EINVAL, "unknown ticket");
  auto ready = [&] { return s->book.settled(ticket, s->err_code); };
  if (timeout_ms != 0 && !ready()) {
    if (timeout_ms < 0)
      s->cv_done.wait(lk, ready);
    else
      s->cv_done.wait_for(lk, std::chrono::milliseconds(timeout_ms), ready);
  }
  const Req& r = s->book.reqs[ticket];
  if (r.state == RELEASED) return fail(PRNG_EINVAL, "ticket already released");
  const int st = s->book.status(ticket, s->err_code);
  if (st < 0) {
    if (r.state == FAILED) return fail(st, "request failed: %s", s->err_msg.c_str());
    return fail(st, "server stopped: %s", s->err_msg.c_str());
  }
  if (st == 0) return 0;
  if (d_out) *d_out = s->pool + r.out_off;
  if (bytes) *bytes = r.out_bytes;
  return 1;
}

PRNG_API int prng_server_release(prng_server* s, uint64_t ticket) {
  if (!s) return fail(PRNG_EINVAL, "s is NULL");
  std::lock_guard<std::mutex> lk(s->mu);
  if (ticket >= s->book.reqs.size()) return fail(PRNG_EINVAL, "unknown ticket");
  if (!s->book.release(ticket)) return fail(PRNG_EINVAL, "ticket not completed or already released");
  s->cv_work.notify_all();
  return PRNG_OK;
}

PRNG_API int prng_server_times(const prng_server* s, uint64_t n, const uint64_t* tickets, int64_t* arrive_ns,
                               int64_t* admit_ns, int64_t* done_ns) {
  if (!s) return fail(PRNG_EINVAL, "s is NULL");
  std::lock_guard<std::mutex> lk(const_cast<prng_server*>(s)->mu);
  for (uint64_t i = 0; i < n; ++i) {
    if (tickets[i] >= s->book.reqs.size()) return fail(PRNG_EINVAL, "unknown ticket");
    const Req& r = s->book.reqs[tickets[i]];
    if (arrive_ns) arrive_ns[i] = r.t_arrive;
    if (admit_ns) admit_ns[i] = r.t_admit;
    if (done_ns) done_ns[i] = r.t_done;
  }
  return PRNG_OK;
}

PRNG_API int prng_server_timing(const prng_server* s, int64_t* host_plan_ns, double* device_ms) {
  if (!s) return fail(PRNG_EINVAL, "s is NULL");
  std::lock_guard<std::mutex> lk(const_cast<prng_server*>(s)->mu);
  if (host_plan_ns) *host_plan_ns = s->plan_ns;
  if (device_ms) *device_ms = s->gpu_ms;
  return PRNG_OK;
}

PRNG_API int prng_server_stats(const prng_server* s, uint64_t* submitted, uint64_t* completed, uint64_t* batches,
                               size_t* pool_in_use) {
  if (!s) return fail(PRNG_EINVAL, "s is NULL");
  std::lock_guard<std::mutex> lk(const_cast<prng_server*>(s)->mu);
  if (submitted) *submitted = s->book.reqs.size();
  if (completed) *completed = s->book.n_completed;
  if (batches) *batches = s->n_batches;
  if (pool_in_use) *pool_in_use = s->book.arena.used();
  if (s->err_code) return fail(s->err_code, "server stopped: %s", s->err_msg.c_str());
  return PRNG_OK;
}
