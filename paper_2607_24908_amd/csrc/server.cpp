// Flow server behind frg_submit / frg_poll.
//
// Admission: a submitted flow waits in a FIFO queue until a slot is free
// and its device footprint (its share of a staging buffer: U, dU/dt and the
// 7 Jacobian bands of one call) fits the context's HBM budget, so the
// batches in flight, which never share a flow, stay within the budget
// together.
//
// Execution: every admitted flow runs the FP64 host stepper in its own
// thread.  Its right-hand-side calls are handed to one dispatcher thread,
// which takes ALL calls pending at that moment -- from any mix of flows,
// grid sizes and N -- and serves them with one batched LPA launch on the
// a stream of the server's (continuous batching: flows join and leave at the
// granularity of a right-hand-side call, and calls that arrive while a batch
// is on the GPU form the next batch).  A flow's result does not depend on
// which flows shared its launches: the kernel evaluates each grid point of
// each flow independently, in a fixed order.
//
// Round trip of a batch: the U of every flow and zeroed domain flags are packed
// into one pinned host buffer; the kernel reads them there and writes the
// flags and every flow's outputs back into it (zero copy; knob
// server_zero_copy), or the packed head goes up in one copy and the flags and
// outputs come back in one (a device mirror of the buffer).  In zero copy the
// kernel's last workgroup sets a word in host memory that the dispatcher polls.  A
// flow that polls for its answer copies its outputs from the buffer itself,
// beside the other flows and the dispatcher; for a sleeping one the dispatcher
// copies.  There are two such buffers, each with its stream, so that two batches
// run side by side; a buffer is staged again when its batch is back and its last
// reader is done.  Six flows of up to 1024 points submitted at once: 26 ms; with
// an event recorded and waited for per batch, one stream and every copy made by
// the dispatcher 42 ms.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <chrono>
#include <cmath>
#include <condition_variable>
#include <cstdlib>
#include <cstring>
#include <deque>
#include <map>
#include <mutex>
#include <thread>
#include <vector>

#include "frg_ctx.h"

namespace frg {

int solve_flow(const frg_request &rq, frg_rhs_fn rhs, void *user, frg_result *res);

struct Server;

struct Flow {
  Server *srv = nullptr;
  uint64_t ticket = 0;
  frg_request req{};
  frg_result res{};
  int64_t n = 0;
  int64_t bytes = 0;
  // right-hand-side hand-off: the stepper's buffers, valid while it waits
  double t = 0.0;
  const double *U_src = nullptr;
  double *dUdt_dst = nullptr;
  double *jac_dst = nullptr;
  bool want_jac = false;
  bool spin = false;                    // polls for its answer, and copies it
  const double *out = nullptr;          // its outputs in the staging buffer
  std::atomic<int> *readers = nullptr;  // of that buffer, to count down
  bool ready = false;
  std::atomic<bool> ready_a{false};  // mirror of ready for waiting without the lock
  int rc = FRG_OK;
  bool done = false;
  std::condition_variable cv;
  std::thread th;
};

// One staging buffer: the batch's descriptors, inputs, flags and outputs.
struct Stage {
  char *h = nullptr;   // pinned, mapped, coherent
  char *hd = nullptr;  // its device address
  char *d = nullptr;   // device mirror (copy mode)
  size_t cap = 0;
  hipStream_t stream = nullptr;
  hipEvent_t done = nullptr;     // copy mode: recorded after the batch's last operation
  volatile unsigned *word = nullptr;  // zero copy: pinned, set by the batch's last workgroup
  LpaDone signal{};              // its device address, the workgroup counter
  std::atomic<int> readers{0};   // flows that still copy their outputs
};

// A launched batch, until its outputs are handed back.
struct Batch {
  std::vector<Flow *> flows;
  std::vector<size_t> o_o;  // each flow's outputs in the staging buffer
  size_t o_flags = 0;
  bool zero_copy = false;
  unsigned polls = 0;
  int rc = FRG_OK;
};

// With more running flows than spin_flows (environment FRG_SERVER_SPIN_FLOWS,
// default kSpinFlows), the steppers sleep on their condition variables at
// once: a spinning thread per flow would take the cores that the others'
// steppers need.
constexpr int kSpinFlows = 12;

constexpr int kStages = 2;
constexpr int kWordStride = 32;  // unsigneds: words and counters on lines of their own

struct Server {
  Context *ctx = nullptr;
  Stage stg[kStages];
  unsigned *words = nullptr;   // pinned, kWordStride apart
  unsigned *counts = nullptr;  // device
  std::mutex m;
  std::condition_variable cv_disp;
  std::deque<Flow *> queue;
  std::vector<Flow *> pending;
  std::atomic<int> n_pending{0};  // size of pending, for waiting without the lock
  std::map<uint64_t, Flow *> flows;
  uint64_t next_ticket = 1;
  int active = 0;
  int max_active = 64;
  int spin_flows = kSpinFlows;
  size_t max_queue = 65536;
  uint64_t budget = 0;
  uint64_t used = 0;
  bool stop = false;
  std::thread disp;
  int64_t flows_done = 0, launches = 0, batched = 0;

  int start();
  void shutdown();
  void release();
  void dispatch_loop();
  void admit_locked();
  static int rhs_cb(void *user, double t, const double *U, int64_t n, double *dUdt, double *jac);
  void run_flow(Flow *f);
  bool grow_stage(Stage &g, size_t bytes);
  void launch_batch(Batch &b, Stage &g);
  bool batch_done(Batch &b, Stage &g, bool block);
  void finish_batch(Batch &b, Stage &g);
  static void take_outputs(Flow *f, const double *o);
};

// A right-hand side comes back, and the next call arrives, within tens of
// microseconds while flows run; the dispatcher and the steppers poll for
// that long before they sleep on their condition variables (a wake-up
// through the kernel costs about as much as the call itself).
constexpr double kSpinSeconds = 200e-6;

template <class Cond>
static bool spin_until(Cond cond) {
  const auto t0 = std::chrono::steady_clock::now();
  for (int i = 0;; ++i) {
    if (cond()) return true;
    if ((i & 63) == 63 && std::chrono::duration<double>(std::chrono::steady_clock::now() - t0)
                                  .count() > kSpinSeconds)
      return false;
  }
}

int Server::start() {
  const size_t bytes = sizeof(unsigned) * kStages * kWordStride;
  void *dev_words = nullptr;
  if (hipHostMalloc((void **)&words, bytes, hipHostMallocMapped | hipHostMallocCoherent) !=
          hipSuccess ||
      hipHostGetDevicePointer(&dev_words, words, 0) != hipSuccess ||
      hipMalloc((void **)&counts, bytes) != hipSuccess ||
      hipMemset(counts, 0, bytes) != hipSuccess || hipDeviceSynchronize() != hipSuccess) {
    release();
    return fail(FRG_E_DEVICE, "server completion words");
  }
  std::memset(words, 0, bytes);
  for (int i = 0; i < kStages; ++i) {
    Stage &g = stg[i];
    g.word = words + i * kWordStride;
    g.signal = LpaDone{counts + i * kWordStride, (unsigned *)dev_words + i * kWordStride, 0};
    if (hipStreamCreateWithFlags(&g.stream, hipStreamNonBlocking) != hipSuccess ||
        hipEventCreateWithFlags(&g.done, hipEventDisableTiming) != hipSuccess) {
      release();
      return fail(FRG_E_DEVICE, "server stream");
    }
  }
  if (const char *e = std::getenv("FRG_SERVER_SLOTS")) max_active = std::max(1, std::atoi(e));
  if (const char *e = std::getenv("FRG_SERVER_SPIN_FLOWS")) spin_flows = std::max(0, std::atoi(e));
  disp = std::thread([this] { dispatch_loop(); });
  return FRG_OK;
}

void Server::shutdown() {
  {
    std::lock_guard<std::mutex> lk(m);
    stop = true;
    for (auto &kv : flows) kv.second->cv.notify_all();
  }
  cv_disp.notify_all();
  if (disp.joinable()) disp.join();
  // `flows` owns every flow that has not been polled, admitted or still
  // queued; `queue` only lists the queued ones, so it is cleared without
  // deleting anything
  for (auto &kv : flows) {
    if (kv.second->th.joinable()) kv.second->th.join();
    delete kv.second;
  }
  flows.clear();
  queue.clear();
  release();
}

// The buffers, streams and words (no batch in flight, no dispatcher).
void Server::release() {
  for (Stage &g : stg) {
    if (g.stream) (void)hipStreamSynchronize(g.stream);
    if (g.d) (void)hipFree(g.d);
    if (g.h) (void)hipHostFree(g.h);
    if (g.done) (void)hipEventDestroy(g.done);
    if (g.stream) (void)hipStreamDestroy(g.stream);
  }
  if (words) (void)hipHostFree(words);
  if (counts) (void)hipFree(counts);
}

// Dispatcher thread only (no batch of this buffer in flight): make the
// staging buffer hold `bytes`.
bool Server::grow_stage(Stage &g, size_t bytes) {
  if (bytes <= g.cap) return true;
  const size_t cap = std::max(bytes, 2 * g.cap);
  if (g.d) (void)hipFree(g.d);
  if (g.h) (void)hipHostFree(g.h);
  g.d = g.h = g.hd = nullptr;
  g.cap = 0;
  if (hipMalloc((void **)&g.d, cap) != hipSuccess) return false;
  if (hipHostMalloc((void **)&g.h, cap, hipHostMallocMapped | hipHostMallocCoherent) !=
          hipSuccess ||
      hipHostGetDevicePointer((void **)&g.hd, g.h, 0) != hipSuccess) {
    if (g.h) (void)hipHostFree(g.h);
    (void)hipFree(g.d);
    g.d = g.h = g.hd = nullptr;
    return false;
  }
  g.cap = cap;
  return true;
}

// Under m: start queued flows while slots and budget allow (strict FIFO).
void Server::admit_locked() {
  while (!queue.empty() && active < max_active && !stop) {
    Flow *f = queue.front();
    // the context's own device buffers count against the same budget (a flow
    // is always admitted when none runs: it fitted on its own at submission)
    if (active > 0 && used + (uint64_t)f->bytes + ctx->hbm.used.load() > budget) break;
    queue.pop_front();
    used += f->bytes;
    ++active;
    f->res.start_s = now_s();
    f->th = std::thread([this, f] { run_flow(f); });
  }
}

int Server::rhs_cb(void *user, double t, const double *U, int64_t n, double *dUdt, double *jac) {
  TraceRange trace_("frg_server_rhs");  // a flow thread's right-hand side, queued to its answer
  Flow *f = static_cast<Flow *>(user);
  Server *s = f->srv;
  if (n != f->n) return FRG_E_INVAL;
  bool spin;
  {
    std::lock_guard<std::mutex> lk(s->m);
    if (s->stop) return FRG_E_DEVICE;
    spin = s->active <= s->spin_flows;
    f->spin = spin;
    f->t = t;
    f->U_src = U;
    f->dUdt_dst = dUdt;
    f->jac_dst = jac;
    f->want_jac = jac != nullptr;
    f->ready = false;
    f->ready_a.store(false, std::memory_order_relaxed);
    s->pending.push_back(f);
    s->n_pending.fetch_add(1, std::memory_order_release);
  }
  s->cv_disp.notify_one();
  if (!spin || !spin_until([&] { return f->ready_a.load(std::memory_order_acquire); })) {
    // a stop ends the wait of a call that still queues; one that a batch has
    // taken is waited for, since the dispatcher reads and writes its vectors
    std::unique_lock<std::mutex> lk(s->m);
    auto queued = [&] { return std::find(s->pending.begin(), s->pending.end(), f); };
    f->cv.wait(lk, [&] { return f->ready || (s->stop && queued() != s->pending.end()); });
    if (!f->ready) {
      s->pending.erase(queued());
      s->n_pending.fetch_sub(1, std::memory_order_relaxed);
      return FRG_E_DEVICE;
    }
  }
  if (f->readers) {
    take_outputs(f, f->out);
    f->readers->fetch_sub(1, std::memory_order_release);
  }
  return f->rc;
}

// Copy a flow's outputs into its stepper's vectors.  Of the bands -3, -2, 2, 3
// only the first and last row's entries are written (LpaJob::far_bands); the
// stepper's vector holds zeros in the others from the start.
void Server::take_outputs(Flow *f, const double *o) {
  const int64_t n = f->n;
  std::memcpy(f->dUdt_dst, o, n * sizeof(double));
  if (!f->want_jac) return;
  const double *src = o + n;
  std::memcpy(f->jac_dst + 2 * n, src + 2 * n, 3 * n * sizeof(double));
  for (int b : {0, 1, 5, 6})
    for (int64_t i : {(int64_t)0, n - 1}) f->jac_dst[b * n + i] = src[b * n + i];
}

void Server::run_flow(Flow *f) {
  frg_result r{};
  solve_flow(f->req, &Server::rhs_cb, f, &r);
  std::lock_guard<std::mutex> lk(m);
  f->res.status = r.status;
  f->res.steps = r.steps;
  f->res.rejected = r.rejected;
  f->res.rhs_calls = r.rhs_calls;
  f->res.t_reached = r.t_reached;
  f->res.done_s = now_s();
  f->done = true;
  used -= f->bytes;
  --active;
  ++flows_done;
  admit_locked();
}

// Stage the batch's right-hand sides into its buffer and enqueue it on the
// buffer's stream.  Layout: jobs (of more flows than a launch takes as
// arguments) | U of each flow | flags | outputs of each flow (dU/dt, then the 7
// bands when asked); [0, o_out) goes up and [o_flags, end) comes back (copy
// mode, then the buffer's event), or the kernel reads and writes the pinned
// buffer in place and sets its word (zero copy).
void Server::launch_batch(Batch &b, Stage &g) {
  TraceRange trace_("frg_server_batch");  // staging and enqueueing one launch
  auto up8 = [](size_t x) { return (x + 7) & ~(size_t)7; };
  const int nb = (int)b.flows.size();
  std::vector<frg_lpa> lpas(nb);
  std::vector<double> ts(nb);
  std::vector<const double *> Us(nb);
  std::vector<double *> Ds(nb), Js(nb);
  std::vector<LpaJob> jobs(nb);
  std::vector<size_t> o_u(nb);
  b.o_o.resize(nb);
  const bool by_args = nb <= kLpaArgs;
  size_t cu = by_args ? 0 : up8(nb * sizeof(LpaJob));
  for (int i = 0; i < nb; ++i) {
    o_u[i] = cu;
    cu += b.flows[i]->n * sizeof(double);
  }
  b.o_flags = cu;
  size_t co = up8(b.o_flags + nb * sizeof(int));
  const size_t o_out = co;
  for (int i = 0; i < nb; ++i) {
    b.o_o[i] = co;
    co += (b.flows[i]->want_jac ? 8 : 1) * b.flows[i]->n * sizeof(double);
  }
  const size_t end = co;
  if (!grow_stage(g, end)) {
    b.rc = FRG_E_NOMEM;
    return;
  }
  {
    std::lock_guard<std::mutex> lk(ctx->mu);
    b.zero_copy = ctx->tune.server_zero_copy != 0;
  }
  char *dev = b.zero_copy ? g.hd : g.d;  // where the kernel finds the buffer
  for (int i = 0; i < nb; ++i) {
    Flow *f = b.flows[i];
    lpas[i] = f->req.lpa;
    ts[i] = f->t;
    std::memcpy(g.h + o_u[i], f->U_src, f->n * sizeof(double));
    Us[i] = (const double *)(dev + o_u[i]);
    Ds[i] = (double *)(dev + b.o_o[i]);
    Js[i] = f->want_jac ? Ds[i] + f->n : nullptr;
  }
  std::memset(g.h + b.o_flags, 0, o_out - b.o_flags);
  int64_t blocks;
  {
    std::lock_guard<std::mutex> lk(ctx->mu);
    b.rc = ctx->lpa_job_table(nb, lpas.data(), ts.data(), Us.data(), Ds.data(), Js.data(),
                              (int *)(dev + b.o_flags), jobs.data(), &blocks);
  }
  if (b.rc != FRG_OK) return;
  for (LpaJob &j : jobs) j.far_bands = 0;
  if (!by_args) std::memcpy(g.h, jobs.data(), nb * sizeof(LpaJob));
  auto launch = [&](const LpaDone &done) {
    return (by_args ? launch_lpa_args(jobs.data(), nb, blocks, done, g.stream)
                    : launch_lpa_table((const LpaJob *)dev, nb, blocks, done, g.stream)) == 0;
  };
  bool ok;
  if (b.zero_copy) {
    ++g.signal.value;
    ok = launch(g.signal);
  } else {
    ok = hipMemcpyAsync(g.d, g.h, o_out, hipMemcpyHostToDevice, g.stream) == hipSuccess &&
         launch(LpaDone{}) &&
         hipMemcpyAsync(g.h + b.o_flags, g.d + b.o_flags, end - b.o_flags,
                        hipMemcpyDeviceToHost, g.stream) == hipSuccess &&
         hipEventRecord(g.done, g.stream) == hipSuccess;
  }
  if (!ok) b.rc = FRG_E_DEVICE;
}

// Whether a launched batch has come back (block: wait until it has).  A kernel
// that ended without setting its word, or an error of the stream, makes it one
// that failed.
bool Server::batch_done(Batch &b, Stage &g, bool block) {
  if (b.rc != FRG_OK) return true;
  for (int i = 1;; ++i, ++b.polls) {
    if (b.zero_copy && *g.word == g.signal.value) {
      std::atomic_thread_fence(std::memory_order_acquire);
      return true;
    }
    if (!b.zero_copy || b.polls % (1u << 20) == (1u << 20) - 1) {
      const hipError_t e = b.zero_copy ? hipStreamQuery(g.stream) : hipEventQuery(g.done);
      if (e == hipSuccess && b.zero_copy && *g.word != g.signal.value) b.rc = FRG_E_DEVICE;
      if (e != hipSuccess && e != hipErrorNotReady) b.rc = FRG_E_DEVICE;
      if (e != hipErrorNotReady) return true;
      (void)hipGetLastError();
    }
    if (!block && i % 64 == 0) return false;
  }
}

// Hand the outputs of a batch that has come back to its flows.
void Server::finish_batch(Batch &b, Stage &g) {
  const int nb = (int)b.flows.size();
  int readers = 0;
  for (int i = 0; i < nb; ++i) {
    Flow *f = b.flows[i];
    f->out = (const double *)(g.h + b.o_o[i]);
    const bool reads = b.rc == FRG_OK && f->spin;
    f->readers = reads ? &g.readers : nullptr;
    readers += reads;
    if (b.rc == FRG_OK && !reads) take_outputs(f, f->out);
  }
  g.readers.store(readers, std::memory_order_relaxed);
  const int *flags = b.rc == FRG_OK ? (const int *)(g.h + b.o_flags) : nullptr;
  std::lock_guard<std::mutex> lk(m);
  ++launches;
  batched += nb;
  for (int i = 0; i < nb; ++i) {
    Flow *f = b.flows[i];
    f->rc = b.rc != FRG_OK ? b.rc : (flags[i] ? FRG_E_DOMAIN : FRG_OK);
    f->ready = true;
    f->ready_a.store(true, std::memory_order_release);
    f->cv.notify_one();
  }
}

// Batches of the pending right-hand sides: with no batch in flight the
// dispatcher waits for work; otherwise it hands back batches as they come back
// and takes whatever is pending as soon as a buffer is free.
void Server::dispatch_loop() {
  (void)hipSetDevice(ctx->device);
  Batch fly[kStages];
  bool busy[kStages] = {};
  for (;;) {
    bool any = false;
    for (int s = 0; s < kStages; ++s) {
      if (busy[s] && batch_done(fly[s], stg[s], false)) {
        finish_batch(fly[s], stg[s]);
        busy[s] = false;
      }
      any |= busy[s];
    }
    if (!any) spin_until([&] { return n_pending.load(std::memory_order_acquire) > 0; });
    int free_slot = -1;
    for (int s = kStages - 1; s >= 0; --s)
      if (!busy[s] && stg[s].readers.load(std::memory_order_acquire) == 0) free_slot = s;
    if (any && (free_slot < 0 || n_pending.load(std::memory_order_acquire) == 0)) continue;
    Batch next;
    bool stopping;
    {
      std::unique_lock<std::mutex> lk(m);
      if (!any) cv_disp.wait(lk, [&] { return !pending.empty() || stop; });
      stopping = stop;
      if (!stopping && free_slot >= 0) {
        next.flows.swap(pending);
        n_pending.store(0, std::memory_order_relaxed);
      }
    }
    if (stopping) {
      for (int s = 0; s < kStages; ++s)
        if (busy[s]) {
          (void)batch_done(fly[s], stg[s], true);
          finish_batch(fly[s], stg[s]);
        }
      return;
    }
    if (!next.flows.empty()) {
      launch_batch(next, stg[free_slot]);
      fly[free_slot] = std::move(next);
      busy[free_slot] = true;
    }
  }
}

void Context::stop_server() {
  if (!server) return;
  server->shutdown();
  delete server;
  server = nullptr;
}

}  // namespace frg

using namespace frg;

extern "C" {

int frg_submit(frg_ctx *ctx, const frg_request *req, uint64_t *ticket) {
  frg::TraceRange trace_("frg_submit");
  if (!ctx || !req || !ticket) return fail(FRG_E_INVAL, "NULL argument");
  int rc = check_lpa(req->lpa);
  if (rc) return rc;
  if (!req->U_out) return fail(FRG_E_INVAL, "U_out is NULL");
  if (!std::isfinite(req->t_end) || req->t_end > 0.0) return fail(FRG_E_INVAL, "t_end must be <= 0");
  if (!std::isfinite(req->lambda) || !std::isfinite(req->rho0))
    return fail(FRG_E_INVAL, "bad initial potential");
  Server *s;
  {
    std::lock_guard<std::mutex> lk(ctx->mu);
    if (!ctx->server) {
      auto *ns = new Server();
      ns->ctx = ctx;
      ns->budget = ctx->hbm_budget;
      (void)hipSetDevice(ctx->device);
      rc = ns->start();
      if (rc) {
        delete ns;
        return rc;
      }
      ctx->server = ns;
    }
    s = ctx->server;
  }
  const int64_t bytes = frg_flow_footprint(&req->lpa);
  {
    std::lock_guard<std::mutex> lk(ctx->mu);
    if ((uint64_t)bytes + ctx->hbm.used + ctx->hbm.extra > s->budget) ctx->hbm.give_back();
  }
  std::lock_guard<std::mutex> lk(s->m);
  if ((uint64_t)bytes + ctx->hbm.used.load() > s->budget)
    return fail(FRG_E_NOMEM, "flow footprint %lld B and the context's buffers exceed the HBM budget",
                (long long)bytes);
  if (s->queue.size() >= s->max_queue) return fail(FRG_E_AGAIN, "submission queue full");
  Flow *f = new Flow();
  f->srv = s;
  f->ticket = s->next_ticket++;
  f->req = *req;
  f->n = req->lpa.n_grid;
  f->bytes = bytes;
  f->res.status = FRG_PENDING;
  f->res.submit_s = now_s();
  s->flows[f->ticket] = f;
  s->queue.push_back(f);
  s->admit_locked();
  *ticket = f->ticket;
  clear_error();
  return FRG_OK;
}

int frg_poll(frg_ctx *ctx, uint64_t ticket, frg_result *out) {
  if (!ctx || !out) return fail(FRG_E_INVAL, "NULL argument");
  Server *s = ctx->server;
  if (!s) return fail(FRG_E_NOTFOUND, "unknown ticket %llu", (unsigned long long)ticket);
  Flow *f;
  {
    std::lock_guard<std::mutex> lk(s->m);
    auto it = s->flows.find(ticket);
    if (it == s->flows.end()) return fail(FRG_E_NOTFOUND, "unknown ticket %llu", (unsigned long long)ticket);
    f = it->second;
    if (!f->done) {
      *out = f->res;
      out->status = FRG_PENDING;
      return FRG_PENDING;
    }
    s->flows.erase(it);
  }
  if (f->th.joinable()) f->th.join();
  *out = f->res;
  delete f;
  clear_error();
  return FRG_OK;
}

int frg_server_stats(frg_ctx *ctx, int64_t *flows_done, int64_t *launches, double *mean_batch) {
  if (!ctx) return fail(FRG_E_INVAL, "ctx is NULL");
  Server *s = ctx->server;
  int64_t d = 0, l = 0, b = 0;
  if (s) {
    std::lock_guard<std::mutex> lk(s->m);
    d = s->flows_done;
    l = s->launches;
    b = s->batched;
  }
  if (flows_done) *flows_done = d;
  if (launches) *launches = l;
  if (mean_batch) *mean_batch = l ? (double)b / (double)l : 0.0;
  return FRG_OK;
}

}  // extern "C"
