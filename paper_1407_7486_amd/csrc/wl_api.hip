// Host side of the C ABI declared in include/wl.h: argument checks, device
// buffers, work decomposition and the launches (kernels in wl_kernels.hip).
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdarg.h>
#include <stdio.h>
#include <string.h>

#include <mutex>
#include <string>
#include <utility>
#include <vector>

#include "wl_host.h"

namespace wl {

int fail(wl_ctx* ctx, int code, const char* fmt, ...) {
  if (ctx) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof(buf), fmt, ap);
    va_end(ap);
    ctx->err = buf;
  }
  return code;
}

int hip_fail(wl_ctx* ctx, hipError_t e, const char* what) {
  return fail(ctx, WL_EHIP, "%s: %s", what, hipGetErrorString(e));
}

// The live contexts, whose idle device memory serves any of them.
struct Contexts {
  std::mutex mu;
  std::vector<wl_ctx*> live;
};
static Contexts& contexts() {
  static Contexts* c = new Contexts;  // outlives every static destructor
  return *c;
}

// Gives back what the contexts of a device hold without using it: the blocks of
// freed ensembles and the scratch that no call is working with.
static void give_back(int device) {
  Contexts& all = contexts();
  std::lock_guard<std::mutex> lock(all.mu);
  for (wl_ctx* c : all.live) {
    if (c->device != device) continue;
    std::lock_guard<std::mutex> idle(c->cache_mu);
    for (const auto& b : c->ens_cache) (void)hipFree(b.first);
    c->ens_cache.clear();
    if (c->d_work && !c->work_busy) {
      (void)hipFree(c->d_work);
      c->d_work = nullptr;
      c->work_bytes = 0;
    }
  }
}

hipError_t dev_malloc(wl_ctx* ctx, void** p, size_t bytes) {
  hipError_t e = hipMalloc(p, bytes);
  if (e == hipSuccess) return e;
  (void)hipGetLastError();
  give_back(ctx->device);
  e = hipMalloc(p, bytes);
  if (e != hipSuccess) {
    *p = nullptr;
    (void)hipGetLastError();
  }
  return e;
}

static int ensure(wl_ctx* ctx, void** p, size_t* have, size_t need, const char* what) {
  if (need <= *have) return WL_OK;
  if (*p) {
    // pending work may still read the old buffer
    hipError_t e = hipStreamSynchronize(ctx->stream);
    if (e != hipSuccess) return hip_fail(ctx, e, "hipStreamSynchronize");
    (void)hipFree(*p);
    *p = nullptr;
    *have = 0;
  }
  if (dev_malloc(ctx, p, need) != hipSuccess)
    return fail(ctx, WL_ENOMEM, "hipMalloc(%zu bytes) for %s failed", need, what);
  *have = need;
  return WL_OK;
}

Work::Work(wl_ctx* ctx, size_t bytes, const char* what) {
  if (bytes <= kWorkKeep) {
    {
      std::lock_guard<std::mutex> lock(ctx->cache_mu);
      ctx->work_busy = true;
    }
    holder = ctx;
    if (ensure(ctx, &ctx->d_work, &ctx->work_bytes, bytes, what) == WL_OK) p = ctx->d_work;
    return;
  }
  temporary = true;
  if (dev_malloc(ctx, &p, bytes) != hipSuccess) {
    p = nullptr;
    fail(ctx, WL_ENOMEM, "hipMalloc(%zu bytes) for %s failed", bytes, what);
  }
}

Work::~Work() {
  if (temporary && p) (void)hipFree(p);
  if (holder) {
    std::lock_guard<std::mutex> lock(holder->cache_mu);
    holder->work_busy = false;
  }
}

// While it lives, this thread's allocations do not end the capture of another
// stream (torch captures in the global mode, in which any hipMalloc would): for
// buffers made on first use, which calls of the same kind did without before.
struct RelaxedCapture {
  hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
  RelaxedCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
  ~RelaxedCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
  RelaxedCapture(const RelaxedCapture&) = delete;
  RelaxedCapture& operator=(const RelaxedCapture&) = delete;
};

// Makes the staging buffer and its events; false (and nothing left behind, so
// that the next call tries again) where they cannot be had.
static bool pin_make(wl_ctx* ctx) {
  if (ctx->h_pin) return true;
  const RelaxedCapture relaxed;
  char* p = nullptr;
  hipEvent_t ev[2] = {nullptr, nullptr};
  bool ok = hipHostMalloc((void**)&p, 2 * kPinHalf, hipHostMallocDefault) == hipSuccess;
  for (int k = 0; k < 2 && ok; ++k)
    ok = hipEventCreateWithFlags(&ev[k], hipEventDisableTiming) == hipSuccess;
  if (!ok) {
    (void)hipGetLastError();
    for (hipEvent_t e : ev)
      if (e) (void)hipEventDestroy(e);
    if (p) (void)hipHostFree(p);
    return false;
  }
  ctx->h_pin = p;
  for (int k = 0; k < 2; ++k) ctx->pin_ev[k] = ev[k];
  return true;
}

// Which pieces go without staging: all where it cannot be had, and arrays of at
// least kPinDirect bytes that the device reaches itself (pinned by the caller):
// the staging's memcpy is slower than the copy (wl_per_loop, three pinned arrays
// of 1 MiB 108 us, staged 200; of 64 MiB 3.6 ms, staged 7.2).  Pageable arrays
// the runtime copies piece by piece itself (three of 1 MiB 205 us, staged 187;
// of 64 MiB 11.3 ms, staged 7.3).
static bool mark_direct(wl_ctx* ctx, Piece* pieces, int n) {
  const bool staging = pin_make(ctx);
  bool any_staged = false;
  for (int i = 0; i < n; ++i) {
    Piece& q = pieces[i];
    if (!q.host || !q.bytes) continue;
    q.direct = !staging;
    if (staging && q.bytes >= kPinDirect) {
      hipPointerAttribute_t a;
      if (hipPointerGetAttributes(&a, q.host) != hipSuccess) (void)hipGetLastError();
      else q.direct = a.type != hipMemoryTypeUnregistered;
    }
    any_staged |= !q.direct;
  }
  return any_staged;
}

hipError_t copy_in(wl_ctx* ctx, void* d_base, Piece* pieces, int n) {
  hipError_t e = hipSuccess;
  if (mark_direct(ctx, pieces, n) && ctx->pin_busy) {
    // copies of an earlier call that failed later on
    e = hipStreamSynchronize(ctx->stream);
    if (e == hipSuccess) ctx->pin_busy = false;
  }
  // halves are filled in turn; pieces that lie side by side on the device and
  // fit a half together travel in one copy
  int half = 0;
  bool used[2] = {false, false};
  size_t fill = 0, start = 0;  // staged bytes of the half, their device offset
  auto flush = [&](bool last) {
    if (fill == 0) return hipSuccess;
    hipError_t r = hipMemcpyAsync((char*)d_base + start, ctx->h_pin + half * kPinHalf, fill,
                                  hipMemcpyHostToDevice, ctx->stream);
    ctx->pin_busy = true;
    if (last) return r;
    if (r == hipSuccess) r = hipEventRecord(ctx->pin_ev[half], ctx->stream);
    used[half] = true;
    half ^= 1;
    if (r == hipSuccess && used[half]) r = hipEventSynchronize(ctx->pin_ev[half]);
    fill = 0;
    return r;
  };
  for (int i = 0; i < n && e == hipSuccess; ++i) {
    const Piece& q = pieces[i];
    if (q.direct) {
      e = hipMemcpyAsync((char*)d_base + q.off, q.host, q.bytes, hipMemcpyHostToDevice,
                         ctx->stream);
      continue;
    }
    size_t done = 0;
    while (done < q.bytes && e == hipSuccess) {
      const size_t off = q.off + done;
      if (fill > 0 && (off != start + fill || fill == kPinHalf)) e = flush(false);
      if (e != hipSuccess) break;
      if (fill == 0) start = off;
      const size_t left = q.bytes - done, room = kPinHalf - fill;
      const size_t take = left < room ? left : room;
      memcpy(ctx->h_pin + half * kPinHalf + fill, (const char*)q.host + done, take);
      fill += take;
      done += take;
    }
  }
  if (e == hipSuccess) e = flush(true);
  if (!ctx->h_pin) {  // pageable arrays: the caller may reuse them now
    const hipError_t w = hipStreamSynchronize(ctx->stream);
    if (e == hipSuccess) e = w;
  }
  return e;
}

// The staged pieces of a copy_out as chunks of at most a half, from one piece's
// start or the last chunk's end: pieces whose gap is small share a chunk.
namespace {
struct Chunk {
  size_t a, b;  // device offsets
  bool none() const { return a == b; }
};
struct Chunks {
  const Piece* pieces;
  int n;
  int at = 0;       // the next piece,
  size_t done = 0;  // its bytes in earlier chunks
  static bool skip(const Piece& q) { return !q.host || !q.bytes || q.direct; }
  Chunk next() {
    Chunk c{0, 0};
    for (; at < n; ++at, done = 0) {
      const Piece& q = pieces[at];
      if (skip(q)) continue;
      const size_t from = q.off + done;
      if (c.a == c.b) c.a = c.b = from;
      const size_t room = c.a + kPinHalf;
      if (from > c.b + kPinGap || from >= room) break;
      const size_t left = q.bytes - done, fit = room - from;
      c.b = from + (left < fit ? left : fit);
      if (left > fit) {
        done += fit;
        break;
      }
    }
    return c;
  }
};
}  // namespace

hipError_t copy_out(wl_ctx* ctx, const void* d_base, Piece* pieces, int n) {
  hipError_t e = hipSuccess;
  const bool staged = mark_direct(ctx, pieces, n);
  for (int i = 0; i < n && e == hipSuccess; ++i)
    if (pieces[i].direct)
      e = hipMemcpyAsync(pieces[i].host, (const char*)d_base + pieces[i].off, pieces[i].bytes,
                         hipMemcpyDeviceToHost, ctx->stream);
  if (staged && e == hipSuccess) {
    // (copy_in's copies are ahead on the same stream: their half may be reused)
    ctx->pin_busy = true;
    // A chunk into its half; its event at once (recorded when it is waited for,
    // it is 15 us late).
    auto ask = [&](const Chunk& c, int half, bool event) {
      hipError_t r = hipMemcpyAsync(ctx->h_pin + half * kPinHalf, (const char*)d_base + c.a,
                                    c.b - c.a, hipMemcpyDeviceToHost, ctx->stream);
      if (r == hipSuccess && event) r = hipEventRecord(ctx->pin_ev[half], ctx->stream);
      return r;
    };
    Chunks rest{pieces, n};
    Chunk c = rest.next(), more = rest.next();
    // A lone chunk of more than 16 KiB is waited for with the stream: such a copy
    // runs on a DMA engine, whose event comes 7 us after it (an 18 KiB result 77.1
    // us, with the stream 70.1); a smaller one runs as a kernel, and the stream's
    // wait is then late by up to 25 us (0.2 KiB of 256 x 512 loops 66.6 us, with
    // the event 40.6; 13.5 KiB 63.6 both).
    const bool by_stream = more.none() && c.b - c.a > kPinEvent;
    e = ask(c, 0, !by_stream);
    int first = 0;  // pieces before it are complete
    for (int half = 0; !c.none() && e == hipSuccess; half ^= 1) {
      const Chunk after = rest.next();
      if (!more.none()) e = ask(more, half ^ 1, true);
      if (e == hipSuccess)
        e = by_stream ? hipStreamSynchronize(ctx->stream)
                      : hipEventSynchronize(ctx->pin_ev[half]);
      if (e != hipSuccess) break;
      for (int i = first; i < n; ++i) {
        const Piece& q = pieces[i];
        if (q.off >= c.b) break;
        if (q.off + q.bytes <= c.b && i == first) ++first;
        if (Chunks::skip(q) || q.off + q.bytes <= c.a) continue;
        const size_t from = q.off > c.a ? q.off : c.a;
        const size_t to = q.off + q.bytes < c.b ? q.off + q.bytes : c.b;
        memcpy((char*)q.host + (from - q.off), ctx->h_pin + half * kPinHalf + (from - c.a),
               to - from);
      }
      c = more;
      more = after;
    }
  } else {
    const hipError_t w = hipStreamSynchronize(ctx->stream);
    if (e == hipSuccess) e = w;
  }
  if (e == hipSuccess) ctx->pin_busy = false;
  return e;
}

// Device block of an ensemble: a kept one that fits without wasting more than
// a quarter of it, or a new allocation.  (hipMalloc and hipFree of a GB take
// 1 ms here and, after some hundred GB of them, 20 to 40: 16384 x 4096 points
// generated, evaluated and freed again and again took 8 to 45 ms, 3.4 with the
// block kept.)
constexpr size_t kEnsCacheBytes = (size_t)8 << 30;
static void* ens_block(wl_ctx* ctx, size_t bytes, size_t* got) {
  {
    std::lock_guard<std::mutex> lock(ctx->cache_mu);
    auto best = ctx->ens_cache.end();  // the smallest that fits
    for (auto b = ctx->ens_cache.begin(); b != ctx->ens_cache.end(); ++b)
      if (b->second >= bytes && b->second - bytes <= b->second / 4 &&
          (best == ctx->ens_cache.end() || b->second < best->second))
        best = b;
    if (best != ctx->ens_cache.end()) {
      void* p = best->first;
      *got = best->second;
      ctx->ens_cache.erase(best);
      return p;
    }
  }
  void* p = nullptr;
  *got = bytes;
  return dev_malloc(ctx, &p, bytes) == hipSuccess ? p : nullptr;
}
// Takes back a block (the caller has waited for the device).  Kept are at most
// kEnsCacheBytes and, since other allocators of the process do not see them, a
// quarter of the memory that is free beside them (asked for, which takes 10 us,
// for larger blocks and whenever 64 MiB have come together since); the oldest
// go first.
static void ens_block_free(wl_ctx* ctx, void* p, size_t bytes) {
  if (!p) return;
  std::lock_guard<std::mutex> lock(ctx->cache_mu);
  constexpr size_t kAsk = (size_t)64 << 20;
  size_t held = bytes, most = kEnsCacheBytes;
  for (const auto& b : ctx->ens_cache) held += b.second;
  const bool ask = bytes > kAsk || held > ctx->cache_asked + kAsk;
  if (ask) {
    size_t avail = 0, total = 0;
    if (hipMemGetInfo(&avail, &total) != hipSuccess) {
      (void)hipGetLastError();
      avail = 0;
    }
    if (avail / 4 < most) most = avail / 4;
  }
  size_t drop = 0;  // kept blocks that go
  for (; drop < ctx->ens_cache.size() && held > most; ++drop) {
    held -= ctx->ens_cache[drop].second;
    (void)hipFree(ctx->ens_cache[drop].first);
  }
  ctx->ens_cache.erase(ctx->ens_cache.begin(), ctx->ens_cache.begin() + drop);
  if (ask) ctx->cache_asked = held <= most ? held : held - bytes;
  try {
    if (held <= most) {
      ctx->ens_cache.emplace_back(p, bytes);
      return;
    }
  } catch (const std::bad_alloc&) {
  }
  (void)hipFree(p);
}
// The arrays of an ensemble of the given shape, in one block.
static bool ens_alloc(wl_ctx* ctx, wl_ens* e) {
  const size_t npts = (size_t)(e->n_loops * e->n_ppl);
  auto up = [](size_t b) { return (b + 255) & ~(size_t)255; };
  const size_t x = up(npts * sizeof(float)), s = up(npts * sizeof(float4));
  e->block = ens_block(ctx, 2 * x + s + (size_t)e->n_loops * sizeof(float2), &e->block_bytes);
  if (!e->block) return false;
  char* p = (char*)e->block;
  e->d_seg = (float4*)p;
  e->d_x = (float*)(p + s);
  e->d_y = (float*)(p + s + x);
  e->d_norm = (float2*)(p + s + 2 * x);
  return true;
}

int check_field(wl_ctx* ctx, const wl_field* f, wl::FieldArgs* a) {
  if (!f) return fail(ctx, WL_EINVAL, "field is NULL");
  if (f->kind < WL_CONST || f->kind > WL_RATIONAL)
    return fail(ctx, WL_EINVAL, "unknown field kind %d", f->kind);
  if (f->reserved != 0) return fail(ctx, WL_EINVAL, "field.reserved must be 0");
  if (!isfinite(f->eB0)) return fail(ctx, WL_EINVAL, "field.eB0 not finite");
  const double lam = f->lambda;
  if (f->kind != WL_CONST && !(isfinite(lam) && lam > 0.0))
    return fail(ctx, WL_EINVAL, "field.lambda must be finite and > 0");
  const double l = (f->kind == WL_CONST) ? 1.0 : lam;
  const double log2e = 1.4426950408889634074;
  a->kind = f->kind;
  a->inv_lam_d = 1.0 / l;
  // constants that all segments share: one rounding each
  const long double ll = (long double)l * l, log2el = 1.44269504088896340736L;
  a->inv_lam2_d = (double)(1.0L / ll);
  a->exp2_scale_d = 0.0;
  a->rad2_d = (double)ll;
  a->inv_lam2 = (float)(1.0 / (l * l));
  a->lam2 = (float)(l * l);
  a->lam2_lo = (float)(l * l - (double)a->lam2);
  a->thr = 0.0f;
  double e2 = 0.0;
  switch (f->kind) {
    case WL_CONST:  // g = eB0/2, b = eB0
      a->cphi = 0.5 * f->eB0;
      a->cspin = f->eB0;
      break;
    case WL_SECH2:  // g = eB0 lam^2 ln2 qa, b = eB0 * 4 * E/(1+E)^2; the FP32
      // walks work in units scaled by gs = 2 log2(e)/lambda (qa is divided by
      // gs^2 and the cross product multiplied by it)
      a->cphi = (double)(f->eB0 * ll * 0.69314718055994530942L);
      a->cspin = 4.0 * f->eB0;
      a->exp2_scale_d = (double)(2.0L * log2el / l);
      a->rad2_d = (double)(0.25L * ll);  // u < 1/2
      break;
    case WL_GAUSS:  // g = (eB0 lam^2/2) (1-E)/rho^2, b = eB0 E
      e2 = -log2e / (l * l);
      a->cphi = (double)(0.5L * f->eB0 * ll);
      a->cspin = f->eB0;
      a->thr = (float)(0.25 * l * l);  // v < 1/4
      a->exp2_scale_d = (double)(log2el / ll);
      a->rad2_d = (double)(0.5L * ll);  // v < 1/2
      break;
    case WL_RATIONAL:  // g = (eB0 lam^2/2) r, b = eB0 lam^4 r^2
      a->cphi = (double)(0.5L * f->eB0 * ll);
      a->cspin = f->eB0 * l * l * l * l;
      break;
  }
  a->exp2_scale = (float)e2;
  a->exp2_scale_lo = (float)(e2 - (double)a->exp2_scale);
  return WL_OK;
}

int check_grid(wl_ctx* ctx, const double* rho, int32_t n_rho, const double* T,
               int32_t n_T) {
  if (n_rho < 0 || n_T < 0) return fail(ctx, WL_EINVAL, "negative grid size");
  if ((int64_t)n_rho * n_T > (int64_t)INT32_MAX)
    return fail(ctx, WL_EINVAL, "grid has more than 2^31-1 points");
  if ((n_rho > 0 && !rho) || (n_T > 0 && !T))
    return fail(ctx, WL_EINVAL, "grid pointer is NULL");
  for (int32_t j = 0; j < n_rho; ++j)
    if (!(isfinite(rho[j]) && rho[j] >= 0.0))
      return fail(ctx, WL_EINVAL, "rho[%d] must be finite and >= 0", j);
  for (int32_t k = 0; k < n_T; ++k)
    if (!(isfinite(T[k]) && T[k] > 0.0))
      return fail(ctx, WL_EINVAL, "T[%d] must be finite and > 0", k);
  return WL_OK;
}

int check_common(wl_ctx* ctx, const wl_ens* ens, int32_t spin, int32_t precision) {
  if (!ens) return fail(ctx, WL_EINVAL, "ensemble is NULL");
  if (ens->ctx != ctx) return fail(ctx, WL_EINVAL, "ensemble belongs to another context");
  if (spin != 0 && spin != 1) return fail(ctx, WL_EINVAL, "spin must be 0 or 1");
  if (precision < WL_FP32C || precision > WL_FP32K)
    return fail(ctx, WL_EINVAL, "unknown precision %d", precision);
  return WL_OK;
}

int check_not_study(wl_ctx* ctx, int32_t precision) {
  if (precision == WL_FP32K)
    return fail(ctx, WL_EINVAL,
                "WL_FP32K is a precision-study mode of wl_average and the per-loop calls only");
  return WL_OK;
}

wl::Sched make_sched(const wl_ctx* ctx, const wl_ens* e, int32_t n_pts) {
  wl::Sched s{};
  s.loops_per_group = e->n_loops / e->n_groups;
  s.n_chunks = (n_pts + wl::kWave - 1) / wl::kWave;
  // Split each group's loops into sub-ranges until there are wavefronts for
  // ~16 rounds of 8 per SIMD (4 SIMDs per CU): the items have equal cost,
  // and with many short workgroups the hardware dispatcher keeps every SIMD
  // busy to the end (with one or two rounds, the last one runs part-empty).
  // At most 64 sub-ranges, of at least 8 loops each; the partial sums cost
  // G n_sub n_pts doubles.  The rule depends only on the request and the
  // ensemble, so a request is decomposed the same way alone and in a batch.
  const int64_t target = (int64_t)ctx->num_cu * 4 * 8 * 16;
  const int64_t base = (int64_t)e->n_groups * s.n_chunks;
  int64_t n_sub = (target + base - 1) / base;
  if (n_sub > 64) n_sub = 64;
  if (n_sub > s.loops_per_group / 8) n_sub = s.loops_per_group / 8;
  if (n_sub < 1) n_sub = 1;
  s.loops_per_sub = (s.loops_per_group + n_sub - 1) / n_sub;
  // no empty sub-ranges
  n_sub = (s.loops_per_group + s.loops_per_sub - 1) / s.loops_per_sub;
  s.n_sub = (int32_t)n_sub;
  s.n_items = base * n_sub;
  s.n_wg = 0;  // set by the launcher (workgroup size depends on precision)
  s.n_xcd = 8;  // MI355X: 8 XCDs; workgroups are dealt round-robin
  s.split = 1;  // set by the launcher
  return s;
}

// Waves to an item of a wide batch (a power of two, one per loop): the
// workgroup's 8 waves hold 8 / team items, a bundle.
static int32_t wide_team(int64_t loops_per_sub) {
  return loops_per_sub >= 8 ? 8 : loops_per_sub >= 4 ? 4 : loops_per_sub >= 2 ? 2 : 1;
}

static int64_t bundles(const wl::Sched& s) {
  const int32_t per = kSplitWaves / wide_team(s.loops_per_sub);
  return (s.n_items + per - 1) / per;
}

ReqPlan plan_request(const wl_ctx* ctx, const wl_ens* ens, const wl_request& q) {
  ReqPlan p;
  p.n_pts = q.n_rho * q.n_T;
  if (p.n_pts == 0) return p;
  p.s = make_sched(ctx, ens, p.n_pts);
  const int64_t G = ens->n_groups;
  p.in_bytes = sizeof(ReqDesc) + 8 * (size_t)(q.n_rho + q.n_T);
  // group sums, mean, err, scale, fp_err, escalation flags (one byte per
  // point, padded to 8 with the other requests'), the item scale and
  // rounding accumulators, the item partial sums of w when split, the
  // compacted list of flagged points with its count, and the request's
  // entry of the FP64 recomputation table (64 bytes are set aside for it, 64
  // more and 32 for the table's last entry and the alignments, also for a
  // batch of one)
  const size_t part = (size_t)G * p.s.n_sub * p.n_pts;
  p.res_bytes = 8 * ((size_t)G * p.n_pts + 4 * (size_t)p.n_pts + 2 * part +
                     (p.s.n_sub > 1 ? part : 0)) +
                (size_t)p.n_pts + 8 + 4 * (size_t)p.n_pts + 8 + 2 * 8 * 8 + 32;
  return p;
}

bool build_batch(const wl_ens* ens, const wl_request* const* reqs, const FieldArgs* fa,
                 const ReqPlan* plans, int32_t n, void* h_in, size_t cap_in, void* d_in,
                 void* d_res, size_t cap_res, BatchLayout* lay) {
  const int64_t G = ens->n_groups;
  *lay = BatchLayout();
  int64_t grid_n = 0;
  // Wide (k_batch_wide) or narrow: an item per wave ends in a part-empty round
  // of whole items; bundles cost a few percent, more where a last round of
  // loops leaves waves of a team idle, and in FP64, whose bundle kernel holds
  // half as many waves.  Time of the wide form over the narrow one's, by the
  // rounds of the chip's wave slots (sech^2 and Gaussian spinor; in brackets
  // constant and rational):
  //   rows of 8, FP32C  0.06: 0.35  0.5: 0.89  2: 0.95  4: 0.98  8: 1.02 (1.04)
  //   rows of 1         0.25: 0.99  2: 1.08 (0.82)  8: 1.02 (0.83)
  //   rows of 13        0.06: 0.48  0.5: 0.93  2: 0.96 (0.91)
  //   rows of 9         0.12: 0.78  0.23: 0.89  0.35: 1.07  0.47: 0.98 (1.12)  3.8: 1.14
  //   rows of 6         0.17: 0.91  0.33: 0.97  0.5: 1.21  2: 1.13  4: 1.15
  //   rows of 8, FP64   0.06: 0.30  0.25: 0.80 (0.83)  0.5: 1.02 (1.61)  2: 1.05 (1.94)
  //   rows of 9, FP64   0.03: 0.24  0.12: 0.72 (0.61)  0.23: 1.10 (1.17)  1.9: 1.37
  //   rows of 6, FP64   0.17: 0.79 (0.83)  0.33: 1.14 (1.19)
  // Plain FP32 lies within 0.05 of FP32C.
  int64_t items_n = 0, turns = 0, loops = 0;
  for (int32_t i = 0; i < n; ++i) {
    const int64_t lps = plans[i].s.loops_per_sub, team = wide_team(lps);
    items_n += plans[i].s.n_items;
    turns += plans[i].s.n_items * ((lps + team - 1) / team * team);
    loops += plans[i].s.n_items * lps;
  }
  const int64_t round = 32 * (int64_t)ens->ctx->num_cu;
  const int64_t idle = 100 * turns / loops - 100;  // waves' turns without a loop, percent
  const int64_t limit = reqs[0]->precision == WL_FP64 ? (idle <= 25 ? 30 : 20)
                        : idle <= 15                  ? 1000
                        : idle <= 25                  ? 300
                                                      : 45;  // percent of a round
  const bool wide = 100 * items_n < limit * round;
  for (int32_t i = 0; i < n; ++i) {
    lay->items += wide ? bundles(plans[i].s) : plans[i].s.n_items;
    lay->sums_n += G * plans[i].n_pts;
    lay->pts_n += plans[i].n_pts;
    lay->acc_n += G * plans[i].s.n_sub * plans[i].n_pts;
    if (plans[i].s.n_sub > 1) lay->part_n += G * plans[i].s.n_sub * plans[i].n_pts;
    grid_n += reqs[i]->n_rho + reqs[i]->n_T;
  }
  const size_t grids_off = kBatchDescOffset + (((size_t)n * sizeof(ReqDesc) + 255) & ~(size_t)255);
  lay->in_bytes = grids_off + 8 * (size_t)grid_n;
  lay->head_bytes = 8 * (size_t)(lay->sums_n + 4 * lay->pts_n) +
                    (((size_t)lay->pts_n + 7) & ~(size_t)7);
  lay->res_bytes = lay->head_bytes + 8 * (size_t)(2 * lay->acc_n + lay->part_n) +
                   4 * (size_t)(lay->pts_n + n) + 8 + 8 * 8 * ((size_t)n + 1);
  if (lay->in_bytes > cap_in || lay->res_bytes > cap_res) return false;
  char* hb = (char*)h_in;
  BatchHeader* hdr = (BatchHeader*)hb;
  hdr->n_reqs = n;
  hdr->wide = wide ? 1 : 0;
  hdr->total_items = lay->items;
  hdr->total_sums = lay->sums_n;
  hdr->total_pts = lay->pts_n;
  ReqDesc* desc = (ReqDesc*)(hb + kBatchDescOffset);
  double* h_grid = (double*)(hb + grids_off);
  const double* d_grid = (const double*)((const char*)d_in + grids_off);
  // [sums | mean | err | scale | fp_err | flags (bytes) | acc a | acc v | partials]
  double* d_sums = (double*)d_res;
  double* d_scale = d_sums + lay->sums_n + 2 * lay->pts_n;
  double* d_fperr = d_scale + lay->pts_n;
  uint8_t* d_flags = (uint8_t*)(d_fperr + lay->pts_n);
  double* d_acc_a = (double*)((char*)d_res + lay->head_bytes);
  double* d_acc_v = d_acc_a + lay->acc_n;
  double* d_part = d_acc_v + lay->acc_n;
  int32_t* d_list = (int32_t*)(d_part + lay->part_n);  // [pts_n] lists, then [n] counts
  int32_t* d_count = d_list + lay->pts_n;
  int64_t* d_esc_begin = (int64_t*)(((uintptr_t)(d_count + n) + 7) & ~(uintptr_t)7);
  hdr->esc_begin = d_esc_begin;
  int64_t items = 0, sums = 0, pts = 0, part = 0, acc = 0, go = 0;
  int32_t tiles = 0;
  for (int32_t i = 0; i < n; ++i) {
    const wl_request& q = *reqs[i];
    const ReqPlan& pl = plans[i];
    ReqDesc e{};
    e.f = fa[i];
    e.rho = d_grid + go;
    e.T = d_grid + go + q.n_rho;
    memcpy(h_grid + go, q.rho, q.n_rho * sizeof(double));
    memcpy(h_grid + go + q.n_rho, q.T, q.n_T * sizeof(double));
    go += q.n_rho + q.n_T;
    e.out = pl.s.n_sub > 1 ? d_part + part : d_sums + sums;
    e.out_a = d_acc_a + acc;
    e.out_v = d_acc_v + acc;
    e.scale = d_scale + pts;
    e.fp_err = d_fperr + pts;
    e.flags = d_flags + pts;
    e.list = d_list + pts;
    e.count = d_count + i;
    e.item_begin = items;
    e.loops_per_sub = pl.s.loops_per_sub;
    e.sums_begin = sums;
    e.pts_begin = pts;
    e.n_sub = pl.s.n_sub;
    e.n_chunks = pl.s.n_chunks;
    e.n_T = q.n_T;
    e.n_pts = pl.n_pts;
    e.spin = (int16_t)q.spin;
    e.team = (int16_t)wide_team(pl.s.loops_per_sub);
    e.tile_begin = tiles;
    tiles += (pl.n_pts + kFinishPts - 1) / kFinishPts;
    desc[i] = e;
    lay->sums_begin.push_back(sums);
    lay->pts_begin.push_back(pts);
    items += wide ? bundles(pl.s) : pl.s.n_items;
    sums += G * pl.n_pts;
    pts += pl.n_pts;
    acc += G * pl.s.n_sub * pl.n_pts;
    if (pl.s.n_sub > 1) part += G * pl.s.n_sub * pl.n_pts;
  }
  return true;
}

void scatter_results(const wl_request& q, const BatchLayout& lay, int32_t i,
                     const double* h_res, int64_t G) {
  const int64_t n_pts = (int64_t)q.n_rho * q.n_T;
  const double* per_pt = h_res + lay.sums_n + lay.pts_begin[i];
  if (q.group_sums)
    memcpy(q.group_sums, h_res + lay.sums_begin[i], G * n_pts * sizeof(double));
  if (q.mean) memcpy(q.mean, per_pt, n_pts * sizeof(double));
  if (q.err) memcpy(q.err, per_pt + lay.pts_n, n_pts * sizeof(double));
  if (q.scale) memcpy(q.scale, per_pt + 2 * lay.pts_n, n_pts * sizeof(double));
  if (q.fp_err) memcpy(q.fp_err, per_pt + 3 * lay.pts_n, n_pts * sizeof(double));
  if (q.escalated)
    memcpy(q.escalated,
           (const uint8_t*)(h_res + lay.sums_n + 4 * lay.pts_n) + lay.pts_begin[i], n_pts);
}

// Event pair for the next timed launch (created on first use).
hipError_t next_events(wl_ctx* ctx, hipEvent_t* a, hipEvent_t* b) {
  if (ctx->n_timed == ctx->events.size()) {
    hipEvent_t e0, e1;
    hipError_t e = hipEventCreate(&e0);
    if (e != hipSuccess) return e;
    e = hipEventCreate(&e1);
    if (e != hipSuccess) {
      (void)hipEventDestroy(e0);
      return e;
    }
    ctx->events.emplace_back(e0, e1);
  }
  *a = ctx->events[ctx->n_timed].first;
  *b = ctx->events[ctx->n_timed].second;
  return hipSuccess;
}

// FP64 segment array of the ensemble, built on first use (on `stream`, which
// is then synchronized, so the array is complete for every stream once the
// pointer is published).  One lock serialises the builders of all ensembles:
// a server thread and a caller of the same ensemble may both ask.
hipError_t ensure_seg64(const wl_ens* ens, hipStream_t stream) {
  static std::mutex mu;
  std::lock_guard<std::mutex> lock(mu);
  if (ens->d_seg64) return hipSuccess;
  const int64_t nseg = ens->n_loops * ens->n_ppl;
  double4* d = nullptr;
  hipError_t e = dev_malloc(ens->ctx, (void**)&d, nseg * sizeof(double4));
  if (e != hipSuccess) return hipErrorOutOfMemory;
  e = launch_prep64(ens->d_x, ens->d_y, ens->n_loops, ens->n_ppl, d, stream);
  if (e == hipSuccess) e = hipStreamSynchronize(stream);
  if (e != hipSuccess) {
    (void)hipStreamSynchronize(stream);
    (void)hipFree(d);
    return e;
  }
  ens->d_seg64 = d;
  return hipSuccess;
}


// Scratch of the allocation-free evaluation (wl_average_async_noalloc):
// one copy per device, reserved when the code object is loaded on it and
// held until the process ends.  In host code `scratch` names a host-side
// stand-in, never the device memory: the device address is obtained once
// per device with hipGetSymbolAddress (noalloc_scratch_ptr) and only that
// address is handed to kernels.
static __device__ __align__(256) unsigned char scratch[WL_NOALLOC_SCRATCH_BYTES];

// Device address of `scratch` on the current device, looked up on the
// first call for each device and kept.
static hipError_t noalloc_scratch_ptr(int device, void** out) {
  constexpr int kMaxDev = 64;
  static std::mutex mu;
  static void* ptr[kMaxDev] = {};
  static hipError_t status[kMaxDev] = {};
  static bool done[kMaxDev] = {};
  *out = nullptr;
  if (device < 0 || device >= kMaxDev) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!done[device]) {
    void* p = nullptr;
    status[device] = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (status[device] != hipSuccess) {
      (void)hipGetLastError();
      p = nullptr;
    }
    ptr[device] = p;
    done[device] = true;
  }
  *out = ptr[device];
  return status[device];
}

}  // namespace wl

using namespace wl;

extern "C" {

const char* wl_version(void) { return "wl 0.1 (gfx950)"; }

const char* wl_strerror(int code) {
  switch (code) {
    case WL_OK: return "ok";
    case WL_EINVAL: return "invalid argument";
    case WL_ENOMEM: return "out of memory";
    case WL_EHIP: return "HIP runtime error";
    case WL_ENODEV: return "no usable gfx950 device";
  }
  return "unknown error code";
}

const char* wl_last_error(const wl_ctx* ctx) { return ctx ? ctx->err.c_str() : ""; }

int wl_create(wl_ctx** out, int device, void* hip_stream) {
  if (!out) return WL_EINVAL;
  *out = nullptr;
  int n = 0;
  if (hipGetDeviceCount(&n) != hipSuccess || n <= 0) {
    (void)hipGetLastError();
    return WL_ENODEV;
  }
  if (device < 0 || device >= n) return WL_ENODEV;
  hipDeviceProp_t prop;
  if (hipGetDeviceProperties(&prop, device) != hipSuccess) return WL_ENODEV;
  if (strncmp(prop.gcnArchName, "gfx950", 6) != 0) return WL_ENODEV;
  wl_ctx* c = new (std::nothrow) wl_ctx();
  if (!c) return WL_ENOMEM;
  c->device = device;
  c->stream = (hipStream_t)hip_stream;
  c->num_cu = prop.multiProcessorCount;
  DeviceGuard g(device);
  if (g.status != hipSuccess || dev_malloc(c, (void**)&c->d_flag, sizeof(int)) != hipSuccess ||
      dev_malloc(c, (void**)&c->d_counter, kBatchCounters * sizeof(unsigned int)) !=
          hipSuccess) {
    wl_destroy(c);
    return WL_ENOMEM;
  }
  try {
    std::lock_guard<std::mutex> lock(contexts().mu);
    contexts().live.push_back(c);
  } catch (const std::bad_alloc&) {
    wl_destroy(c);
    return WL_ENOMEM;
  }
  // with the context's device current: the allocation-free entry point's
  // scratch address on this device (a failure is reported by that entry
  // point only)
  c->noalloc_status = noalloc_scratch_ptr(device, &c->d_noalloc);
  *out = c;
  return WL_OK;
}

int wl_destroy(wl_ctx* ctx) {
  if (!ctx) return WL_OK;
  {
    Contexts& all = contexts();
    std::lock_guard<std::mutex> lock(all.mu);
    for (size_t i = 0; i < all.live.size(); ++i)
      if (all.live[i] == ctx) {
        all.live.erase(all.live.begin() + i);
        break;
      }
  }
  {
    DeviceGuard g(ctx->device);
    if (ctx->stream) (void)hipStreamSynchronize(ctx->stream);
    else (void)hipDeviceSynchronize();
    if (ctx->d_grid) (void)hipFree(ctx->d_grid);
    if (ctx->d_out) (void)hipFree(ctx->d_out);
    if (ctx->d_partial) (void)hipFree(ctx->d_partial);
    for (void* p : ctx->d_terms)
      if (p) (void)hipFree(p);
    if (ctx->d_flag) (void)hipFree(ctx->d_flag);
    if (ctx->d_counter) (void)hipFree(ctx->d_counter);
    if (ctx->d_batch) (void)hipFree(ctx->d_batch);
    if (ctx->d_work) (void)hipFree(ctx->d_work);
    for (const auto& b : ctx->ens_cache) (void)hipFree(b.first);
    if (ctx->h_pin) (void)hipHostFree(ctx->h_pin);
    for (hipEvent_t ev : ctx->pin_ev)
      if (ev) (void)hipEventDestroy(ev);
    for (auto& pr : ctx->events) {
      (void)hipEventDestroy(pr.first);
      (void)hipEventDestroy(pr.second);
    }
  }
  delete ctx;
  return WL_OK;
}

int wl_ensemble_upload(wl_ctx* ctx, const float* y_x, const float* y_y,
                       int64_t n_loops, int32_t n_ppl, int32_t n_groups,
                       int32_t flags, wl_ens** out) {
  if (!ctx) return WL_EINVAL;
  ctx->err.clear();
  if (!out) return fail(ctx, WL_EINVAL, "out is NULL");
  *out = nullptr;
  if (!y_x || !y_y) return fail(ctx, WL_EINVAL, "coordinate pointer is NULL");
  if (n_loops < 1) return fail(ctx, WL_EINVAL, "n_loops must be >= 1");
  if (n_ppl < 2) return fail(ctx, WL_EINVAL, "n_ppl must be >= 2");
  if (n_groups < 1 || n_loops % n_groups != 0)
    return fail(ctx, WL_EINVAL, "n_groups must be >= 1 and divide n_loops");
  if (flags != WL_HOST_PTR && flags != WL_DEVICE_PTR)
    return fail(ctx, WL_EINVAL, "unknown flags %d", flags);
  if (n_loops > ((int64_t)1 << 40) / n_ppl)
    return fail(ctx, WL_EINVAL, "ensemble too large");
  DeviceGuard g(ctx->device);
  if (g.status != hipSuccess) return hip_fail(ctx, g.status, "hipSetDevice");
  const int64_t npts = n_loops * n_ppl;
  wl_ens* e = new (std::nothrow) wl_ens();
  if (!e) return fail(ctx, WL_ENOMEM, "host allocation failed");
  e->ctx = ctx;
  e->n_loops = n_loops;
  e->n_ppl = n_ppl;
  e->n_groups = n_groups;
  auto cleanup = [&](int code) {
    if (e->block) {
      (void)hipStreamSynchronize(ctx->stream);
      (void)hipFree(e->block);
    }
    delete e;
    return code;
  };
  if (!ens_alloc(ctx, e))
    return cleanup(fail(ctx, WL_ENOMEM, "device allocation of %lld points failed",
                        (long long)npts));
  const hipMemcpyKind kind =
      flags == WL_DEVICE_PTR ? hipMemcpyDeviceToDevice : hipMemcpyHostToDevice;
  hipError_t err = hipMemcpyAsync(e->d_x, y_x, npts * sizeof(float), kind, ctx->stream);
  if (err == hipSuccess)
    err = hipMemcpyAsync(e->d_y, y_y, npts * sizeof(float), kind, ctx->stream);
  if (err == hipSuccess) err = hipMemsetAsync(ctx->d_flag, 0, sizeof(int), ctx->stream);
  if (err == hipSuccess)
    err = wl::launch_prep(e->d_x, e->d_y, n_loops, n_ppl, e->d_seg, e->d_norm, ctx->d_flag,
                           ctx->stream);
  int bad = 0;
  if (err == hipSuccess)
    err = hipMemcpyAsync(&bad, ctx->d_flag, sizeof(int), hipMemcpyDeviceToHost, ctx->stream);
  if (err == hipSuccess) err = hipStreamSynchronize(ctx->stream);
  if (err != hipSuccess) return cleanup(hip_fail(ctx, err, "ensemble upload"));
  if (bad) return cleanup(fail(ctx, WL_EINVAL, "non-finite loop coordinate"));
  *out = e;
  return WL_OK;
}

int wl_ensemble_generate(wl_ctx* ctx, uint64_t seed, int64_t first_loop, int64_t n_loops,
                         int32_t n_ppl, int32_t n_groups, wl_ens** out) {
  if (!ctx) return WL_EINVAL;
  ctx->err.clear();
  if (!out) return fail(ctx, WL_EINVAL, "out is NULL");
  *out = nullptr;
  if (n_loops < 1) return fail(ctx, WL_EINVAL, "n_loops must be >= 1");
  if (first_loop < 0) return fail(ctx, WL_EINVAL, "first_loop must be >= 0");
  if (n_ppl < 2 || n_ppl > 8192 || (n_ppl & (n_ppl - 1)))
    return fail(ctx, WL_EINVAL, "d-loops need n_ppl a power of two in [2, 8192]");
  if (n_groups < 1 || n_loops % n_groups != 0)
    return fail(ctx, WL_EINVAL, "n_groups must be >= 1 and divide n_loops");
  if (n_loops > ((int64_t)1 << 40) / n_ppl) return fail(ctx, WL_EINVAL, "ensemble too large");
  DeviceGuard g(ctx->device);
  if (g.status != hipSuccess) return hip_fail(ctx, g.status, "hipSetDevice");
  const int64_t npts = n_loops * n_ppl;
  wl_ens* e = new (std::nothrow) wl_ens();
  if (!e) return fail(ctx, WL_ENOMEM, "host allocation failed");
  e->ctx = ctx;
  e->n_loops = n_loops;
  e->n_ppl = n_ppl;
  e->n_groups = n_groups;
  auto cleanup = [&](int code) {
    if (e->block) {
      (void)hipStreamSynchronize(ctx->stream);
      (void)hipFree(e->block);
    }
    delete e;
    return code;
  };
  if (!ens_alloc(ctx, e))
    return cleanup(fail(ctx, WL_ENOMEM, "device allocation of %lld points failed",
                        (long long)npts));
  hipEvent_t ev0 = nullptr, ev1 = nullptr;
  hipError_t err = hipSuccess;
  if (ctx->timing) {
    err = next_events(ctx, &ev0, &ev1);
    if (err == hipSuccess) err = hipEventRecord(ev0, ctx->stream);
  }
  if (err == hipSuccess)
    err = wl::launch_generate(seed, first_loop, n_loops, n_ppl, e->d_x, e->d_y, e->d_seg,
                              e->d_norm, ctx->stream);
  if (err == hipSuccess && ctx->timing) {
    err = hipEventRecord(ev1, ctx->stream);
    if (err == hipSuccess) ctx->n_timed++;
  }
  if (err == hipSuccess) err = hipStreamSynchronize(ctx->stream);
  if (err != hipSuccess) return cleanup(hip_fail(ctx, err, "ensemble generation"));
  *out = e;
  return WL_OK;
}

int wl_ensemble_download(const wl_ens* ens, float* y_x, float* y_y, int64_t loop0,
                         int64_t n_loops) {
  if (!ens) return WL_EINVAL;
  wl_ctx* ctx = ens->ctx;
  ctx->err.clear();
  if (loop0 < 0 || n_loops < 0 || loop0 + n_loops > ens->n_loops)
    return fail(ctx, WL_EINVAL, "loop range [%lld, %lld) outside the ensemble",
                (long long)loop0, (long long)(loop0 + n_loops));
  if (n_loops == 0) return WL_OK;
  DeviceGuard g(ctx->device);
  if (g.status != hipSuccess) return hip_fail(ctx, g.status, "hipSetDevice");
  const size_t off = (size_t)(loop0 * ens->n_ppl), cnt = (size_t)(n_loops * ens->n_ppl);
  hipError_t e = hipSuccess;
  if (y_x)
    e = hipMemcpyAsync(y_x, ens->d_x + off, cnt * sizeof(float), hipMemcpyDeviceToHost,
                       ctx->stream);
  if (e == hipSuccess && y_y)
    e = hipMemcpyAsync(y_y, ens->d_y + off, cnt * sizeof(float), hipMemcpyDeviceToHost,
                       ctx->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
  if (e != hipSuccess) return hip_fail(ctx, e, "wl_ensemble_download");
  return WL_OK;
}

int wl_ensemble_free(wl_ens* ens) {
  if (!ens) return WL_OK;
  DeviceGuard g(ens->ctx->device);
  // the points may be in use on any stream (a captured launch replayed on
  // another than the context's): what hipFree waits for itself, the next
  // ensemble in a kept block would not
  if (hipDeviceSynchronize() == hipSuccess) {
    ens_block_free(ens->ctx, ens->block, ens->block_bytes);
  } else {
    (void)hipGetLastError();
    if (ens->block) (void)hipFree(ens->block);
  }
  if (ens->d_sub) (void)hipFree(ens->d_sub);
  if (ens->d_seg64) (void)hipFree(ens->d_seg64);
  if (ens->d_sub64) (void)hipFree(ens->d_sub64);
  delete ens;
  return WL_OK;
}

int wl_ensemble_info(const wl_ens* ens, int64_t* n_loops, int32_t* n_ppl,
                     int32_t* n_groups) {
  if (!ens) return WL_EINVAL;
  if (n_loops) *n_loops = ens->n_loops;
  if (n_ppl) *n_ppl = ens->n_ppl;
  if (n_groups) *n_groups = ens->n_groups;
  return WL_OK;
}

int wl_set_timing(wl_ctx* ctx, int32_t enable) {
  if (!ctx) return WL_EINVAL;
  ctx->timing = enable != 0;
  ctx->n_timed = 0;
  return WL_OK;
}

static int elapsed(wl_ctx* ctx, size_t i, double* ms) {
  hipError_t e = hipEventSynchronize(ctx->events[i].second);
  float f = 0.0f;
  if (e == hipSuccess) e = hipEventElapsedTime(&f, ctx->events[i].first, ctx->events[i].second);
  if (e != hipSuccess) return hip_fail(ctx, e, "hipEventElapsedTime");
  *ms = f;
  return WL_OK;
}

int wl_last_kernel_ms(wl_ctx* ctx, double* ms) {
  if (!ctx || !ms) return WL_EINVAL;
  ctx->err.clear();
  if (ctx->n_timed == 0) return fail(ctx, WL_EINVAL, "no timed launch recorded");
  DeviceGuard g(ctx->device);
  return elapsed(ctx, ctx->n_timed - 1, ms);
}

int wl_kernel_ms_total(wl_ctx* ctx, double* total_ms, int64_t* count) {
  if (!ctx || !total_ms || !count) return WL_EINVAL;
  ctx->err.clear();
  if (ctx->n_timed == 0) return fail(ctx, WL_EINVAL, "no timed launch recorded");
  DeviceGuard g(ctx->device);
  double tot = 0.0;
  for (size_t i = 0; i < ctx->n_timed; ++i) {
    double ms;
    int rc = elapsed(ctx, i, &ms);
    if (rc) return rc;
    tot += ms;
  }
  *total_ms = tot;
  *count = (int64_t)ctx->n_timed;
  return WL_OK;
}


static int need_seg64(wl_ctx* ctx, const wl_ens* ens) {
  const hipError_t e = wl::ensure_seg64(ens, ctx->stream);
  if (e == hipErrorOutOfMemory)
    return fail(ctx, WL_ENOMEM, "device allocation of the FP64 segments (%lld bytes) failed",
                (long long)(ens->n_loops * ens->n_ppl * (int64_t)sizeof(double4)));
  if (e != hipSuccess) return hip_fail(ctx, e, "FP64 segments");
  return WL_OK;
}

// Device outputs of one evaluation (each may be NULL but sums).
struct DevOut {
  double* sums;   // [G][n_pts]
  double* mean;   // [n_pts]
  double* err;
  double* scale;
  double* fp_err;
  uint8_t* escalated;
};

// Scratch of one evaluation: the item partial sums of w (when a group's
// loops are split), of the scale and rounding accumulators, the FP64
// recomputation flags and the compacted list of flagged points with its
// count.
static size_t flag_bytes(int32_t n_pts) { return ((size_t)n_pts + 7) & ~(size_t)7; }
// The sub-range partial sums of w (when split), the scale and rounding
// accumulators, the scale of each mean (read by the FP64 recomputation,
// also when the caller does not ask for it), one flag byte and one list
// entry per grid point.
static size_t eval_scratch_bytes(const wl::Sched& s, int64_t n_groups, int32_t n_pts) {
  const size_t part = (size_t)n_groups * s.n_sub * n_pts;
  return 8 * part * (s.n_sub > 1 ? 3 : 2) + 8 * (size_t)n_pts + flag_bytes(n_pts) +
         4 * ((size_t)n_pts + 1);
}

// Waves to a loop (launch_walk), or 0: a wave per loop (launch_average), by
// the walks (loops x chunks) per SIMD.  Up to one walk, 8 waves: sech^2 spinor
// at 1003 points 111 -> 62 us, rational 53 -> 42, constant 34 -> 27; loops of
// under 256 points have too few blocks for 8, and below 128 (384 for the
// fields whose block costs little) the terms' pass costs more (130 points:
// constant 10.2 -> 12.9 us, sech^2 20.8 -> 17.4).  Beyond, only the fields with
// costly blocks gain, with 4 waves (rational 56 -> 65 us at 2 walks).  Rows
// of even rounds: up to 3 walks (sech^2 118 -> 85 us at 1.5, Gaussian 150 ->
// 119 at 3 and equal at 4 and 6), sech^2 loops from 768 points that several
// chunks read also beyond (8: 354 -> 320 us, 16: 656 -> 589; with one chunk
// 2.42 -> 2.51 ms).  Rows whose last round leaves k_average's waves idle gain
// most (9 loops: 5.4 walks 295 -> 178 us, 18: 638 -> 534, 42: 1614 -> 1508);
// at kWalkMost walks the terms take 38 MB, where this stops.  512 points are the
// shortest with a gain there (256: sech^2 124 -> 132 us at 12).
static int32_t walk_waves(const wl_ctx* ctx, const wl::Sched& s, int32_t kind, int32_t n_ppl) {
  const int64_t walks = s.n_items * s.loops_per_sub, simds = 4 * (int64_t)ctx->num_cu;
  const bool costly = kind == WL_SECH2 || kind == WL_GAUSS;
  if (walks <= simds) return n_ppl < (costly ? 128 : 384) ? 0 : n_ppl < 256 ? 4 : 8;
  if (!costly || n_ppl < 512) return 0;
  const bool uneven = 100 * ((s.loops_per_sub + 7) / 8 * 8) > 115 * s.loops_per_sub;
  const bool more = uneven || (kind == WL_SECH2 && n_ppl >= 768 && s.n_chunks > 1);
  return walks <= (more ? kWalkMost : kWalkFew) * simds ? 4 : 0;
}
static size_t walk_terms_bytes(const wl::Sched& s, int32_t n_pts) {
  return (size_t)(s.n_items / s.n_chunks) * s.loops_per_sub * 3 * n_pts * sizeof(double);
}
// The context's room for the loops' terms: two buffers, for the launches of up
// to kWalkFew and kWalkMost walks per SIMD, each allocated by the first call
// that needs it and never moved, so that no later call takes it from under a
// captured one.  NULL where it cannot be had (under capture, or out of memory).
static double* walk_terms(wl_ctx* ctx, const wl::Sched& s) {
  const int64_t simds = 4 * (int64_t)ctx->num_cu;
  const bool few = s.n_items * s.loops_per_sub <= kWalkFew * simds;
  void** p = &ctx->d_terms[few ? 0 : 1];
  if (!*p) {
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(ctx->stream, &st) != hipSuccess) (void)hipGetLastError();
    else if (st == hipStreamCaptureStatusNone) {
      const RelaxedCapture relaxed;
      // (not dev_malloc: the walk can do without, so kept blocks stay)
      if (hipMalloc(p, (size_t)(few ? kWalkFew : kWalkMost) * simds * kWave * 3 *
                           sizeof(double)) != hipSuccess) {
        *p = nullptr;
        (void)hipGetLastError();
      }
    }
  }
  return (double*)*p;
}

// Enqueue one evaluation; grid and outputs are device memory: the main
// kernel, then the group sums, statistics, scale and rounding estimate per
// point (and for WL_FP32C the FP64 recomputation of the flagged points).  With `noalloc` the call allocates nothing: the scratch
// is the static array (ctx->d_noalloc), the FP64 segment array must exist
// already, and no timing events are recorded.
static int average_device(wl_ctx* ctx, const wl_ens* ens, const wl::FieldArgs& fa,
                          const double* d_rho, int32_t n_rho, const double* d_T,
                          int32_t n_T, int32_t spin, int32_t precision, const DevOut& o,
                          bool noalloc = false) {
  const int32_t n_pts = n_rho * n_T;
  if (precision == WL_FP64) {
    if (noalloc) {
      if (!ens->d_seg64)
        return fail(ctx, WL_EINVAL,
                    "the ensemble's FP64 segment array does not exist yet (an FP64 "
                    "wl_average or wl_average_async derives it)");
    } else {
      int rc = need_seg64(ctx, ens);
      if (rc) return rc;
    }
  }
  wl::Sched s = make_sched(ctx, ens, n_pts);
  const size_t need = eval_scratch_bytes(s, ens->n_groups, n_pts);
  double* terms = nullptr;
  if (precision == WL_FP32C) {
    // without room for the loops' terms, the walk of a wave per loop
    s.walk = walk_waves(ctx, s, fa.kind, ens->n_ppl);
    const size_t off = (need + 7) & ~(size_t)7;
    if (s.walk && !noalloc)
      terms = walk_terms(ctx, s);
    else if (s.walk && off + walk_terms_bytes(s, n_pts) <= WL_NOALLOC_SCRATCH_BYTES)
      terms = (double*)((char*)ctx->d_noalloc + off);
    if (!terms) s.walk = 0;
  }
  void* buf;
  if (noalloc) {
    if (need > WL_NOALLOC_SCRATCH_BYTES)
      return fail(ctx, WL_EINVAL,
                  "the evaluation needs %zu bytes of scratch, above the %zu-byte array of "
                  "the allocation-free evaluation", need, (size_t)WL_NOALLOC_SCRATCH_BYTES);
    buf = ctx->d_noalloc;
  } else {
    int rc = ensure(ctx, &ctx->d_partial, &ctx->partial_bytes, need, "evaluation scratch");
    if (rc) return rc;
    buf = ctx->d_partial;
  }
  const size_t part = (size_t)ens->n_groups * s.n_sub * n_pts;
  double* p_w = s.n_sub > 1 ? (double*)buf : o.sums;
  double* p_a = (double*)buf + (s.n_sub > 1 ? part : 0);
  double* p_v = p_a + part;
  double* scale = o.scale ? o.scale : p_v + part;
  uint8_t* flags = (uint8_t*)(p_v + part + n_pts);
  int32_t* list = (int32_t*)(flags + flag_bytes(n_pts));
  hipError_t e = hipSuccess;
  hipEvent_t ev0 = nullptr, ev1 = nullptr;
  if (ctx->timing && !noalloc) {
    e = next_events(ctx, &ev0, &ev1);
    if (e == hipSuccess) e = hipEventRecord(ev0, ctx->stream);
  }
  if (e == hipSuccess)
    e = s.walk ? wl::launch_walk(spin, fa, ens->d_seg, ens->d_norm, ens->n_ppl, d_rho, d_T, n_T,
                                 n_pts, s, terms, p_w, p_a, p_v, ctx->stream)
               : wl::launch_average(precision, spin, fa, ens->d_seg, ens->d_seg64, ens->d_norm,
                                    ens->n_ppl, d_rho, d_T, n_T, n_pts, s, p_w, p_a, p_v,
                                    ctx->stream);
  if (e == hipSuccess && ctx->timing && !noalloc) {
    e = hipEventRecord(ev1, ctx->stream);
    if (e == hipSuccess) ctx->n_timed++;
  }
  if (e == hipSuccess)
    e = wl::launch_finish(precision, spin, fa, ens->d_x, ens->d_y, ens->n_ppl, d_rho, d_T, n_T,
                          n_pts, s, ens->n_groups, ens->n_loops, p_w, p_a, p_v, o.sums, o.mean,
                          o.err, scale, o.fp_err, flags, o.escalated, list, ctx->stream);
  if (e != hipSuccess) return hip_fail(ctx, e, "kernel launch");
  return WL_OK;
}

// Host grids to d_rho [n_rho], then [n_T] right behind it.
static hipError_t grids_in(wl_ctx* ctx, double* d_rho, const double* rho, int32_t n_rho,
                           const double* T, int32_t n_T) {
  const size_t rb = n_rho * sizeof(double);
  Piece p[] = {{(void*)rho, 0, rb}, {(void*)T, rb, n_T * sizeof(double)}};
  return copy_in(ctx, d_rho, p, 2);
}

static int average_impl(wl_ctx* ctx, const wl_ens* ens, const wl_field* field,
                        const double* rho, int32_t n_rho, const double* T, int32_t n_T,
                        int32_t spin, int32_t precision, int32_t flags, const wl_result* out,
                        bool noalloc) {
  if (!ctx) return WL_EINVAL;
  ctx->err.clear();
  if (!out) return fail(ctx, WL_EINVAL, "result is NULL");
  if (flags != WL_HOST_PTR && flags != WL_DEVICE_PTR)
    return fail(ctx, WL_EINVAL, "unknown flags %d", flags);
  int rc = check_common(ctx, ens, spin, precision);
  if (rc) return rc;
  wl::FieldArgs fa;
  if ((rc = check_field(ctx, field, &fa))) return rc;
  if (flags == WL_DEVICE_PTR) {
    if (n_rho < 0 || n_T < 0) return fail(ctx, WL_EINVAL, "negative grid size");
    if ((int64_t)n_rho * n_T > (int64_t)INT32_MAX)
      return fail(ctx, WL_EINVAL, "grid has more than 2^31-1 points");
    if ((int64_t)n_rho * n_T == 0) return WL_OK;
    if (!rho || !T || !out->group_sums)
      return fail(ctx, WL_EINVAL, "device pointer is NULL");
    if (noalloc && !ctx->d_noalloc)
      return hip_fail(ctx, ctx->noalloc_status, "address of the allocation-free scratch");
    DeviceGuard g(ctx->device);
    if (g.status != hipSuccess) return hip_fail(ctx, g.status, "hipSetDevice");
    const DevOut o{out->group_sums, out->mean, out->err, out->scale, out->fp_err,
                   out->escalated};
    return average_device(ctx, ens, fa, rho, n_rho, T, n_T, spin, precision, o, noalloc);
  }
  if ((rc = check_grid(ctx, rho, n_rho, T, n_T))) return rc;
  const int64_t n_pts = (int64_t)n_rho * n_T;
  if (n_pts == 0) return WL_OK;
  DeviceGuard g(ctx->device);
  if (g.status != hipSuccess) return hip_fail(ctx, g.status, "hipSetDevice");
  const size_t gbytes = (size_t)(n_rho + n_T) * sizeof(double);
  const size_t sums_n = (size_t)ens->n_groups * n_pts;
  // [group sums | mean | err | scale | fp_err | escalation flags]
  const size_t obytes = (sums_n + 4 * (size_t)n_pts) * sizeof(double) + (size_t)n_pts;
  if ((rc = ensure(ctx, &ctx->d_grid, &ctx->grid_bytes, gbytes, "grid"))) return rc;
  if ((rc = ensure(ctx, &ctx->d_out, &ctx->out_bytes, obytes, "results"))) return rc;
  double* d_rho = (double*)ctx->d_grid;
  double* d_T = d_rho + n_rho;
  DevOut o;
  o.sums = (double*)ctx->d_out;
  o.mean = o.sums + sums_n;
  o.err = o.mean + n_pts;
  o.scale = o.err + n_pts;
  o.fp_err = o.scale + n_pts;
  o.escalated = (uint8_t*)(o.fp_err + n_pts);
  hipError_t e = grids_in(ctx, d_rho, rho, n_rho, T, n_T);
  if (e != hipSuccess) return hip_fail(ctx, e, "grid upload");
  if ((rc = average_device(ctx, ens, fa, d_rho, n_rho, d_T, n_T, spin, precision, o)))
    return rc;
  auto off = [&](const void* p) { return (size_t)((const char*)p - (const char*)ctx->d_out); };
  const size_t pt = n_pts * sizeof(double);
  Piece pieces[] = {{out->group_sums, off(o.sums), sums_n * sizeof(double)},
                          {out->mean, off(o.mean), pt},
                          {out->err, off(o.err), pt},
                          {out->scale, off(o.scale), pt},
                          {out->fp_err, off(o.fp_err), pt},
                          {out->escalated, off(o.escalated), (size_t)n_pts}};
  e = copy_out(ctx, ctx->d_out, pieces, 6);
  if (e != hipSuccess) return hip_fail(ctx, e, "wl_average");
  return WL_OK;
}

int wl_average_ex(wl_ctx* ctx, const wl_ens* ens, const wl_field* field, const double* rho,
                  int32_t n_rho, const double* T, int32_t n_T, int32_t spin,
                  int32_t precision, int32_t flags, const wl_result* out) {
  return average_impl(ctx, ens, field, rho, n_rho, T, n_T, spin, precision, flags, out,
                      false);
}

int wl_average_async(wl_ctx* ctx, const wl_ens* ens, const wl_field* field,
                     const double* d_rho, int32_t n_rho, const double* d_T,
                     int32_t n_T, int32_t spin, int32_t precision,
                     double* d_mean, double* d_err, double* d_group_sums) {
  const wl_result r{d_mean, d_err, d_group_sums, nullptr, nullptr, nullptr};
  return average_impl(ctx, ens, field, d_rho, n_rho, d_T, n_T, spin, precision,
                      WL_DEVICE_PTR, &r, false);
}

int wl_average_async_noalloc(wl_ctx* ctx, const wl_ens* ens, const wl_field* field,
                             const double* d_rho, int32_t n_rho, const double* d_T,
                             int32_t n_T, int32_t spin, int32_t precision,
                             double* d_mean, double* d_err, double* d_group_sums) {
  const wl_result r{d_mean, d_err, d_group_sums, nullptr, nullptr, nullptr};
  return average_impl(ctx, ens, field, d_rho, n_rho, d_T, n_T, spin, precision,
                      WL_DEVICE_PTR, &r, true);
}

int wl_average(wl_ctx* ctx, const wl_ens* ens, const wl_field* field,
               const double* rho, int32_t n_rho, const double* T, int32_t n_T,
               int32_t spin, int32_t precision, double* mean, double* err,
               double* group_sums) {
  const wl_result r{mean, err, group_sums, nullptr, nullptr, nullptr};
  return average_impl(ctx, ens, field, rho, n_rho, T, n_T, spin, precision, WL_HOST_PTR, &r,
                      false);
}

int wl_average_batch(wl_ctx* ctx, const wl_ens* ens, const wl_request* reqs,
                     int32_t n_reqs) {
  if (!ctx) return WL_EINVAL;
  ctx->err.clear();
  if (n_reqs < 0 || (n_reqs > 0 && !reqs)) return fail(ctx, WL_EINVAL, "bad request list");
  int rc = check_common(ctx, ens, 0, WL_FP32C);
  if (rc) return rc;
  std::vector<wl::FieldArgs> fa(n_reqs);
  for (int32_t r = 0; r < n_reqs; ++r) {
    const wl_request& q = reqs[r];
    if ((rc = check_common(ctx, ens, q.spin, q.precision)) ||
        (rc = check_not_study(ctx, q.precision)) ||
        (rc = check_field(ctx, &q.field, &fa[r])) ||
        (rc = check_grid(ctx, q.rho, q.n_rho, q.T, q.n_T))) {
      std::string m = ctx->err;
      return fail(ctx, rc, "request %d: %s", r, m.c_str());
    }
  }
  DeviceGuard g(ctx->device);
  if (g.status != hipSuccess) return hip_fail(ctx, g.status, "hipSetDevice");
  for (int prec = WL_FP32C; prec <= WL_FP64; ++prec) {
    std::vector<const wl_request*> rq;
    std::vector<wl::FieldArgs> rf;
    std::vector<ReqPlan> pl;
    size_t in_b = kBatchDescOffset + 256, res_b = 0;
    for (int32_t r = 0; r < n_reqs; ++r) {
      if (reqs[r].precision != prec || (int64_t)reqs[r].n_rho * reqs[r].n_T == 0) continue;
      rq.push_back(&reqs[r]);
      rf.push_back(fa[r]);
      pl.push_back(plan_request(ctx, ens, reqs[r]));
      in_b += pl.back().in_bytes;
      res_b += pl.back().res_bytes;
    }
    if (rq.empty()) continue;
    if (prec == WL_FP64 && (rc = need_seg64(ctx, ens))) return rc;
    int64_t items = 0;
    for (const ReqPlan& p : pl) items += p.s.n_items;
    if (items > 0xffffffffll)
      return fail(ctx, WL_EINVAL, "batch of %lld work items is too large", (long long)items);
    in_b = (in_b + 255) & ~(size_t)255;
    if ((rc = ensure(ctx, &ctx->d_batch, &ctx->batch_bytes, in_b + res_b, "batch buffer")))
      return rc;
    void* d_in = ctx->d_batch;
    double* d_res = (double*)((char*)ctx->d_batch + in_b);
    std::vector<char> h_in(in_b);
    wl::BatchLayout lay;
    if (!build_batch(ens, rq.data(), rf.data(), pl.data(), (int32_t)rq.size(), h_in.data(),
                     in_b, d_in, d_res, res_b, &lay))
      return fail(ctx, WL_EINVAL, "internal: batch layout exceeds its buffer");
    Piece in{h_in.data(), 0, lay.in_bytes};
    hipError_t e = copy_in(ctx, d_in, &in, 1);
    if (e == hipSuccess)
      e = wl::launch_batch(prec, ens->d_seg, ens->d_seg64, ens->d_norm, ens->d_x, ens->d_y,
                           ens->n_ppl, d_in, ens->n_groups, ens->n_loops, ctx->d_counter,
                           d_res, ctx->num_cu, ctx->stream);
    // every request's arrays, in the order of the result region's head
    std::vector<Piece> pieces;
    pieces.reserve(6 * rq.size());
    const size_t n_rq = rq.size(), G = ens->n_groups;
    for (size_t i = 0; i < n_rq; ++i)
      pieces.push_back({rq[i]->group_sums, 8 * (size_t)lay.sums_begin[i],
                        8 * G * (size_t)pl[i].n_pts});
    for (size_t k = 0; k < 5; ++k)
      for (size_t i = 0; i < n_rq; ++i) {
        double* const dst[] = {rq[i]->mean, rq[i]->err, rq[i]->scale, rq[i]->fp_err};
        const size_t at = 8 * (size_t)(lay.sums_n + (int64_t)k * lay.pts_n);
        if (k < 4)
          pieces.push_back({dst[k], at + 8 * (size_t)lay.pts_begin[i], 8 * (size_t)pl[i].n_pts});
        else
          pieces.push_back({rq[i]->escalated, at + (size_t)lay.pts_begin[i],
                            (size_t)pl[i].n_pts});
      }
    if (e == hipSuccess) e = copy_out(ctx, d_res, pieces.data(), (int)pieces.size());
    if (e != hipSuccess) return hip_fail(ctx, e, "wl_average_batch");
  }
  return WL_OK;
}

// Sub-loop segment array of the discretisation estimate, derived once per
// ensemble on the ctx stream.
static int ensure_sub(wl_ctx* ctx, const wl_ens* ens) {
  if (ens->d_sub) return WL_OK;
  const int64_t npts = ens->n_loops * ens->n_ppl;
  float4* d = nullptr;
  if (dev_malloc(ctx, (void**)&d, npts * sizeof(float4)) != hipSuccess) {
    return fail(ctx, WL_ENOMEM, "device allocation of the sub-loop segments (%lld bytes) failed",
                (long long)(npts * (int64_t)sizeof(float4)));
  }
  hipError_t e = wl::launch_prep_sub(ens->d_x, ens->d_y, ens->n_loops, ens->n_ppl, d,
                                     ctx->stream);
  if (e != hipSuccess) {
    (void)hipStreamSynchronize(ctx->stream);
    (void)hipFree(d);
    return hip_fail(ctx, e, "sub-loop segments");
  }
  ens->d_sub = d;
  return WL_OK;
}

// FP64 sub-loop segment array, derived once per ensemble on the ctx stream.
static int ensure_sub64(wl_ctx* ctx, const wl_ens* ens) {
  if (ens->d_sub64) return WL_OK;
  const int64_t npts = ens->n_loops * ens->n_ppl;
  double4* d = nullptr;
  if (dev_malloc(ctx, (void**)&d, npts * sizeof(double4)) != hipSuccess) {
    return fail(ctx, WL_ENOMEM,
                "device allocation of the FP64 sub-loop segments (%lld bytes) failed",
                (long long)(npts * (int64_t)sizeof(double4)));
  }
  hipError_t e = wl::launch_prep_sub64(ens->d_x, ens->d_y, ens->n_loops, ens->n_ppl, d,
                                       ctx->stream);
  if (e != hipSuccess) {
    (void)hipStreamSynchronize(ctx->stream);
    (void)hipFree(d);
    return hip_fail(ctx, e, "FP64 sub-loop segments");
  }
  ens->d_sub64 = d;
  return WL_OK;
}

static int check_subloops(wl_ctx* ctx, const wl_ens* ens) {
  if (ens->n_ppl % 4 != 0 || ens->n_ppl < 8)
    return fail(ctx, WL_EINVAL, "sub-loops need n_ppl divisible by 4 and >= 8 (have %d)",
                ens->n_ppl);
  return WL_OK;
}

// Per-loop values of the part of each loop that `sl` names (segments of
// `seg` for the FP32 paths, of `seg64` for FP64).
static int per_loop_impl(wl_ctx* ctx, const wl_ens* ens, const wl::FieldArgs& fa,
                         const float4* seg, const double4* seg64, const wl::SubLoop& sl,
                         const double* rho,
                         int32_t n_rho, const double* T, int32_t n_T, int32_t spin,
                         int32_t precision, int64_t loop0, int64_t n_loops, double* phase,
                         double* spin_exp, double* w);

int wl_per_loop(wl_ctx* ctx, const wl_ens* ens, const wl_field* field,
                const double* rho, int32_t n_rho, const double* T, int32_t n_T,
                int32_t spin, int32_t precision, int64_t loop0, int64_t n_loops,
                double* phase, double* spin_exp, double* w) {
  if (!ctx) return WL_EINVAL;
  ctx->err.clear();
  int rc = check_common(ctx, ens, spin, precision);
  if (rc) return rc;
  wl::FieldArgs fa;
  if ((rc = check_field(ctx, field, &fa))) return rc;
  if ((rc = check_grid(ctx, rho, n_rho, T, n_T))) return rc;
  DeviceGuard g(ctx->device);
  if (g.status != hipSuccess) return hip_fail(ctx, g.status, "hipSetDevice");
  const wl::SubLoop sl{0, ens->n_ppl, 0, 1};
  if (precision == WL_FP64 && (rc = need_seg64(ctx, ens))) return rc;
  return per_loop_impl(ctx, ens, fa, ens->d_seg, ens->d_seg64, sl, rho, n_rho, T, n_T, spin,
                       precision, loop0, n_loops, phase, spin_exp, w);
}

int wl_subloop_per_loop(wl_ctx* ctx, const wl_ens* ens, const wl_field* field,
                        const double* rho, int32_t n_rho, const double* T, int32_t n_T,
                        int32_t spin, int32_t precision, int32_t subloop, int64_t loop0,
                        int64_t n_loops, double* phase, double* spin_exp, double* w) {
  if (!ctx) return WL_EINVAL;
  ctx->err.clear();
  int rc = check_common(ctx, ens, spin, precision);
  if (rc) return rc;
  wl::FieldArgs fa;
  if ((rc = check_field(ctx, field, &fa))) return rc;
  if ((rc = check_grid(ctx, rho, n_rho, T, n_T))) return rc;
  if ((rc = check_subloops(ctx, ens))) return rc;
  const int32_t h = ens->n_ppl / 2, q = ens->n_ppl / 4;
  wl::SubLoop sl;
  switch (subloop) {
    case WL_SUB_CIRCLE: sl = wl::SubLoop{0, h, 0, 2}; break;
    case WL_SUB_SQUARE: sl = wl::SubLoop{h, q, 1, 4}; break;
    case WL_SUB_TRIANGLE: sl = wl::SubLoop{h + q, q, 3, 4}; break;
    default: return fail(ctx, WL_EINVAL, "unknown sub-loop %d", subloop);
  }
  if (loop0 < 0 || n_loops < 0 || loop0 + n_loops > ens->n_loops)
    return fail(ctx, WL_EINVAL, "loop range [%lld, %lld) outside the ensemble",
                (long long)loop0, (long long)(loop0 + n_loops));
  DeviceGuard g(ctx->device);
  if (g.status != hipSuccess) return hip_fail(ctx, g.status, "hipSetDevice");
  if ((rc = precision == WL_FP64 ? ensure_sub64(ctx, ens) : ensure_sub(ctx, ens))) return rc;
  return per_loop_impl(ctx, ens, fa, ens->d_sub, ens->d_sub64, sl, rho, n_rho, T, n_T, spin,
                       precision, loop0, n_loops, phase, spin_exp, w);
}

static int per_loop_impl(wl_ctx* ctx, const wl_ens* ens, const wl::FieldArgs& fa,
                         const float4* seg, const double4* seg64, const wl::SubLoop& sl,
                         const double* rho, int32_t n_rho, const double* T, int32_t n_T,
                         int32_t spin, int32_t precision, int64_t loop0, int64_t n_loops,
                         double* phase, double* spin_exp, double* w) {
  int rc;
  if (loop0 < 0 || n_loops < 0 || loop0 + n_loops > ens->n_loops)
    return fail(ctx, WL_EINVAL, "loop range [%lld, %lld) outside the ensemble",
                (long long)loop0, (long long)(loop0 + n_loops));
  const int64_t n_pts = (int64_t)n_rho * n_T;
  if (n_pts == 0 || n_loops == 0) return WL_OK;
  if (n_loops * n_pts > ((int64_t)1 << 27))
    return fail(ctx, WL_EINVAL, "n_loops * grid points above 2^27 in one call");
  const size_t gbytes = (size_t)(n_rho + n_T) * sizeof(double);
  const size_t each = (size_t)(n_loops * n_pts);
  if ((rc = ensure(ctx, &ctx->d_grid, &ctx->grid_bytes, gbytes, "grid"))) return rc;
  if ((rc = ensure(ctx, &ctx->d_out, &ctx->out_bytes, 3 * each * sizeof(double),
                   "per-loop results")))
    return rc;
  double* d_rho = (double*)ctx->d_grid;
  double* d_T = d_rho + n_rho;
  double* d_ph = (double*)ctx->d_out;
  double* d_sp = d_ph + each;
  double* d_w = d_sp + each;
  hipError_t e = grids_in(ctx, d_rho, rho, n_rho, T, n_T);
  if (e == hipSuccess)
    e = wl::launch_per_loop(precision, spin, fa, seg, seg64, ens->d_x, ens->d_y, ens->n_ppl, sl,
                            d_rho, d_T, n_T, (int32_t)n_pts, loop0, n_loops, d_ph, d_sp, d_w,
                            ctx->stream);
  const size_t eb = each * sizeof(double);
  Piece pieces[] = {{phase, 0, eb}, {spin_exp, eb, eb}, {w, 2 * eb, eb}};
  if (e == hipSuccess) e = copy_out(ctx, d_ph, pieces, 3);
  if (e != hipSuccess) return hip_fail(ctx, e, "per-loop evaluation");
  return WL_OK;
}

int wl_discretisation(wl_ctx* ctx, const wl_ens* ens, const wl_field* field,
                      const double* rho, int32_t n_rho, const double* T, int32_t n_T,
                      int32_t spin, int32_t precision, int32_t mode, double* mean,
                      double* err, double* delta, double* group_sums) {
  if (!ctx) return WL_EINVAL;
  ctx->err.clear();
  int rc = check_common(ctx, ens, spin, precision);
  if (rc) return rc;
  if ((rc = check_not_study(ctx, precision))) return rc;
  wl::FieldArgs fa;
  if ((rc = check_field(ctx, field, &fa))) return rc;
  if ((rc = check_grid(ctx, rho, n_rho, T, n_T))) return rc;
  if ((rc = check_subloops(ctx, ens))) return rc;
  if (mode != WL_DISC_PAPER && mode != WL_DISC_FULL)
    return fail(ctx, WL_EINVAL, "unknown discretisation mode %d", mode);
  const int64_t n_pts = (int64_t)n_rho * n_T;
  if (n_pts == 0) return WL_OK;
  DeviceGuard g(ctx->device);
  if (g.status != hipSuccess) return hip_fail(ctx, g.status, "hipSetDevice");
  if ((rc = precision == WL_FP64 ? ensure_sub64(ctx, ens) : ensure_sub(ctx, ens))) return rc;
  if (precision == WL_FP64 && mode == WL_DISC_FULL && (rc = need_seg64(ctx, ens))) return rc;
  const int64_t G = ens->n_groups;
  const size_t gbytes = (size_t)(n_rho + n_T) * sizeof(double);
  const size_t sums_n = 4 * (size_t)G * n_pts;
  const size_t obytes = (sums_n + 9 * (size_t)n_pts) * sizeof(double);
  if ((rc = ensure(ctx, &ctx->d_grid, &ctx->grid_bytes, gbytes, "grid"))) return rc;
  if ((rc = ensure(ctx, &ctx->d_out, &ctx->out_bytes, obytes, "results"))) return rc;
  const wl::Sched s = make_sched(ctx, ens, (int32_t)n_pts);
  double* level_out = nullptr;
  if (s.n_sub > 1) {
    const size_t need = 3 * (size_t)G * s.n_sub * n_pts * sizeof(double);
    if ((rc = ensure(ctx, &ctx->d_partial, &ctx->partial_bytes, need, "partial sums")))
      return rc;
    level_out = (double*)ctx->d_partial;
  }
  double* d_rho = (double*)ctx->d_grid;
  double* d_T = d_rho + n_rho;
  double* d_sums = (double*)ctx->d_out;
  double* d_mean = d_sums + sums_n;
  double* d_err = d_mean + 4 * n_pts;
  double* d_delta = d_err + 4 * n_pts;
  if (!level_out) level_out = d_sums;
  hipError_t e = grids_in(ctx, d_rho, rho, n_rho, T, n_T);
  hipEvent_t ev0 = nullptr, ev1 = nullptr;
  if (e == hipSuccess && ctx->timing) {
    e = next_events(ctx, &ev0, &ev1);
    if (e == hipSuccess) e = hipEventRecord(ev0, ctx->stream);
  }
  if (e == hipSuccess)
    e = wl::launch_disc(precision, spin, fa, ens->d_seg, ens->d_sub, ens->d_seg64,
                        ens->d_sub64, ens->n_ppl, d_rho, d_T, n_T, (int32_t)n_pts, s,
                        mode == WL_DISC_FULL ? 1 : 0, level_out, ctx->stream);
  if (e == hipSuccess && ctx->timing) {
    e = hipEventRecord(ev1, ctx->stream);
    if (e == hipSuccess) ctx->n_timed++;
  }
  if (e == hipSuccess)
    e = wl::launch_disc_finish(level_out, d_sums, (int32_t)G, s.n_sub, (int32_t)n_pts,
                               ens->n_loops, d_mean, d_err, d_delta, ctx->stream);
  const size_t sb = sums_n * sizeof(double), pb = n_pts * sizeof(double);
  Piece pieces[] = {{group_sums, 0, sb},
                          {mean, sb, 4 * pb},
                          {err, sb + 4 * pb, 4 * pb},
                          {delta, sb + 8 * pb, pb}};
  if (e == hipSuccess) e = copy_out(ctx, d_sums, pieces, 4);
  if (e != hipSuccess) return hip_fail(ctx, e, "wl_discretisation");
  return WL_OK;
}

}  // extern "C"
