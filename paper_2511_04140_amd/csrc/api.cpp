// api.cpp -- C ABI of the Falcon codec (declared in include/falcon.h):
// context life cycle and the device-resident compress / decompress calls.
//
// A context owns a main lane (a HIP stream, a small pinned staging buffer
// for the few bytes read back per call, the scratch of its launches, and the
// control block) and, once the host pipeline is used, one lane per pipeline
// stream.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <string.h>

#include <new>

#include "context.hpp"

using namespace falcon_dev;

namespace falcon_host {

void write_header(uint8_t* h, falcon_dtype dt, uint64_t n, uint64_t payload) {
  memset(h, 0, 32);
  memcpy(h, "FLCN", 4);
  h[4] = 1;
  h[5] = (uint8_t)dt;
  const uint32_t cn = (uint32_t)kChunkN;
  memcpy(h + 8, &cn, 4);
  memcpy(h + 16, &n, 8);
  memcpy(h + 24, &payload, 8);
}

falcon_status lane_init(Lane& l) {
  if (hipStreamCreateWithFlags(&l.stream, hipStreamNonBlocking) != hipSuccess ||
      hipHostMalloc(&l.ctl, 64, hipHostMallocDefault) != hipSuccess ||
      hipHostMalloc(&l.stage, kStageBytes, hipHostMallocDefault) != hipSuccess) {
    lane_free(l);
    return FALCON_ERR_DEVICE;
  }
  memset(l.stage, 0, kStageBytes);
  memset(l.ctl, 0, 64);
  return FALCON_OK;
}

void lane_free(Lane& l) {
  if (l.stream) (void)hipStreamSynchronize(l.stream);
  if (l.offsets) (void)hipFree(l.offsets);
  if (l.local) (void)hipFree(l.local);
  if (l.tiles) (void)hipFree(l.tiles);
  if (l.meta) (void)hipFree(l.meta);
  if (l.gsizes) (void)hipFree(l.gsizes);
  queue_free(l.q);
  if (l.ctl) (void)hipHostFree(l.ctl);
  if (l.stage) (void)hipHostFree(l.stage);
  if (l.stream) (void)hipStreamDestroy(l.stream);
  l = Lane();
}

namespace {

// Grows a device array to at least n elements (contents undefined).
template <class P>
falcon_status grow_raw(P** arr, size_t* cap, uint64_t n, hipStream_t s) {
  if (n <= *cap && *arr) return FALCON_OK;
  size_t c = *cap ? *cap : 1024;
  while (c < n) c *= 2;
  if (*arr) {
    if (hipStreamSynchronize(s) != hipSuccess) return FALCON_ERR_DEVICE;
    (void)hipFree(*arr);
  }
  *arr = nullptr;
  *cap = 0;
  if (hipMalloc(reinterpret_cast<void**>(arr), c * sizeof(P)) != hipSuccess) return FALCON_ERR_OUT_OF_MEMORY;
  *cap = c;
  return FALCON_OK;
}

int grid_for(int max_grid, uint64_t nchunks, int waves_per_block) {
  uint64_t want = (nchunks + waves_per_block - 1) / waves_per_block;
  if (want < 1) want = 1;
  return (int)(want < (uint64_t)max_grid ? want : (uint64_t)max_grid);
}

}  // namespace

falcon_status queue_prepare(Queue& q, uint64_t nchunks, hipStream_t s) {
  if (q.ctr && nchunks + kQueueSlack <= q.cap && !q.dirty) return FALCON_OK;
  q.dirty = true;  // until everything below has worked
  if (!q.ctr && hipMalloc(&q.ctr, 8 * kQueueWords) != hipSuccess) return FALCON_ERR_OUT_OF_MEMORY;
  // room for as many chunks as the other scratch then has: the next power of two
  uint64_t room = 1024;
  while (room < nchunks) room *= 2;
  room += kQueueSlack;
  const size_t had = q.cap, cap = had > room ? had : room;
  falcon_status st = FALCON_OK;
  if (cap > had) {
    q.cap = 0;
    if ((q.size || q.off) && hipStreamSynchronize(s) != hipSuccess) return FALCON_ERR_DEVICE;
    if (q.size) (void)hipFree(q.size);
    if (q.off) (void)hipFree(q.off);
    q.size = nullptr;
    q.off = nullptr;
    if (hipMalloc(&q.size, cap * sizeof(*q.size)) != hipSuccess || hipMalloc(&q.off, cap * sizeof(*q.off)) != hipSuccess)
      return FALCON_ERR_OUT_OF_MEMORY;
  }
  // Cleared now and not by a recorded fill, where s is being captured: calls
  // that are not recorded use the words too, and may come before any replay.
  hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
  if ((st = dev_err(hipStreamIsCapturing(s, &capture))) != FALCON_OK) return st;
  const bool recording = capture != hipStreamCaptureStatusNone;
  hipStream_t at = s;
  if (recording && (st = dev_err(hipStreamCreateWithFlags(&at, hipStreamNonBlocking))) != FALCON_OK) return st;
  if ((st = dev_err(launch_fill_u64(q.ctr, kQueueWords, 0, at))) == FALCON_OK &&
      (st = dev_err(launch_fill_u64(reinterpret_cast<uint64_t*>(q.size), cap / 2, 0, at))) == FALCON_OK)
    st = dev_err(launch_fill_u64(q.off, cap, 0, at));
  if (recording) {
    if (hipStreamSynchronize(at) != hipSuccess && st == FALCON_OK) st = FALCON_ERR_DEVICE;
    (void)hipStreamDestroy(at);
  }
  if (st != FALCON_OK) return st;
  q.cap = cap;
  q.dirty = false;
  return FALCON_OK;
}

void queue_free(Queue& q) {
  if (q.ctr) (void)hipFree(q.ctr);
  if (q.size) (void)hipFree(q.size);
  if (q.off) (void)hipFree(q.off);
  q = Queue();
}

// Up to one 4-wave workgroup per CU (1,024 chunks), small workgroups spread
// the chunks over more CUs; beyond that, larger ones (queue_large) draw from
// as many ticket counters and scan more sizes a round.  Decimals, us a call:
// float64, 4 against 8 waves, 98 chunks 10.8 / 12.5, 1,024 15.3 / 15.7, 1,200 16.9
// / 16.3, 2,047 20.9 / 19.5, 16,369 76 / 56; float32, 4 against 12, 98 10.2 / 13.1,
// 1,024 13.9 / 15.8, 2,047 18.7 / 17.1, 16,369 82 / 46.
int queue_waves(uint64_t nchunks) { return nchunks <= 1024 ? 4 : 8; }

// Moves the timing ring to a fresh slot for a timed call; the slot counts
// once the call sets its kind, when everything is enqueued.
static void begin_timed(falcon_ctx* ctx) {
  ctx->ev_slot = (ctx->ev_slot + 1) % FALCON_TIMED_CALLS;
  ctx->ev_kind[ctx->ev_slot] = falcon_ctx::kNotTimed;
  ctx->done_recorded[ctx->ev_slot] = false;
  ctx->call_slot = ctx->ev_slot;
}

// The scratch of a decompression of nc chunks, but for its counters.
static falcon_status grow_decompress(Lane& l, uint64_t nc, hipStream_t s) {
  if (nc <= kDirectChunks) return FALCON_OK;
  const falcon_status st = grow_raw(&l.local, &l.local_cap, nc, s);
  return st != FALCON_OK ? st : grow_raw(&l.tiles, &l.tiles_cap, scan_tiles(nc) + 1, s);
}

// Compression: one launch in which waves take chunks from a work queue and
// one workgroup turns their sizes into offsets (k_compress_queue).  The ablation
// variants run in two passes: a size pass, a scan of the chunk sizes into
// offsets, a write pass that redoes a4-a7 and writes each chunk at its
// offset.
falcon_status enqueue_compress(falcon_ctx* ctx, Lane& l, const void* d_in, uint64_t n, falcon_dtype dt, void* d_out,
                               hipStream_t s, bool timed, int variant, uint64_t* d_len) {
  const uint64_t nc = chunks_of(n);
  falcon_status st = FALCON_OK;
  CompressArgs a{};
  a.one.in = d_in;
  a.one.out = static_cast<uint8_t*>(d_out);
  a.one.n = n;
  a.one.chunk0 = 0;
  a.one.dtype = (uint32_t)dt;
  a.one.idx = 0;
  a.many = nullptr;
  a.nseries = 1;
  a.total_chunks = nc;
  a.lens = d_len;
  if (timed) begin_timed(ctx);
  // a decompression of this size is to find its scratch grown: it may be
  // recorded into a graph, where nothing can be allocated
  if ((st = queue_prepare(l.q, variant == 0 ? nc : 0, s)) != FALCON_OK ||
      (st = grow_decompress(l, nc, s)) != FALCON_OK)
    return st;
  if (variant == 0) {
    const int nw = queue_nw((int)dt, queue_waves(nc));
    a.qctr = l.q.ctr;
    a.qsize = l.q.size;
    a.qoff = l.q.off;
    a.ctl = l.ctl;
    a.times = timed ? ctx->times + (size_t)ctx->ev_slot * kTimeWords : nullptr;
    // one workgroup scans
    if ((st = dev_err(launch_compress_queue(a, (int)dt, nw, grid_for(max_grid_q(ctx, dt, nw), nc + nw, nw), s))) !=
        FALCON_OK)
      return st;
    if (timed) ctx->ev_kind[ctx->ev_slot] = falcon_ctx::kStamps;
    return FALCON_OK;
  }
  hipEvent_t* ev = ctx->ev[ctx->ev_slot];
  auto mark = [&](int i) { return timed ? dev_err(hipEventRecord(ev[i], s)) : FALCON_OK; };
  st = grow_raw(&l.offsets, &l.offsets_cap, nc ? nc : 1, s);
  if (st == FALCON_OK) st = grow_raw(&l.tiles, &l.tiles_cap, scan_tiles(nc) + 1, s);
  if (st == FALCON_OK) st = grow_raw(&l.meta, &l.meta_cap, nc ? nc : 1, s);
  if (st == FALCON_OK) st = grow_raw(&l.gsizes, &l.gsizes_cap, nc ? nc : 1, s);
  if (st != FALCON_OK) return st;
  a.meta = l.meta;
  a.gsizes = l.gsizes;
  a.offsets = l.offsets;
  const int nw = kVariantWaves;
  auto launch = [&](int pass) {
    const int grid = grid_for(ctx->grid_v[dt][variant][pass], nc, nw);
    a.total_waves = (uint32_t)(grid * nw);
    return dev_err(launch_compress_variant(a, (int)dt, variant, pass, grid, s));
  };
  if ((st = mark(0)) != FALCON_OK) return st;
  if (nc && (st = launch(1)) != FALCON_OK) return st;
  if ((st = mark(1)) != FALCON_OK) return st;
  if (nc && (st = dev_err(launch_scan_sizes(l.gsizes, nc, l.tiles, l.offsets, s))) != FALCON_OK) return st;
  if ((st = mark(2)) != FALCON_OK) return st;
  if ((st = launch(2)) != FALCON_OK) return st;
  if ((st = mark(3)) != FALCON_OK) return st;
  if (timed) ctx->ev_kind[ctx->ev_slot] = falcon_ctx::kEvents;
  return FALCON_OK;
}

falcon_status enqueue_decompress(falcon_ctx* ctx, Lane& l, const uint8_t* d_in, uint64_t in_len, uint64_t n,
                                 falcon_dtype dt, uint64_t payload, void* d_out, hipStream_t s, bool timed) {
  const uint64_t nc = chunks_of(n);
  falcon_status st = FALCON_OK;
  const bool direct = nc <= kDirectChunks;
  if ((st = grow_decompress(l, nc, s)) != FALCON_OK) return st;
  // the value a failing launch leaves in the error word
  l.epoch += 1;
  if (l.epoch == 0) l.epoch = 1;
  if (timed) begin_timed(ctx);
  DecompressArgs a{};
  a.one.in = d_in;
  a.one.out = static_cast<uint8_t*>(d_out);
  a.one.n = n;
  a.one.chunk0 = 0;
  a.one.payload_bytes = payload;
  a.one.in_len = in_len;
  a.one.dtype = (uint32_t)dt;
  a.many = nullptr;
  a.nseries = 1;
  a.total_chunks = nc;
  a.ctl = l.ctl;
  a.epoch = l.epoch;
  a.times = timed ? ctx->times + (size_t)ctx->ev_slot * kTimeWords : nullptr;
  const int grid = grid_for(max_grid_d(ctx, dt), nc, kDecompressWaves);
  a.total_waves = (uint32_t)(grid * kDecompressWaves);
  if (!direct || nc > kDrawFrom * a.total_waves) {
    if ((st = queue_prepare(l.q, 0, s)) != FALCON_OK) return st;
    a.qctr = l.q.ctr;
  }
  if (!direct && (st = dev_err(launch_scan_local(&a, nc, l.local, l.tiles, s))) != FALCON_OK) return st;
  if ((st = dev_err(launch_decompress(a, (int)dt, direct, grid, s))) != FALCON_OK) return st;
  if (timed) ctx->ev_kind[ctx->ev_slot] = falcon_ctx::kStamps;
  return FALCON_OK;
}

namespace {

// ---- asynchronous device calls --------------------------------------------
// A device call runs in three steps: begin_call (stream choice, ordering
// after the previous call), the enqueue, end_call (with FALCON_OPT_BLOCKING
// synchronises and reports at once).

hipStream_t call_stream(falcon_ctx* ctx, void* stream) {
  return stream ? static_cast<hipStream_t>(stream) : ctx->main.stream;
}

falcon_status begin_call(falcon_ctx* ctx, hipStream_t s) {
  if (hipSetDevice(ctx->device) != hipSuccess) return FALCON_ERR_DEVICE;
  ctx->call_slot = FALCON_TIMED_CALLS;
  if (!ctx->unsynced || ctx->last_stream == s) return FALCON_OK;
  if (!ctx->last_event) {  // the last call's stream is the context's own
    ctx->last_event = ctx->done[FALCON_TIMED_CALLS];
    if (hipEventRecord(ctx->last_event, ctx->last_stream) != hipSuccess) return FALCON_ERR_DEVICE;
  }
  if (hipStreamWaitEvent(s, ctx->last_event, 0) == hipSuccess) return FALCON_OK;
  (void)hipGetLastError();  // reported here, not to the program's next call
  return FALCON_ERR_DEVICE;
}

falcon_status end_call(falcon_ctx* ctx, hipStream_t s, falcon_status st) {
  // also after an error, so that a later call or falcon_sync still orders
  // after the work enqueued so far
  ctx->last_stream = s;
  ctx->last_event = nullptr;
  ctx->unsynced = true;
  if (ctx->opt_flags & FALCON_OPT_BLOCKING) {
    const falcon_status sy = falcon_sync(ctx);
    if (st == FALCON_OK) st = sy;
  } else if (s != ctx->main.stream) {
    ctx->last_event = ctx->done[ctx->call_slot];
    ctx->done_recorded[ctx->call_slot] = hipEventRecord(ctx->last_event, s) == hipSuccess;
    if (!ctx->done_recorded[ctx->call_slot] && st == FALCON_OK) st = FALCON_ERR_DEVICE;
  }
  return st;
}

// A pinned word that the kernels of one compression fill with its stream
// length, reported to *dst at falcon_sync.
falcon_status pending_length(falcon_ctx* ctx, size_t* dst, uint64_t** d_len) {
  const size_t slot = ctx->pending.size();
  const size_t b = slot / kLenBlock;
  if (b == ctx->len_blocks.size()) {
    void* p = nullptr;
    if (hipHostMalloc(&p, kLenBlock * 8, hipHostMallocDefault) != hipSuccess) return FALCON_ERR_OUT_OF_MEMORY;
    ctx->len_blocks.push_back(static_cast<uint64_t*>(p));
  }
  *d_len = ctx->len_blocks[b] + slot % kLenBlock;
  ctx->pending.push_back({dst, slot});
  return FALCON_OK;
}

// Writes 32 (the stream length of n = 0, which no kernel writes) to a
// length word.
falcon_status empty_length(uint64_t* d_len, hipStream_t s) { return dev_err(launch_fill_u64(d_len, 1, 32, s)); }

}  // namespace

}  // namespace falcon_host

using namespace falcon_host;

extern "C" {

const char* falcon_status_str(falcon_status st) {
  switch (st) {
    case FALCON_OK: return "ok";
    case FALCON_ERR_INVALID_ARG: return "invalid argument";
    case FALCON_ERR_BUFFER_TOO_SMALL: return "buffer too small";
    case FALCON_ERR_CORRUPT_STREAM: return "corrupt stream";
    case FALCON_ERR_DEVICE: return "device error";
    case FALCON_ERR_OUT_OF_MEMORY: return "out of memory";
  }
  return "unknown status";
}

size_t falcon_compress_bound(size_t n, falcon_dtype dt) {
  const size_t per = max_chunk_bytes(dt);
  if (per == 0) return 0;
  return 32 + chunks_of(n) * (4 + per);
}

falcon_status falcon_create(int device, const falcon_opts* opts, falcon_ctx** out) {
  if (!out) return FALCON_ERR_INVALID_ARG;
  *out = nullptr;
  const unsigned flags = opts ? opts->flags : 0u;
  const int form = opts ? opts->compress_form : 0;
  if ((flags & ~(unsigned)(FALCON_OPT_BLOCKING | FALCON_OPT_DEVICE_LENGTHS)) ||
      (form != FALCON_FORM_TWO_PASS && form != FALCON_FORM_SINGLE_PASS))
    return FALCON_ERR_INVALID_ARG;
  int ndev = 0;
  if (hipGetDeviceCount(&ndev) != hipSuccess || device < 0 || device >= ndev) return FALCON_ERR_DEVICE;
  if (hipSetDevice(device) != hipSuccess) return FALCON_ERR_DEVICE;
  falcon_ctx* ctx = new (std::nothrow) falcon_ctx();
  if (!ctx) return FALCON_ERR_OUT_OF_MEMORY;
  ctx->device = device;
  ctx->opt_flags = flags;
  bool ok = lane_init(ctx->main) == FALCON_OK;
  for (int c = 0; ok && c <= FALCON_TIMED_CALLS; ++c)
    ok = hipEventCreateWithFlags(&ctx->done[c], hipEventDisableTiming) == hipSuccess;
  for (int c = 0; ok && c < FALCON_TIMED_CALLS; ++c)
    for (int i = 0; ok && i < 4; ++i) ok = hipEventCreate(&ctx->ev[c][i]) == hipSuccess;
  constexpr size_t kTimeBytes = (size_t)kTimeWords * 8;
  ok = ok && hipMalloc(&ctx->times, FALCON_TIMED_CALLS * kTimeBytes) == hipSuccess &&
       launch_fill_u64(ctx->times, (size_t)FALCON_TIMED_CALLS * kTimeWords, 0, ctx->main.stream) == hipSuccess &&
       hipStreamSynchronize(ctx->main.stream) == hipSuccess &&
       hipHostMalloc(&ctx->times_host, kTimeBytes, hipHostMallocDefault) == hipSuccess &&
       hipDeviceGetAttribute(&ctx->tick_khz, hipDeviceAttributeWallClockRate, device) == hipSuccess;
  if (!ok) {
    falcon_destroy(ctx);
    return FALCON_ERR_DEVICE;
  }
  for (int form_ = 1; form_ <= 3; ++form_) {
    ctx->grid_d[form_] = max_grid_decompress(device, form_);
    ctx->grid_q[form_][0] = max_grid_compress_queue(device, form_, 4);
    ctx->grid_q[form_][1] = max_grid_compress_queue(device, form_, queue_large(form_));
  }
  for (int f = 1; f <= 2; ++f)
    for (int v = 1; v <= 3; ++v)
      for (int pass = 1; pass <= 2; ++pass) ctx->grid_v[f][v][pass] = max_grid_compress_variant(device, f, v, pass);
  if (noalloc_setup(device) != FALCON_OK) {
    falcon_destroy(ctx);
    return FALCON_ERR_DEVICE;
  }
  *out = ctx;
  return FALCON_OK;
}

falcon_status falcon_sync(falcon_ctx* ctx) {
  if (!ctx) return FALCON_ERR_INVALID_ARG;
  if (!ctx->unsynced) return FALCON_OK;
  if (hipSetDevice(ctx->device) != hipSuccess) return FALCON_ERR_DEVICE;
  Lane& l = ctx->main;
  falcon_status st = dev_err(hipStreamSynchronize(ctx->last_stream));
  if (st == FALCON_OK) {
    // lengths and error words lie in pinned memory: nothing is copied
    for (const auto& p : ctx->pending)
      *p.dst = (size_t)ctx->len_blocks[p.slot / kLenBlock][p.slot % kLenBlock];
    // the decompression error word holds the epoch of the last launch whose
    // chunk failed: a launch since the last sync has a larger one
    const uint32_t err = l.ctl->error;
    if (err != 0 && err > ctx->sync_epoch && err <= l.epoch) st = FALCON_ERR_CORRUPT_STREAM;
    if (compress_failed(l)) {
      // cleared here and not before the next call, which may be the replay of
      // a recorded one
      st = FALCON_ERR_DEVICE;
      if (queue_prepare(l.q, 0, ctx->last_stream) == FALCON_OK) (void)hipStreamSynchronize(ctx->last_stream);
    }
  }
  ctx->pending.clear();
  ctx->sync_epoch = l.epoch;
  ctx->unsynced = false;
  return st;
}

void falcon_destroy(falcon_ctx* ctx) {
  if (!ctx) return;
  (void)hipSetDevice(ctx->device);
  pipe_release(ctx);
  if (ctx->main.stream) (void)hipStreamSynchronize(ctx->main.stream);
  if (ctx->last_stream) (void)hipStreamSynchronize(ctx->last_stream);
  batch_free(ctx->batch);
  lane_free(ctx->main);
  for (auto& call : ctx->ev)
    for (hipEvent_t e : call)
      if (e) (void)hipEventDestroy(e);
  for (hipEvent_t e : ctx->done)
    if (e) (void)hipEventDestroy(e);
  for (uint64_t* b : ctx->len_blocks) (void)hipHostFree(b);
  if (ctx->times) (void)hipFree(ctx->times);
  if (ctx->times_host) (void)hipHostFree(ctx->times_host);
  delete ctx;
}

falcon_status falcon_stream_info(const void* h_hdr, size_t len, size_t* n, falcon_dtype* dt) {
  if (!h_hdr || !n || !dt) return FALCON_ERR_INVALID_ARG;
  const uint8_t* h = static_cast<const uint8_t*>(h_hdr);
  if (len < 32 || memcmp(h, "FLCN", 4) != 0 || h[4] != 1 || (h[5] != 1 && h[5] != 2) || h[6] || h[7] ||
      rd32(h + 8) != kChunkN || rd32(h + 12) != 0)
    return FALCON_ERR_CORRUPT_STREAM;
  *n = (size_t)rd64(h + 16);
  *dt = (falcon_dtype)h[5];
  return FALCON_OK;
}

falcon_status falcon_compress(falcon_ctx* ctx, const void* d_in, size_t n, falcon_dtype dt, void* d_out,
                              size_t out_cap, size_t* out_len, void* stream) {
  return falcon_compress_variant(ctx, d_in, n, dt, FALCON_VARIANT_FALCON, d_out, out_cap, out_len, stream);
}

size_t falcon_compress_bound_variant(size_t n, falcon_dtype dt, falcon_variant v) {
  if (v < FALCON_VARIANT_FALCON || v > FALCON_VARIANT_DENSE) return 0;
  if (v != FALCON_VARIANT_SPARSE) return falcon_compress_bound(n, dt);
  const size_t per = dt == FALCON_FLOAT64 ? 11 + 8 + 64 * 144 : dt == FALCON_FLOAT32 ? 7 + 4 + 32 * 144 : 0;
  if (per == 0) return 0;
  return 32 + chunks_of(n) * (4 + per);
}

falcon_status falcon_compress_variant(falcon_ctx* ctx, const void* d_in, size_t n, falcon_dtype dt, falcon_variant v,
                                      void* d_out, size_t out_cap, size_t* out_len, void* stream) {
  if (!ctx || !d_out || !out_len || (n && !d_in)) return FALCON_ERR_INVALID_ARG;
  if (v < FALCON_VARIANT_FALCON || v > FALCON_VARIANT_DENSE) return FALCON_ERR_INVALID_ARG;
  const size_t es = elem_size(dt);
  if (es == 0) return FALCON_ERR_INVALID_ARG;
  if (((uintptr_t)d_in % es) || ((uintptr_t)d_out % 4)) return FALCON_ERR_INVALID_ARG;
  const bool dev_len = (ctx->opt_flags & FALCON_OPT_DEVICE_LENGTHS) != 0;
  if (dev_len && ((uintptr_t)out_len % 8)) return FALCON_ERR_INVALID_ARG;
  if (out_cap < falcon_compress_bound_variant(n, dt, v)) return FALCON_ERR_BUFFER_TOO_SMALL;
  const uint64_t nc = chunks_of(n);
  if (nc >= 0xFFFFFFF0ull) return FALCON_ERR_INVALID_ARG;
  hipStream_t s = call_stream(ctx, stream);
  falcon_status st = begin_call(ctx, s);
  if (st != FALCON_OK) return st;
  uint64_t* d_len = nullptr;
  if (dev_len) d_len = reinterpret_cast<uint64_t*>(out_len);
  else if (n) st = pending_length(ctx, out_len, &d_len);
  else *out_len = 32;
  if (st == FALCON_OK)
    st = enqueue_compress(ctx, ctx->main, d_in, n, dt, d_out, s, true, (int)v, d_len);
  if (st == FALCON_OK && dev_len && n == 0) st = empty_length(d_len, s);
  return end_call(ctx, s, st);
}

falcon_status falcon_decompress_n(falcon_ctx* ctx, const void* d_in, size_t in_len, size_t n, falcon_dtype dt,
                                  void* d_out, size_t out_cap_bytes, void* stream) {
  if (!ctx || !d_in || ((uintptr_t)d_in % 4)) return FALCON_ERR_INVALID_ARG;
  const size_t es = elem_size(dt);
  if (es == 0) return FALCON_ERR_INVALID_ARG;
  const uint64_t nc = chunks_of(n);
  if (nc >= 0xFFFFFFF0ull || in_len < 32 || (in_len - 32) / 4 < nc) return FALCON_ERR_CORRUPT_STREAM;
  if (out_cap_bytes / es < n) return FALCON_ERR_BUFFER_TOO_SMALL;
  if (n && (!d_out || ((uintptr_t)d_out % es))) return FALCON_ERR_INVALID_ARG;
  hipStream_t s = call_stream(ctx, stream);
  falcon_status st = begin_call(ctx, s);
  if (st != FALCON_OK) return st;
  // an empty stream has no chunk to check its header: nothing to launch
  if (n) st = enqueue_decompress(ctx, ctx->main, static_cast<const uint8_t*>(d_in), in_len, n, dt,
                                 kPayloadFromHeader, d_out, s, true);
  return end_call(ctx, s, st);
}

falcon_status falcon_decompress(falcon_ctx* ctx, const void* d_in, size_t in_len, void* d_out, size_t out_cap_bytes,
                                size_t* n_out, void* stream) {
  if (!ctx || !d_in || !n_out || ((uintptr_t)d_in % 4)) return FALCON_ERR_INVALID_ARG;
  if (in_len < 32) return FALCON_ERR_CORRUPT_STREAM;
  Lane& l = ctx->main;
  hipStream_t s = call_stream(ctx, stream);
  falcon_status st = begin_call(ctx, s);
  if (st != FALCON_OK) return st;
  // the header, read after the work already on the stream
  if ((st = dev_err(hipMemcpyAsync(l.stage, d_in, 32, hipMemcpyDeviceToHost, s))) != FALCON_OK ||
      (st = dev_err(hipStreamSynchronize(s))) != FALCON_OK)
    return end_call(ctx, s, st);
  size_t n = 0;
  falcon_dtype dt;
  if ((st = falcon_stream_info(l.stage, 32, &n, &dt)) != FALCON_OK) return end_call(ctx, s, st);
  const uint64_t payload = rd64(l.stage + 24);
  const uint64_t nc = chunks_of(n);
  if (nc >= 0xFFFFFFF0ull || (in_len - 32) / 4 < nc || payload > in_len - 32 - 4 * nc ||
      (n == 0 && payload != 0))
    return end_call(ctx, s, FALCON_ERR_CORRUPT_STREAM);
  *n_out = n;
  const size_t es = elem_size(dt);
  if (out_cap_bytes / es < n) return end_call(ctx, s, FALCON_ERR_BUFFER_TOO_SMALL);
  if (n && (!d_out || ((uintptr_t)d_out % es))) return end_call(ctx, s, FALCON_ERR_INVALID_ARG);
  if (n)
    st = enqueue_decompress(ctx, l, static_cast<const uint8_t*>(d_in), in_len, n, dt, payload, d_out, s, true);
  return end_call(ctx, s, st);
}

// The one-series-per-launch path over many series: one asynchronous call per
// series, lengths written by the kernels to pinned memory, one wait.
falcon_status falcon_compress_each(falcon_ctx* ctx, falcon_series* ss, size_t count, void* stream) {
  if (!ctx || (count && !ss)) return FALCON_ERR_INVALID_ARG;
  for (size_t i = 0; i < count; ++i) {
    const falcon_status st = batch_check(FALCON_OP_COMPRESS, ss[i]);
    if (st != FALCON_OK) return st;
  }
  if (count == 0) return FALCON_OK;
  hipStream_t s = call_stream(ctx, stream);
  falcon_status st = begin_call(ctx, s);
  if (st != FALCON_OK) return st;
  std::vector<uint64_t*> dl(count);
  for (size_t i = 0; i < count && st == FALCON_OK; ++i) {
    st = pending_length(ctx, &ss[i].out_len, &dl[i]);
    if (st == FALCON_OK)
      st = enqueue_compress(ctx, ctx->main, ss[i].d_in, ss[i].n, ss[i].dtype, ss[i].d_out, s, false, 0,
                            dl[i]);
    if (st == FALCON_OK && ss[i].n == 0) st = empty_length(dl[i], s);
  }
  st = end_call(ctx, s, st);
  const falcon_status sy = falcon_sync(ctx);
  return st != FALCON_OK ? st : sy;
}

falcon_status falcon_decompress_each(falcon_ctx* ctx, falcon_series* ss, size_t count, void* stream) {
  if (!ctx || (count && !ss)) return FALCON_ERR_INVALID_ARG;
  for (size_t i = 0; i < count; ++i) {
    const falcon_status st = batch_check(FALCON_OP_DECOMPRESS, ss[i]);
    if (st != FALCON_OK) return st;
  }
  if (count == 0) return FALCON_OK;
  hipStream_t s = call_stream(ctx, stream);
  falcon_status st = begin_call(ctx, s);
  if (st != FALCON_OK) return st;
  for (size_t i = 0; i < count && st == FALCON_OK; ++i) {
    if (ss[i].n)
      st = enqueue_decompress(ctx, ctx->main, static_cast<const uint8_t*>(ss[i].d_in), ss[i].in_len, ss[i].n,
                              ss[i].dtype, kPayloadFromHeader, ss[i].d_out, s, false);
    ss[i].out_len = ss[i].n;
  }
  st = end_call(ctx, s, st);
  const falcon_status sy = falcon_sync(ctx);
  return st != FALCON_OK ? st : sy;
}

falcon_status falcon_call_stage_ms(falcon_ctx* ctx, unsigned back, float* ms) {
  if (!ctx || !ms || back >= FALCON_TIMED_CALLS) return FALCON_ERR_INVALID_ARG;
  const int slot = (ctx->ev_slot + FALCON_TIMED_CALLS - (int)back) % FALCON_TIMED_CALLS;
  if (ctx->ev_kind[slot] == falcon_ctx::kNotTimed) return FALCON_ERR_INVALID_ARG;
  if (ctx->ev_kind[slot] == falcon_ctx::kEvents) {
    hipEvent_t* ev = ctx->ev[slot];
    if (hipEventSynchronize(ev[3]) != hipSuccess) return FALCON_ERR_DEVICE;
    for (int i = 0; i < 3; ++i)
      if (hipEventElapsedTime(ms + i, ev[i], ev[i + 1]) != hipSuccess) return FALCON_ERR_DEVICE;
    return FALCON_OK;
  }
  // the call, unless a falcon_sync has waited for it already: its event, or
  // the context's own stream
  if (hipSetDevice(ctx->device) != hipSuccess ||
      (ctx->unsynced && ctx->done_recorded[slot] && hipEventSynchronize(ctx->done[slot]) != hipSuccess) ||
      hipMemcpyAsync(ctx->times_host, ctx->times + (size_t)slot * kTimeWords, (size_t)kTimeWords * 8,
                     hipMemcpyDeviceToHost, ctx->main.stream) != hipSuccess ||
      hipStreamSynchronize(ctx->main.stream) != hipSuccess)
    return FALCON_ERR_DEVICE;
  const uint64_t* w = ctx->times_host;
  uint64_t end = w[2];
  for (int i = 1; i <= kTimeEnds; ++i) end = w[kTimeStride * i] > end ? w[kTimeStride * i] : end;
  const double per_ms = (double)ctx->tick_khz;
  ms[0] = (float)((double)(w[1] - w[0]) / per_ms);
  ms[1] = (float)((double)(w[2] - w[1]) / per_ms);
  ms[2] = (float)((double)(end - w[2]) / per_ms);
  return FALCON_OK;
}

falcon_status falcon_last_stage_ms(falcon_ctx* ctx, float* ms) { return falcon_call_stage_ms(ctx, 0, ms); }

falcon_status falcon_last_kernel_ms(falcon_ctx* ctx, float* ms) {
  if (!ms) return FALCON_ERR_INVALID_ARG;
  float st[3];
  const falcon_status s = falcon_call_stage_ms(ctx, 0, st);
  if (s == FALCON_OK) *ms = st[0] + st[1] + st[2];
  return s;
}

}  // extern "C"
