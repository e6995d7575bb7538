// batch.cpp -- many series in one launch: batch calls, reusable plans with
// an autotuned launch geometry, captured as a HIP graph.
//
// Every chunk of every series gets a launch chunk index t: the float64
// series come first, then the float32 ones, each series' chunks
// consecutive.  Each series' offsets are counted from its own first chunk, so
// series are independent and each output is byte-identical to a one-series
// call.  Two launch forms exist: split (one launch per dtype,
// each over its own contiguous range of t) and mixed (one launch over all
// of t, the wave branching on the dtype of the chunk's series).
//
// Compression takes the chunks of all series from one work queue per launch,
// and its scanning workgroup starts every series' offsets at 0 (see
// codec_kernels.hpp).  A run never depends on host state beyond its
// descriptors: the queue's words are clear before and after every launch,
// the error words are cleared on the host before each run, and the launch
// epoch is fixed, so a recorded graph can be replayed (no memset nodes).
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <string.h>

#include <algorithm>
#include <new>
#include <vector>

#include "context.hpp"

using namespace falcon_dev;

namespace falcon_host {

namespace {

constexpr uint32_t kBatchEpoch = 1;

// Grows a device (pinned = false) or pinned host array to at least need
// elements, waiting for stream s before freeing the old one.
template <class P>
falcon_status grow(P** p, size_t* cap, size_t need, size_t elem, bool pinned, hipStream_t s) {
  if (need <= *cap && *p) return FALCON_OK;
  size_t c = *cap ? *cap : 64;
  while (c < need) c *= 2;
  if (*p) {
    if (hipStreamSynchronize(s) != hipSuccess) return FALCON_ERR_DEVICE;
    if (pinned) (void)hipHostFree(*p);
    else (void)hipFree(*p);
    *p = nullptr;
    *cap = 0;
  }
  void* q = nullptr;
  const hipError_t e = pinned ? hipHostMalloc(&q, c * elem, hipHostMallocDefault) : hipMalloc(&q, c * elem);
  if (e != hipSuccess) return FALCON_ERR_OUT_OF_MEMORY;
  *p = static_cast<P*>(q);
  *cap = c;
  return FALCON_OK;
}

int grid_of(int maxg, const BatchGeom& g, uint64_t waves, int per) {
  int grid = (int)((int64_t)maxg * g.grid_pct / 100);
  if (grid < 1) grid = 1;
  const uint64_t want = (waves + per - 1) / per;
  if (want < (uint64_t)grid) grid = (int)(want ? want : 1);
  return grid;
}

}  // namespace

falcon_status batch_check(int op, const falcon_series& d) {
  const size_t es = elem_size(d.dtype);
  if (es == 0) return FALCON_ERR_INVALID_ARG;
  const uint64_t nc = chunks_of(d.n);
  // a decompression output may be null only when there is nothing to write
  if (nc >= 0xFFFFFFF0ull || (!d.d_out && (op == FALCON_OP_COMPRESS || d.n != 0)) ||
      ((uintptr_t)d.d_out % (op == FALCON_OP_COMPRESS ? 4 : es)))
    return FALCON_ERR_INVALID_ARG;
  if (op == FALCON_OP_COMPRESS) {
    if (d.n && (!d.d_in || ((uintptr_t)d.d_in % es))) return FALCON_ERR_INVALID_ARG;
    if (d.out_cap < falcon_compress_bound(d.n, d.dtype)) return FALCON_ERR_BUFFER_TOO_SMALL;
  } else {
    if (!d.d_in || ((uintptr_t)d.d_in % 4)) return FALCON_ERR_INVALID_ARG;
    if (d.in_len < 32 + 4 * nc) return FALCON_ERR_CORRUPT_STREAM;
    if (d.out_cap / es < d.n) return FALCON_ERR_BUFFER_TOO_SMALL;
  }
  return FALCON_OK;
}

falcon_status batch_layout(BatchScratch& b, int op, const falcon_series* s, size_t count, BatchLayout& L,
                           hipStream_t st) {
  L = BatchLayout();
  L.op = op;
  L.count = count;
  const size_t dsz = op == FALCON_OP_COMPRESS ? sizeof(CompressSeries) : sizeof(DecompressSeries);
  uint64_t total = 0;
  for (size_t i = 0; i < count; ++i) total += chunks_of(s[i].n);
  const uint64_t nindex = (total >> kIndexShift) + 2;
  L.index_at = count * dsz;
  L.desc_bytes = L.index_at + 4 * nindex;
  falcon_status r = grow(&b.h_desc, &b.h_desc_cap, L.desc_bytes, 1, true, st);
  if (r != FALCON_OK) return r;
  uint64_t t = 0;
  size_t k = 0;
  for (int pass = 0; pass < 2; ++pass) {  // float64 series first, then float32
    for (size_t i = 0; i < count; ++i) {
      const falcon_series& d = s[i];
      if ((d.dtype == FALCON_FLOAT64) != (pass == 0)) continue;
      const uint64_t nc = chunks_of(d.n);
      if (op == FALCON_OP_COMPRESS) {
        CompressSeries c{};
        c.in = d.d_in;
        c.out = static_cast<uint8_t*>(d.d_out);
        c.n = d.n;
        c.chunk0 = t;
        c.dtype = (uint32_t)d.dtype;
        c.idx = (uint32_t)i;
        memcpy(b.h_desc + k * dsz, &c, dsz);
        if (k == 0) L.one_c = c;
      } else {
        DecompressSeries c{};
        c.in = static_cast<const uint8_t*>(d.d_in);
        c.out = static_cast<uint8_t*>(d.d_out);
        c.n = d.n;
        c.chunk0 = t;
        c.payload_bytes = kPayloadFromHeader;
        c.in_len = d.in_len;
        c.dtype = (uint32_t)d.dtype;
        c.idx = (uint32_t)i;
        memcpy(b.h_desc + k * dsz, &c, dsz);
        if (k == 0) L.one_d = c;
      }
      ++k;
      if (d.dtype == FALCON_FLOAT64) {
        L.t64 += nc;
        L.has64 |= nc > 0;
      } else {
        L.has32 |= nc > 0;
      }
      t += nc;
      L.longest = std::max(L.longest, nc);
    }
  }
  L.total = t;
  // the index: the last series with chunk0 <= 64 k
  uint32_t* const index = reinterpret_cast<uint32_t*>(b.h_desc + L.index_at);
  uint64_t c = 0, filled = 0;
  k = 0;
  for (int pass = 0; pass < 2; ++pass) {
    for (size_t i = 0; i < count; ++i) {
      if ((s[i].dtype == FALCON_FLOAT64) != (pass == 0)) continue;
      c += chunks_of(s[i].n);
      for (; filled < nindex && filled << kIndexShift < c; ++filled) index[filled] = (uint32_t)k;
      ++k;
    }
  }
  for (; filled < nindex; ++filled) index[filled] = (uint32_t)(count - 1);
  if ((r = grow(&b.many, &b.many_cap, L.desc_bytes, 1, false, st)) != FALCON_OK ||
      (r = grow(&b.lens, &b.lens_cap, count, 8, true, st)) != FALCON_OK)
    return r;
  if (op == FALCON_OP_DECOMPRESS && L.longest > kDirectChunks &&
      ((r = grow(&b.local, &b.local_cap, t, 4, false, st)) != FALCON_OK ||
       (r = grow(&b.tiles, &b.tiles_cap, scan_tiles(t), 8, false, st)) != FALCON_OK))
    return r;
  if ((r = queue_prepare(b.q, op == FALCON_OP_COMPRESS ? t : 0, st)) != FALCON_OK) return r;
  if (!b.ctl) {
    if (hipHostMalloc(&b.ctl, 64, hipHostMallocDefault) != hipSuccess) return FALCON_ERR_OUT_OF_MEMORY;
    memset(b.ctl, 0, 64);
  }
  return FALCON_OK;
}

// Nothing of an earlier run may reach this one's result, also where that
// run's was never asked for (the tuner's runs, an enqueue or a wait that
// failed): the error words are cleared, and the queue's words again if it
// gave up.  The scratch never grows here.
falcon_status batch_begin(BatchScratch& b, const BatchLayout& L, hipStream_t s) {
  b.ctl->error = 0;
  (void)queue_failed(b.ctl, b.q);
  return queue_prepare(b.q, L.op == FALCON_OP_COMPRESS ? L.total : 0, s);
}

falcon_status batch_enqueue(const falcon_ctx* ctx, BatchScratch& b, const BatchLayout& L, const BatchGeom& g,
                            hipStream_t s, bool upload) {
  falcon_status st = batch_begin(b, L, s);
  if (st != FALCON_OK) return st;
  if (upload && (st = dev_err(hipMemcpyAsync(b.many, b.h_desc, L.desc_bytes, hipMemcpyHostToDevice, s))) !=
                    FALCON_OK)
    return st;
  struct Part { int form; uint64_t t0, chunks; };
  Part parts[2];
  int np = 0;
  if (L.has64 && L.has32 && !g.split) {
    parts[np++] = {kFormMixed, 0, L.total};
  } else {
    if (L.has64) parts[np++] = {2, 0, L.t64};
    if (L.has32) parts[np++] = {1, L.t64, L.total - L.t64};
  }
  if (L.op == FALCON_OP_COMPRESS) {
    if (np == 0) parts[np++] = {2, 0, 0};  // only empty series: the launch writes their headers
    CompressArgs a{};
    a.one = L.one_c;
    a.many = static_cast<const CompressSeries*>(b.many);
    a.nseries = (uint32_t)L.count;
    a.index = reinterpret_cast<const uint32_t*>(static_cast<const uint8_t*>(b.many) + L.index_at);
    a.lens = b.lens;
    a.qctr = b.q.ctr;
    a.qsize = b.q.size;
    a.qoff = b.q.off;
    a.ctl = b.ctl;
    // launches run one after the other on s, each leaving the queue's words
    // clear for the next
    for (int i = 0; i < np; ++i) {
      a.total_chunks = parts[i].chunks;
      a.t0 = parts[i].t0;
      const int nw = queue_nw(parts[i].form, g.nw ? g.nw : queue_waves(parts[i].chunks));
      const int grid = grid_of(max_grid_q(ctx, parts[i].form, nw), g, parts[i].chunks + nw, nw);
      if ((st = dev_err(launch_compress_queue(a, parts[i].form, nw, grid, s))) != FALCON_OK) return st;
    }
    return FALCON_OK;
  }
  if (np == 0) parts[np++] = {2, 0, 0};  // only empty series: the launch checks their headers
  DecompressArgs a{};
  a.one = L.one_d;
  a.many = static_cast<const DecompressSeries*>(b.many);
  a.nseries = (uint32_t)L.count;
  a.index = reinterpret_cast<const uint32_t*>(static_cast<const uint8_t*>(b.many) + L.index_at);
  a.ctl = b.ctl;
  a.epoch = kBatchEpoch;
  a.qctr = b.q.ctr;
  const bool direct = L.longest <= kDirectChunks;
  if (!direct && (st = dev_err(launch_scan_local(&a, L.total, b.local, b.tiles, s))) != FALCON_OK) return st;
  for (int i = 0; i < np; ++i) {
    a.total_chunks = parts[i].chunks;
    a.t0 = parts[i].t0;
    const int grid = grid_of(max_grid_d(ctx, parts[i].form), g, parts[i].chunks, kDecompressWaves);
    a.total_waves = (uint32_t)(grid * kDecompressWaves);
    if ((st = dev_err(launch_decompress(a, parts[i].form, direct, grid, s))) != FALCON_OK) return st;
  }
  return FALCON_OK;
}

falcon_status batch_result(BatchScratch& b, const BatchLayout& L, const falcon_series* src,
                           falcon_series* dst) {
  if (L.op == FALCON_OP_DECOMPRESS && b.ctl->error == kBatchEpoch) return FALCON_ERR_CORRUPT_STREAM;
  if (queue_failed(b.ctl, b.q)) return FALCON_ERR_DEVICE;
  if (dst)
    for (size_t i = 0; i < L.count; ++i) dst[i].out_len = L.op == FALCON_OP_COMPRESS ? b.lens[i] : src[i].n;
  return FALCON_OK;
}

void batch_free(BatchScratch& b) {
  if (b.many) (void)hipFree(b.many);
  if (b.h_desc) (void)hipHostFree(b.h_desc);
  if (b.tiles) (void)hipFree(b.tiles);
  if (b.local) (void)hipFree(b.local);
  if (b.ctl) (void)hipHostFree(b.ctl);
  if (b.lens) (void)hipHostFree(b.lens);
  queue_free(b.q);
  b = BatchScratch();
}

}  // namespace falcon_host

using namespace falcon_host;

struct falcon_plan {
  falcon_ctx* ctx = nullptr;
  std::vector<falcon_series> series;  // caller's descriptors (by caller index)
  BatchLayout layout;
  BatchScratch scratch;               // never grows after creation (the graph holds its pointers)
  BatchGeom geom;
  hipStream_t stream = nullptr;
  int candidates = 0;
  bool from_cache = false;
  float best_ms = 0.f, default_ms = 0.f;
  hipGraph_t graph = nullptr;
  hipGraphExec_t exec = nullptr;
};

namespace {

void plan_free(falcon_plan* p) {
  if (p->stream) (void)hipStreamSynchronize(p->stream);
  if (p->exec) (void)hipGraphExecDestroy(p->exec);
  if (p->graph) (void)hipGraphDestroy(p->graph);
  batch_free(p->scratch);
  if (p->stream) (void)hipStreamDestroy(p->stream);
  delete p;
}

// Times the plan's current geometry: best of reps - 1 runs after a warm-up.
falcon_status time_runs(falcon_plan* p, int reps, float* best) {
  hipEvent_t e0, e1;
  if (hipEventCreate(&e0) != hipSuccess) return FALCON_ERR_DEVICE;
  if (hipEventCreate(&e1) != hipSuccess) {
    (void)hipEventDestroy(e0);
    return FALCON_ERR_DEVICE;
  }
  falcon_status st = FALCON_OK;
  *best = 1e30f;
  for (int r = 0; r < reps && st == FALCON_OK; ++r) {
    float ms = 0.f;
    if ((st = dev_err(hipEventRecord(e0, p->stream))) != FALCON_OK ||
        (st = batch_enqueue(p->ctx, p->scratch, p->layout, p->geom, p->stream, false)) != FALCON_OK ||
        (st = dev_err(hipEventRecord(e1, p->stream))) != FALCON_OK ||
        (st = dev_err(hipEventSynchronize(e1))) != FALCON_OK ||
        (st = dev_err(hipEventElapsedTime(&ms, e0, e1))) != FALCON_OK)
      break;
    if (r > 0 || reps == 1) *best = std::min(*best, ms);
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  return st;
}

// Shape class of a plan for the tuning record: operation, dtypes present,
// log2 of the chunk count and of the series count.
uint64_t shape_class(const BatchLayout& L) {
  auto lg = [](uint64_t v) {
    uint64_t k = 0;
    while (v > 1) {
      v >>= 1;
      ++k;
    }
    return k;
  };
  return (uint64_t)L.op | (uint64_t)L.has64 << 1 | (uint64_t)L.has32 << 2 | lg(L.total + 1) << 3 |
         lg(L.count) << 16;
}

// Autotuner: times every candidate geometry on the plan's own series and
// keeps the fastest.  Compression: launch form (split / mixed) x 8 or 4
// waves per workgroup x full or half grid; decompression: launch form x
// grid.  All
// candidates produce the same bytes (the launch geometry never changes a
// stream).  The choice is recorded in the context by shape class, and a
// later plan of the same class takes it without timing.
falcon_status autotune(falcon_plan* p) {
  const uint64_t key = shape_class(p->layout);
  auto hit = p->ctx->tuned.find(key);
  if (hit != p->ctx->tuned.end()) {
    p->geom = hit->second;
    p->from_cache = true;
    return FALCON_OK;
  }
  std::vector<BatchGeom> cands;
  const bool both = p->layout.has64 && p->layout.has32;
  const bool comp = p->layout.op == FALCON_OP_COMPRESS;
  for (int split = 1; split >= (both ? 0 : 1); --split)
    for (int nw : {8, 4})
      for (int pct : {100, 50}) {
        if (!comp && nw != 8) continue;  // no workgroup size choice there
        BatchGeom g;
        g.split = split;
        g.nw = nw;
        g.grid_pct = pct;
        cands.push_back(g);
      }
  // the default geometry, which default_ms stands for, is the candidate with
  // the workgroups that its launches take by themselves; where those of the
  // two dtypes differ, it is one more
  size_t def = 0;
  if (comp) {
    const int w64 = queue_waves(p->layout.t64), w32 = queue_waves(p->layout.total - p->layout.t64);
    const int nw = !p->layout.has32 ? w64 : !p->layout.has64 || w32 == w64 ? w32 : 0;
    while (def < cands.size() && cands[def].nw != nw) ++def;
    if (def == cands.size()) cands.push_back(BatchGeom());
  }
  float best = 1e30f;
  BatchGeom pick = cands[def];
  for (size_t i = 0; i < cands.size(); ++i) {
    p->geom = cands[i];
    float ms;
    falcon_status st = time_runs(p, 3, &ms);
    if (st != FALCON_OK) return st;
    if (i == def) p->default_ms = ms;
    if (ms < best) {
      best = ms;
      pick = cands[i];
    }
  }
  p->geom = pick;
  p->best_ms = best;
  p->candidates = (int)cands.size();
  p->ctx->tuned[key] = pick;
  return FALCON_OK;
}

// One-shot batch calls run with the context's batch scratch (grown on
// demand) and the default geometry.
falcon_status batch_call(falcon_ctx* ctx, int op, falcon_series* s, size_t count, void* stream) {
  if (!ctx || (count && !s)) return FALCON_ERR_INVALID_ARG;
  if (count == 0) return FALCON_OK;
  if (count > 0x7FFFFFFFull) return FALCON_ERR_INVALID_ARG;
  for (size_t i = 0; i < count; ++i) {
    falcon_status st = batch_check(op, s[i]);
    if (st != FALCON_OK) return st;
  }
  if (hipSetDevice(ctx->device) != hipSuccess) return FALCON_ERR_DEVICE;
  hipStream_t hs = stream ? static_cast<hipStream_t>(stream) : ctx->main.stream;
  BatchLayout L;
  BatchGeom g;
  falcon_status st = batch_layout(ctx->batch, op, s, count, L, hs);
  if (st == FALCON_OK) st = batch_enqueue(ctx, ctx->batch, L, g, hs, true);
  if (st == FALCON_OK) st = dev_err(hipStreamSynchronize(hs));
  if (st == FALCON_OK) st = batch_result(ctx->batch, L, s, s);
  return st;
}

}  // namespace

extern "C" {

falcon_status falcon_plan_create(falcon_ctx* ctx, falcon_op op, const falcon_series* s, size_t count,
                                 unsigned flags, falcon_plan** out) {
  if (!ctx || !out || !s || (op != FALCON_OP_COMPRESS && op != FALCON_OP_DECOMPRESS) || count == 0 ||
      count > 0x7FFFFFFFull)
    return FALCON_ERR_INVALID_ARG;
  *out = nullptr;
  for (size_t i = 0; i < count; ++i) {
    falcon_status st = batch_check(op, s[i]);
    if (st != FALCON_OK) return st;
  }
  if (hipSetDevice(ctx->device) != hipSuccess) return FALCON_ERR_DEVICE;
  falcon_plan* p = new (std::nothrow) falcon_plan();
  if (!p) return FALCON_ERR_OUT_OF_MEMORY;
  p->ctx = ctx;
  p->series.assign(s, s + count);
  falcon_status st = FALCON_OK;
  if (hipStreamCreateWithFlags(&p->stream, hipStreamNonBlocking) != hipSuccess) st = FALCON_ERR_DEVICE;
  if (st == FALCON_OK) st = batch_layout(p->scratch, op, s, count, p->layout, p->stream);
  // descriptors go up once; runs reuse them
  if (st == FALCON_OK)
    st = dev_err(hipMemcpyAsync(p->scratch.many, p->scratch.h_desc, p->layout.desc_bytes, hipMemcpyHostToDevice,
                                p->stream));
  if (st == FALCON_OK) st = dev_err(hipStreamSynchronize(p->stream));
  if (st == FALCON_OK && (flags & FALCON_PLAN_TUNE)) st = autotune(p);
  if (st == FALCON_OK && (flags & FALCON_PLAN_GRAPH)) {
    st = batch_begin(p->scratch, p->layout, p->stream);  // what it may have to clear is not recorded
    if (st == FALCON_OK) st = dev_err(hipStreamBeginCapture(p->stream, hipStreamCaptureModeThreadLocal));
    if (st == FALCON_OK) {
      const falcon_status est = batch_enqueue(ctx, p->scratch, p->layout, p->geom, p->stream, false);
      const hipError_t ce = hipStreamEndCapture(p->stream, &p->graph);
      if (est != FALCON_OK) st = est;
      else if (ce != hipSuccess || hipGraphInstantiate(&p->exec, p->graph, nullptr, nullptr, 0) != hipSuccess)
        st = FALCON_ERR_DEVICE;
    }
  }
  if (st != FALCON_OK) {
    plan_free(p);
    return st;
  }
  *out = p;
  return FALCON_OK;
}

falcon_status falcon_plan_run(falcon_plan* p, falcon_series* s, void* stream) {
  if (!p) return FALCON_ERR_INVALID_ARG;
  if (hipSetDevice(p->ctx->device) != hipSuccess) return FALCON_ERR_DEVICE;
  hipStream_t hs = stream ? static_cast<hipStream_t>(stream) : p->stream;
  falcon_status st = FALCON_OK;
  if (p->exec) {
    if ((st = batch_begin(p->scratch, p->layout, hs)) == FALCON_OK) st = dev_err(hipGraphLaunch(p->exec, hs));
  } else {
    st = batch_enqueue(p->ctx, p->scratch, p->layout, p->geom, hs, false);
  }
  if (st != FALCON_OK) return st;
  if ((st = dev_err(hipStreamSynchronize(hs))) != FALCON_OK) return st;
  return batch_result(p->scratch, p->layout, p->series.data(), s);
}

falcon_status falcon_plan_describe(const falcon_plan* p, falcon_plan_info* info) {
  if (!p || !info) return FALCON_ERR_INVALID_ARG;
  info->split = p->geom.split;
  const bool comp = p->layout.op == FALCON_OP_COMPRESS;
  info->waves_per_group = !comp ? kDecompressWaves : p->geom.nw ? p->geom.nw : queue_waves(p->layout.total);
  info->grid_percent = p->geom.grid_pct;
  info->candidates = p->candidates;
  info->best_ms = p->best_ms;
  info->default_ms = p->default_ms;
  info->graph = p->exec != nullptr;
  info->total_chunks = p->layout.total;
  info->form = comp ? 1 : 0;
  info->from_cache = p->from_cache ? 1 : 0;
  return FALCON_OK;
}

void falcon_plan_destroy(falcon_plan* p) {
  if (!p) return;
  (void)hipSetDevice(p->ctx->device);
  plan_free(p);
}

falcon_status falcon_compress_batch(falcon_ctx* ctx, falcon_series* s, size_t count, void* stream) {
  return batch_call(ctx, FALCON_OP_COMPRESS, s, count, stream);
}

falcon_status falcon_decompress_batch(falcon_ctx* ctx, falcon_series* s, size_t count, void* stream) {
  return batch_call(ctx, FALCON_OP_DECOMPRESS, s, count, stream);
}

}  // extern "C"
