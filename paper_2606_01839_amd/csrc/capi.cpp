// C ABI of the library (declared in include/conserve_attn.h): argument validation, host metadata
// (pages, conversations, plans), metadata upload through a pinned ring, kernel launches.
#include "conserve_attn.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>
#include <string>
#include <vector>

#include "host/host_state.hpp"
#include "kernels.hpp"

namespace {

thread_local std::string g_err;

cs_status fail(cs_status code, const std::string& msg) {
  g_err = msg;
  return code;
}

constexpr size_t kAlign = 256;
constexpr size_t kRingBytes = size_t(8) << 20;  // metadata ring (device + pinned host), 4 quarters
constexpr size_t kQuarter = kRingBytes / 4;
constexpr int kItemKeys = 128;  // the workspace has room for a decode record per this many keys (an item has 256 or more)
// Splits (waves) a decode launch aims for (16 per CU). Half as many (longer splits, fewer items to
// merge) made the 32-layer mixed trace 5% slower, twice as many 1% slower.
constexpr int64_t kDecodeTargetItems = 4096;

size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

constexpr int kMaxLayersPerLaunch = 32768;  // a grid dimension
// Records of cut extend tiles one layer may write: two per CU.
constexpr int kExtendRecords = 2 * cs::kCus;
// Tiles and merges of a plan that split_extend has cut: at most two rounds of tiles, each a tile or a
// merge, and a piece for every record.
constexpr size_t kMaxCutBytes = 2 * cs::kCus * (sizeof(cs::ExtendTile) + sizeof(cs::ExtendMerge)) +
                                kExtendRecords * sizeof(cs::ExtendTile) + kAlign;
// Records the workspace holds (69 MB at head dim 128; 208 MB in a multi-layer pool, whose overlapped
// steps put as many layers into one launch as have room: 28 layers of a 4-conversation step in one
// launch instead of three 395 -> 374 us, 32 of an 8-conversation one 1614 -> 1527 us).
int extend_records(const cs_pool_desc& d) { return (d.n_layers > 1 ? 3 : 1) * kExtendRecords; }

struct WsLayout {
  size_t page_table, partials, ext_parts, ring, total;
  // decode records: one layer of any batch, two in a multi-layer pool, and every layer of a batch whose
  // items fit the CUs in one round (17 MB at 32 layers, 32 query heads, head dim 128)
  size_t partial_floats;
};

int64_t max_decode_items(const cs_pool_desc& d) {
  // sum_b ceil(L_b / kItemKeys) <= total tokens / kItemKeys + batch
  return d.n_pages * cs::kPage / kItemKeys + d.max_convs;
}

WsLayout ws_layout(const cs_pool_desc& d) {
  WsLayout w{};
  w.page_table = 0;
  size_t pt_bytes = static_cast<size_t>(d.max_convs) * static_cast<size_t>(d.max_pages_per_conv) * 4;
  w.partials = align_up(pt_bytes, kAlign);
  const int64_t one_round = std::max(1, cs::kCus / d.n_kv_heads) * std::min<int64_t>(d.n_layers, 128);
  w.partial_floats = static_cast<size_t>(std::max(max_decode_items(d) * (d.n_layers > 1 ? 2 : 1), one_round)) *
                     d.n_q_heads * cs::partial_floats(d.head_dim);
  w.ext_parts = align_up(w.partials + w.partial_floats * 4, kAlign);
  // a pool whose longest conversation is too short to be cut needs no records
  const int64_t longest = std::min<int64_t>(d.max_pages_per_conv, d.n_pages) * cs::kPage;
  const size_t records = longest > cs::kExtendKeyTile * cs::kMinPiece ? extend_records(d) : 0;
  w.ring = align_up(w.ext_parts + records * cs::extend_part_floats(d.head_dim) * 4, kAlign);
  w.total = w.ring + kRingBytes;
  return w;
}

const char* desc_problem(const cs_pool_desc* d) {
  if (!d) return "null descriptor";
  if (d->n_layers < 1) return "n_layers must be >= 1";
  if (d->n_kv_heads < 1 || d->n_q_heads < 1 || d->n_q_heads % d->n_kv_heads != 0)
    return "n_q_heads must be a positive multiple of n_kv_heads";
  const int group = d->n_q_heads / d->n_kv_heads;
  if (d->head_dim != 64 && d->head_dim != 128) return "head_dim must be 64 or 128";
  if (group != 1 && group != 2 && group != 4 && group != 8)
    return "n_q_heads/n_kv_heads must be 1, 2, 4 or 8";
  if (d->max_convs < 1 || d->max_convs > (1 << cs::ConvTable::kSlotBits))
    return "max_convs must be in [1, 2^20]";
  if (d->max_pages_per_conv < 1 || d->max_pages_per_conv > (1 << 26))
    return "max_pages_per_conv must be in [1, 2^26]";
  if (d->n_pages < 1 || d->n_pages > INT32_MAX) return "n_pages must be in [1, 2^31)";
  return nullptr;
}

}  // namespace

struct cs_pool {
  cs_pool_desc desc;
  char* kv;
  size_t kv_bytes;
  char* ws;
  size_t ws_bytes;
  WsLayout lay;
  cs::PagePool pages;
  cs::ConvTable convs;
  // device resources, created on first use
  bool dev_ready = false;
  int device = -1;
  char* h_ring = nullptr;
  size_t ring_head = 0;
  int cur_quarter = -1;
  hipEvent_t quarter_ev[4] = {};
  bool quarter_used[4] = {};
  hipEvent_t switch_ev = nullptr;
  hipStream_t stream = nullptr;
  bool have_stream = false;
  // second stream of cs_mixed_step (extend chunks run on it concurrently with the decode batch)
  hipStream_t side = nullptr;
  hipEvent_t fork_ev = nullptr, join_ev = nullptr;
  // instrumentation: timing events around each kernel launch while enabled
  struct ProfEvent {
    hipEvent_t start, stop;
    int kind;
    int launches;
  };
  bool prof_on = false;
  int64_t fail_after = -1;  // cs_debug_fail_launches: launches left before the injected failure
  // an open span: one pair of events brackets a run of launches of one kind on one stream
  bool span_open = false;
  hipEvent_t span_start = nullptr;
  hipStream_t span_stream = nullptr;
  int span_kind = 0, span_launches = 0;
  // check_convs: the batch that last named each conversation slot
  std::vector<uint32_t> seen;
  uint32_t batch = 0;
  std::vector<hipEvent_t> ev_free;
  std::vector<ProfEvent> prof_events;

  cs_pool(const cs_pool_desc& d, char* kvp, size_t kvb, char* wsp, size_t wsb, uint64_t seed)
      : desc(d), kv(kvp), kv_bytes(kvb), ws(wsp), ws_bytes(wsb), lay(ws_layout(d)),
        pages(d.n_pages, seed), convs(d.max_convs, d.max_pages_per_conv) {}

  cs::PoolGeom geom() const {
    cs::PoolGeom g;
    g.pool = kv;
    g.n_pages = desc.n_pages;
    g.n_layers = desc.n_layers;
    g.n_kv_heads = desc.n_kv_heads;
    g.n_q_heads = desc.n_q_heads;
    g.head_dim = desc.head_dim;
    g.page_table = reinterpret_cast<int32_t*>(ws + lay.page_table);
    g.max_pages = desc.max_pages_per_conv;
    return g;
  }
  float* partials() const { return reinterpret_cast<float*>(ws + lay.partials); }
  float* ext_parts() const { return reinterpret_cast<float*>(ws + lay.ext_parts); }
};

namespace {

cs_status hip_fail(hipError_t e, const char* what) {
  return fail(CS_EHIP, std::string(what) + ": " + hipGetErrorString(e));
}

#define CS_HIP(call, what)                        \
  do {                                            \
    hipError_t e_ = (call);                       \
    if (e_ != hipSuccess) return hip_fail(e_, what); \
  } while (0)

cs_status ensure_device(cs_pool* p) {
  if (p->dev_ready) return CS_OK;
  int dev = 0;
  CS_HIP(hipGetDevice(&dev), "hipGetDevice");
  void* h = nullptr;
  CS_HIP(hipHostMalloc(&h, kRingBytes, hipHostMallocDefault), "hipHostMalloc(metadata ring)");
  for (int i = 0; i < 4; ++i) {
    hipError_t e = hipEventCreateWithFlags(&p->quarter_ev[i], hipEventDisableTiming);
    if (e != hipSuccess) {
      for (int k = 0; k < i; ++k) (void)hipEventDestroy(p->quarter_ev[k]);
      (void)hipHostFree(h);
      return hip_fail(e, "hipEventCreate");
    }
  }
  hipError_t e = hipEventCreateWithFlags(&p->switch_ev, hipEventDisableTiming);
  if (e != hipSuccess) {
    for (int k = 0; k < 4; ++k) (void)hipEventDestroy(p->quarter_ev[k]);
    (void)hipHostFree(h);
    return hip_fail(e, "hipEventCreate");
  }
  p->h_ring = static_cast<char*>(h);
  p->device = dev;
  p->dev_ready = true;
  return CS_OK;
}

// All of a pool's work is chained on one stream at a time; a new stream first waits for the old.
cs_status use_stream(cs_pool* p, hipStream_t s) {
  if (p->have_stream && s != p->stream) {
    CS_HIP(hipEventRecord(p->switch_ev, p->stream), "hipEventRecord");
    CS_HIP(hipStreamWaitEvent(s, p->switch_ev, 0), "hipStreamWaitEvent");
  }
  p->stream = s;
  p->have_stream = true;
  return CS_OK;
}

hipError_t take_event(cs_pool* p, hipEvent_t* e) {
  if (!p->ev_free.empty()) {
    *e = p->ev_free.back();
    p->ev_free.pop_back();
    return hipSuccess;
  }
  return hipEventCreate(e);
}

// Launch a kernel on stream `s`; while profiling, bracket it with timing events on that stream
// (inside an open span the span's events cover it and it only counts as one more launch).
template <typename F>
cs_status timed_launch_on(cs_pool* p, hipStream_t s, int kind, const char* what, F&& launch) {
  if (p->fail_after == 0) return fail(CS_EHIP, std::string(what) + ": failure injected by cs_debug_fail_launches");
  if (p->fail_after > 0) --p->fail_after;
  if (p->prof_on && p->span_open) {
    CS_HIP(launch(), what);
    ++p->span_launches;
    return CS_OK;
  }
  hipEvent_t a = nullptr, b = nullptr;
  if (p->prof_on) {
    CS_HIP(take_event(p, &a), "hipEventCreate");
    CS_HIP(take_event(p, &b), "hipEventCreate");
    CS_HIP(hipEventRecord(a, s), "hipEventRecord");
  }
  CS_HIP(launch(), what);
  if (p->prof_on) {
    CS_HIP(hipEventRecord(b, s), "hipEventRecord");
    p->prof_events.push_back({a, b, kind, 1});
  }
  return CS_OK;
}

// Open a timing span of `kind` on stream `s` (no-op while profiling is off). A run of launches
// then records two events in all instead of two per launch, which keeps the instrumentation's own
// cost out of multi-layer steps; the span's time includes the short gaps between its launches.
cs_status span_begin(cs_pool* p, hipStream_t s, int kind) {
  if (!p->prof_on) return CS_OK;
  hipEvent_t a = nullptr;
  CS_HIP(take_event(p, &a), "hipEventCreate");
  const hipError_t e = hipEventRecord(a, s);
  if (e != hipSuccess) {
    p->ev_free.push_back(a);
    return hip_fail(e, "hipEventRecord");
  }
  p->span_start = a;
  p->span_open = true;
  p->span_stream = s;
  p->span_kind = kind;
  p->span_launches = 0;
  return CS_OK;
}

// Close the open span (no-op if none is open); called on error paths too.
cs_status span_end(cs_pool* p) {
  if (!p->span_open) return CS_OK;
  p->span_open = false;
  hipEvent_t b = nullptr;
  hipError_t e = take_event(p, &b);
  if (e == hipSuccess) {
    e = hipEventRecord(b, p->span_stream);
    if (e != hipSuccess) p->ev_free.push_back(b);
  }
  if (e != hipSuccess) {
    p->ev_free.push_back(p->span_start);
    return hip_fail(e, "hipEventRecord");
  }
  p->prof_events.push_back({p->span_start, b, p->span_kind, p->span_launches});
  return CS_OK;
}

template <typename F>
cs_status timed_launch(cs_pool* p, int kind, const char* what, F&& launch) {
  return timed_launch_on(p, p->stream, kind, what, launch);
}

// The second stream and its fork/join events, created on first use.
cs_status ensure_side(cs_pool* p) {
  if (p->side) return CS_OK;
  hipStream_t s = nullptr;
  CS_HIP(hipStreamCreateWithFlags(&s, hipStreamNonBlocking), "hipStreamCreate");
  hipEvent_t f = nullptr, j = nullptr;
  hipError_t e = hipEventCreateWithFlags(&f, hipEventDisableTiming);
  if (e == hipSuccess) e = hipEventCreateWithFlags(&j, hipEventDisableTiming);
  if (e != hipSuccess) {
    if (f) (void)hipEventDestroy(f);
    (void)hipStreamDestroy(s);
    return hip_fail(e, "hipEventCreate");
  }
  p->side = s;
  p->fork_ev = f;
  p->join_ev = j;
  return CS_OK;
}

// Reserve `n` bytes of the metadata ring inside one quarter. Entering a quarter records an event
// closing the previous one (everything enqueued so far) and waits for the event that closed the
// entered quarter last time round, so a region is never rewritten while a copy or kernel of an
// earlier call may still read it.
cs_status ring_reserve(cs_pool* p, size_t n, size_t* off_out) {
  n = align_up(std::max<size_t>(n, 1), kAlign);
  if (n > kQuarter) return fail(CS_ENOMEM, "metadata for one launch exceeds the upload ring");
  size_t off = p->ring_head;
  if (off / kQuarter != (off + n - 1) / kQuarter || off + n > kRingBytes)
    off = ((off + kQuarter - 1) / kQuarter) * kQuarter;
  if (off + n > kRingBytes) off = 0;
  const int q = static_cast<int>(off / kQuarter);
  if (q != p->cur_quarter) {
    if (p->cur_quarter >= 0) {
      CS_HIP(hipEventRecord(p->quarter_ev[p->cur_quarter], p->stream), "hipEventRecord");
      p->quarter_used[p->cur_quarter] = true;
    }
    if (p->quarter_used[q]) CS_HIP(hipEventSynchronize(p->quarter_ev[q]), "hipEventSynchronize");
    p->cur_quarter = q;
  }
  p->ring_head = off + n;
  *off_out = off;
  return CS_OK;
}

// Copy host bytes into the ring and enqueue their upload; returns the device address.
cs_status upload(cs_pool* p, const void* src, size_t n, void** dev_out) {
  size_t off = 0;
  cs_status st = ring_reserve(p, n, &off);
  if (st != CS_OK) return st;
  std::memcpy(p->h_ring + off, src, n);
  char* d = p->ws + p->lay.ring + off;
  CS_HIP(hipMemcpyAsync(d, p->h_ring + off, n, hipMemcpyHostToDevice, p->stream), "hipMemcpyAsync");
  *dev_out = d;
  return CS_OK;
}

// Launch metadata being laid out on the host: arrays at 16-byte offsets of one block.
struct Blob {
  std::vector<char> bytes;
  template <typename T>
  size_t push(const T* a, size_t n) {
    const size_t off = align_up(bytes.size(), 16);
    bytes.resize(align_up(off + n * sizeof(T), 16));
    if (n > 0) std::memcpy(bytes.data() + off, a, n * sizeof(T));
    return off;
  }
};

// The block as a launch reads it: in the launch's own arguments if it fits there, else uploaded.
cs_status place_meta(cs_pool* p, const Blob& b, cs::Meta* m) {
  m->host = b.bytes.data();
  m->bytes = b.bytes.size();
  m->dev = nullptr;
  if (b.bytes.size() <= cs::kMetaBytes) return CS_OK;
  void* d = nullptr;
  cs_status st = upload(p, b.bytes.data(), b.bytes.size(), &d);
  m->dev = d;
  return st;
}

// Part of an uploaded block.
cs::Meta meta_part(const void* dev, size_t off, size_t bytes) {
  cs::Meta m;
  m.dev = static_cast<const char*>(dev) + off;
  m.bytes = bytes;
  return m;
}

cs_status check_convs(cs_pool* p, int32_t n, const cs_conv* convs, std::vector<const cs::Conv*>& out) {
  if (n < 0) return fail(CS_EINVAL, "negative batch size");
  if (n > 0 && !convs) return fail(CS_EINVAL, "null conversation array");
  out.clear();
  out.reserve(static_cast<size_t>(n));
  // Slots of this batch are stamped with its number (one slot has one valid handle at a time); the
  // stamps start over when the counter wraps.
  if (p->seen.empty()) p->seen.assign(static_cast<size_t>(p->desc.max_convs), 0);
  if (++p->batch == 0) {
    std::fill(p->seen.begin(), p->seen.end(), 0u);
    p->batch = 1;
  }
  for (int32_t i = 0; i < n; ++i) {
    const cs::Conv* c = p->convs.find(convs[i]);
    if (!c) return fail(CS_ENOENT, "unknown conversation handle " + std::to_string(convs[i]));
    uint32_t& mark = p->seen[static_cast<size_t>(cs::ConvTable::slot_of(convs[i]))];
    if (mark == p->batch)
      return fail(CS_EINVAL, "conversation " + std::to_string(convs[i]) + " appears twice in a batch");
    mark = p->batch;
    out.push_back(c);
  }
  return CS_OK;
}

size_t wire_size(const cs_pool_desc& d, int64_t len) {
  return static_cast<size_t>(d.n_layers) * static_cast<size_t>(cs::pages_for(len)) *
         static_cast<size_t>(d.n_kv_heads) * 2 * cs::kPage * static_cast<size_t>(d.head_dim) * 2;
}

hipStream_t as_stream(cs_stream s) { return reinterpret_cast<hipStream_t>(s); }

// Extend/prefill work, launchable for any layer: one part, or several where the tiles exceed one
// quarter of the ring. `blobs` keeps the bytes of parts that travel in the launch arguments.
struct ExtendWork {
  std::vector<cs::ExtendLaunch> parts;
  std::vector<Blob> blobs;
};

cs::ExtendPlan plan_extend_batch(const cs_pool* p, const std::vector<int32_t>& slots,
                                 const std::vector<int64_t>& lens, const std::vector<int32_t>& q_lens) {
  const int tile = cs::extend_query_tile(p->desc.n_q_heads / p->desc.n_kv_heads);
  cs::ExtendPlan plan = cs::plan_extend(slots, lens, q_lens, tile);
  // A cut plan is one part: a part's merges follow its launch and read every piece of their tiles. Beside
  // the descriptors of some 129,000 conversations (nearly all without queries) there is no room for it.
  if (plan.convs.size() * sizeof(cs::ExtendConvDesc) + kMaxCutBytes <= kQuarter)
    cs::split_extend(plan, p->desc.n_kv_heads, cs::kCus, kExtendRecords);
  return plan;
}

// Tiles [t0, t1) of a plan with its conversations, laid out at the end of the block; offsets of
// the launch are relative to *off.
cs::ExtendLaunch push_extend(const cs::ExtendPlan& plan, size_t t0, size_t t1, Blob* b, size_t* off) {
  cs::ExtendLaunch e;
  *off = b->push(plan.convs.data(), plan.convs.size());
  e.tiles_off = b->push(plan.tiles.data() + t0, t1 - t0) - *off;
  e.merges_off = b->push(plan.merges.data(), plan.merges.size()) - *off;
  e.n_tiles = static_cast<int>(t1 - t0);
  e.n_merges = static_cast<int>(plan.merges.size());
  e.piece = plan.piece;
  e.n_parts = plan.n_parts;
  e.chained = plan.n_parts > 0 && plan.merges.empty();
  e.q_rows = plan.convs.empty() ? 0 : plan.convs.back().q_row + plan.convs.back().q_len;
  return e;
}

// Tiles one part of a plan holds, beside its conversations (0: not even one).
size_t extend_part_tiles(const cs::ExtendPlan& plan) {
  const size_t desc_bytes = align_up(plan.convs.size() * sizeof(cs::ExtendConvDesc), 16);
  if (desc_bytes + kAlign + sizeof(cs::ExtendTile) > kQuarter) return 0;
  return (kQuarter - desc_bytes - kAlign) / sizeof(cs::ExtendTile);
}

// Tiles [t0, t1) of a plan as one more part of `w`.
cs_status place_extend(cs_pool* p, const cs::ExtendPlan& plan, size_t t0, size_t t1, ExtendWork* w) {
  Blob b;
  size_t off = 0;
  cs::ExtendLaunch e = push_extend(plan, t0, std::min(plan.tiles.size(), t1), &b, &off);
  const cs_status st = place_meta(p, b, &e.meta);
  if (st != CS_OK) return st;
  w->parts.push_back(e);
  w->blobs.push_back(std::move(b));   // moving a vector keeps its buffer, which e.meta.host points to
  return CS_OK;
}

// Layers [0, n_layers) of a step from `layer` on; q and out hold them one after the other. The layers
// of one launch are as many as the records of their cut tiles have room for.
cs_status launch_extend_layers(cs_pool* p, const ExtendWork& w, int layer, int n_layers, const void* q, void* out,
                               hipStream_t s) {
  const cs::PoolGeom g = p->geom();
  const size_t row_bytes = static_cast<size_t>(g.n_q_heads) * g.head_dim * 2;
  for (const auto& e : w.parts) {
    const int per = std::min(kMaxLayersPerLaunch,
                             e.n_parts == 0 ? n_layers : std::max(1, extend_records(p->desc) / (e.n_parts * g.n_kv_heads)));
    for (int l = 0; l < n_layers; l += per) {
      const int nl = std::min(per, n_layers - l);
      const char* ql = static_cast<const char*>(q) + l * e.q_rows * row_bytes;
      char* ol = static_cast<char*>(out) + l * e.q_rows * row_bytes;
      cs_status st = timed_launch_on(p, s, CS_PROF_ATTN_FWD, "attention launch", [&] {
        return cs::launch_extend(g, layer + l, nl, e, ql, ol, p->ext_parts(), s);
      });
      if (st == CS_OK && e.n_merges > 0)
        st = timed_launch_on(p, s, CS_PROF_ATTN_FWD, "attention merge launch",
                             [&] { return cs::launch_extend_merge(g, nl, e, ol, p->ext_parts(), s); });
      if (st != CS_OK) return st;
    }
  }
  return CS_OK;
}

// Layers [0, n_layers) of a plan of any number of parts, each launched before the next is uploaded: the
// ring holds four quarters, so a part that waited for the fourth after it would be gone.
cs_status run_extend(cs_pool* p, const cs::ExtendPlan& plan, int layer, int n_layers, const void* q, void* out) {
  const size_t per = extend_part_tiles(plan);
  if (per == 0) return fail(CS_ENOMEM, "batch descriptor exceeds the metadata ring");
  for (size_t t0 = 0; t0 < plan.tiles.size(); t0 += per) {
    ExtendWork w;
    cs_status st = place_extend(p, plan, t0, t0 + per, &w);
    if (st == CS_OK) st = launch_extend_layers(p, w, layer, n_layers, q, out, p->stream);
    if (st != CS_OK) return st;
  }
  return CS_OK;
}

struct DecodeWork {
  cs::DecodeLaunch w;
  Blob blob;
  bool single = false;  // one work item per conversation: the split writes the output directly
};

cs::DecodePlan plan_decode_batch(const cs_pool* p, const std::vector<int32_t>& slots,
                                 const std::vector<int64_t>& lens) {
  return cs::plan_decode_filling(slots, lens, p->desc.n_kv_heads, kDecodeTargetItems, cs::kCus);
}

// Descriptors and launch order of a decode plan, as laid out back to back.
size_t decode_upload_bytes(const cs::DecodePlan& plan) {
  return align_up(plan.convs.size() * sizeof(cs::DecodeConvDesc), 16) + plan.order.size() * sizeof(int32_t);
}

cs_status check_decode_plan(const cs_pool* p, const cs::DecodePlan& plan) {
  if (plan.n_items > max_decode_items(p->desc)) return fail(CS_ENOMEM, "decode partials exceed the workspace");
  if (decode_upload_bytes(plan) > kQuarter) return fail(CS_ENOMEM, "batch descriptor exceeds the metadata ring");
  return CS_OK;
}

// A plan laid out at the end of the block; offsets of the launch are relative to *off.
cs::DecodeLaunch push_decode(const cs::DecodePlan& plan, Blob* b, size_t* off) {
  cs::DecodeLaunch w;
  *off = b->push(plan.convs.data(), plan.convs.size());
  w.order_off = b->push(plan.order.data(), plan.order.size()) - *off;
  w.n_convs = static_cast<int>(plan.convs.size());
  w.n_items = plan.n_items;
  w.split = plan.split_tokens;
  return w;
}

cs_status place_decode(cs_pool* p, const cs::DecodePlan& plan, DecodeWork* dw) {
  size_t off = 0;
  dw->w = push_decode(plan, &dw->blob, &off);
  dw->single = plan.single_item;
  return place_meta(p, dw->blob, &dw->w.meta);
}

// Split, then merge, of n_layers layers from `layer` on (q and out hold them one after the other); when
// every conversation is one work item the split writes the output itself. The layers of one launch
// are as many as their records have room for.
cs_status launch_decode_layers(cs_pool* p, const DecodeWork& w, int layer, int n_layers, const void* q, void* out) {
  const cs::PoolGeom g = p->geom();
  const size_t row_bytes = static_cast<size_t>(g.n_q_heads) * g.head_dim * 2;
  const size_t records = static_cast<size_t>(w.w.n_items) * g.n_q_heads * cs::partial_floats(g.head_dim);
  const int room = static_cast<int>(std::min<size_t>(kMaxLayersPerLaunch, p->lay.partial_floats / records));
  const int per = w.single ? kMaxLayersPerLaunch : room;   // room >= 1: check_decode_plan
  for (int l = 0; l < n_layers; l += per) {
    const int nl = std::min(per, n_layers - l);
    const char* ql = static_cast<const char*>(q) + l * w.w.n_convs * row_bytes;
    char* ol = static_cast<char*>(out) + l * w.w.n_convs * row_bytes;
    cs_status st = timed_launch(p, CS_PROF_DECODE_SPLIT, "decode split launch", [&] {
      return cs::launch_decode_split(g, layer + l, nl, w.w, ql, p->partials(), w.single ? ol : nullptr, p->stream);
    });
    if (st == CS_OK && !w.single)
      st = timed_launch(p, CS_PROF_DECODE_MERGE, "decode merge launch",
                        [&] { return cs::launch_decode_merge(g, nl, w.w, p->partials(), ol, p->stream); });
    if (st != CS_OK) return st;
  }
  return CS_OK;
}

cs_status attend(cs_pool* p, int32_t n, const cs_conv* convs, const int32_t* q_lens, int32_t layer,
                 const void* q, void* out, cs_stream stream, bool turn1) {
  if (!p) return fail(CS_EINVAL, "null pool");
  std::vector<const cs::Conv*> cv;
  cs_status st = check_convs(p, n, convs, cv);
  if (st != CS_OK) return st;
  if (n > 0 && !q_lens) return fail(CS_EINVAL, "null q_lens");
  if (layer < 0 || layer >= p->desc.n_layers) return fail(CS_ERANGE, "layer out of range");
  int64_t rows = 0;
  for (int32_t i = 0; i < n; ++i) {
    if (q_lens[i] < 0) return fail(CS_EINVAL, "negative q_len");
    if (q_lens[i] > cv[i]->len)
      return fail(CS_ESTATE, "q_len " + std::to_string(q_lens[i]) + " exceeds conversation length " +
                                 std::to_string(cv[i]->len));
    if (turn1 && q_lens[i] != cv[i]->len)
      return fail(CS_ESTATE, "turn-1 prefill needs q_len == conversation length (append the prompt first)");
    rows += q_lens[i];
  }
  if (rows == 0) return CS_OK;
  if (rows > INT32_MAX) return fail(CS_EINVAL, "too many query rows");
  if (!q || !out) return fail(CS_EINVAL, "null q/out");
  if ((st = ensure_device(p)) != CS_OK) return st;
  if ((st = use_stream(p, as_stream(stream))) != CS_OK) return st;

  std::vector<int32_t> slots(n), ql(q_lens, q_lens + n);
  std::vector<int64_t> lens(n);
  for (int32_t i = 0; i < n; ++i) {
    slots[i] = cs::ConvTable::slot_of(convs[i]);
    lens[i] = cv[i]->len;
  }
  return run_extend(p, plan_extend_batch(p, slots, lens, ql), layer, 1, q, out);
}

// Whether the conversations can take n_new[i] tokens each (nothing is changed); *total = their sum.
cs_status check_append(const cs_pool* p, const std::vector<const cs::Conv*>& cv, const int32_t* n_new, const void* k,
                       const void* v, int64_t* total_out) {
  int64_t total = 0, need_pages = 0;
  for (size_t i = 0; i < cv.size(); ++i) {
    if (n_new[i] < 0) return fail(CS_EINVAL, "negative token count");
    const int64_t nl = cv[i]->len + n_new[i];
    if (cs::pages_for(nl) > p->desc.max_pages_per_conv)
      return fail(CS_ERANGE, "conversation would exceed max_pages_per_conv");
    need_pages += cs::pages_for(nl) - cs::pages_for(cv[i]->len);
    total += n_new[i];
  }
  *total_out = total;
  if (total == 0) return CS_OK;
  if (total > INT32_MAX) return fail(CS_EINVAL, "too many tokens in one append");
  if (!k || !v) return fail(CS_EINVAL, "null k/v");
  if (need_pages > p->pages.free_count())
    return fail(CS_ENOMEM, "KV pool exhausted: need " + std::to_string(need_pages) + " pages, " +
                               std::to_string(p->pages.free_count()) + " free");
  return CS_OK;
}

// `carry` (may be null): metadata of the launches that follow the append in the same call; on success
// *carry_dev is its device address.
cs_status append_impl(cs_pool* p, int32_t n, const cs_conv* convs, const int32_t* n_new,
                      const void* k, const void* v, cs_stream stream, const Blob* carry = nullptr,
                      void** carry_dev = nullptr) {
  if (!p) return fail(CS_EINVAL, "null pool");
  std::vector<const cs::Conv*> cv;
  cs_status st = check_convs(p, n, convs, cv);
  if (st != CS_OK) return st;
  if (n > 0 && !n_new) return fail(CS_EINVAL, "null n_new");
  int64_t total = 0;
  if ((st = check_append(p, cv, n_new, k, v, &total)) != CS_OK || total == 0) return st;
  if ((st = ensure_device(p)) != CS_OK) return st;
  if ((st = use_stream(p, as_stream(stream))) != CS_OK) return st;

  // Reserve pages (cannot fail now) and build the chunks; lengths are committed only after every
  // upload and launch has been issued. If one of those fails, the reserved pages go back to the
  // free list in their old order and nothing about the conversations changes. (Launches already
  // issued may have written the new tokens into the reserved pages and into unused slots past a
  // conversation's end; no kernel reads those: attention masks keys past the length, pack writes
  // zeros there, and the pages return to the free list.)
  std::vector<int32_t> slots(n), nn(n_new, n_new + n);
  std::vector<int64_t> old_lens(n);
  std::vector<size_t> old_pages(n);
  std::vector<const std::vector<int32_t>*> lists(n);
  for (int32_t i = 0; i < n; ++i) {
    cs::Conv* c = p->convs.find(convs[i]);
    slots[i] = cs::ConvTable::slot_of(convs[i]);
    old_lens[i] = c->len;
    old_pages[i] = c->pages.size();
    p->pages.alloc(cs::pages_for(c->len + n_new[i]) - cs::pages_for(c->len), c->pages);
    lists[i] = &c->pages;
  }
  std::vector<cs::PageChunk> chunks = cs::plan_append(slots, old_lens, nn, lists);
  auto roll_back = [&] {
    std::vector<int32_t> taken;
    for (int32_t i = 0; i < n; ++i) {
      cs::Conv* c = p->convs.find(convs[i]);
      taken.insert(taken.end(), c->pages.begin() + static_cast<std::ptrdiff_t>(old_pages[i]), c->pages.end());
      c->pages.resize(old_pages[i]);
    }
    p->pages.unalloc(taken);
  };

  const cs::PoolGeom g = p->geom();
  const size_t carry_bytes = carry ? carry->bytes.size() : 0;
  auto launch = [&](const cs::Meta& m, int n_chunks, const cs::AppendCarry& c) {
    return timed_launch(p, CS_PROF_APPEND, "append launch",
                        [&] { return cs::launch_append(g, m, n_chunks, c, k, v, total, p->stream); });
  };
  if (chunks.size() * sizeof(cs::PageChunk) + carry_bytes <= cs::kMetaBytes) {
    // small: the chunks travel in the launch's arguments, and so does the metadata of the launches
    // that follow, which the append kernel stores to the ring's device half.
    Blob b;
    b.push(chunks.data(), chunks.size());
    cs::AppendCarry c;
    if (carry_bytes > 0) {
      size_t off = 0;
      st = ring_reserve(p, carry_bytes, &off);
      c.dst = p->ws + p->lay.ring + off;
      c.bytes = carry_bytes;
      c.off = b.push(carry->bytes.data(), carry_bytes);
      *carry_dev = c.dst;
    }
    cs::Meta m;
    m.host = b.bytes.data();
    m.bytes = b.bytes.size();
    if (st == CS_OK) st = launch(m, static_cast<int>(chunks.size()), c);
  } else {
    const size_t per = kQuarter / sizeof(cs::PageChunk) - 1;
    for (size_t c0 = 0; c0 < chunks.size() && st == CS_OK; c0 += per) {
      const size_t c1 = std::min(chunks.size(), c0 + per);
      void* d = nullptr;
      st = upload(p, chunks.data() + c0, (c1 - c0) * sizeof(cs::PageChunk), &d);
      if (st == CS_OK)
        st = launch(meta_part(d, 0, (c1 - c0) * sizeof(cs::PageChunk)), static_cast<int>(c1 - c0), {});
    }
    // After the chunks, which may go round the ring: nothing of it is reused before the launches that read
    // the carried metadata are issued.
    if (carry_bytes > 0 && st == CS_OK) st = upload(p, carry->bytes.data(), carry_bytes, carry_dev);
  }
  if (st != CS_OK) {
    roll_back();
    return st;
  }
  for (int32_t i = 0; i < n; ++i) p->convs.find(convs[i])->len += n_new[i];
  return CS_OK;
}

}  // namespace

extern "C" {

const char* cs_last_error(void) { return g_err.c_str(); }

size_t cs_pool_kv_bytes(const cs_pool_desc* d) {
  if (desc_problem(d)) return 0;
  return static_cast<size_t>(d->n_layers) * static_cast<size_t>(d->n_pages) *
         static_cast<size_t>(d->n_kv_heads) * 2 * cs::kPage * static_cast<size_t>(d->head_dim) * 2;
}

size_t cs_pool_workspace_bytes(const cs_pool_desc* d) {
  if (desc_problem(d)) return 0;
  return ws_layout(*d).total;
}

cs_status cs_pool_create(const cs_pool_desc* d, void* kv_base, size_t kv_bytes, void* ws_base,
                         size_t ws_bytes, uint64_t seed, cs_pool** out) {
  if (const char* why = desc_problem(d)) return fail(CS_EINVAL, why);
  if (!out) return fail(CS_EINVAL, "null out");
  if (!kv_base || !ws_base) return fail(CS_EINVAL, "null kv or workspace base");
  if (reinterpret_cast<uintptr_t>(kv_base) % kAlign || reinterpret_cast<uintptr_t>(ws_base) % kAlign)
    return fail(CS_EINVAL, "kv and workspace bases must be 256-byte aligned");
  if (kv_bytes < cs_pool_kv_bytes(d)) return fail(CS_EINVAL, "kv buffer smaller than cs_pool_kv_bytes");
  if (ws_bytes < cs_pool_workspace_bytes(d))
    return fail(CS_EINVAL, "workspace smaller than cs_pool_workspace_bytes");
  cs_pool* p = new (std::nothrow)
      cs_pool(*d, static_cast<char*>(kv_base), kv_bytes, static_cast<char*>(ws_base), ws_bytes, seed);
  if (!p) return fail(CS_ENOMEM, "host allocation failed");
  *out = p;
  return CS_OK;
}

cs_status cs_pool_destroy(cs_pool* p) {
  if (!p) return fail(CS_EINVAL, "null pool");
  cs_status st = CS_OK;
  if (p->dev_ready) {
    if (p->have_stream && hipStreamSynchronize(p->stream) != hipSuccess)
      st = fail(CS_EHIP, "hipStreamSynchronize failed while destroying the pool");
    for (auto& e : p->quarter_ev) (void)hipEventDestroy(e);
    for (auto& e : p->ev_free) (void)hipEventDestroy(e);
    for (auto& pe : p->prof_events) {
      (void)hipEventDestroy(pe.start);
      (void)hipEventDestroy(pe.stop);
    }
    (void)hipEventDestroy(p->switch_ev);
    if (p->side) {
      if (hipStreamSynchronize(p->side) != hipSuccess)
        st = fail(CS_EHIP, "hipStreamSynchronize failed while destroying the pool");
      (void)hipEventDestroy(p->fork_ev);
      (void)hipEventDestroy(p->join_ev);
      (void)hipStreamDestroy(p->side);
    }
    (void)hipHostFree(p->h_ring);
  }
  delete p;
  return st;
}

cs_status cs_pool_occupancy(const cs_pool* p, int64_t* used, int64_t* free_pages) {
  if (!p || !used || !free_pages) return fail(CS_EINVAL, "null argument");
  *used = p->pages.used_count();
  *free_pages = p->pages.free_count();
  return CS_OK;
}

cs_status cs_conv_create(cs_pool* p, cs_conv* out) {
  if (!p || !out) return fail(CS_EINVAL, "null argument");
  if (!p->convs.create(out)) return fail(CS_ENOMEM, "all conversation slots are live");
  return CS_OK;
}

cs_status cs_conv_destroy(cs_pool* p, cs_conv conv) {
  if (!p) return fail(CS_EINVAL, "null pool");
  if (!p->convs.find(conv)) return fail(CS_ENOENT, "unknown conversation handle");
  p->convs.destroy(conv, p->pages);
  return CS_OK;
}

cs_status cs_conv_len(const cs_pool* p, cs_conv conv, int64_t* tokens) {
  if (!p || !tokens) return fail(CS_EINVAL, "null argument");
  const cs::Conv* c = p->convs.find(conv);
  if (!c) return fail(CS_ENOENT, "unknown conversation handle");
  *tokens = c->len;
  return CS_OK;
}

cs_status cs_conv_pages(const cs_pool* p, cs_conv conv, int32_t* out, int64_t cap, int64_t* n) {
  if (!p || !n) return fail(CS_EINVAL, "null argument");
  const cs::Conv* c = p->convs.find(conv);
  if (!c) return fail(CS_ENOENT, "unknown conversation handle");
  *n = static_cast<int64_t>(c->pages.size());
  if (cap < *n) return fail(CS_ERANGE, "output capacity smaller than the page count");
  if (*n > 0 && !out) return fail(CS_EINVAL, "null output");
  std::copy(c->pages.begin(), c->pages.end(), out);
  return CS_OK;
}

cs_status cs_kv_append(cs_pool* p, cs_conv conv, int32_t n_new, const void* k, const void* v,
                       cs_stream stream) {
  return append_impl(p, 1, &conv, &n_new, k, v, stream);
}

cs_status cs_kv_append_batch(cs_pool* p, int32_t n_convs, const cs_conv* convs, const int32_t* n_new,
                             const void* k, const void* v, cs_stream stream) {
  return append_impl(p, n_convs, convs, n_new, k, v, stream);
}

cs_status cs_attn_prefill_turn1(cs_pool* p, int32_t n, const cs_conv* convs, const int32_t* q_lens,
                                int32_t layer, const void* q, void* out, cs_stream stream) {
  return attend(p, n, convs, q_lens, layer, q, out, stream, true);
}

cs_status cs_attn_extend(cs_pool* p, int32_t n, const cs_conv* convs, const int32_t* q_lens,
                         int32_t layer, const void* q, void* out, cs_stream stream) {
  return attend(p, n, convs, q_lens, layer, q, out, stream, false);
}

cs_status cs_attn_decode_batch(cs_pool* p, int32_t n, const cs_conv* convs, int32_t layer,
                               const void* q, void* out, cs_stream stream) {
  if (!p) return fail(CS_EINVAL, "null pool");
  std::vector<const cs::Conv*> cv;
  cs_status st = check_convs(p, n, convs, cv);
  if (st != CS_OK) return st;
  if (layer < 0 || layer >= p->desc.n_layers) return fail(CS_ERANGE, "layer out of range");
  for (int32_t i = 0; i < n; ++i)
    if (cv[i]->len < 1) return fail(CS_ESTATE, "decode on an empty conversation");
  if (n == 0) return CS_OK;
  if (!q || !out) return fail(CS_EINVAL, "null q/out");
  if ((st = ensure_device(p)) != CS_OK) return st;
  if ((st = use_stream(p, as_stream(stream))) != CS_OK) return st;
  std::vector<int32_t> slots(n);
  std::vector<int64_t> lens(n);
  for (int32_t i = 0; i < n; ++i) {
    slots[i] = cs::ConvTable::slot_of(convs[i]);
    lens[i] = cv[i]->len;
  }
  const cs::DecodePlan plan = plan_decode_batch(p, slots, lens);
  if ((st = check_decode_plan(p, plan)) != CS_OK) return st;
  DecodeWork w;
  if ((st = place_decode(p, plan, &w)) != CS_OK) return st;
  return launch_decode_layers(p, w, layer, 1, q, out);
}

cs_status cs_attn_decode_batch_noalloc(cs_pool* p, int32_t n, const cs_conv* convs, int32_t layer,
                                       const void* q, void* out, cs_stream stream) {
  if (!p) return fail(CS_EINVAL, "null pool");
  std::vector<const cs::Conv*> cv;
  cs_status st = check_convs(p, n, convs, cv);
  if (st != CS_OK) return st;
  if (layer < 0 || layer >= p->desc.n_layers) return fail(CS_ERANGE, "layer out of range");
  for (int32_t i = 0; i < n; ++i)
    if (cv[i]->len < 1) return fail(CS_ESTATE, "decode on an empty conversation");
  if (n == 0) return CS_OK;
  if (!q || !out) return fail(CS_EINVAL, "null q/out");
  // The pool's device state (metadata ring) is created by its first device call, which allocates;
  // every pool holding a non-empty conversation has made one (an append or an unpack).
  if (!p->dev_ready) return fail(CS_ESTATE, "pool has no device state yet (no append or unpack ran)");
  int dev = -1;
  CS_HIP(hipGetDevice(&dev), "hipGetDevice");
  if (dev != p->device) return fail(CS_EINVAL, "the current device is not the pool's device");
  std::vector<int32_t> slots(n);
  std::vector<int64_t> lens(n);
  for (int32_t i = 0; i < n; ++i) {
    slots[i] = cs::ConvTable::slot_of(convs[i]);
    lens[i] = cv[i]->len;
  }
  const cs::DecodePlan plan = plan_decode_batch(p, slots, lens);
  const size_t need = plan.single_item ? 0
      : static_cast<size_t>(plan.n_items) * p->desc.n_q_heads * cs::partial_floats(p->desc.head_dim);
  if (need > cs::kStaticScratchFloats)
    return fail(CS_ENOMEM, "decode partials (" + std::to_string(need * 4) + " bytes) exceed the " +
                               std::to_string(cs::kStaticScratchFloats * 4) + "-byte static scratch");
  if (decode_upload_bytes(plan) > kQuarter) return fail(CS_ENOMEM, "batch descriptor exceeds the metadata ring");
  float* scratch = nullptr;
  CS_HIP(cs::static_decode_scratch(&scratch), "hipGetSymbolAddress(decode scratch)");
  if ((st = use_stream(p, as_stream(stream))) != CS_OK) return st;
  DecodeWork w;
  if ((st = place_decode(p, plan, &w)) != CS_OK) return st;
  const cs::PoolGeom g = p->geom();
  // untimed launches: the timing events of cs_profile_* would be created on demand
  CS_HIP(cs::launch_decode_split(g, layer, 1, w.w, q, scratch, w.single ? out : nullptr, p->stream),
         "decode split launch");
  if (w.single) return CS_OK;
  CS_HIP(cs::launch_decode_merge(g, 1, w.w, scratch, out, p->stream), "decode merge launch");
  return CS_OK;
}

cs_status cs_kv_pack_size(const cs_pool* p, cs_conv conv, size_t* bytes) {
  if (!p || !bytes) return fail(CS_EINVAL, "null argument");
  const cs::Conv* c = p->convs.find(conv);
  if (!c) return fail(CS_ENOENT, "unknown conversation handle");
  *bytes = wire_size(p->desc, c->len);
  return CS_OK;
}

cs_status cs_kv_pack(const cs_pool* pc, cs_conv conv, void* dst, size_t dst_bytes, cs_stream stream) {
  cs_pool* p = const_cast<cs_pool*>(pc);  // host metadata is unchanged; stream/ring state is not
  if (!p) return fail(CS_EINVAL, "null pool");
  const cs::Conv* c = p->convs.find(conv);
  if (!c) return fail(CS_ENOENT, "unknown conversation handle");
  if (dst_bytes != wire_size(p->desc, c->len)) return fail(CS_EINVAL, "dst_bytes != cs_kv_pack_size");
  if (c->len == 0) return CS_OK;
  if (!dst) return fail(CS_EINVAL, "null dst");
  cs_status st;
  if ((st = ensure_device(p)) != CS_OK) return st;
  if ((st = use_stream(p, as_stream(stream))) != CS_OK) return st;
  return timed_launch(p, CS_PROF_PACK, "pack launch", [&] {
    return cs::launch_pack(p->geom(), cs::ConvTable::slot_of(conv), c->len, dst, p->stream);
  });
}

cs_status cs_kv_unpack(cs_pool* p, const void* src, size_t src_bytes, int64_t n_tokens,
                       cs_conv* out_conv, cs_stream stream) {
  if (!p || !out_conv) return fail(CS_EINVAL, "null argument");
  if (n_tokens < 1) return fail(CS_EINVAL, "n_tokens must be >= 1");
  if (!src) return fail(CS_EINVAL, "null src");
  const int64_t np = cs::pages_for(n_tokens);
  if (np > p->desc.max_pages_per_conv) return fail(CS_ERANGE, "conversation exceeds max_pages_per_conv");
  if (src_bytes != wire_size(p->desc, n_tokens))
    return fail(CS_EINVAL, "src_bytes does not match the wire size of n_tokens for this pool");
  if (p->convs.live_count() >= p->convs.max_convs()) return fail(CS_ENOMEM, "all conversation slots are live");
  if (np > p->pages.free_count()) return fail(CS_ENOMEM, "KV pool exhausted");
  cs_status st;
  if ((st = ensure_device(p)) != CS_OK) return st;
  if ((st = use_stream(p, as_stream(stream))) != CS_OK) return st;
  cs_conv h;
  p->convs.create(&h);
  cs::Conv* c = p->convs.find(h);
  p->pages.alloc(np, c->pages);
  c->len = n_tokens;
  *out_conv = h;
  const size_t per = kQuarter / sizeof(int32_t) - 64;
  for (size_t p0 = 0; p0 < c->pages.size(); p0 += per) {
    const size_t p1 = std::min(c->pages.size(), p0 + per);
    Blob b;
    b.push(c->pages.data() + p0, p1 - p0);
    cs::Meta m;
    if ((st = place_meta(p, b, &m)) != CS_OK) return st;
    st = timed_launch(p, CS_PROF_UNPACK, "unpack launch", [&] {
      return cs::launch_unpack(p->geom(), src, m, cs::ConvTable::slot_of(h),
                               n_tokens, static_cast<int>(p0), static_cast<int>(p1 - p0), p->stream);
    });
    if (st != CS_OK) return st;
  }
  return CS_OK;
}

cs_status cs_mixed_step(cs_pool* p, int32_t n_ext, const cs_conv* ext_convs, const int32_t* ext_lens,
                        int32_t n_dec, const cs_conv* dec_convs, const void* k, const void* v,
                        const void* q_ext, void* out_ext, const void* q_dec, void* out_dec,
                        uint32_t flags, cs_stream stream) {
  if (!p) return fail(CS_EINVAL, "null pool");
  if (n_ext < 0 || n_dec < 0) return fail(CS_EINVAL, "negative batch size");
  if (flags & ~static_cast<uint32_t>(CS_MIXED_LAYER_ORDERED)) return fail(CS_EINVAL, "unknown flags");
  if ((n_ext > 0 && (!ext_convs || !ext_lens)) || (n_dec > 0 && !dec_convs))
    return fail(CS_EINVAL, "null conversation or length array");
  std::vector<cs_conv> all;
  if (n_ext > 0) all.assign(ext_convs, ext_convs + n_ext);
  if (n_dec > 0) all.insert(all.end(), dec_convs, dec_convs + n_dec);
  std::vector<const cs::Conv*> cv;
  cs_status st = check_convs(p, static_cast<int32_t>(all.size()), all.data(), cv);
  if (st != CS_OK) return st;
  std::vector<int32_t> n_new;
  int64_t ext_rows = 0;
  for (int32_t i = 0; i < n_ext; ++i) {
    if (ext_lens[i] < 1) return fail(CS_EINVAL, "an extend chunk must hold at least one token");
    ext_rows += ext_lens[i];
    n_new.push_back(ext_lens[i]);
  }
  if (ext_rows > INT32_MAX) return fail(CS_EINVAL, "too many extend tokens");
  n_new.insert(n_new.end(), static_cast<size_t>(n_dec), 1);
  if (all.empty()) return CS_OK;
  if ((ext_rows > 0 && (!q_ext || !out_ext)) || (n_dec > 0 && (!q_dec || !out_dec)))
    return fail(CS_EINVAL, "null q/out");
  if (align_up(static_cast<size_t>(n_ext) * sizeof(cs::ExtendConvDesc), 16) + kAlign +
          sizeof(cs::ExtendTile) > kQuarter)
    return fail(CS_ENOMEM, "batch descriptor exceeds the metadata ring");
  // The decode plan covers each decoding conversation with its new token; it is checked before
  // the append so that a batch it cannot take leaves the pool unchanged.
  std::vector<int32_t> d_slots(n_dec);
  std::vector<int64_t> d_lens(n_dec);
  for (int32_t i = 0; i < n_dec; ++i) {
    d_slots[i] = cs::ConvTable::slot_of(dec_convs[i]);
    d_lens[i] = cv[n_ext + i]->len + 1;
  }
  cs::DecodePlan d_plan;
  if (n_dec > 0) {
    d_plan = plan_decode_batch(p, d_slots, d_lens);
    if ((st = check_decode_plan(p, d_plan)) != CS_OK) return st;
  }
  int64_t total = 0;
  if ((st = check_append(p, cv, n_new.data(), k, v, &total)) != CS_OK) return st;
  // The step's plans, laid out in one block that goes to the device with the append.
  std::vector<int32_t> e_slots(n_ext), e_q(n_new.begin(), n_new.begin() + n_ext);
  std::vector<int64_t> e_lens(n_ext);
  for (int32_t i = 0; i < n_ext; ++i) {
    e_slots[i] = cs::ConvTable::slot_of(ext_convs[i]);
    e_lens[i] = cv[i]->len + ext_lens[i];
  }
  cs::ExtendPlan e_plan = plan_extend_batch(p, e_slots, e_lens, e_q);
  const bool ordered = (flags & CS_MIXED_LAYER_ORDERED) != 0;
  const float dec_steps = cs::decode_steps(d_lens, p->desc.n_kv_heads, p->desc.head_dim, cs::kCus);
  if (cs::chain_pays(e_plan, p->desc.n_kv_heads, cs::kCus, ordered ? 1 : p->desc.n_layers, dec_steps))
    cs::chain_extend(e_plan);
  Blob blob;
  ExtendWork ew;
  DecodeWork dw;
  size_t e_off = 0, d_off = 0;
  if (n_dec > 0) {
    dw.w = push_decode(d_plan, &blob, &d_off);
    dw.single = d_plan.single_item;
  }
  const size_t d_bytes = blob.bytes.size();
  // an extend plan that does not fit beside the decode plan is uploaded by itself, maybe in parts
  const bool e_carried = n_ext > 0 && d_bytes + e_plan.convs.size() * sizeof(cs::ExtendConvDesc) +
                                              e_plan.tiles.size() * sizeof(cs::ExtendTile) +
                                              e_plan.merges.size() * sizeof(cs::ExtendMerge) + 64 <= kQuarter;
  if (e_carried) ew.parts.push_back(push_extend(e_plan, 0, e_plan.tiles.size(), &blob, &e_off));
  // append every new token (all layers); validates capacity and commits the host metadata
  void* dev = nullptr;
  if ((st = append_impl(p, static_cast<int32_t>(all.size()), all.data(), n_new.data(), k, v, stream, &blob, &dev)) !=
      CS_OK)
    return st;
  if (n_dec > 0) dw.w.meta = meta_part(dev, d_off, d_bytes);
  if (e_carried) ew.parts[0].meta = meta_part(dev, e_off, blob.bytes.size() - e_off);
  // Up to three parts stay in the ring beside the carried plan until the last launch that reads them is
  // issued; more are uploaded again where they are launched.
  const size_t per = n_ext > 0 ? extend_part_tiles(e_plan) : 1;   // > 0: checked above
  const bool e_held = e_carried || (e_plan.tiles.size() + per - 1) / per <= 3;
  if (n_ext > 0 && !e_carried && e_held)
    for (size_t t0 = 0; t0 < e_plan.tiles.size(); t0 += per)
      if ((st = place_extend(p, e_plan, t0, t0 + per, &ew)) != CS_OK) return st;
  const size_t row_bytes = static_cast<size_t>(p->desc.n_q_heads) * p->desc.head_dim * 2;
  const int nl = p->desc.n_layers;
  const size_t ext_layer_bytes = static_cast<size_t>(ext_rows) * row_bytes;
  const size_t dec_layer_bytes = static_cast<size_t>(n_dec) * row_bytes;
  auto q_e = [&](int l) { return static_cast<const char*>(q_ext) + l * ext_layer_bytes; };
  auto o_e = [&](int l) { return static_cast<char*>(out_ext) + l * ext_layer_bytes; };
  auto q_d = [&](int l) { return static_cast<const char*>(q_dec) + l * dec_layer_bytes; };
  auto o_d = [&](int l) { return static_cast<char*>(out_dec) + l * dec_layer_bytes; };
  if (!e_held) {
    // More metadata than the ring holds (100,000 chunks and more): everything on one stream, the decode
    // first, whose carried plan the parts of the extend plan go over; in layer order it is uploaded again.
    if (!(flags & CS_MIXED_LAYER_ORDERED)) {
      if (n_dec > 0) st = launch_decode_layers(p, dw, 0, nl, q_d(0), o_d(0));
      return st != CS_OK ? st : run_extend(p, e_plan, 0, nl, q_e(0), o_e(0));
    }
    for (int layer = 0; layer < nl && st == CS_OK; ++layer) {
      DecodeWork again;
      if (n_dec > 0) st = place_decode(p, d_plan, &again);
      if (n_dec > 0 && st == CS_OK) st = launch_decode_layers(p, again, layer, 1, q_d(layer), o_d(layer));
      if (st == CS_OK) st = run_extend(p, e_plan, layer, 1, q_e(layer), o_e(layer));
    }
    return st;
  }
  // Extend chunks and decode tokens are independent once their K/V is appended: with both present
  // the extend launches go to a second stream (forked from `stream`, joined back before the call
  // returns), so the matrix-core-bound extend work overlaps the HBM-bound decode work.
  const bool fork = n_ext > 0 && n_dec > 0;
  // layer order with one launch per layer (extend tiles + decode split) needs no second stream
  const bool fused_layers = (flags & CS_MIXED_LAYER_ORDERED) && fork && ew.parts.size() == 1;
  hipStream_t ext_stream = p->stream;
  if (fork && !fused_layers && (st = ensure_side(p)) != CS_OK) return st;
  if (fork && !fused_layers) ext_stream = p->side;
  auto fork_side = [&]() -> cs_status {
    CS_HIP(hipEventRecord(p->fork_ev, p->stream), "hipEventRecord");
    CS_HIP(hipStreamWaitEvent(p->side, p->fork_ev, 0), "hipStreamWaitEvent");
    return CS_OK;
  };
  auto join_side = [&]() -> cs_status {
    CS_HIP(hipEventRecord(p->join_ev, p->side), "hipEventRecord");
    CS_HIP(hipStreamWaitEvent(p->stream, p->join_ev, 0), "hipStreamWaitEvent");
    return CS_OK;
  };
  if (fused_layers) {
    // As in a model forward pass, one layer after the other; each layer is one launch with its
    // extend tiles and its decode split, then one that merges what they left in pieces.
    const cs::PoolGeom g = p->geom();
    const auto& e = ew.parts[0];
    for (int layer = 0; layer < nl && st == CS_OK; ++layer) {
      st = timed_launch(p, CS_PROF_MIXED_LAYER, "mixed layer launch", [&] {
        return cs::launch_mixed_layer(g, layer, e, q_e(layer), o_e(layer), p->ext_parts(), dw.w, q_d(layer),
                                      p->partials(), dw.single ? o_d(layer) : nullptr, p->stream);
      });
      if (st == CS_OK && (e.n_merges > 0 || !dw.single))
        st = timed_launch(p, CS_PROF_DECODE_MERGE, "mixed merge launch", [&] {
          return cs::launch_mixed_merge(g, e, o_e(layer), p->ext_parts(), dw.w, p->partials(),
                                        dw.single ? nullptr : o_d(layer), p->stream);
        });
    }
    return st;
  }
  if (flags & CS_MIXED_LAYER_ORDERED) {
    // As in a model forward pass: layer l's extend and decode overlap each other, and layer l+1
    // starts only once both are complete.
    for (int layer = 0; layer < nl && st == CS_OK; ++layer) {
      if (fork && (st = fork_side()) != CS_OK) return st;
      if (n_ext > 0) st = launch_extend_layers(p, ew, layer, 1, q_e(layer), o_e(layer), ext_stream);
      if (n_dec > 0 && st == CS_OK) st = launch_decode_layers(p, dw, layer, 1, q_d(layer), o_d(layer));
      if (fork) {  // join even after a failed launch, so later work never overtakes the side stream
        const cs_status sj = join_side();
        if (st == CS_OK) st = sj;
      }
    }
    return st;
  }
  // Every layer's queries are inputs of this call, so no layer waits for another: one launch takes the
  // extend tiles of all layers on the side stream while one on the main stream decodes all layers
  // (each followed by its merge). Against a launch per layer this leaves no half-empty last round and
  // no gap per layer.
  if (fork && (st = fork_side()) != CS_OK) return st;
  if (n_ext > 0) st = span_begin(p, ext_stream, CS_PROF_ATTN_FWD);
  if (n_ext > 0 && st == CS_OK) st = launch_extend_layers(p, ew, 0, nl, q_e(0), o_e(0), ext_stream);
  if (const cs_status se = span_end(p); st == CS_OK) st = se;
  if (n_dec > 0 && st == CS_OK) st = launch_decode_layers(p, dw, 0, nl, q_d(0), o_d(0));
  if (fork) {  // join even after a failed launch, so later work never overtakes the side stream
    const cs_status sj = join_side();
    if (st == CS_OK) st = sj;
  }
  return st;
}

cs_status cs_device_info(int32_t device, cs_device_info_t* out) {
  if (!out) return fail(CS_EINVAL, "null out");
  hipDeviceProp_t pr;
  CS_HIP(hipGetDeviceProperties(&pr, device), "hipGetDeviceProperties");
  std::memset(out, 0, sizeof(*out));
  std::strncpy(out->name, pr.name, sizeof(out->name) - 1);
  std::strncpy(out->arch, pr.gcnArchName, sizeof(out->arch) - 1);
  out->cu_count = pr.multiProcessorCount;
  out->clock_khz = pr.clockRate;
  out->memory_clock_khz = pr.memoryClockRate;
  out->memory_bus_width_bits = pr.memoryBusWidth;
  out->lds_per_cu_bytes = static_cast<int64_t>(pr.maxSharedMemoryPerMultiProcessor);
  out->lds_per_block_bytes = static_cast<int64_t>(pr.sharedMemPerBlock);
  out->l2_bytes = pr.l2CacheSize;
  out->total_mem_bytes = static_cast<int64_t>(pr.totalGlobalMem);
  return CS_OK;
}

cs_status cs_probe_stream_read(const void* src, size_t bytes, void* sink, cs_stream stream) {
  if (!src || !sink) return fail(CS_EINVAL, "null src or sink");
  if (bytes % 16) return fail(CS_EINVAL, "bytes must be a multiple of 16");
  int dev = 0, cus = 0;
  CS_HIP(hipGetDevice(&dev), "hipGetDevice");
  CS_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev), "hipDeviceGetAttribute");
  CS_HIP(cs::launch_stream_read_probe(src, bytes, static_cast<uint32_t*>(sink), cus, as_stream(stream)),
         "stream read probe launch");
  return CS_OK;
}

cs_status cs_debug_fail_launches(cs_pool* p, int64_t after) {
  if (!p) return fail(CS_EINVAL, "null pool");
  p->fail_after = after < 0 ? -1 : after;
  return CS_OK;
}

cs_status cs_profile_start(cs_pool* p) {
  if (!p) return fail(CS_EINVAL, "null pool");
  for (auto& pe : p->prof_events) {
    p->ev_free.push_back(pe.start);
    p->ev_free.push_back(pe.stop);
  }
  p->prof_events.clear();
  p->prof_on = true;
  return CS_OK;
}

cs_status cs_profile_stop(cs_pool* p, double* ms, int64_t* launches) {
  if (!p || !ms || !launches) return fail(CS_EINVAL, "null argument");
  for (int k = 0; k < CS_PROF_KINDS; ++k) {
    ms[k] = 0.0;
    launches[k] = 0;
  }
  p->prof_on = false;
  for (auto& pe : p->prof_events) {
    CS_HIP(hipEventSynchronize(pe.stop), "hipEventSynchronize");
    float t = 0.f;
    CS_HIP(hipEventElapsedTime(&t, pe.start, pe.stop), "hipEventElapsedTime");
    ms[pe.kind] += t;
    launches[pe.kind] += pe.launches;
    p->ev_free.push_back(pe.start);
    p->ev_free.push_back(pe.stop);
  }
  p->prof_events.clear();
  return CS_OK;
}

}  // extern "C"
namespace cs {
// Error reporting shared with the other C-ABI translation units (sched_capi.cpp).
cs_status api_fail(cs_status code, const char* msg) { return fail(code, msg); }
}  // namespace cs
