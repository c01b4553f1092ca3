// Host-callable launchers of the gfx950 kernels (defined in the .hip files).
#pragma once

#include <hip/hip_runtime.h>

#include <cstring>

#include "host/host_state.hpp"

namespace cs {

struct PoolGeom {
  void* pool;          // device base of the KV pool
  int64_t n_pages;
  int n_layers;
  int n_kv_heads;
  int n_q_heads;
  int head_dim;
  int32_t* page_table;  // device mirror [max_convs][max_pages]
  int max_pages;
};

// Metadata of one launch (descriptors, work lists, page ids): `bytes` bytes laid out on the host at
// `host`, or already on the device at `dev` (a stream-ordered upload; `host` is then unused). A plan
// of at most kMetaBytes travels in the launch's own kernel arguments (dev = nullptr): an upload is a
// copy kernel of 2-5 us that the launch waits for (~8 us apart when nothing else is queued). Decode of
// 16 conversations of 1k-9k tokens 29.4 -> 25.6 us, one of 24k 25.6 -> 23.3, prefill of 1.4k tokens
// 39.4 -> 37.3; the larger argument block costs a launch of 690 us nothing measurable. Larger plans
// are uploaded: they belong to launches of many tiles. 3 KiB keeps every kernel's arguments inside
// the 4 KiB a launch may pass.
constexpr size_t kMetaBytes = 3072;
struct LaunchMeta {
  alignas(16) uint32_t w[kMetaBytes / 4];
};
struct Meta {
  const void* host = nullptr;
  const void* dev = nullptr;
  size_t bytes = 0;
  // false: neither uploaded nor small enough to travel with the launch
  bool ok() const { return dev != nullptr || (host != nullptr && bytes <= kMetaBytes); }
};

// The argument block of a launch whose plan is not on the device: the plan's bytes. (The rest of the
// block is not read.)
inline void fill_meta(const Meta& m, LaunchMeta* out) {
  if (m.dev == nullptr) std::memcpy(out->w, m.host, m.bytes);
}

// KV append: write chunks (meta: PageChunk[n_chunks]) of k,v [n_layers][src_rows][Hkv][D]. With
// carry_bytes > 0 the metadata travels in the kernel arguments and its bytes [carry_off, carry_off +
// carry_bytes) (multiples of 16) are also stored to carry_dst, for the launches that follow.
struct AppendCarry {
  void* dst = nullptr;
  size_t off = 0, bytes = 0;
};
hipError_t launch_append(const PoolGeom& g, const Meta& meta, int n_chunks, const AppendCarry& carry,
                         const void* k, const void* v, int64_t src_rows, hipStream_t stream);

// Pack: conversation pages (page-table row `slot`) -> wire [layer][lpage][head] blocks.
hipError_t launch_pack(const PoolGeom& g, int slot, int64_t len, void* wire, hipStream_t stream);

// Unpack: wire logical pages [lp0, lp0 + n_lp) -> physical pages (meta: int32[n_lp]) of the
// conversation in page-table row `slot` (length len).
hipError_t launch_unpack(const PoolGeom& g, const void* wire, const Meta& meta, int slot,
                         int64_t len, int lp0, int n_lp, hipStream_t stream);

// Decode partial record of one (work item, query head): o[d], running max m, sum l, two unused
// floats, so records stay 16-byte aligned.
constexpr int partial_floats(int head_dim) { return head_dim + 4; }

// A decode plan as the kernels read it: meta = DecodeConvDesc[n_convs], then (16-byte aligned, at
// order_off) the launch order of its n_items items (a permutation).
struct DecodeLaunch {
  Meta meta;
  size_t order_off = 0;
  int n_convs = 0, n_items = 0, split = 0;
};

// Decode of n_layers consecutive layers from `layer` on in one launch: split kernel over plan items
// (partials: n_layers x n_items x n_q_heads records), then the merge kernel (output). q and out:
// [n_layers][n_convs][n_q_heads][head_dim].
// direct_out != nullptr (only when every conversation is one item, n_items == n_convs): the split
// writes the final output there and no merge follows.
hipError_t launch_decode_split(const PoolGeom& g, int layer, int n_layers, const DecodeLaunch& w, const void* q,
                               float* partials, void* direct_out, hipStream_t stream);
hipError_t launch_decode_merge(const PoolGeom& g, int n_layers, const DecodeLaunch& w, const float* partials,
                               void* out, hipStream_t stream);

// Streaming-read probe: read `bytes` (a multiple of 16) of device memory once with non-temporal
// 16-byte loads on 8 workgroups per CU; `sink` is 4 bytes of device memory (almost never written).
hipError_t launch_stream_read_probe(const void* src, size_t bytes, uint32_t* sink, int n_cus,
                                    hipStream_t stream);

// Capacity of the static decode scratch (floats): 16 MiB on each GPU.
constexpr size_t kStaticScratchFloats = size_t(4) << 20;
// Device address of the static decode scratch on the current device (looked up once per device
// with hipGetSymbolAddress and cached; allocates nothing).
hipError_t static_decode_scratch(float** out);

// Query rows (query tokens x query heads of the kv head) of an extend tile.
constexpr int kExtendTileRows = 256;
// Record of one piece of a cut extend tile and one kv head: o[256 rows][d] in accumulator order, then
// (maximum, sum) for each of the 8 x 64 lanes.
constexpr int extend_part_floats(int head_dim) { return kExtendTileRows * head_dim + 2 * 512; }

// An extend plan as the kernels read it: meta = ExtendConvDesc[..], then (16-byte aligned, at
// tiles_off) ExtendTile[n_tiles] and (at merges_off) ExtendMerge[n_merges].
struct ExtendLaunch {
  Meta meta;
  size_t tiles_off = 0, merges_off = 0;
  int n_tiles = 0, n_merges = 0;
  int piece = 0, n_parts = 0;
  bool chained = false;  // some tiles hold their pieces (ExtendTile::k0 < 0)
  int64_t q_rows = 0;  // query rows of a layer
};

// One layer of a mixed step in one launch: the extend tiles of the layer and its decode split
// (partials); launch_mixed_merge then combines the pieces of cut extend tiles and (out_dec !=
// nullptr) the decode records in one launch. Both plans uploaded.
hipError_t launch_mixed_layer(const PoolGeom& g, int layer, const ExtendLaunch& e, const void* q_ext,
                              void* out_ext, float* parts, const DecodeLaunch& w, const void* q_dec,
                              float* partials, void* direct_out, hipStream_t stream);
hipError_t launch_mixed_merge(const PoolGeom& g, const ExtendLaunch& e, void* out_ext, float* parts,
                              const DecodeLaunch& w, const float* partials, void* out_dec, hipStream_t stream);

// Query tokens per extend/prefill work tile for this GQA group (the host plan must match).
int extend_query_tile(int group);

// Extend / prefill of n_layers consecutive layers from `layer` on: one workgroup per (tile or piece, kv
// head, layer); then, where tiles are cut (n_merges > 0), the merge of their pieces. q and out:
// [n_layers][q_rows][n_q_heads][head_dim]; parts: n_layers x n_parts x n_kv_heads records.
hipError_t launch_extend(const PoolGeom& g, int layer, int n_layers, const ExtendLaunch& e, const void* q, void* out,
                         float* parts, hipStream_t stream);
hipError_t launch_extend_merge(const PoolGeom& g, int n_layers, const ExtendLaunch& e, void* out, float* parts,
                               hipStream_t stream);

}  // namespace cs
