// Host-side metadata of a KV page pool: free-page list with seeded random placement, the
// conversation table (length + logical->physical page list per conversation), and the work plans
// the attention kernels are launched with. No HIP here: everything compiles and is tested on a CPU.
#pragma once

#include <cstdint>
#include <deque>
#include <string>
#include <vector>

namespace cs {

constexpr int kPage = 16;  // tokens per KV page
constexpr int kCus = 256;  // compute units of the part, which the plans fill

inline int64_t pages_for(int64_t tokens) { return (tokens + kPage - 1) / kPage; }

// SplitMix64 (Steele, Lea, Flood 2014) -- seeds the page-placement shuffle.
struct SplitMix64 {
  uint64_t s;
  explicit SplitMix64(uint64_t seed) : s(seed) {}
  uint64_t next() {
    uint64_t z = (s += 0x9E3779B97F4A7C15ull);
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
  }
  uint64_t below(uint64_t n) { return next() % n; }  // modulo bias is irrelevant for placement
};

// Fixed set of physical pages handed out in a seeded random order.
class PagePool {
 public:
  PagePool(int64_t n_pages, uint64_t seed);
  int64_t capacity() const { return n_pages_; }
  int64_t free_count() const { return static_cast<int64_t>(free_.size()); }
  int64_t used_count() const { return n_pages_ - free_count(); }
  // All-or-nothing: appends n page ids to `out` and returns true, or changes nothing.
  bool alloc(int64_t n, std::vector<int32_t>& out);
  void release(const std::vector<int32_t>& pages);
  // Undo the latest alloc calls exactly: `pages` are the ids they handed out, in order (the free
  // list then holds the same ids in the same order as before them).
  void unalloc(const std::vector<int32_t>& pages);

 private:
  int64_t n_pages_;
  std::vector<int32_t> free_;
  SplitMix64 rng_;
};

struct Conv {
  bool live = false;
  uint32_t gen = 0;
  int64_t len = 0;
  std::vector<int32_t> pages;  // logical page i -> physical page id
};

// Conversation handles are slot | (generation << 20): a destroyed handle stays invalid after its
// slot is reused (until the 11-bit generation wraps). Freed slots are reused first-in first-out.
class ConvTable {
 public:
  static constexpr int kSlotBits = 20;
  ConvTable(int32_t max_convs, int32_t max_pages_per_conv);
  int32_t max_convs() const { return max_convs_; }
  int32_t max_pages_per_conv() const { return max_pages_; }
  int32_t live_count() const { return live_; }
  bool create(int32_t* handle);               // false when every slot is live
  Conv* find(int32_t handle);                  // nullptr if unknown / destroyed
  const Conv* find(int32_t handle) const;
  static int32_t slot_of(int32_t handle) { return handle & ((1 << kSlotBits) - 1); }
  void destroy(int32_t handle, PagePool& pool);  // handle must be valid

 private:
  int32_t max_convs_, max_pages_, live_ = 0;
  std::vector<Conv> slots_;
  std::deque<int32_t> free_slots_;
};

// ---------------------------------------------------------------------------------------------
// Work plans (plain structs uploaded to the device as-is; layouts shared with the kernels).
// ---------------------------------------------------------------------------------------------

// Decode: one work item = (conversation b, item s, kv head) covers keys [s*K, min(len, (s+1)*K))
// with K = kDecodeSubSplits * split_tokens, shared out evenly over its waves in whole page pairs.
// Items of conversation b are numbered item_start[b] + s.
struct DecodeConvDesc {
  int32_t slot;        // row of the device page-table mirror
  int32_t len;         // tokens
  int32_t item_start;  // first work item of this conversation
  int32_t n_splits;    // work items: ceil(len / (kDecodeSubSplits * split_tokens))
};

// Waves per decode work item: each takes one split of keys; the item's waves merge their partial
// results on chip and write one partial record per query head.
constexpr int kDecodeSubSplits = 8;

struct DecodePlan {
  int32_t split_tokens = 0;  // keys per wave (one split), multiple of 32, <= 1024
  int32_t n_items = 0;       // work items over the batch (per kv head)
  bool single_item = false;  // every conversation is one work item (no merge of items needed)
  std::vector<DecodeConvDesc> convs;
  // Launch order: workgroup w takes item order[w / n_kv_heads]. Full items (K keys) come first, in
  // conversation order, then the shorter last items by decreasing key count, so the last round
  // of workgroups on the chip holds the shortest ones.
  std::vector<int32_t> order;
};

// Choose the split size: the largest candidate for which the splits holding keys, over all kv
// heads, number at least `target_items` (the waves that read), else the smallest candidate. A
// work item is kDecodeSubSplits consecutive splits of one conversation.
DecodePlan plan_decode(const std::vector<int32_t>& slots, const std::vector<int64_t>& lens,
                       int32_t n_kv_heads, int64_t target_items);

// The same, but a batch whose work items (over all kv heads) would leave CUs without one gets the
// smallest splits, in steps of a page pair, whose items still fit the CUs in one round: one
// conversation of 2000 tokens 14.2 -> 11.3 us, 6000 (24 items instead of 6) 15.1 -> 11.1, four of
// 1100-4000 18.1 -> 13.1, 24.6k 20.3 -> 19.1; a second round that is not full costs more than it gives
// (24.6k tokens as 48 items of 64-key splits 26.3 us, as 24 of 128 23.2). A batch with a conversation of
// one item keeps its plan: where all are, the split writes the outputs without a merge (600 tokens 9.7
// us, cut 12.3). A conversation of at most 1024 tokens is one item in every plan of plan_decode, so its
// bits do not depend on the batch it is decoded in; a longer one's do.
DecodePlan plan_decode_filling(const std::vector<int32_t>& slots, const std::vector<int64_t>& lens,
                               int32_t n_kv_heads, int64_t target_items, int32_t n_cus);

// Extend / prefill: queries are the last q_len tokens of each conversation, cut into tiles of q_tile
// query tokens; one tile = (conversation, query block) x one kv head.
struct ExtendConvDesc {
  int32_t slot;
  int32_t len;    // tokens (keys) of the conversation
  int32_t q_len;  // queries = positions len-q_len .. len-1
  int32_t q_row;  // first row of this conversation in the q/out tensors
};

constexpr int kExtendKeyTile = 64;  // keys per step of the attention kernel
// Key tiles of the smallest piece; below, a piece is mostly start-up and records. One 64-token chunk on
// 3000 tokens takes 19.6 us with 4, 22.0 with 8, but a step of 8 conversations over 32 layers 979 / 839 us,
// one of 4 over 28 layers 407 / 337, and one of 8 over 16 layers in layer order 627 / 593, where other work
// fills the CUs.
constexpr int kMinPiece = 8;
constexpr int kPieceStep = 4;       // a piece is a multiple of the buffers of the kernel's LDS ring

struct ExtendTile {
  int32_t conv;       // index into the batch
  int32_t q0;         // first query index (0-based within the conversation's q_len)
  int32_t k0 = 0;     // first key tile; -1 - part0 < 0: a cut tile whose pieces part0, part0 + 1, ... one
                      // workgroup takes one after the other (part = -1)
  int32_t part = -1;  // -1: every key tile the queries see; else piece `part` of the launch: key
                      // tiles [k0, k0 + ExtendPlan::piece) of them
};

// The pieces part0 .. part0 + n_parts - 1 of a cut tile, in key order.
struct ExtendMerge {
  int32_t conv;
  int32_t q0;
  int32_t part0;
  int32_t n_parts;
};

struct ExtendPlan {
  int32_t q_tile = 64;
  std::vector<ExtendConvDesc> convs;
  std::vector<ExtendTile> tiles;  // conversation-major (longest conversation first), heaviest tile first
  // after split_extend:
  int32_t piece = 0;    // key tiles per piece
  int32_t n_parts = 0;  // pieces (per kv head)
  std::vector<ExtendMerge> merges;
};

ExtendPlan plan_extend(const std::vector<int32_t>& slots, const std::vector<int64_t>& lens,
                       const std::vector<int32_t>& q_lens, int32_t q_tile);

// Cut the keys of a launch's tiles into pieces where the tiles alone would leave CUs idle; at most
// max_records pieces over all kv heads. Changes nothing where the tiles fill the chip. Pieces are
// counted from key tile 0 and all tiles of a launch are cut at multiples of one size, so a query's
// result depends on that size and its position only.
void split_extend(ExtendPlan& plan, int32_t n_kv_heads, int32_t n_cus, int32_t max_records);

// The same cuts, but one workgroup for each tile: it takes the tile's pieces one after the other and
// combines them itself (bit for bit what separate pieces and their merge give, without their start-up,
// their merge launch and most of their records' way to memory).
void chain_extend(ExtendPlan& plan);

// A decode batch's share of the CUs in steps of one key tile of the attention kernel (1.3 us on a busy chip
// at head dim 128), for each layer and kv head: its K and V at 6 TB/s.
float decode_steps(const std::vector<int64_t>& lens, int32_t n_kv_heads, int32_t head_dim, int32_t n_cus);

// Whether chain_extend makes the launch shorter where other work waits for the CUs too: other_steps of
// it for each layer and kv head (in CU-steps of a key tile), n_layers layers in the launch.
bool chain_pays(const ExtendPlan& plan, int32_t n_kv_heads, int32_t n_cus, int32_t n_layers, float other_steps);

// Append / unpack: one chunk = the part of one logical page a call writes.
struct PageChunk {
  int32_t conv;      // index into the batch
  int32_t slot;      // page-table row
  int32_t lpage;     // logical page index within the conversation
  int32_t page;      // physical page id
  int32_t t0, t1;    // token slots [t0, t1) of the page receive data; when t0 = 0, [t1, 16) are zeroed
  int32_t src_row;   // row (token) of the first written slot in the source tensor
  int32_t new_page;  // 1 if this page was just allocated (the mirror entry must be written)
};

// Chunks for appending n_new[i] tokens to conversations whose lengths are lens[i] and whose page
// lists already include the newly reserved pages.
std::vector<PageChunk> plan_append(const std::vector<int32_t>& slots,
                                   const std::vector<int64_t>& lens,
                                   const std::vector<int32_t>& n_new,
                                   const std::vector<const std::vector<int32_t>*>& page_lists);

}  // namespace cs
