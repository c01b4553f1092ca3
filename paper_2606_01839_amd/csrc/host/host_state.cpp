#include "host_state.hpp"

#include <algorithm>
#include <functional>
#include <numeric>

namespace cs {

PagePool::PagePool(int64_t n_pages, uint64_t seed) : n_pages_(n_pages), rng_(seed) {
  free_.resize(static_cast<size_t>(n_pages));
  std::iota(free_.begin(), free_.end(), 0);
  // Fisher-Yates shuffle: physical placement of logical pages is random.
  for (int64_t i = n_pages - 1; i > 0; --i) {
    int64_t j = static_cast<int64_t>(rng_.below(static_cast<uint64_t>(i + 1)));
    std::swap(free_[i], free_[j]);
  }
}

bool PagePool::alloc(int64_t n, std::vector<int32_t>& out) {
  if (n < 0 || n > free_count()) return false;
  out.reserve(out.size() + static_cast<size_t>(n));
  for (int64_t i = 0; i < n; ++i) {
    out.push_back(free_.back());
    free_.pop_back();
  }
  return true;
}

void PagePool::release(const std::vector<int32_t>& pages) {
  for (int32_t p : pages) {
    free_.push_back(p);
    // keep the free list in random order: swap the returned page to a random position
    size_t j = static_cast<size_t>(rng_.below(free_.size()));
    std::swap(free_[j], free_.back());
  }
}

void PagePool::unalloc(const std::vector<int32_t>& pages) {
  for (auto it = pages.rbegin(); it != pages.rend(); ++it) free_.push_back(*it);
}

ConvTable::ConvTable(int32_t max_convs, int32_t max_pages_per_conv)
    : max_convs_(max_convs), max_pages_(max_pages_per_conv), slots_(static_cast<size_t>(max_convs)) {
  for (int32_t i = 0; i < max_convs; ++i) free_slots_.push_back(i);
}

bool ConvTable::create(int32_t* handle) {
  if (free_slots_.empty()) return false;
  int32_t s = free_slots_.front();
  free_slots_.pop_front();
  Conv& c = slots_[static_cast<size_t>(s)];
  c.live = true;
  c.len = 0;
  c.pages.clear();
  ++live_;
  *handle = s | static_cast<int32_t>((c.gen & 0x7FFu) << kSlotBits);
  return true;
}

Conv* ConvTable::find(int32_t handle) {
  if (handle < 0) return nullptr;
  int32_t s = slot_of(handle);
  if (s >= max_convs_) return nullptr;
  Conv& c = slots_[static_cast<size_t>(s)];
  if (!c.live) return nullptr;
  if (static_cast<uint32_t>(handle >> kSlotBits) != (c.gen & 0x7FFu)) return nullptr;
  return &c;
}

const Conv* ConvTable::find(int32_t handle) const {
  return const_cast<ConvTable*>(this)->find(handle);
}

void ConvTable::destroy(int32_t handle, PagePool& pool) {
  int32_t s = slot_of(handle);
  Conv& c = slots_[static_cast<size_t>(s)];
  pool.release(c.pages);
  c.pages.clear();
  c.pages.shrink_to_fit();
  c.len = 0;
  c.live = false;
  c.gen = (c.gen + 1) & 0x7FFu;
  --live_;
  free_slots_.push_back(s);
}

// The items and launch order of a plan with splits of `split` keys.
static DecodePlan decode_plan_of(const std::vector<int32_t>& slots, const std::vector<int64_t>& lens, int32_t split) {
  DecodePlan plan;
  plan.split_tokens = split;
  const int64_t item_keys = static_cast<int64_t>(kDecodeSubSplits) * split;
  int32_t start = 0;
  plan.convs.reserve(lens.size());
  for (size_t i = 0; i < lens.size(); ++i) {
    int32_t ns = static_cast<int32_t>((lens[i] + item_keys - 1) / item_keys);
    plan.convs.push_back({slots[i], static_cast<int32_t>(lens[i]), start, ns});
    start += ns;
  }
  plan.n_items = start;
  plan.single_item = start == static_cast<int32_t>(lens.size());
  std::vector<int64_t> keys(static_cast<size_t>(start));
  for (const DecodeConvDesc& c : plan.convs)
    for (int32_t s = 0; s < c.n_splits; ++s) keys[c.item_start + s] = std::min<int64_t>(item_keys, c.len - s * item_keys);
  plan.order.resize(static_cast<size_t>(start));
  std::iota(plan.order.begin(), plan.order.end(), 0);
  std::stable_sort(plan.order.begin(), plan.order.end(),
                   [&](int32_t x, int32_t y) { return keys[x] > keys[y]; });
  return plan;
}

DecodePlan plan_decode(const std::vector<int32_t>& slots, const std::vector<int64_t>& lens,
                       int32_t n_kv_heads, int64_t target_items) {
  static const int32_t kCandidates[] = {1024, 512, 256, 128};
  int32_t split = 0;
  for (int32_t c : kCandidates) {
    int64_t items = 0;
    for (int64_t L : lens) items += (L + c - 1) / c;
    split = c;
    if (items * n_kv_heads >= target_items) break;
  }
  return decode_plan_of(slots, lens, split);
}

DecodePlan plan_decode_filling(const std::vector<int32_t>& slots, const std::vector<int64_t>& lens,
                               int32_t n_kv_heads, int64_t target_items, int32_t n_cus) {
  DecodePlan plan = plan_decode(slots, lens, n_kv_heads, target_items);
  if (static_cast<int64_t>(plan.n_items) * n_kv_heads >= n_cus) return plan;
  for (const DecodeConvDesc& c : plan.convs)
    if (c.n_splits < 2) return plan;
  for (int32_t split = 32; split < plan.split_tokens; split += 32) {
    int64_t items = 0;
    const int64_t item_keys = static_cast<int64_t>(kDecodeSubSplits) * split;
    for (int64_t L : lens) items += (L + item_keys - 1) / item_keys;
    if (items * n_kv_heads <= n_cus) return decode_plan_of(slots, lens, split);
  }
  return plan;
}

ExtendPlan plan_extend(const std::vector<int32_t>& slots, const std::vector<int64_t>& lens,
                       const std::vector<int32_t>& q_lens, int32_t q_tile) {
  ExtendPlan plan;
  plan.q_tile = q_tile;
  int32_t row = 0;
  std::vector<std::pair<int64_t, ExtendTile>> work;
  for (size_t i = 0; i < lens.size(); ++i) {
    plan.convs.push_back({slots[i], static_cast<int32_t>(lens[i]), q_lens[i], row});
    row += q_lens[i];
    for (int32_t q0 = 0; q0 < q_lens[i]; q0 += q_tile) {
      int64_t keys = lens[i] - q_lens[i] + std::min(q_lens[i], q0 + q_tile);
      work.push_back({keys, {static_cast<int32_t>(i), q0, 0, -1}});
    }
  }
  // Conversation-major order: longest conversation first, its heaviest tiles first. Workgroups that
  // run at the same time on one XCD then mostly belong to one conversation and sweep the same
  // prefix K/V, so it stays in that XCD's L2; the heaviest tiles still start first.
  std::vector<int64_t> conv_keys(lens.size(), 0);
  for (auto& w : work) conv_keys[w.second.conv] = std::max(conv_keys[w.second.conv], w.first);
  std::stable_sort(work.begin(), work.end(), [&](const auto& a, const auto& b) {
    const int64_t ka = conv_keys[a.second.conv], kb = conv_keys[b.second.conv];
    if (ka != kb) return ka > kb;
    if (a.second.conv != b.second.conv) return a.second.conv < b.second.conv;
    return a.first > b.first;
  });
  plan.tiles.reserve(work.size());
  for (auto& w : work) plan.tiles.push_back(w.second);
  return plan;
}

// The line between cutting and not cutting is an estimate of the launch's time, in steps of one key
// tile (1.16 us at head dim 128 on a part-filled chip): the CUs one kv head gets (n_cus / n_kv_heads) take
// the workgroups longest first; each costs its key tiles plus kStartSteps (measured 9 us: plan, pages,
// queries and first tiles one after the other from memory, the refresh of the first tile's maximum, the
// last stores), and cutting costs the merge launch plus the records' way to memory and back. The same
// numbers serve head dim 64, where a step is shorter against start-up and merge: of 93 launches (prompts
// of 300 to 9000 tokens, chunks of 1 to 1000 on 600 to 20,000) none is slower than with whole tiles and 59
// are 1.2 to 10 times faster; of 24 layer-ordered steps beside a decode three are slower, by 1, 2 and 5%,
// all with 1000-token chunks.
constexpr float kStartSteps = 8.f;
constexpr float kMergeSteps = 6.f;
constexpr float kRecordSteps = 0.03f;
// A launch that is this much longer for fewer pieces is preferred (513 tokens on 2948: 49 us in two pieces
// a tile instead of 42.5 in three, but the 32-layer mixed step they arrive in 2.95 ms instead of 3.05;
// uncut 79 us and 2.93 ms).
constexpr float kFewerSteps = 6.f;

// Time of workgroups of the given key tiles (longest first) on `slots` CUs: each goes to the CU that is
// free first.
static float makespan(const std::vector<int32_t>& keys, size_t slots) {
  if (keys.empty()) return 0.f;
  if (keys.size() <= slots) return static_cast<float>(keys[0]) + kStartSteps;
  // min-heap of the CUs' end times; after one workgroup each, last to first, they are in order
  std::vector<float> end(slots);
  for (size_t i = 0; i < slots; ++i) end[i] = static_cast<float>(keys[slots - 1 - i]) + kStartSteps;
  float last = end.back();
  for (size_t i = slots; i < keys.size(); ++i) {
    const float e = end[0] + static_cast<float>(keys[i]) + kStartSteps;
    last = std::max(last, e);
    size_t at = 0;
    for (size_t c = 1; c < slots; c = 2 * at + 1) {
      if (c + 1 < slots && end[c + 1] < end[c]) ++c;
      if (end[c] >= e) break;
      end[at] = end[c];
      at = c;
    }
    end[at] = e;
  }
  return last;
}

void split_extend(ExtendPlan& plan, int32_t n_kv_heads, int32_t n_cus, int32_t max_records) {
  const int n = static_cast<int>(plan.tiles.size());
  const int slots = std::max(1, n_cus / n_kv_heads);
  const int max_parts = max_records / n_kv_heads;
  // Beyond two rounds of tiles cutting could win back only part of the last.
  if (n == 0 || n > 2 * slots || max_parts < 2) return;
  std::vector<int32_t> keys(static_cast<size_t>(n));
  int64_t total = 0;
  for (int i = 0; i < n; ++i) {
    const ExtendConvDesc& c = plan.convs[static_cast<size_t>(plan.tiles[i].conv)];
    const int32_t seen = c.len - c.q_len + std::min(c.q_len, plan.tiles[i].q0 + plan.q_tile);
    keys[i] = (seen + kExtendKeyTile - 1) / kExtendKeyTile;
    total += keys[i];
  }
  std::vector<int32_t> sorted = keys;
  std::sort(sorted.begin(), sorted.end(), std::greater<int32_t>());
  const int32_t longest = sorted[0];
  if (longest <= kMinPiece) return;
  const float limit = 0.9f * makespan(sorted, static_cast<size_t>(slots));  // cut only for a clear gain
  // What `pieces` workgroups and their merge take at the least, with every CU busy to the end. Where that is
  // no gain nothing is scheduled: 250 tiles of an 8000-token prompt at 2 kv heads 53 -> 3 us of planning, 500
  // tiles at one kv head 70 -> 6.
  const auto at_least = [&](int pieces, int parts) {
    return 0.999f * (static_cast<float>(total) + kStartSteps * static_cast<float>(pieces)) / static_cast<float>(slots) +
           kMergeSteps + kRecordSteps * static_cast<float>(parts * n_kv_heads);
  };
  if (at_least(n + 1, 2) >= limit) return;
  struct Cut {
    int32_t c;
    int parts;
    float time;
  };
  std::vector<Cut> cuts;
  std::vector<int32_t> work_keys;
  // Sizes: the smallest whose pieces fit in one to four rounds of the CUs (and their records), and half
  // the longest tile.
  for (int rounds = 0; rounds <= 4; ++rounds) {
    int32_t c = std::max<int32_t>(
        kMinPiece, rounds == 0 ? (longest + 1) / 2 : static_cast<int32_t>(total / (static_cast<int64_t>(rounds) * slots)));
    c = (c + kPieceStep - 1) / kPieceStep * kPieceStep;
    int pieces = 0, parts = 0;
    for (;; c += std::max(1, c / 16 / kPieceStep) * kPieceStep) {
      pieces = parts = 0;
      for (int32_t k : keys) {
        const int np = (k + c - 1) / c;
        pieces += np;
        parts += np > 1 ? np : 0;
      }
      if (c >= longest || (parts <= max_parts && (rounds == 0 || pieces <= rounds * slots))) break;
    }
    if (c >= longest || at_least(pieces, parts) >= limit) continue;
    work_keys.clear();
    size_t whole = 0;
    for (int32_t k : keys) whole += static_cast<size_t>(k / c);
    work_keys.assign(whole, c);
    for (int32_t k : keys)
      if (k % c) work_keys.push_back(k % c);
    std::sort(work_keys.begin() + static_cast<std::ptrdiff_t>(whole), work_keys.end(), std::greater<int32_t>());
    const float t = makespan(work_keys, static_cast<size_t>(slots)) + kMergeSteps + kRecordSteps * static_cast<float>(parts * n_kv_heads);
    if (t < limit) cuts.push_back({c, parts, t});
  }
  if (cuts.empty()) return;
  // Of the cuts within kFewerSteps of the best the one with the fewest pieces: beside a decode, which
  // takes the CUs that cutting would fill, each piece only costs.
  float best = limit;
  for (const Cut& x : cuts) best = std::min(best, x.time);
  const Cut* pick = nullptr;
  for (const Cut& x : cuts)
    if (x.time <= best + kFewerSteps && (pick == nullptr || x.parts < pick->parts ||
                                         (x.parts == pick->parts && x.time < pick->time)))
      pick = &x;
  const int32_t best_c = pick->c;
  plan.piece = best_c;
  std::vector<std::pair<int32_t, ExtendTile>> work;
  for (int i = 0; i < n; ++i) {
    ExtendTile t = plan.tiles[i];
    if (keys[i] <= best_c) {
      work.push_back({keys[i], t});
      continue;
    }
    const int np = (keys[i] + best_c - 1) / best_c;
    plan.merges.push_back({t.conv, t.q0, plan.n_parts, np});
    for (int s = 0; s < np; ++s) {
      t.k0 = s * best_c;
      t.part = plan.n_parts++;
      work.push_back({std::min(best_c, keys[i] - t.k0), t});
    }
  }
  // longest first, so the last round holds the shortest
  std::stable_sort(work.begin(), work.end(), [](const auto& a, const auto& b) { return a.first > b.first; });
  plan.tiles.clear();
  for (auto& w : work) plan.tiles.push_back(w.second);
}

void chain_extend(ExtendPlan& plan) {
  std::vector<std::pair<int32_t, ExtendTile>> work;
  auto keys_of = [&](const ExtendTile& t) {
    const ExtendConvDesc& c = plan.convs[static_cast<size_t>(t.conv)];
    return c.len - c.q_len + std::min(c.q_len, t.q0 + plan.q_tile);
  };
  for (const ExtendTile& t : plan.tiles)
    if (t.part < 0) work.push_back({keys_of(t), t});
  for (const ExtendMerge& m : plan.merges) {
    const ExtendTile t{m.conv, m.q0, -1 - m.part0, -1};
    work.push_back({keys_of(t), t});
  }
  std::stable_sort(work.begin(), work.end(), [](const auto& a, const auto& b) { return a.first > b.first; });
  plan.tiles.clear();
  for (auto& w : work) plan.tiles.push_back(w.second);
  plan.merges.clear();
}

float decode_steps(const std::vector<int64_t>& lens, int32_t n_kv_heads, int32_t head_dim, int32_t n_cus) {
  double tokens = 0;
  for (int64_t L : lens) tokens += static_cast<double>(L);
  const double us = tokens * n_kv_heads * head_dim * 4 / 6e6;
  return static_cast<float>(us / 1.3 * std::max(1, n_cus / n_kv_heads));
}

bool chain_pays(const ExtendPlan& plan, int32_t n_kv_heads, int32_t n_cus, int32_t n_layers, float other_steps) {
  if (plan.merges.empty()) return false;
  const float slots = static_cast<float>(std::max(1, n_cus / n_kv_heads));
  float keys = 0.f, longest = 0.f;
  int whole = static_cast<int>(plan.merges.size());
  auto add = [&](int32_t conv, int32_t q0, bool cut) {
    const ExtendConvDesc& c = plan.convs[static_cast<size_t>(conv)];
    const int32_t seen = c.len - c.q_len + std::min(c.q_len, q0 + plan.q_tile);
    const float k = static_cast<float>((seen + kExtendKeyTile - 1) / kExtendKeyTile);
    keys += k;
    // a chained tile writes and reads back a record (about two steps) for every piece but its last
    longest = std::max(longest, k + (cut ? 2.f * k / static_cast<float>(plan.piece) : 0.f));
  };
  for (const ExtendMerge& m : plan.merges) add(m.conv, m.q0, true);
  for (const ExtendTile& t : plan.tiles)
    if (t.part < 0) {
      add(t.conv, t.q0, false);
      ++whole;
    }
  const float nl = static_cast<float>(n_layers);
  const float work = nl * (keys + other_steps) / slots, start = nl * kStartSteps / slots;
  const float chained = std::max(longest + kStartSteps, work + start * static_cast<float>(whole) +
                                                             nl * 2.f * static_cast<float>(plan.n_parts) / slots);
  const float apart = work + start * static_cast<float>(plan.tiles.size()) +
                      kMergeSteps / 2 + nl * kRecordSteps * static_cast<float>(plan.n_parts * n_kv_heads);
  return chained <= apart;
}

std::vector<PageChunk> plan_append(const std::vector<int32_t>& slots,
                                   const std::vector<int64_t>& lens,
                                   const std::vector<int32_t>& n_new,
                                   const std::vector<const std::vector<int32_t>*>& page_lists) {
  std::vector<PageChunk> chunks;
  int64_t row_base = 0;
  for (size_t i = 0; i < lens.size(); ++i) {
    const int64_t pos0 = lens[i], n = n_new[i];
    if (n > 0) {
      const int64_t old_pages = pages_for(pos0);
      for (int64_t p = pos0 / kPage; p <= (pos0 + n - 1) / kPage; ++p) {
        const int64_t a = std::max(pos0, p * kPage), b = std::min(pos0 + n, (p + 1) * kPage);
        PageChunk c;
        c.conv = static_cast<int32_t>(i);
        c.slot = slots[i];
        c.lpage = static_cast<int32_t>(p);
        c.page = (*page_lists[i])[static_cast<size_t>(p)];
        c.t0 = static_cast<int32_t>(a - p * kPage);
        c.t1 = static_cast<int32_t>(b - p * kPage);
        c.src_row = static_cast<int32_t>(row_base + (a - pos0));
        c.new_page = p >= old_pages ? 1 : 0;
        chunks.push_back(c);
      }
    }
    row_base += n;
  }
  return chunks;
}

}  // namespace cs
