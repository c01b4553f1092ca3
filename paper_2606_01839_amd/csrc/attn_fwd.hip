// Turn-1 prefill and turn-N extend-prefill attention over paged KV (flash-attention forward).
//
// A workgroup owns one (conversation, query block, kv head) tile; its waves cover the G query
// heads of that kv head (the GQA group), so every K/V tile in LDS serves all the query rows of
// the group (256 rows at head_dim 128).
// Each wave computes the transposed score tile on the matrix cores (v_mfma_f32_32x32x16_bf16):
//   S^T[key][query] = K[key][:] . Q[query][:]       A = K rows from LDS, B = Q kept in registers
//   O^T[dim][query] += V^T[dim][key] . P^T[key][query]   A = V^T rows from LDS, B = P registers
// With the transposed formulation every lane owns one query row (32 rows of a 32x32 tile, the two
// 32-lane halves holding different keys), so the online-softmax max/sum are in-lane except for
// one exchange between the halves, and the P accumulator registers are directly the B operand of
// the PV product: the key order of K or V^T in LDS is arranged so the two contractions agree.
//
// Eight waves, G query heads x 8/G blocks of 32 queries (a 64-query tile at G = 4, 128 queries at
// G = 2), two waves per SIMD.
// K/V tiles of 64 keys (4 pages) are copied from HBM straight into a four-deep LDS ring with
// global_load_lds_dwordx4 (no staging registers, no LDS store instructions), three tiles ahead;
// the K operands of tile j+1 are read into registers while the PV product of tile j runs.
// Diagonal tiles apply the causal mask and fully visible tiles skip it.
//
// A workgroup sweeps its tile's keys one after another, so a launch with fewer tiles than the chip
// has CUs takes as long as its longest tile. The host then cuts the tiles' keys into pieces
// (split_extend in host_state.cpp): each piece is a workgroup that writes its unnormalised output, row
// maximum and row sum, and extend_merge_kernel combines the pieces of a tile in their order. Where other
// work fills the CUs (a mixed step's decode, many layers in one launch) one workgroup takes a tile's
// pieces one after the other instead and combines them itself, with the same result bit for bit.
// A 301-token chunk on 41k tokens (40 workgroups, 646 key tiles each) 802 -> 200 us, a 1437-token prompt
// 39.4 -> 25.7 us.
//
// Bound: large launches by the matrix cores at the part's power limit (1.24-1.29 PFLOP/s at head dim
// 128; a library product of 8192^3 reaches 1.37). Small ones by a workgroup's start-up, 9 us at head dim
// 128 of which 0.5 is the plan, 1.5 pages, queries and first copies, 1.0 their arrival, 2.5 the first
// tile (mask, weights taken twice) and 2.0-3.7 were 8-byte output stores into 32 rows at a time.
// Head dim 64 against a kernel that staged tiles through registers, one wave per SIMD: six prompts of
// 300-9000 tokens 361 -> 229 us.
#include <cfloat>
#include <cmath>
#include <type_traits>

#include "decode_split.hpp"
#include "device_common.hpp"
#include "kernels.hpp"

namespace cs {

struct ExtendArgs {
  const uint16_t* pool;
  int64_t n_pages;
  int n_kv_heads;
  int layer;
  const int32_t* page_table;
  int max_pages;
  const void* meta;  // device copy of the plan, or nullptr: in the kernel's arguments
  uint32_t tiles_off;
  const uint16_t* q;
  uint16_t* out;
  float scale_log2;
  int piece;              // key tiles of a whole piece of a cut tile
  float* parts;           // records of the pieces: [part][kv head] of extend_part_floats(D)
  uint32_t merges_off;
  size_t q_stride;        // elements of q (and out) from one layer to the next
  size_t part_stride;     // floats of parts from one layer to the next
  __device__ __forceinline__ ExtendTile tile(int i) const {
    const auto* p = meta_at<ExtendTile>(meta, tiles_off) + i;
    return {p->conv, p->q0, p->k0, p->part};
  }
  __device__ __forceinline__ ExtendMerge merge(int i) const {
    const auto* p = meta_at<ExtendMerge>(meta, merges_off) + i;
    return {p->conv, p->q0, p->part0, p->n_parts};
  }
  __device__ __forceinline__ ExtendConvDesc conv(int i) const {
    const auto* p = meta_at<ExtendConvDesc>(meta, 0) + i;
    return {p->slot, p->len, p->q_len, p->q_row};
  }
};

constexpr int kBN = 64;  // keys per tile
static_assert(kBN == kExtendKeyTile, "the plan counts the kernel's key tiles");

// Per-lane bound on the sum of a tile's weights (32 keys per lane) before the max is refreshed.
constexpr float kSumLimit = 256.f;

// ------------------------------------------------------------------------------------------------
// K/V copied from HBM straight into LDS.
// LDS ring of four tiles: the K parts of the four buffers first, their V^T parts after them, so every
// operand read reaches its buffer through the instruction's 16-bit offset field (no address
// arithmetic per read). K as 64 rows of 2 D bytes, the 16-byte chunk index XOR-swizzled by the row
// (D = 128: chunk ^ (row & 15); D = 64, where two rows share 256 bytes: chunk ^ ((row >> 1) & 7));
// V^T page by page, D dims x 32 B (16 keys) per page, the two 16-byte halves of a dim swapped when
// bit 2 xor bit 3 of the dim is set. A 16-byte operand read is served 16 lanes at a time over 256
// bytes of banks: the 16 rows (K) or dims (V^T) such a group reads then fall in 16 distinct 16-byte
// bank groups (rocprofv3 SQ_LDS_BANK_CONFLICT counts about 100 cycles a wave, those of the output rows
// at the end), while every copy instruction still writes 1 KiB of consecutive LDS bytes.
// ------------------------------------------------------------------------------------------------
__device__ __forceinline__ uint32_t lds_u32(const void* p) {
  return static_cast<uint32_t>(reinterpret_cast<uintptr_t>((const __attribute__((address_space(3))) void*)p));
}
// Copy 16 bytes per lane from global memory (wave-uniform base + per-lane byte offset) straight
// into LDS: lane l writes LDS bytes lds + 16 l .. +15 (global_load_lds_dwordx4, destination base in
// M0). The copy is tracked by the vector-memory counter only; M0 is saved and restored around it.
__device__ __forceinline__ void dma16(uint32_t lds, const void* gbase, uint32_t voff) {
  uint32_t saved;
  asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\tglobal_load_lds_dwordx4 %2, %3\n\ts_mov_b32 m0, %0"
               : "=&s"(saved) : "s"(lds), "v"(voff), "s"(gbase) : "memory");
}
// Wait until at most N of this wave's vector-memory operations (its copies) are in flight, then a
// workgroup barrier: afterwards every wave's copies issued before its own last N have landed. A barrier
// after which a buffer is copied over must also have that buffer's operand reads of every wave behind it,
// and the matrix instructions that wait for them may be scheduled after the barrier: with READS the wave's
// LDS reads return first.
template <int N, bool READS = false>
__device__ __forceinline__ void dma_wait_barrier() {
  if constexpr (READS) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"(N) : "memory");
  else asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" :: "n"(N) : "memory");
}

// One (tile or piece, kv head) workgroup (`block` = its index in the layer's grid, `dl` = its layer
// counted from a.layer).
//
// PRE: the K operands of the next tile and the V operands of this one are read from LDS ahead of the
// matrix instructions that use them (two waves per SIMD have little else to cover the LDS latency).
// Without it a head_dim 64 wave needs 121 registers and two workgroups fit a CU.
// CHAIN: tiles may hold pieces to take one after the other (a form of its own, since the code around
// the loop costs launches without such tiles 1.5%).
template <int D, int G, bool PRE, bool CHAIN>
__device__ __forceinline__ void attn_fwd_block(const ExtendArgs& a, const int block, const int dl) {
  constexpr int NW = 8;                   // waves: G query heads x (8 / G) blocks of 32 queries
  constexpr int BM = 32 * (NW / G);       // queries per workgroup
  static_assert(NW % G == 0, "the group must divide the eight waves");
  constexpr int KS = D / 16;
  constexpr int DT = D / 32;
  constexpr int HALF_TILE = kBN * D * 2;  // K (or V^T) bytes per buffer
  constexpr int NB = HALF_TILE / 1024;    // 1 KiB blocks per K (and per V^T) tile
  constexpr int BPP = NB / 4;             // ... and per page of it
  constexpr int BPW = NB / NW;            // blocks per wave
  constexpr int CPR = D / 8;              // 16-byte chunks per K row
  constexpr int RPB = 64 / CPR;           // K rows per block
  static_assert(NB % NW == 0 && BPP % BPW == 0, "a wave's blocks must lie in one page");
  // chunk swizzle of LDS row r
  auto swz = [](int r) { return D == 128 ? r & 15 : (r >> 1) & 7; };
  constexpr int NBUF = 4;                 // LDS ring: tile j read, j+1 landed, j+2 and j+3 in flight
  constexpr int VBASE = NBUF * HALF_TILE; // V^T parts after the K parts of all buffers
  __shared__ __attribute__((aligned(1024))) uint8_t smem[2 * NBUF * HALF_TILE];

  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int tile_idx = block / a.n_kv_heads, g = block % a.n_kv_heads;
  const ExtendTile tile = a.tile(tile_idx);
  const ExtendConvDesc cd = a.conv(tile.conv);
  const int prefix = cd.len - cd.q_len;
  const int q_hi = min(cd.q_len, tile.q0 + BM);
  const int pos_min = prefix + tile.q0, pos_max = prefix + q_hi - 1;
  // key tiles [kt0, n_kt): all that the tile sees, or one piece of them
  const bool chained = CHAIN && tile.k0 < 0;                  // a cut tile's pieces one after the other
  const int kt0 = chained ? 0 : tile.k0;
  int part = chained ? -1 - tile.k0 : tile.part;     // record of the piece
  const int n_kt = tile.part < 0 ? pos_max / kBN + 1 : min(pos_max / kBN + 1, kt0 + a.piece);
  const int n_pg = (cd.len + kPageTokens - 1) / kPageTokens;
  const int32_t* pt = a.page_table + static_cast<size_t>(cd.slot) * a.max_pages;
  const int h = g * G + wave % G;
  const int qblk = wave / G;
  const int n_q_heads = a.n_kv_heads * G;
  const size_t head_stride = static_cast<size_t>(2 * kPageTokens * D);
  const size_t layer_base = static_cast<size_t>(a.layer + dl) * a.n_pages * a.n_kv_heads * head_stride +
                            static_cast<size_t>(g) * head_stride;
  const size_t page_stride = static_cast<size_t>(a.n_kv_heads) * head_stride;
  const float c = a.scale_log2;
  const auto* ptc = as_const(pt);

  // ---- copy side: block kb (1 KiB) of a tile = K rows RPB kb .. of page kb / BPP and V^T dims
  // 32 (kb % BPP) .. +31 of the same page; this wave copies blocks BPW*wave .. BPW*wave + BPW-1, all
  // of one page. The per-lane global offsets are fixed; only the page base changes per tile.
  const int q_w = (BPW * wave) / BPP;
  uint32_t koff[BPW], voff[BPW];
#pragma unroll
  for (int i = 0; i < BPW; ++i) {
    const int part = (BPW * wave + i) % BPP;
    const int row = RPB * part + lane / CPR;                 // LDS row within the page
    const int chunk = (lane % CPR) ^ swz(row);               // logical 16-byte chunk of that row
    // LDS row 8a + 4h + b holds key 8h + 4a + b (bits 2 and 3 swapped): the S^T accumulator
    // of lane half h then holds keys 8h .. 8h+7 of each 16-key step, the order of V^T in LDS.
    const int key = (row & 3) | ((row >> 3) & 1) << 2 | ((row >> 2) & 1) << 3;
    koff[i] = static_cast<uint32_t>(k_elem(key, chunk) * 2);
    const int dim = 32 * part + lane / 2;
    const int hv = (lane & 1) ^ ((dim >> 2) & 1) ^ ((dim >> 3) & 1);
    voff[i] = static_cast<uint32_t>(2 * kPageTokens * D + dim * 32 + hv * 16);
  }
  const uint32_t smem_base = lds_u32(smem);
  // Copies for tiles past the end are issued too (of the last tile, whose pages past the
  // conversation's end are its last page), so every step issues the same number and the counter
  // waits below stay exact. Those keys are masked by the causal mask.
  auto page_of = [&](int j) { return ptc[min(4 * min(j, n_kt - 1) + q_w, n_pg - 1)]; };
  auto copy_tile = [&](int page, int buf) {
    const uint16_t* blk = a.pool + layer_base + static_cast<size_t>(page) * page_stride;
#pragma unroll
    for (int i = 0; i < BPW; ++i) {
      const int kb = BPW * wave + i;
      dma16(smem_base + buf * HALF_TILE + kb * 1024, blk, koff[i]);
      dma16(smem_base + VBASE + buf * HALF_TILE + kb * 1024, blk, voff[i]);
    }
  };

  // ---- read side: MFMA operand addresses (bytes within a buffer) -------------------------------
  // K operand of lane (col, half) for k-step ks: LDS row col (+32 kt2), logical chunk 2 ks + half,
  // stored at chunk (2 ks + half) ^ swz(row). V^T operand for (kt2, j2, t): page 2 kt2 + j2,
  // dims 32 t + col, keys 8 half .. +7, stored in the block DT (2 kt2 + j2) + t at col * 32 +
  // 16 (half ^ bit 2 of col ^ bit 3 of col).
  const int half = lane >> 5, col = lane & 31;
  uint32_t kaddr[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks)
    kaddr[ks] = static_cast<uint32_t>(col * (2 * D) + (((2 * ks + half) ^ swz(col)) * 16));
  const uint32_t vaddr =
      static_cast<uint32_t>(col * 32 + ((half ^ ((col >> 2) & 1) ^ ((col >> 3) & 1)) * 16));

  // Q first, then the copies of the first three tiles, so that both are on their way together.
  bf16x8 qop[KS];
  const int qrow0 = tile.q0 + 32 * qblk;
  const bool valid = qrow0 + col < cd.q_len;
  const int qpos = prefix + (valid ? qrow0 + col : cd.q_len - 1);
  const uint16_t* qrow =
      a.q + dl * a.q_stride + (static_cast<size_t>(cd.q_row + (valid ? qrow0 + col : 0)) * n_q_heads + h) * D;
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) qop[ks] = as_bf16x8(ld16(qrow + 16 * ks + 8 * half));  // padding rows: row 0
  // (one vector load of the first four tiles' pages: one trip to memory instead of four)
  const int pages = pt[min(4 * min(kt0 + (lane & 3), n_kt - 1) + q_w, n_pg - 1)];
#pragma unroll
  for (int i = 0; i < 3; ++i) copy_tile(__builtin_amdgcn_readlane(pages, i), i);
  int page_next = __builtin_amdgcn_readlane(pages, 3);
  __builtin_amdgcn_sched_barrier(0);   // no wait for Q before the copies are issued
  // Q must have arrived before the loop: a wait of the compiler's at the loop head would drain the copies
  // that the loop keeps in flight. Here too its waits do not count the copies (made in asm) and so wait
  // for all three tiles behind Q, though the barrier below needs only two.
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    if (!valid) qop[ks] = bf16x8{};
    asm volatile("" ::"v"(qop[ks]));
  }
  f32x16 o[DT];
#pragma unroll
  for (int t = 0; t < DT; ++t)
#pragma unroll
    for (int e = 0; e < 16; ++e) o[t][e] = 0.f;
  // The running maximum starts at the lowest finite value: weights against it overflow for every
  // score but that value itself, so a row's first visible tile always refreshes it, and a row that
  // sees no key of a piece's first tiles keeps weights of 0 (no inf - inf).
  float m_s = -FLT_MAX, l_run = 0.f;
  const bf16x2 ones = {static_cast<__bf16>(1.f), static_cast<__bf16>(1.f)};

  dma_wait_barrier<2 * BPW>();   // tiles 0 and 1 landed
  if (qrow0 >= cd.q_len) {
    // A wave whose 32 query rows all lie past the chunk's end only does its share of the copies and
    // leaves the matrix cores to the others (17 tokens on 1007 at G = 4: 29.2 -> 19.6 us).
    for (int j = kt0; j < n_kt; ++j) {
      copy_tile(page_next, (j - kt0 + 3) % NBUF);
      page_next = page_of(j + 4);
      dma_wait_barrier<2 * BPW>();
    }
    dma_wait_barrier<0>();
    return;
  }
  auto k_operand = [&](int buf, int ks, int kt2) {
    return as_bf16x8(ld16(smem + buf * HALF_TILE + kaddr[ks] + kt2 * (HALF_TILE / 2)));
  };
  auto v_operand = [&](int buf, int kt2, int j2, int t) {
    return as_bf16x8(ld16(smem + VBASE + buf * HALF_TILE + vaddr + (DT * (2 * kt2 + j2) + t) * 1024));
  };
  // With PRE the K operands of the next tile are read into registers during the current tile's PV product.
  bf16x8 kop[KS][2];
  auto read_k = [&](int buf) {
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int kt2 = 0; kt2 < 2; ++kt2) kop[ks][kt2] = k_operand(buf, ks, kt2);
  };
  if constexpr (PRE) read_k(0);

  auto tile_step = [&](const int j, const int buf) {
    copy_tile(page_next, (buf + 3) % NBUF);
    f32x16 s[2];
#pragma unroll
    for (int kt2 = 0; kt2 < 2; ++kt2)
#pragma unroll
      for (int e = 0; e < 16; ++e) s[kt2][e] = 0.f;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int kt2 = 0; kt2 < 2; ++kt2)
        s[kt2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(PRE ? kop[ks][kt2] : k_operand(buf, ks, kt2), qop[ks], s[kt2],
                                                         0, 0, 0);

    bf16x8 vop[2][2][DT];
#pragma unroll
    for (int kt2 = 0; kt2 < 2; ++kt2)
#pragma unroll
      for (int j2 = 0; j2 < 2; ++j2)
#pragma unroll
        for (int t = 0; t < DT; ++t)
          if constexpr (PRE) vop[kt2][j2][t] = v_operand(buf, kt2, j2, t);

    page_next = page_of(j + 4);    // for the next step's copy; it arrives behind the softmax

    if (kBN * j + kBN - 1 > pos_min) {
#pragma unroll
      for (int kt2 = 0; kt2 < 2; ++kt2)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int key = kBN * j + 32 * kt2 + 16 * (e >> 3) + 8 * half + 4 * ((e >> 2) & 1) + (e & 3);
          if (key > qpos) s[kt2][e] = -INFINITY;
        }
    }
    // Weights against the running max m. If a lane's partial sum over its 32 keys of the tile
    // exceeds 2^8 or is not finite (always on a row's first visible tile), the wave takes the
    // tile's row max, rescales O and l and recomputes the weights: every weight stays <= 2^8
    // without a max reduction on the common path.
    bf16x8 pop[2][2];
    auto weights = [&](float neg_m) {
      float ps0 = 0.f, ps1 = 0.f;
#pragma unroll
      for (int kt2 = 0; kt2 < 2; ++kt2) {
        float p[16];
#pragma unroll
        for (int e = 0; e < 16; ++e) p[e] = fast_exp2(__builtin_fmaf(s[kt2][e], c, neg_m));
#pragma unroll
        for (int j2 = 0; j2 < 2; ++j2) {
          const uint4 pw = make_uint4(pack_bf16x2(p[8 * j2 + 0], p[8 * j2 + 1]),
                                      pack_bf16x2(p[8 * j2 + 2], p[8 * j2 + 3]),
                                      pack_bf16x2(p[8 * j2 + 4], p[8 * j2 + 5]),
                                      pack_bf16x2(p[8 * j2 + 6], p[8 * j2 + 7]));
          // the denominator sums the same bf16-rounded weights the PV product uses
          ps0 = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pw.x), ones, ps0, false);
          ps1 = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pw.y), ones, ps1, false);
          ps0 = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pw.z), ones, ps0, false);
          ps1 = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pw.w), ones, ps1, false);
          pop[kt2][j2] = __builtin_bit_cast(bf16x8, pw);
        }
      }
      return ps0 + ps1;
    };
    float ps = weights(-m_s);
    if (__builtin_amdgcn_ballot_w64(!(ps <= kSumLimit)) != 0) {
      float mx = -INFINITY;
#pragma unroll
      for (int kt2 = 0; kt2 < 2; ++kt2)
#pragma unroll
        for (int e = 0; e < 16; ++e) mx = fmaxf(mx, s[kt2][e]);
      const float m_new = fmaxf(m_s, halves_max(mx) * c);
      const float alpha = fast_exp2(m_s - m_new);
      m_s = m_new;
      l_run *= alpha;
#pragma unroll
      for (int t = 0; t < DT; ++t) o[t] *= alpha;
      ps = weights(-m_new);
    }
    l_run += ps;
#pragma unroll
    for (int kt2 = 0; kt2 < 2; ++kt2)
#pragma unroll
      for (int j2 = 0; j2 < 2; ++j2)
#pragma unroll
        for (int t = 0; t < DT; ++t)
          o[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(PRE ? vop[kt2][j2][t] : v_operand(buf, kt2, j2, t),
                                                         pop[kt2][j2], o[t], 0, 0, 0);
    if constexpr (PRE) read_k((buf + 1) % NBUF);      // tile j+1 is in LDS (waited at the end of step j-1)
    // this wave's copies of tile j+2 have landed (those of tile j+3 may still fly); after the
    // barrier every wave's have. The next step copies over this step's buffer. With PRE its V^T operands
    // were read before the softmax and the reads still in flight are the next tile's K, a buffer that is
    // copied over a step later; without PRE the last V^T reads are waited for here.
    dma_wait_barrier<2 * BPW, !PRE>();
  };
  // One piece's record: the accumulators as they lie in the registers (every store 1 KiB of consecutive
  // bytes per wave), then (maximum, sum) of each lane's row.
  auto record = [&](int pt_) {
    return a.parts + dl * a.part_stride + (static_cast<size_t>(pt_) * a.n_kv_heads + g) * extend_part_floats(D);
  };
  auto write_record = [&]() {
    float* rec = record(part);
    f32x4* ow = reinterpret_cast<f32x4*>(rec) + wave * (4 * DT * 64) + lane;
#pragma unroll
    for (int t = 0; t < DT; ++t)
#pragma unroll
      for (int e4 = 0; e4 < 4; ++e4)
        ow[(4 * t + e4) * 64] = f32x4{o[t][4 * e4], o[t][4 * e4 + 1], o[t][4 * e4 + 2], o[t][4 * e4 + 3]};
    reinterpret_cast<f32x2*>(rec + kExtendTileRows * D)[wave * 64 + lane] = f32x2{m_s, halves_sum(l_run)};
  };
  float m_all = -FLT_MAX;   // over the pieces already recorded
  int kb = kt0, ke = chained ? min(n_kt, a.piece) : n_kt;   // a.piece is a multiple of the ring's four buffers
  for (;;) {
    for (int j = kb; j < ke; j += 4) {
      tile_step(j, 0);
      if (j + 1 < ke) tile_step(j + 1, 1);
      if (j + 2 < ke) tile_step(j + 2, 2);
      if (j + 3 < ke) tile_step(j + 3, 3);
    }
    if (!CHAIN || ke == n_kt) break;
    // The stores stay in flight: the loop's waits count them too and so only wait for more (loads return
    // in order among themselves: with at most N operations left, the loads left are the newest N).
    write_record();
    m_all = fmaxf(m_all, m_s);
    ++part;
#pragma unroll
    for (int t = 0; t < DT; ++t)
#pragma unroll
      for (int e = 0; e < 16; ++e) o[t][e] = 0.f;
    m_s = -FLT_MAX;
    l_run = 0.f;
    kb = ke;
    ke = min(n_kt, ke + a.piece);
  }
  // no copy may land after the workgroup ends, nor in what follows
  dma_wait_barrier<0>();

  if (tile.part >= 0) {
    write_record();
    return;
  }
  float l_tot = halves_sum(l_run);
  if (chained) {
    // Combine with the records of the pieces before, as extend_merge_body does (this wave wrote them
    // and has waited for the stores).
    const int part0 = -1 - tile.k0;
    const size_t stride = static_cast<size_t>(a.n_kv_heads) * extend_part_floats(D);
    const float* ml = record(part0) + kExtendTileRows * D + (wave * 64 + lane) * 2;
    const float* src = record(part0) + (wave * 4 * DT * 64 + lane) * 4;
    const float M = fmaxf(m_all, m_s);
    float l = 0.f;
    f32x16 acc[DT];
#pragma unroll
    for (int t = 0; t < DT; ++t)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[t][e] = 0.f;
    for (int i = 0; i < part - part0; ++i) {
      const f32x2 x = *reinterpret_cast<const f32x2*>(ml + i * stride);
      f32x4 v[DT][4];
#pragma unroll
      for (int t = 0; t < DT; ++t)
#pragma unroll
        for (int e4 = 0; e4 < 4; ++e4)
          v[t][e4] = *reinterpret_cast<const f32x4*>(src + i * stride + (4 * t + e4) * 256);
      const float wt = fast_exp2(x.x - M);
      l = __builtin_fmaf(wt, x.y, l);
#pragma unroll
      for (int t = 0; t < DT; ++t)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[t][e] = __builtin_fmaf(wt, v[t][e / 4][e % 4], acc[t][e]);
    }
    const float w_last = fast_exp2(m_s - M);
    l_tot = __builtin_fmaf(w_last, l_tot, l);
#pragma unroll
    for (int t = 0; t < DT; ++t)
#pragma unroll
      for (int e = 0; e < 16; ++e) o[t][e] = __builtin_fmaf(w_last, o[t][e], acc[t][e]);
  }
  // Through the wave's own part of LDS (rows padded by 16 bytes), so that a store writes whole rows (64
  // lanes: RPB rows of 2 D bytes) instead of 8 bytes in each of 32 rows (a 1437-token prompt 28.6 -> 25.9
  // us).
  constexpr int ORS = 2 * D + 16;
  static_assert(NW * 32 * ORS <= 2 * NBUF * HALF_TILE, "the output rows of all waves fit the ring");
  uint8_t* obuf = smem + wave * (32 * ORS);
  const float inv = 1.f / l_tot;
#pragma unroll
  for (int t = 0; t < DT; ++t)
#pragma unroll
    for (int e4 = 0; e4 < 4; ++e4)
      st8(obuf + col * ORS + 2 * (32 * t + 8 * e4 + 4 * half),
          make_uint2(pack_bf16x2(o[t][4 * e4 + 0] * inv, o[t][4 * e4 + 1] * inv),
                     pack_bf16x2(o[t][4 * e4 + 2] * inv, o[t][4 * e4 + 3] * inv)));
  uint16_t* orow = a.out + dl * a.q_stride + (static_cast<size_t>(cd.q_row + qrow0) * n_q_heads + h) * D + 8 * (lane % CPR);
  const int rows = cd.q_len - qrow0;
#pragma unroll
  for (int i = 0; i < 32 / RPB; ++i) {
    const int r = RPB * i + lane / CPR;
    const uint4 x = ld16(obuf + r * ORS + 16 * (lane % CPR));
    if (r < rows) st16(orow + static_cast<size_t>(r) * n_q_heads * D, x);
  }
}

// Merge of the pieces of one cut tile: one of 8 workgroups per (tile, kv head), 256 threads; kv heads
// fastest, as in the grid that wrote the records. Workgroup w takes the rows of wave w, thread `tid` the accumulators of lane tid % 64, DT of its
// 4 DT groups of 4 dims; the pieces are added in their order (bitwise deterministic). A piece in which
// a row sees no key has maximum -FLT_MAX and sum 0 and adds 0.
template <int D, int G>
__device__ __forceinline__ void extend_merge_body(const ExtendArgs& a, const int block, const int dl,
                                                  const int tid) {
  constexpr int DT = D / 32;
  const int g = block % a.n_kv_heads, w = (block / a.n_kv_heads) % 8;
  const ExtendMerge mg = a.merge(block / 8 / a.n_kv_heads);
  const ExtendConvDesc cd = a.conv(mg.conv);
  if (mg.q0 + 32 * (w / G) >= cd.q_len) return;   // rows past the chunk's end have no records
  const int lane = tid & 63, sub = tid >> 6, half = lane >> 5;
  const size_t stride = static_cast<size_t>(a.n_kv_heads) * extend_part_floats(D);
  const float* rec = a.parts + dl * a.part_stride +
                     (static_cast<size_t>(mg.part0) * a.n_kv_heads + g) * extend_part_floats(D);
  const float* ml = rec + kExtendTileRows * D + (w * 64 + lane) * 2;
  const float* src = rec + ((w * 4 * DT + sub * DT) * 64 + lane) * 4;
  // The first kAhead records are loaded whole before the maximum is known: one trip to memory less.
  constexpr int kAhead = 4;
  f32x2 x0[kAhead];
  f32x4 v0[kAhead][DT];
#pragma unroll
  for (int i = 0; i < kAhead; ++i) {
    const size_t at = (i < mg.n_parts ? i : 0) * stride;
    x0[i] = *reinterpret_cast<const f32x2*>(ml + at);
#pragma unroll
    for (int k = 0; k < DT; ++k) v0[i][k] = *reinterpret_cast<const f32x4*>(src + at + k * 256);
  }
  float M = -FLT_MAX;
#pragma unroll
  for (int i = 0; i < kAhead; ++i) M = fmaxf(M, x0[i].x);
#pragma unroll 4
  for (int i = kAhead; i < mg.n_parts; ++i) M = fmaxf(M, ml[i * stride]);
  f32x4 acc[DT];
#pragma unroll
  for (int k = 0; k < DT; ++k) acc[k] = f32x4{0.f, 0.f, 0.f, 0.f};
  float l = 0.f;
  auto add = [&](f32x2 x, const f32x4 (&v)[DT]) {
    const float wt = fast_exp2(x.x - M);
    l = __builtin_fmaf(wt, x.y, l);
#pragma unroll
    for (int k = 0; k < DT; ++k)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[k][r] = __builtin_fmaf(wt, v[k][r], acc[k][r]);
  };
#pragma unroll
  for (int i = 0; i < kAhead; ++i)
    if (i < mg.n_parts) add(x0[i], v0[i]);
#pragma unroll 2
  for (int i = kAhead; i < mg.n_parts; ++i) {
    f32x4 v[DT];
#pragma unroll
    for (int k = 0; k < DT; ++k) v[k] = *reinterpret_cast<const f32x4*>(src + i * stride + k * 256);
    add(*reinterpret_cast<const f32x2*>(ml + i * stride), v);
  }
  const int qi = mg.q0 + 32 * (w / G) + (lane & 31);
  if (qi >= cd.q_len) return;
  const float inv = 1.f / l;
  uint16_t* orow = a.out + dl * a.q_stride +
                   (static_cast<size_t>(cd.q_row + qi) * (a.n_kv_heads * G) + g * G + w % G) * D;
#pragma unroll
  for (int k = 0; k < DT; ++k) {
    const int c = sub * DT + k;     // 32-dim tile c / 4, group c % 4 of its accumulators
    st8(orow + 32 * (c / 4) + 8 * (c % 4) + 4 * half,
        make_uint2(pack_bf16x2(acc[k][0] * inv, acc[k][1] * inv), pack_bf16x2(acc[k][2] * inv, acc[k][3] * inv)));
  }
}

// blockIdx.y: layer (consecutive layers of one launch share the plan)
template <int D, int G, bool PRE, bool CHAIN>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(PRE ? 2 : 4)))
void attn_fwd_kernel(LaunchMeta, ExtendArgs a) {
  attn_fwd_block<D, G, PRE, CHAIN>(a, blockIdx.x, blockIdx.y);
}

template <int D, int G>
__global__ __launch_bounds__(256) void extend_merge_kernel(LaunchMeta, ExtendArgs a) {
  extend_merge_body<D, G>(a, blockIdx.x, blockIdx.y, threadIdx.x);
}

// One layer of a mixed step in one launch: extend tiles (or pieces) and work items of the decode split
// (8 waves, as in the split kernel), one workgroup each. Every workgroup gets the attention kernel's LDS
// ring and register budget, one workgroup (two waves per SIMD) a CU; at head dim 128 the decode split has no
// more by itself. At 64 it has three workgroups a CU by itself: 16 conversations of 10k tokens and a 20-token
// chunk take 64 us a layer here, 61 with the decode in its own launch.
// Units of n_kv_heads workgroups are taken in an order that spreads the extend units evenly over the
// first n_mix units, so that at any time some CUs use the matrix cores while others read HBM; n_mix =
// their number puts them all in front (tiles longer than everything else).
template <int D, int G, bool CHAIN>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2)))
void mixed_layer_kernel(ExtendArgs ea, int n_ext, int n_mix, DecodeArgs da) {
  static_assert(kDecodeItemThreads == 512, "a decode work item fills one attention workgroup");
  __shared__ float xch[split_exchange_floats<D>()];
  const int unit = blockIdx.x / ea.n_kv_heads, head = blockIdx.x % ea.n_kv_heads;
  const int before = unit < n_mix ? static_cast<int>(static_cast<int64_t>(unit) * n_ext / n_mix) : n_ext;
  const int after = unit < n_mix ? static_cast<int>(static_cast<int64_t>(unit + 1) * n_ext / n_mix) : n_ext;
  if (after > before) {
    attn_fwd_block<D, G, true, CHAIN>(ea, before * ea.n_kv_heads + head, 0);
    return;
  }
  split_body<D>(da, (unit - before) * ea.n_kv_heads + head, 0, __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), xch);
}

// What is left of that layer: the first n_ext workgroups merge its cut extend tiles, the others its
// decode records (n_dec of them, 256 threads each).
template <int D, int G>
__global__ __launch_bounds__(256) void mixed_merge_kernel(ExtendArgs ea, int n_ext, DecodeArgs da) {
  __shared__ MergeLds<D> lds;
  const int blk = blockIdx.x;
  if (blk < n_ext) {
    extend_merge_body<D, G>(ea, blk, 0, threadIdx.x);
    return;
  }
  merge_body<D>(da, blk - n_ext, 0, threadIdx.x, lds);
}

int extend_query_tile(int group) { return kExtendTileRows / group; }

static ExtendArgs make_extend_args(const PoolGeom& g, int layer, const ExtendLaunch& e, const void* q, void* out,
                                   float* parts) {
  ExtendArgs a;
  a.pool = static_cast<const uint16_t*>(g.pool);
  a.n_pages = g.n_pages;
  a.n_kv_heads = g.n_kv_heads;
  a.layer = layer;
  a.page_table = g.page_table;
  a.max_pages = g.max_pages;
  a.meta = e.meta.dev;
  a.tiles_off = static_cast<uint32_t>(e.tiles_off);
  a.merges_off = static_cast<uint32_t>(e.merges_off);
  a.q = static_cast<const uint16_t*>(q);
  a.out = static_cast<uint16_t*>(out);
  a.scale_log2 = static_cast<float>(1.4426950408889634 / std::sqrt(static_cast<double>(g.head_dim)));
  a.piece = e.piece;
  a.parts = parts;
  a.q_stride = static_cast<size_t>(e.q_rows) * g.n_q_heads * g.head_dim;
  a.part_stride = static_cast<size_t>(e.n_parts) * g.n_kv_heads * extend_part_floats(g.head_dim);
  return a;
}

// Calls f with std::integral_constant<int, D> and <int, G> of the pool's head dim and GQA group.
template <typename F>
static hipError_t by_shape(const PoolGeom& g, F&& f) {
  const int G = g.n_q_heads / g.n_kv_heads;
  auto by_group = [&](auto d) {
    if (G == 1) return f(d, std::integral_constant<int, 1>{});
    if (G == 2) return f(d, std::integral_constant<int, 2>{});
    if (G == 4) return f(d, std::integral_constant<int, 4>{});
    if (G == 8) return f(d, std::integral_constant<int, 8>{});
    return hipErrorInvalidValue;
  };
  if (g.head_dim == 128) return by_group(std::integral_constant<int, 128>{});
  if (g.head_dim == 64) return by_group(std::integral_constant<int, 64>{});
  return hipErrorInvalidValue;
}

hipError_t launch_extend(const PoolGeom& g, int layer, int n_layers, const ExtendLaunch& e, const void* q, void* out,
                         float* parts, hipStream_t stream) {
  if (e.n_tiles == 0 || n_layers == 0) return hipSuccess;
  if (!e.meta.ok() || (e.n_parts > 0 && (parts == nullptr || e.piece < 1))) return hipErrorInvalidValue;
  const ExtendArgs a = make_extend_args(g, layer, e, q, out, parts);
  LaunchMeta m;
  fill_meta(e.meta, &m);
  const dim3 grid(e.n_tiles * g.n_kv_heads, n_layers);
  // At head_dim 64 a launch of more than 2.5 workgroups per CU runs two at a time on each: one prompt of
  // 9000 tokens (1128 workgroups) 352 -> 339 us, 6000 (752) 168 -> 163; below, one at a time that reads
  // its operands ahead is the faster form: 4500 (568) 98 against 106 us, 2500 (320) 41 against 45. A
  // head_dim 128 workgroup fills its CU's LDS.
  const bool two_per_cu = static_cast<int64_t>(grid.x) * grid.y > 5 * kCus / 2;
  auto launch = [&](auto kernel) {
    kernel<<<grid, 512, 0, stream>>>(m, a);
    return hipGetLastError();
  };
  return by_shape(g, [&](auto d, auto grp) {
    if constexpr (d() == 64) {
      if (two_per_cu)
        return e.chained ? launch(attn_fwd_kernel<d(), grp(), false, true>) : launch(attn_fwd_kernel<d(), grp(), false, false>);
    }
    return e.chained ? launch(attn_fwd_kernel<d(), grp(), true, true>) : launch(attn_fwd_kernel<d(), grp(), true, false>);
  });
}

hipError_t launch_extend_merge(const PoolGeom& g, int n_layers, const ExtendLaunch& e, void* out, float* parts,
                               hipStream_t stream) {
  if (e.n_merges == 0 || n_layers == 0) return hipSuccess;
  if (!e.meta.ok() || parts == nullptr) return hipErrorInvalidValue;
  const ExtendArgs a = make_extend_args(g, 0, e, nullptr, out, parts);
  LaunchMeta m;
  fill_meta(e.meta, &m);
  return by_shape(g, [&](auto d, auto grp) {
    extend_merge_kernel<d(), grp()><<<dim3(e.n_merges * g.n_kv_heads * 8, n_layers), 256, 0, stream>>>(m, a);
    return hipGetLastError();
  });
}

hipError_t launch_mixed_layer(const PoolGeom& g, int layer, const ExtendLaunch& e, const void* q_ext,
                              void* out_ext, float* parts, const DecodeLaunch& w, const void* q_dec,
                              float* partials, void* direct_out, hipStream_t stream) {
  if (e.n_tiles == 0 || w.n_convs == 0) return hipErrorInvalidValue;
  if (e.meta.dev == nullptr || w.meta.dev == nullptr || w.n_items < w.n_convs) return hipErrorInvalidValue;
  if (direct_out != nullptr && w.n_items != w.n_convs) return hipErrorInvalidValue;
  if (e.n_parts > 0 && (parts == nullptr || e.piece < 1)) return hipErrorInvalidValue;
  const ExtendArgs ea = make_extend_args(g, layer, e, q_ext, out_ext, parts);
  DecodeArgs da = make_decode_args(g, layer, w, q_dec, direct_out, partials);
  da.direct = direct_out != nullptr;
  // Pieces of cut tiles (all short) are spread over the first 60% of the decode items; whole and chained
  // tiles go in front of them. Layers of 16 conversations (2k-12k tokens, a 513-token chunk): 4.20-4.33 ms per 32-layer
  // step with the pieces in front, 4.06 spread over 40%, 4.05 over 70%, 4.72 over all; 16 x 4k tokens and
  // a 300-token chunk 3.19, 2.88, 2.70, 2.92.
  const int n_mix = e.n_tiles + (e.n_merges > 0 ? w.n_items * 6 / 10 : 0);
  const int blocks = (e.n_tiles + w.n_items) * g.n_kv_heads;
  return by_shape(g, [&](auto d, auto grp) {
    if (e.chained) mixed_layer_kernel<d(), grp(), true><<<blocks, 512, 0, stream>>>(ea, e.n_tiles, n_mix, da);
    else mixed_layer_kernel<d(), grp(), false><<<blocks, 512, 0, stream>>>(ea, e.n_tiles, n_mix, da);
    return hipGetLastError();
  });
}

hipError_t launch_mixed_merge(const PoolGeom& g, const ExtendLaunch& e, void* out_ext, float* parts,
                              const DecodeLaunch& w, const float* partials, void* out_dec, hipStream_t stream) {
  // out_dec == nullptr: the split wrote the decode outputs
  const int n_ext = e.n_merges * g.n_kv_heads * 8;
  const int blocks = n_ext + (out_dec != nullptr ? w.n_convs * g.n_q_heads : 0);
  if (blocks == 0) return hipSuccess;
  if (e.meta.dev == nullptr || w.meta.dev == nullptr || (n_ext > 0 && parts == nullptr)) return hipErrorInvalidValue;
  const ExtendArgs ea = make_extend_args(g, 0, e, nullptr, out_ext, parts);
  const DecodeArgs da = make_decode_args(g, 0, w, nullptr, out_dec, partials);
  return by_shape(g, [&](auto d, auto grp) {
    mixed_merge_kernel<d(), grp()><<<blocks, 256, 0, stream>>>(ea, n_ext, da);
    return hipGetLastError();
  });
}

}  // namespace cs
