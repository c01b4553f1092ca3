// Batched single-token decode attention over paged KV (split-K "flash decoding").
//
// A work item is up to kDecodeSubSplits splits (`split` keys each) of consecutive keys of one
// (conversation, kv head), taken by one workgroup; its waves share its keys evenly, each reading
// its range once and serving all G query heads of the kv head. Workgroups take the items in the
// plan's launch order (full items first, then shorter ones). The two contractions per page pair are
// done on the matrix cores with v_mfma_f32_16x16x32_bf16, the GQA group as the 16-wide N side:
//   S^T[key][head] = K[key][:] . Q[head][:]          (A = K rows straight from the page,
//                                                     B = Q, 8 consecutive dims per lane)
//   O^T[dim][head] += V^T[dim][key] . P^T[key][head]  (A = V^T rows from the page,
//                                                     B = P from the S^T accumulator registers)
// so K and V^T are used in the layout they are stored in: each K operand load reads one 1 KiB
// sub-block of a page, each V^T load 512 consecutive bytes. The softmax is online in fp32 (exp2
// with log2(e)/sqrt(d) folded into the score scale). The waves of an item merge their (o, m, l) in
// LDS and write one partial record per (item, query head) to a workspace (decode_split.hpp); a
// second kernel merges the items of each (conversation, query head). Both merges run in a fixed
// order and there are no atomics: bitwise deterministic, and split boundaries are logical
// positions, so results do not depend on physical page placement.
// Bound: HBM in large batches (64 conversations of 8k-32k tokens: 6.74 TB/s, 95% of the 7.07 that the
// fastest plain read of 4 GiB in 8 KiB blocks reaches); in small ones the four or fewer page pairs a wave
// reads one after the other and the merge launch (one conversation of 2000 tokens 11.3 us, of 24.6k 19.1
// of which the merge is 3.9).
#include <cmath>
#include <mutex>

#include "decode_split.hpp"

namespace cs {

namespace {
// Static decode scratch of the allocation-free decode entry point: the split partial records live
// here instead of in the pool's workspace. Each GPU the library runs on holds its own copy until
// the process ends. Host code never passes `scratch` itself to a kernel (on the host it is only a
// stand-in symbol): its device address, per device, comes from hipGetSymbolAddress below.
__device__ __align__(256) float scratch[kStaticScratchFloats];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
float* g_scratch_dev[kMaxDevices] = {};
}  // namespace

hipError_t static_decode_scratch(float** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (g_scratch_dev[dev] == nullptr) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));   // with `dev` current: this device's copy
    if (e != hipSuccess) return e;
    g_scratch_dev[dev] = static_cast<float*>(p);
  }
  *out = g_scratch_dev[dev];
  return hipSuccess;
}

// blockIdx.y: layer, counted from a.layer
template <int D>
__global__ __launch_bounds__(kDecodeItemThreads) void decode_split_kernel(LaunchMeta, DecodeArgs a) {
  __shared__ float xch[split_exchange_floats<D>()];
  split_body<D>(a, blockIdx.x, blockIdx.y, __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), xch);
}

template <int D>
__global__ __launch_bounds__(256) void decode_merge_kernel(LaunchMeta, DecodeArgs a) {
  __shared__ MergeLds<D> lds;
  merge_body<D>(a, blockIdx.x, blockIdx.y, threadIdx.x, lds);
}

hipError_t launch_decode_split(const PoolGeom& g, int layer, int n_layers, const DecodeLaunch& w, const void* q,
                               float* partials, void* direct_out, hipStream_t stream) {
  if (w.n_convs == 0 || n_layers == 0) return hipSuccess;
  if (!w.meta.ok() || w.n_items < w.n_convs) return hipErrorInvalidValue;
  DecodeArgs a = make_decode_args(g, layer, w, q, direct_out, partials);
  a.direct = direct_out != nullptr && w.n_items == w.n_convs;
  if (direct_out != nullptr && !a.direct) return hipErrorInvalidValue;
  LaunchMeta m;
  fill_meta(w.meta, &m);
  const dim3 grid(w.n_items * g.n_kv_heads, n_layers);
  if (g.head_dim == 128) decode_split_kernel<128><<<grid, kDecodeItemThreads, 0, stream>>>(m, a);
  else if (g.head_dim == 64) decode_split_kernel<64><<<grid, kDecodeItemThreads, 0, stream>>>(m, a);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_decode_merge(const PoolGeom& g, int n_layers, const DecodeLaunch& w, const float* partials,
                               void* out, hipStream_t stream) {
  if (w.n_convs == 0 || n_layers == 0) return hipSuccess;
  if (!w.meta.ok()) return hipErrorInvalidValue;
  const DecodeArgs a = make_decode_args(g, 0, w, nullptr, out, partials);
  LaunchMeta m;
  fill_meta(w.meta, &m);
  const dim3 grid(w.n_convs * g.n_q_heads, n_layers);
  if (g.head_dim == 128) decode_merge_kernel<128><<<grid, 256, 0, stream>>>(m, a);
  else if (g.head_dim == 64) decode_merge_kernel<64><<<grid, 256, 0, stream>>>(m, a);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace cs
