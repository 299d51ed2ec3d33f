// Mode A of Zarya (MDM sampling with first-hitting denoising, Sec. 5.1):
// the positions a denoising step reveals (gfx950).  The mask budget of a
// generation is host code, in mdm_plan.hip.
//
// What is computed (Sec. 5.1 steps 1-3): a generation with N masks runs T
// diffusion steps that together reveal a Binomial(N, alpha_0) share of the
// masks, then reveals the rest one per step; with T = 0 the draw is skipped
// and T is a quarter of N.  At each step the model's drawn tokens of some
// masked positions are committed -- the most confident ones, the leftmost ones
// (sequential phase) or a uniformly random set (the first-hitting sampler) --
// and those positions join the committed part of the sequence.
//
// The reveal is integer work on at most 8192 positions per row, one workgroup
// per row, bound by the latency of dependent LDS steps.  Up to 512 positions
// every position counts the keys ahead of it (ties: the lower position), which
// is its place in the reveal order: reads that do not depend on each other, and
// two barriers in all.  256 positions: 10.3 us with the sort, 4.3 us; 512: 12.9
// and 9.8 us (16 rows, launches in a graph).  The
// counting grows with the square of the positions, so above 512 each key packs
// the rule's ordering (confidence, position, or a Philox uniform) above the
// position and one ascending bitonic sort in LDS yields the reveal order.
#include <algorithm>

#include "common.hpp"
#include "kernels.hpp"

namespace zarya {

namespace {

constexpr int kThreads = 1024;
constexpr uint64_t kClosed = ~0ull;  // sorts after every open position
constexpr uint32_t kClosedRank = ~0u;  // the same for the ordering alone (no open position's reaches it)
constexpr int kRankMaxN = 512;

// Float32 confidence -> 32-bit key that increases as the confidence falls
// (NaN counts as -inf, -0 as +0), by integer operations only.
__device__ __forceinline__ uint32_t conf_desc_key(float c) {
  uint32_t b = __float_as_uint(c);
  if ((b & 0x7F800000u) == 0x7F800000u && (b & 0x007FFFFFu) != 0) b = 0xFF800000u;  // NaN -> -inf
  if (b == 0x80000000u) b = 0;                                                        // -0 -> +0
  const uint32_t asc = (b & 0x80000000u) ? ~b : (b | 0x80000000u);  // increases with the value
  return ~asc;
}

// Philox uniform of (row, position) as its 23-bit integer (x >> 9): the same
// order as u = ((x >> 9) + 1/2) * 2^-23.
__device__ __forceinline__ uint32_t uniform_bits(const RevealParams& p, int row, int pos) {
  const uint4 r = philox4x32_10_dev((uint32_t)pos >> 2, (uint32_t)row, p.off_lo, p.off_hi, p.seed_lo, p.seed_hi);
  const uint32_t w[4] = {r.x, r.y, r.z, r.w};
  return w[pos & 3] >> 9;
}

// The rule's ordering of an open position.
__device__ __forceinline__ uint32_t order_key(const RevealParams& p, int row, int pos) {
  if (p.rule == 0) return conf_desc_key(p.conf[(size_t)row * p.N + pos]);
  return p.rule == 2 ? uniform_bits(p, row, pos) : 0;
}

}  // namespace

// N <= 512: kThreads / NP neighbouring lanes count for one position, four keys
// at a time.  A key of a lower position is ahead when it is not above mine, one
// of a higher position when it is below: one comparison each, against mine + 1
// or mine (an open position's key is below 2^32 - 1).
__global__ __launch_bounds__(kThreads) void mdm_reveal_rank_kernel(RevealParams p, int lanes) {
  __shared__ __attribute__((aligned(16))) uint32_t keys[kRankMaxN];
  const int b = blockIdx.x, tid = threadIdx.x;
  const size_t base = (size_t)b * p.N;
  const int k = p.k[b];
  const bool open = tid < p.N && p.mask[base + tid] != 0;
  if (tid < kRankMaxN) keys[tid] = open ? order_key(p, b, tid) : kClosedRank;
  const int n = min(max(k, 0), __syncthreads_count(open));
  const int i = tid / lanes, g = tid % lanes;
  const uint32_t mine = keys[min(i, kRankMaxN - 1)];
  int rank = 0;
  for (int j = 4 * g; j < p.N; j += 4 * lanes) {  // keys past N are closed
    const uint4 v = *reinterpret_cast<const uint4*>(&keys[j]);
    const uint32_t limit = mine + (j + 3 < i ? 1 : 0);
    rank += (v.x < limit) + (v.y < limit) + (v.z < limit) + (v.w < limit);
  }
  if (g == 0 && mine != kClosedRank) {  // equal keys of lower positions among my own four
    for (int j = i & ~3; j < i; ++j) rank += keys[j] == mine;
  }
  for (int off = lanes >> 1; off > 0; off >>= 1) rank += __shfl_xor(rank, off);
  if (g == 0 && mine != kClosedRank && rank < n) {
    p.order[base + rank] = i;
    p.mask[base + i] = 0;
    if (p.tokens) p.tokens[base + i] = p.sample_id[base + i];
  }
  if (tid >= n && tid < p.N) p.order[base + tid] = -1;
  if (tid == 0 && p.n_revealed) p.n_revealed[b] = n;
}

__global__ __launch_bounds__(kThreads) void mdm_reveal_kernel(RevealParams p) {
  __shared__ uint64_t keys[kRevealMaxN];
  __shared__ int n_open;
  const int b = blockIdx.x;
  const int tid = threadIdx.x;
  const size_t base = (size_t)b * p.N;
  if (tid == 0) n_open = 0;
  __syncthreads();
  int mine = 0;
  for (int i = tid; i < p.NP; i += kThreads) {
    uint64_t key = kClosed;
    if (i < p.N && p.mask[base + i] != 0) {
      key = ((uint64_t)order_key(p, b, i) << 32) | (uint32_t)i;
      ++mine;
    }
    keys[i] = key;
  }
  atomicAdd(&n_open, mine);  // integer sum: order-free
  __syncthreads();
  // ascending bitonic sort of NP keys (NP a power of two)
  for (int size = 2; size <= p.NP; size <<= 1) {
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      for (int t = tid; t < p.NP / 2; t += kThreads) {
        const int lo = 2 * t - (t & (stride - 1));  // first element of the pair
        const int hi = lo + stride;
        const bool up = (lo & size) == 0;
        const uint64_t a = keys[lo], c = keys[hi];
        if ((a > c) == up) {
          keys[lo] = c;
          keys[hi] = a;
        }
      }
      __syncthreads();
    }
  }
  const int n = min(max(p.k[b], 0), n_open);
  for (int j = tid; j < p.N; j += kThreads) {
    const int pos = j < n ? (int)(uint32_t)keys[j] : -1;
    p.order[base + j] = pos;
    if (j < n) {
      p.mask[base + pos] = 0;
      if (p.tokens) p.tokens[base + pos] = p.sample_id[base + pos];
    }
  }
  if (tid == 0 && p.n_revealed) p.n_revealed[b] = n;
}

hipError_t launch_mdm_reveal(const RevealParams& p, hipStream_t stream) {
  if (p.N <= kRankMaxN) {
    const int lanes = std::min(64, kThreads / p.NP);
    mdm_reveal_rank_kernel<<<dim3(p.B), dim3(std::max(p.NP * lanes, 64)), 0, stream>>>(p, lanes);
    return hipGetLastError();
  }
  mdm_reveal_kernel<<<dim3(p.B), dim3(kThreads), 0, stream>>>(p);
  return hipGetLastError();
}

}  // namespace zarya
