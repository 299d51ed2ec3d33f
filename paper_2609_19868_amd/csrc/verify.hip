// Verification step of slotted speculative decoding (gfx950): token acceptance
// and the KV-cache append of the accepted tokens.
//
// What is computed (Zarya, Sec. 5.2 "Verification phase" and "KV cache
// update"; Sec. 6 token threshold 0.4): in every slot listed as verified, a
// draft token whose probability under the autoregressive verification pass
// exceeds the threshold is accepted -- with the prefix rule only the leading
// run of such tokens -- and the accepted tokens' keys and values are appended
// to the cache after the committed prefix, which grows by their number.
//
// Both kernels are a few KB of integer and copy work per batch row, bound by
// the latency of the dependent steps (list, flags, counts, positions, copy), so
// one workgroup of 1024 threads per batch row takes each step for the whole row
// at once: a thread per list entry, a thread per token, and for the counts and
// positions a power of two of lanes per slot.
#include <algorithm>

#include "common.hpp"
#include "kernels.hpp"

namespace zarya {

namespace {

constexpr int kThreads = 1024;  // at most: one per slot at the largest S

}  // namespace

// One workgroup per batch row.  A verified slot accepts its leading run of
// passing tokens (its length is the lowest failing position) or, token by
// token, every passing one.  B = 16, 8 slots of 8 tokens: 6.6 -> 3.4 us (a
// thread per slot walked its tokens, waiting for each).
template <int MAXT>
__global__ __launch_bounds__(MAXT) void verify_accept_kernel(AcceptParams p) {
  __shared__ int listed[1024], run[1024], count[1024];
  __shared__ int end, total;
  const int b = blockIdx.x, tid = threadIdx.x, threads = MAXT == kThreads ? kThreads : blockDim.x;
  const int32_t* sel = p.selected + (size_t)b * p.S;
  const int mine = tid < p.S ? sel[tid] : 0;
  // f(i, list entry i) over the list, f(s, 0) over the slots: a thread each with kThreads
  auto each = [&](int n, bool entries, auto&& f) {
    if constexpr (MAXT == kThreads) {
      if (tid < n) f(tid, mine);
    } else {
      for (int i = tid; i < n; i += threads) f(i, entries ? sel[i] : 0);
    }
  };
  if (tid == 0) {
    end = p.S;
    total = 0;
  }
  each(p.S, false, [&](int s, int) {
    listed[s] = 0;
    run[s] = p.L;
    count[s] = 0;
  });
  __syncthreads();
  // integer minima and sums in LDS: order-free
  each(p.S, true, [&](int i, int s) {
    if (s < 0) atomicMin(&end, i);  // the first negative entry ends the list
  });
  const float* tp = p.token_prob + (size_t)b * p.S * p.L;
  const int T = p.S * p.L;
  for (int x = tid; x < T; x += threads) {
    const int s = x / p.L;
    if (tp[x] > p.threshold) {
      if (p.rule != 0) atomicAdd(&count[s], 1);
    } else {
      atomicMin(&run[s], x - s * p.L);
    }
  }
  __syncthreads();
  each(end, true, [&](int, int s) {
    if (s < p.S) listed[s] = 1;  // ids >= S are skipped
  });
  __syncthreads();
  uint8_t* acc = p.accepted + (size_t)b * T;
  for (int x = tid; x < T; x += threads) {
    const int s = x / p.L;
    acc[x] = listed[s] && (p.rule == 0 ? x - s * p.L < run[s] : tp[x] > p.threshold) ? 1 : 0;
  }
  each(p.S, false, [&](int s, int) {
    const int n = listed[s] ? (p.rule == 0 ? run[s] : count[s]) : 0;
    p.n_accepted[(size_t)b * p.S + s] = n;
    if (n) atomicAdd(&total, n);
  });
  __syncthreads();
  if (tid == 0 && p.n_total) p.n_total[b] = total;
}

// One workgroup per batch row: list the accepted tokens in append order in
// LDS (a slot listed twice counts at its first position only), check that
// they fit, then copy their K and V rows of every KV head in 16-byte pieces
// and move the row's prefix length.  `lg`: log2 of the lanes per slot.
// B = 16, 8 heads, 4 of 8 slots with 7 of 8 tokens: 9.4 -> 7.2 us (256 threads,
// a serial scan over the slots and a thread per slot reading its flags).
__global__ __launch_bounds__(kThreads) void kv_append_kernel(AppendParams p, int lg) {
  __shared__ int slot_of[1024];   // order position -> slot id (or -1)
  __shared__ int count_of[1024];  // order position -> accepted tokens of that slot
  __shared__ int start_of[1024];  // order position -> first index in `tokens`
  __shared__ int first_pos[1024];  // slot id -> first order position listing it
  __shared__ int wave_sum[kThreads / 64];
  __shared__ uint8_t flags[kAppendMaxTokens];  // the row's accepted flags
  __shared__ int tokens[kAppendMaxTokens];
  __shared__ int end;
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
  const int T = p.S * p.L;
  const int s_mine = tid < p.S ? p.order[(size_t)b * p.S + tid] : -1;
  const int p0 = p.prefix_lens[b];
  const uint8_t* acc = p.accepted + (size_t)b * T;
  for (int x = tid; x < T; x += kThreads) flags[x] = acc[x];
  if (tid == 0) end = p.S;
  first_pos[tid] = p.S;
  __syncthreads();
  if (tid < p.S && s_mine < 0) atomicMin(&end, tid);  // end of the order list
  __syncthreads();
  const bool in_list = tid < end && s_mine < p.S;
  if (in_list) atomicMin(&first_pos[s_mine], tid);  // LDS integer minimum: order-free
  __syncthreads();
  // a slot listed again is skipped: its tokens are committed once
  slot_of[tid] = in_list && first_pos[s_mine] == tid ? s_mine : -1;
  __syncthreads();
  // 1 << lg neighbouring lanes take one slot, a token each (in rounds where the
  // slot is longer); f(position, token, rank of the token in its slot) for the
  // accepted ones
  const int per = 1 << lg, sub = tid & (per - 1);
  const uint64_t group = (lg == 6 ? ~0ull : (1ull << per) - 1) << (lane & ~(per - 1));
  auto each_accepted = [&](auto&& f, auto&& done) {
    for (int i0 = 0; i0 < p.S; i0 += kThreads >> lg) {  // the same trips for every lane
      const int i = i0 + (tid >> lg);
      const int s = i < p.S ? slot_of[i] : -1;
      int n = 0;
      for (int r0 = 0; r0 < p.L; r0 += per) {
        const int r = r0 + sub;
        const bool a = s >= 0 && r < p.L && flags[s * p.L + r] != 0;
        const uint64_t m = __ballot(a) & group;
        if (a) f(i, s * p.L + r, n + __popcll(m & ((1ull << lane) - 1)));
        n += __popcll(m);
      }
      if (sub == 0 && i < p.S) done(i, n);
    }
  };
  each_accepted([](int, int, int) {}, [&](int i, int n) { count_of[i] = n; });
  __syncthreads();
  // exclusive scan of the counts in order
  const int c = tid < p.S ? count_of[tid] : 0;
  int incl = c;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int up = __shfl_up(incl, off);
    if (lane >= off) incl += up;
  }
  if (lane == 63) wave_sum[tid >> 6] = incl;
  __syncthreads();
  int before = 0, n = 0;
#pragma unroll
  for (int w = 0; w < kThreads / 64; ++w) {
    before += w < (tid >> 6) ? wave_sum[w] : 0;
    n += wave_sum[w];
  }
  start_of[tid] = before + incl - c;
  if (p0 < 0 || (long long)p0 + n > p.C) return;  // uniform: the row does not fit and stays unchanged
  __syncthreads();
  each_accepted([&](int i, int token, int rank) { tokens[start_of[i] + rank] = token; }, [](int, int) {});
  __syncthreads();
  const int lp = __builtin_ctz(p.row_bytes / 16);  // 16-byte pieces of a row: 8, 16 or 32
  // one flat loop over (head, token, 16-byte piece): every thread's loads are
  // independent of its stores (the slot K/V and the cache never overlap), so
  // many are in flight at once
  const char* __restrict__ ks = static_cast<const char*>(p.k_slot);
  const char* __restrict__ vs = static_cast<const char*>(p.v_slot);
  char* __restrict__ kc = static_cast<char*>(p.k_cache);
  char* __restrict__ vc = static_cast<char*>(p.v_cache);
  const int total = (p.Hkv * n) << lp;
#pragma unroll 4
  for (int e = tid; e < total; e += kThreads) {
    const int x = e >> lp, c16 = (e & ((1 << lp) - 1)) * 16;
    const int g = x / n, i = x - g * n;
    const size_t src = (((size_t)b * p.Hkv + g) * T + tokens[i]) * p.row_bytes + c16;
    const size_t dst = (((size_t)b * p.Hkv + g) * p.C + p0 + i) * p.row_bytes + c16;
    const uint4 kv = *reinterpret_cast<const uint4*>(ks + src);
    const uint4 vv = *reinterpret_cast<const uint4*>(vs + src);
    *reinterpret_cast<uint4*>(kc + dst) = kv;
    *reinterpret_cast<uint4*>(vc + dst) = vv;
  }
  if (tid == 0) p.prefix_lens[b] = p0 + n;
}

hipError_t launch_verify_accept(const AcceptParams& p, hipStream_t stream) {
  // 1024 threads a row, of which a unit holds two, where the rows alone do not
  // fill the units; with many rows up to 256 and no more than tokens (4096 rows: 64
  // slots of one token 25.0 us with 1024 threads, 8.5 with 64; 256 slots of 4 39.1
  // and 19.5 with 256; 512 rows 7.3 and 7.7)
  if (p.B < 1024) {
    verify_accept_kernel<kThreads><<<dim3(p.B), dim3(kThreads), 0, stream>>>(p);
  } else {
    const int threads = (int)std::min<int64_t>(256, ((int64_t)p.S * p.L + 63) / 64 * 64);
    verify_accept_kernel<256><<<dim3(p.B), dim3(threads), 0, stream>>>(p);
  }
  return hipGetLastError();
}

hipError_t launch_kv_append(const AppendParams& p, hipStream_t stream) {
  int lg = 0;  // a lane per token of a slot, up to a wave
  while (lg < 6 && (1 << lg) < p.L) ++lg;
  kv_append_kernel<<<dim3(p.B), dim3(kThreads), 0, stream>>>(p, lg);
  return hipGetLastError();
}

}  // namespace zarya
