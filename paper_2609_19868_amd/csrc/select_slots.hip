// First-hitting slot selection (Zarya, Sec. 5.2 "Slot selection"; Sec. 6 uses
// slot_threshold = 0.9).  One workgroup per batch row.
//
// Slot confidence is the first token's probability (the paper's rule) or the
// mean over the slot, summed in float64 in token order, divided by L and
// rounded once to float32.  Every open slot gets its rank in first-hitting
// order: the number of open slots with a higher confidence, or an equal one
// and a lower index.  THRESHOLD keeps the open slots whose confidence exceeds
// the threshold (strictly) -- exactly the first ranks -- or, when none does,
// the rank-0 slot; TOP_K keeps ranks below k.  A kept slot is written at its
// rank, so the output is in first-hitting order without a sort.
#include "common.hpp"
#include "kernels.hpp"

namespace zarya {

constexpr int kMaxSlots = 1024;

// A thread per slot and no more waves than slots; bound by latency: 16 rows of
// 8 slots x 8 tokens under the mean rule 4.0 -> 2.9 us (one token's load waited
// for the sum before it).  Closed slots hold NaN in LDS, which compares false with
// everything: they count in no rank.
__global__ __launch_bounds__(kMaxSlots) void select_slots_kernel(SelectParams p) {
  __shared__ __attribute__((aligned(16))) float conf[kMaxSlots];
  __shared__ int n_open, n_above;
  const int b = blockIdx.x, s = threadIdx.x;
  if (s == 0) {
    n_open = 0;
    n_above = 0;
  }
  const bool op = s < p.S && (p.slot_open ? p.slot_open[(size_t)b * p.S + s] != 0 : true);
  float c = __builtin_nanf("");
  if (s < p.S) {
    const float* tc = p.token_conf + ((size_t)b * p.S + s) * p.L;
    if (p.conf_rule == 0) {
      c = tc[0];
    } else {
      // summed in token order; loaded eight at a time, so that the loads
      // overlap instead of each waiting for the sum before it
      double acc = 0.0;
      for (int r0 = 0; r0 < p.L; r0 += 8) {
        float t[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) t[j] = tc[min(r0 + j, p.L - 1)];
#pragma unroll
        for (int j = 0; j < 8; ++j)
          if (r0 + j < p.L) acc = acc + (double)t[j];
      }
      c = (float)(acc / (double)p.L);
    }
    if (c != c) c = -INFINITY;  // a NaN confidence ranks last and never passes the threshold
    p.slot_conf[(size_t)b * p.S + s] = op ? c : -1.f;
  }
  conf[s] = op ? c : __builtin_nanf("");
  __syncthreads();
  if (op) {
    atomicAdd(&n_open, 1);
    if (c > p.threshold) atomicAdd(&n_above, 1);
  }
  int rank = 0;
  if (op) {
    for (int o = 0; o < p.S; o += 4) {  // the block covers S rounded up to 64, so the tail holds NaN
      const f32x4 v = *reinterpret_cast<const f32x4*>(&conf[o]);
#pragma unroll
      for (int j = 0; j < 4; ++j) rank += (v[j] > c) || (v[j] == c && o + j < s);
    }
  }
  __syncthreads();
  const int n_sel = p.rule == 0 ? (n_above > 0 ? n_above : (n_open > 0 ? 1 : 0)) : min(p.k, n_open);
  int32_t* sel = p.selected + (size_t)b * p.S;
  if (op && rank < n_sel) sel[rank] = s;
  if (s >= n_sel && s < p.S) sel[s] = -1;
  if (s == 0) p.n_selected[b] = n_sel;
}

hipError_t launch_select_slots(const SelectParams& p, hipStream_t stream) {
  hipLaunchKernelGGL(select_slots_kernel, dim3(p.B), dim3((p.S + 63) / 64 * 64), 0, stream, p);
  return hipGetLastError();
}

}  // namespace zarya
