// Slot-parallel attention against a reused prefix KV cache (gfx950).
//
// What is computed (Zarya, Sec. 5.1 KV-reuse argument and Sec. 5.2 draft /
// verification phases): every draft token t = s*L + r of query head h attends
// to all P prefix keys of KV head g = h / G and to a contiguous range of the
// draft tokens' own keys -- its own slot (all of it in the DIFFUSION pass, up
// to itself in the AR_INFILL pass), preceded by every earlier slot when
// cross_slot = CAUSAL.
//
// bf16 kernel design (one workgroup = 4 or 8 waves = up to 128 or 256 query
// rows of one GQA group, i.e. G heads x T tokens flattened token-major, so a
// block holds every head of a contiguous token range; one split of the
// prefix keys):
//  * K/V tiles of 64 keys are staged in LDS once and shared by every query
//    row of the group (the prefix is read from HBM once per group and split).
//  * Scores are computed transposed, S^T = K Q^T, with v_mfma_f32_32x32x16_bf16:
//    each lane then owns one query row, so the online-softmax row statistics
//    need a single cross-lane exchange (lane ^ 32) per tile.
//  * O^T += V^T P^T reuses the score accumulators directly as the B operand
//    (the MFMA k-order is chosen to match the accumulator layout); V^T is read
//    from the row-major LDS tile with ds_read_b64_tr_b16.
//  * LDS rows are XOR-swizzled in 16-byte chunks so that both the row reads of
//    K and the transposing reads of V are free of bank conflicts.
//  * The prefix is split into `n_split` ranges handled by separate workgroups
//    (split-K, flash-decoding style); each writes a float32 partial (O, LSE)
//    and a merge kernel combines them exactly.  With one split the kernel
//    writes the final bf16 output itself.  The draft tokens' own keys are
//    processed by the last split, with the mask applied per element.
#include <algorithm>
#include <type_traits>
#include <utility>

#include "common.hpp"
#include "kernels.hpp"

namespace zarya {

#ifndef ZARYA_ATTN_WPE
#define ZARYA_ATTN_WPE 2  // waves per SIMD the register budget is sized for
#endif

namespace {

// f(std::integral_constant<int, 0>{}) ... f(std::integral_constant<int, N - 1>{})
template <class F, int... I>
__device__ __forceinline__ void static_for(std::integer_sequence<int, I...>, F&& f) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for(std::make_integer_sequence<int, N>{}, f);
}

constexpr int KT = 64;          // keys per tile
constexpr float kRescaleLog2 = 8.f;  // growth of a row maximum (log2 units) that forces a rescale

// XOR swizzle of the 16-byte chunk index of LDS row `kr` (D = 128: 16 chunks
// per row; D = 64: 8).  Any 16 consecutive rows (the rows one pass of a
// K-fragment ds_read_b128 serves) get distinct bank groups, and the aligned
// chunk pairs of 4 consecutive rows (one transposing V read) stay aligned
// pairs on distinct banks: the pair index takes the low row bits, the chunk's
// low bit the next one.
template <int D>
__host__ __device__ constexpr int swz(int kr) {
  if constexpr (D == 128) {
    return ((kr & 7) << 1) | ((kr >> 3) & 1);
  } else {
    return (((kr >> 1) & 3) << 1) | ((kr >> 3) & 1);
  }
}

}  // namespace

// NWAVE: waves per workgroup, 32 query rows each; every wave stages its share
// of each K/V tile, one tile ahead (two LDS buffers of 32 KB at D = 128, which
// leaves room for two workgroups per CU).  At D = 64 four waves of a SIMD fit if
// the kernel keeps to 128 registers, which short prefixes of many sequences need
// (71 x 8 groups of 153 rows, 470 keys: 43.4 us, and 54.6 with the 154 registers
// and three waves that the compiler takes when it is left to).
template <int D, int NWAVE>
__global__ __launch_bounds__(NWAVE * 64) __attribute__((amdgpu_waves_per_eu(D == 64 ? 4 : ZARYA_ATTN_WPE))) void slot_attn_bf16_kernel(
    AttnParams p) {
  constexpr int RB = NWAVE * 32;        // query rows per workgroup
  constexpr int ROWB = D * 2;           // bytes per key row
  constexpr int TILEB = KT * ROWB;      // bytes of one K (or V) tile
  constexpr int CPW = TILEB / 1024 / NWAVE;  // 1 KB direct loads per wave per tile (K; same for V)
  constexpr int LPR = ROWB / 16;        // lanes per row in a direct load
  constexpr int RPC = 1024 / ROWB;      // rows per 1 KB chunk
  constexpr int NDB = D / 32;           // 32-wide blocks of the head dim
  constexpr int NKS = D / 16;           // k-steps of the QK^T contraction
  static_assert(CPW * NWAVE * 1024 == TILEB, "tile must split into 1 KB chunks per wave");
  __shared__ __attribute__((aligned(16))) uint8_t lds[2][2][TILEB];

  int rb, split, bg;  // row block, prefix split, b * Hkv + g
  if (p.heavy_first) {
    // Causal launch whose XCDs each hold whole GQA groups (one split): an
    // XCD walks its groups' row blocks heaviest first (the last tokens see
    // the most keys), so the longest work items start first and the short
    // ones fill the tail.
    const int x = blockIdx.x & 7, k = blockIdx.x >> 3;
    const int gpx = p.per_xcd / p.n_rb;  // groups per XCD
    rb = p.n_rb - 1 - k / gpx;
    split = 0;
    bg = x * gpx + k % gpx;
  } else {
    const int w = xcd_work_index(blockIdx.x, p.per_xcd, p.n_items);
    if (w < 0) return;
    rb = w % p.n_rb;
    split = (w / p.n_rb) % p.n_split;
    bg = w / (p.n_rb * p.n_split);
  }
  const int b = bg / p.Hkv;
  // this batch row's prefix length (rows differ after KV-cache appends)
  const int Pb = p.prefix_lens ? min(max(p.prefix_lens[b], 0), p.P) : p.P;

  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int wave_u = __builtin_amdgcn_readfirstlane(wave);
  const int n = lane & 31, hh = lane >> 5;

  // ---- this lane's query row and its visible range [vis_lo, vis_hi) of
  // draft-token keys.  A group's G*T rows are taken token-major (row = t*G +
  // h), so a block's rows cover a contiguous token range of every head of
  // the group and share one visible key range; mrow is the row's place in
  // the head-major [G, T] layout of q and out.
  const int row = rb * RB + wave * 32 + n;
  const bool row_ok = row < p.R;
  const int mrow = (row % p.G) * p.T + row / p.G;
  int vis_lo = 0, vis_hi = 0;
  if (row_ok) {
    const int t = row / p.G;
    const int s = t / p.L, r = t - s * p.L;
    const int pass = p.slot_pass ? (int)p.slot_pass[b * p.S + s] : p.pass;
    const int own_lo = s * p.L;
    vis_hi = own_lo + (pass == 0 ? p.L : r + 1);
    vis_lo = p.cross ? 0 : own_lo;
  }

  // ---- key tiles of this workgroup: a range of prefix tiles, then (last
  // split only) the draft-token tiles covering every row's visible range.
  const int pre_begin = split * p.tiles_per_split;
  const int pre_end = min((Pb + KT - 1) / KT, pre_begin + p.tiles_per_split);
  const int n_pre = max(0, pre_end - pre_begin);
  int slot_lo = 0, n_slot = 0;
  if (split == p.n_split - 1) {
    const int t0 = rb * RB / p.G;                   // tokens of this block's rows
    const int t1 = (min(p.R, rb * RB + RB) - 1) / p.G;
    const int lo = p.cross ? 0 : (t0 / p.L) * p.L;
    const int hi = min(p.T, (t1 / p.L + 1) * p.L);
    slot_lo = (lo / KT) * KT;
    n_slot = (hi - slot_lo + KT - 1) / KT;
  }
  const int nt = n_pre + n_slot;

  // ---- Q fragments (B operand of S^T = K Q^T), kept in registers; loaded
  // and waited for before the direct-load pipeline starts so that the
  // pipeline's counted waits see only its own loads
  bf16x8 qf[NKS];
  {
    const uint4* qrow = reinterpret_cast<const uint4*>(p.q + ((size_t)bg * p.R + (row_ok ? mrow : 0)) * D);
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
      uint4 v = row_ok ? qrow[2 * ks + hh] : make_uint4(0, 0, 0, 0);
      qf[ks] = __builtin_bit_cast(bf16x8, v);
    }
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) lds_tie(qf[ks]);
    wait_vmcnt<0>();
  }

  // ---- direct-to-LDS staging of K and V tiles: load j of a wave fills 1 KB
  // chunk c = NWAVE*j + wave (RPC rows); lane l lands at row RPC*c + l/LPR,
  // physical 16-byte column l%LPR and fetches the logical column the swizzle
  // puts there.  Rows past the valid keys are clamped to the last valid row
  // (their scores are masked, so they contribute exact zeros).
  int my_r[CPW];
  uint32_t my_off[CPW];
#pragma unroll
  for (int j = 0; j < CPW; ++j) {
    my_r[j] = RPC * (NWAVE * j + wave_u) + lane / LPR;
    my_off[j] = (uint32_t)(my_r[j] * ROWB + (((lane % LPR) ^ swz<D>(my_r[j])) << 4));
  }
  const char* kc = reinterpret_cast<const char*>(p.k_cache + (size_t)bg * p.C * D);
  const char* vc = reinterpret_cast<const char*>(p.v_cache + (size_t)bg * p.C * D);
  const char* ks_ = reinterpret_cast<const char*>(p.k_slot + (size_t)bg * p.T * D);
  const char* vs_ = reinterpret_cast<const char*>(p.v_slot + (size_t)bg * p.T * D);
  auto issue = [&](int i, int buf) __attribute__((always_inline)) {
    const char *kp, *vp;
    int key0, valid;
    if (i < n_pre) {
      key0 = (pre_begin + i) * KT;
      kp = kc;
      vp = vc;
      valid = Pb - key0;
    } else {
      key0 = slot_lo + (i - n_pre) * KT;
      kp = ks_;
      vp = vs_;
      valid = p.T - key0;
    }
    kp += (size_t)key0 * ROWB;
    vp += (size_t)key0 * ROWB;
    uint8_t* kd = &lds[buf][0][wave_u * 1024];
    uint8_t* vd = &lds[buf][1][wave_u * 1024];
    if (valid >= KT) {
#pragma unroll
      for (int j = 0; j < CPW; ++j) {
        dma16(kp + my_off[j], kd + NWAVE * j * 1024);
        dma16(vp + my_off[j], vd + NWAVE * j * 1024);
      }
    } else {
#pragma unroll
      for (int j = 0; j < CPW; ++j) {
        const int dr = min(my_r[j], valid - 1) - my_r[j];  // <= 0: clamp to the last valid row
        dma16(kp + my_off[j] + dr * ROWB, kd + NWAVE * j * 1024);
        dma16(vp + my_off[j] + dr * ROWB, vd + NWAVE * j * 1024);
      }
    }
  };

  f32x16 oacc[NDB];
#pragma unroll
  for (int db = 0; db < NDB; ++db) oacc[db] = f32x16{};
  float m_run = kNegBig, l_run = 0.f;  // running max of raw scores; sum of 2^(scaled score - scaled max)
  const float c2 = p.scale_log2;

  // lane-dependent parts of the LDS fragment addresses (the swizzle of every
  // row a lane reads depends on the lane only)
  const uint32_t lds0 = lds_addr(&lds[0][0][0]);
  // K fragment of k-step ks: row n, logical chunk 2*ks + hh, i.e. physical
  // chunk (2*ks) ^ (hh ^ swz(n)) (2*ks is even, hh the low bit)
  const uint32_t k_row = lds0 + n * ROWB;
  const uint32_t k_cx = (uint32_t)((hh ^ swz<D>(n)) << 4);
  uint32_t k_addr[NKS];
#pragma unroll
  for (int ks = 0; ks < NKS; ++ks) k_addr[ks] = k_row + (k_cx ^ ((uint32_t)ks << 5));
  const int q16 = lane >> 4, rr = lane & 15;
  const int vrow = 4 * hh + (rr >> 2);  // first key row of this lane's transposing reads (+16*st, +8)
  // Rows vrow + 16 * step and vrow + 8 + 16 * step: the swizzle repeats every
  // 16 rows and, for vrow < 8, swz(vrow + 8) = swz(vrow) ^ 1, which flips bit
  // 4 of the address (the chunk's low bit): the second half of a step is read
  // at (v_col ^ 16) + 8 rows.
  uint32_t v_addr[NDB][2];  // first and second half-step
#pragma unroll
  for (int db = 0; db < NDB; ++db) {
    const int d = db * 32 + (q16 & 1) * 16 + 4 * (rr & 3);
    const uint32_t v_col = vrow * ROWB + (((d >> 3) ^ swz<D>(vrow)) << 4) + (d & 7) * 2;
    v_addr[db][0] = lds0 + TILEB + v_col;
    v_addr[db][1] = lds0 + TILEB + (v_col ^ 16u) + 8 * ROWB;
  }
  static_assert((swz<D>(8) ^ swz<D>(0)) == 1, "second V half-step addressing assumes swz(r + 8) = swz(r) ^ 1");

  f32x16 sacc[2];   // scores of the tile between its QK^T and its softmax
  bf16x8 pb[4];      // its probabilities (bf16, B operands of the PV steps)
  v4i16 vf[2][NDB][2];  // V^T fragments, double-buffered across PV steps

  // ---- S^T = K Q^T of tile i for two 32-key blocks; register v of block kb
  // holds key kb*32 + 8*(v/4) + 4*hh + v%4 of the tile.  K fragments are read
  // one k-step ahead of their MFMAs (deeper read-ahead measured no faster).
  auto qk = [&](auto buf) __attribute__((always_inline)) {
    constexpr int KB = decltype(buf)::value * 2 * TILEB;
    sacc[0] = f32x16{};
    sacc[1] = f32x16{};
    bf16x8 kf[2][2];
    kf[0][0] = lds_read_b128<KB>(k_addr[0]);
    kf[0][1] = lds_read_b128<KB + 32 * ROWB>(k_addr[0]);
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
      const int sl = ks & 1;
      if (ks + 1 < NKS) {
        kf[sl ^ 1][0] = lds_read_b128<KB>(k_addr[ks + 1]);
        kf[sl ^ 1][1] = lds_read_b128<KB + 32 * ROWB>(k_addr[ks + 1]);
        lds_wait<2>();
      } else {
        lds_wait<0>();
      }
      lds_tie(kf[sl][0]);
      lds_tie(kf[sl][1]);
      sacc[0] = mfma32x32x16(kf[sl][0], qf[ks], sacc[0]);
      sacc[1] = mfma32x32x16(kf[sl][1], qf[ks], sacc[1]);
    }
  };

  // ---- V^T fragments of PV step `stp` of a tile
  auto pv_read = [&](auto buf, auto stp) __attribute__((always_inline)) {
    constexpr int OFF = decltype(buf)::value * 2 * TILEB + 16 * decltype(stp)::value * ROWB;
#pragma unroll
    for (int db = 0; db < NDB; ++db) {
      vf[decltype(stp)::value & 1][db][0] = lds_read_tr16_b64<OFF>(v_addr[db][0]);
      vf[decltype(stp)::value & 1][db][1] = lds_read_tr16_b64<OFF>(v_addr[db][1]);
    }
  };

  // ---- online softmax of tile i's scores; masks only on tiles that need them
  auto softmax = [&](int i) __attribute__((always_inline)) {
    const bool is_slot = i >= n_pre;
    const int key0 = is_slot ? slot_lo + (i - n_pre) * KT : (pre_begin + i) * KT;
    const bool full = !is_slot && key0 + KT <= Pb;
    const int lim_lo = is_slot ? vis_lo : key0;
    const int lim_n = is_slot ? vis_hi - vis_lo : Pb - key0;
    if (!full) {
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int key = key0 + kb * 32 + 8 * (v >> 2) + 4 * hh + (v & 3);
          if ((unsigned)(key - lim_lo) >= (unsigned)lim_n) sacc[kb][v] = -INFINITY;
        }
    }
    // tile maximum of this lane's row: a max3 tree (depth 3 instead of a
    // 16-long chain), then the other lane half of the row
    float mt;
    {
      float t[11];
#pragma unroll
      for (int j = 0; j < 5; ++j) t[j] = max3f(sacc[0][3 * j], sacc[0][3 * j + 1], sacc[0][3 * j + 2]);
      t[5] = max3f(sacc[0][15], sacc[1][0], sacc[1][1]);
#pragma unroll
      for (int j = 0; j < 4; ++j) t[6 + j] = max3f(sacc[1][3 * j + 2], sacc[1][3 * j + 3], sacc[1][3 * j + 4]);
      t[10] = max3f(sacc[1][14], sacc[1][15], sacc[1][15]);
      const float u0 = max3f(t[0], t[1], t[2]), u1 = max3f(t[3], t[4], t[5]);
      const float u2 = max3f(t[6], t[7], t[8]), u3 = max3f(t[9], t[10], t[10]);
      mt = max_xor32(max3f(max3f(u0, u1, u2), u3, u3));
    }
    const float m_new = fmaxf(m_run, mt);
    // Rescale only when the maximum of some row moved by more than 2^8 in
    // probability: until then the exponentials below are taken against the
    // stale maximum and stay <= 2^8 (exact in the float32 sums, same relative
    // rounding in bf16), and the final O / l and LSE do not depend on which
    // maximum was used.  Random scores raise a row's maximum on most early
    // tiles, each time by little; this skips those rescales.  Every PV of the
    // earlier tiles is in oacc before this (the callers keep that order).
    if (__any((m_new - m_run) * c2 > kRescaleLog2)) {
      const float alpha = fast_exp2((m_run - m_new) * c2);
      l_run *= alpha;
#pragma unroll
      for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int v = 0; v < 16; ++v) oacc[db][v] *= alpha;
      m_run = m_new;
    }
    const float mc = m_run * c2;
    float ps[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int half = 0; half < 2; ++half) {
        uint32_t pk[4];
#pragma unroll
        for (int j = 0; j < 8; j += 2) {
          const int v = half * 8 + j;
          const float e0 = fast_exp2(fmaf(sacc[kb][v], c2, -mc));
          const float e1 = fast_exp2(fmaf(sacc[kb][v + 1], c2, -mc));
          ps[j >> 1] += e0 + e1;
          pk[j >> 1] = pack_bf16x2_hw(e0, e1);
        }
        // B operand of PV step 2*kb + half: slot j = accumulator register 8*half + j
        pb[2 * kb + half] = __builtin_bit_cast(bf16x8, make_uint4(pk[0], pk[1], pk[2], pk[3]));
      }
    l_run += (ps[0] + ps[1]) + (ps[2] + ps[3]);
  };

  // ---- O^T += V^T P^T of tile i (after pv_read of step 0).  Step st covers
  // keys 16*st + 4*hh + {0..3} (slots 0-3) and 16*st + 8 + 4*hh + {0..3} (slots
  // 4-7); V^T fragments are read one step ahead with the transposing LDS read.
  auto pv = [&](auto buf) __attribute__((always_inline)) {
    static_for<4>([&](auto stp) __attribute__((always_inline)) {
      constexpr int st = decltype(stp)::value;
      if constexpr (st + 1 < 4) {
        pv_read(buf, std::integral_constant<int, st + 1>{});
        lds_wait<2 * NDB>();
      } else {
        lds_wait<0>();
      }
#pragma unroll
      for (int db = 0; db < NDB; ++db) {
        v4i16(&f)[2] = vf[st & 1][db];
        lds_tie(f[0]);
        lds_tie(f[1]);
        const uint2 l2 = __builtin_bit_cast(uint2, f[0]);
        const uint2 h2 = __builtin_bit_cast(uint2, f[1]);
        const bf16x8 a = __builtin_bit_cast(bf16x8, make_uint4(l2.x, l2.y, h2.x, h2.y));
        oacc[db] = mfma32x32x16(a, pb[st], oacc[db]);
      }
    });
  };

  // The LDS buffer of a tile is a compile-time constant of its half of the
  // loop, so that every fragment address is a register set up once plus an
  // immediate offset (the 40 additions per tile it saves are a tenth of the
  // vector instructions beside the MFMAs, and the two hardly overlap: the 4B
  // shape 308 -> 294 us, the training layout 672 -> 651, 1.7B 118 -> 115.5; at
  // 0.6B, 42.1 us, no difference).
  // a wave of padding rows only helps to load the tiles (520 rows a group in
  // blocks of 128, Mode A: the step 211 -> 207 us)
  const bool live = rb * RB + wave_u * 32 < p.R;
  auto step = [&](int i, auto buf) __attribute__((always_inline)) {
    wait_vmcnt<0>();
    block_barrier();
    if (i + 1 < nt) issue(i + 1, decltype(buf)::value ^ 1);
    if (!live) return;
    qk(buf);
    pv_read(buf, std::integral_constant<int, 0>{});  // in flight during the softmax
    softmax(i);
    pv(buf);
  };
  if (nt > 0) issue(0, 0);
  for (int i = 0; i < nt; i += 2) {
    step(i, std::integral_constant<int, 0>{});
    if (i + 1 < nt) step(i + 1, std::integral_constant<int, 1>{});
  }

  // ---- finalize: combine the two lane halves' partial sums
  const float l_tot = sum_xor32(l_run);
  if (!row_ok) return;
  int orow_in = mrow;
  if constexpr (D == 64) {
    // worked out anew, from a thread index that the compiler does not know to be
    // the same, instead of kept in a register through the loop
    int te = tid;
    asm volatile("" : "+v"(te));
    const int row_e = rb * RB + (te >> 6) * 32 + (te & 31);
    orow_in = (row_e % p.G) * p.T + row_e / p.G;
  }
  const size_t grow = (size_t)bg * p.R + orow_in;  // row of the [B*Hq*T] output
  const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
  const float lse2 = m_run * c2 + __log2f(l_tot);  // log2 units
  if (p.n_split == 1) {
    uint16_t* orow = p.out + grow * D;
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int d = db * 32 + 8 * u + 4 * hh;
        uint2 pk;
        pk.x = pack_bf16x2_hw(oacc[db][4 * u] * inv, oacc[db][4 * u + 1] * inv);
        pk.y = pack_bf16x2_hw(oacc[db][4 * u + 2] * inv, oacc[db][4 * u + 3] * inv);
        *reinterpret_cast<uint2*>(orow + d) = pk;
      }
    if (p.lse && hh == 0) p.lse[grow] = lse2 * kLn2;
  } else {
    float* orow = p.part_o + ((size_t)split * p.rows_total + grow) * D;
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int d = db * 32 + 8 * u + 4 * hh;
        float4 o4 = make_float4(oacc[db][4 * u] * inv, oacc[db][4 * u + 1] * inv, oacc[db][4 * u + 2] * inv,
                                oacc[db][4 * u + 3] * inv);
        *reinterpret_cast<float4*>(orow + d) = o4;
      }
    if (hh == 0) p.part_lse[(size_t)split * p.rows_total + grow] = l_tot > 0.f ? lse2 : -INFINITY;
  }
}

// Exact merge of the prefix splits: O = sum_i w_i O_i / sum_i w_i with
// w_i = 2^(lse_i - max_j lse_j); lse = max + log2(sum w) (natural log on output).
// A lane merges 4 consecutive elements of one row (D/4 lanes per row).  With
// SW = 1 a wave takes all the splits of its rows (up to 8); with SW = 4 the
// four waves of a workgroup share the rows, take a quarter of the splits each
// (up to 16) and meet in LDS, so that every load of a row is in flight at once
// whatever the number of splits (8 heads x 128 rows over 32768 keys, with the
// attention: 64 splits 72.6 -> 45.2 us, 32 splits 46.4 -> 37.3; a wave that walks
// past its first eight waits for each further one).
template <int D, int SW>
__global__ __launch_bounds__(256) void slot_attn_merge_kernel(const float* __restrict__ part_o,
                                                              const float* __restrict__ part_lse, int n_split,
                                                              int rows_total, int row0, uint16_t* __restrict__ out,
                                                              float* __restrict__ lse) {
  constexpr int LPR = D / 4, RPW = 64 / LPR;
  constexpr int MAXS = SW == 1 ? 8 : 16;  // splits of a wave, all loaded before any arithmetic
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int row_in = row0 + (SW == 1 ? blockIdx.x * 4 + wave : blockIdx.x) * RPW + lane / LPR;
  const int row = min(row_in, rows_total - 1);  // lanes past the end follow the last row and store nothing
  const int c = (lane % LPR) * 4;
  const int per = SW == 1 ? n_split : (n_split + SW - 1) / SW;
  const int s0 = SW == 1 ? 0 : wave * per;
  const int ns = max(0, min(n_split - s0, per));
  float l[MAXS];
  float4 o[MAXS];
#pragma unroll
  for (int i = 0; i < MAXS; ++i) {
    if (i < ns) {
      l[i] = part_lse[(size_t)(s0 + i) * rows_total + row];
      o[i] = *reinterpret_cast<const float4*>(part_o + ((size_t)(s0 + i) * rows_total + row) * D + c);
    }
  }
  float mx = -INFINITY;
#pragma unroll
  for (int i = 0; i < MAXS; ++i)
    if (i < ns) mx = fmaxf(mx, l[i]);
  float acc[4] = {0.f, 0.f, 0.f, 0.f};
  float wsum = 0.f;
#pragma unroll
  for (int i = 0; i < MAXS; ++i) {
    if (i < ns) {
      const float wi = l[i] == -INFINITY ? 0.f : fast_exp2(l[i] - mx);
      wsum += wi;
      acc[0] += wi * o[i].x;
      acc[1] += wi * o[i].y;
      acc[2] += wi * o[i].z;
      acc[3] += wi * o[i].w;
    }
  }
  if constexpr (SW > 1) {
    __shared__ float xm[SW][64], xw[SW][64], xa[SW][4][64];
    xm[wave][lane] = mx;
    xw[wave][lane] = wsum;
#pragma unroll
    for (int e = 0; e < 4; ++e) xa[wave][e][lane] = acc[e];
    __syncthreads();
    if (wave != 0) return;
#pragma unroll
    for (int i = 1; i < SW; ++i) mx = fmaxf(mx, xm[i][lane]);
    wsum = 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[e] = 0.f;
#pragma unroll
    for (int i = 0; i < SW; ++i) {
      const float wi = xm[i][lane] == -INFINITY ? 0.f : fast_exp2(xm[i][lane] - mx);
      wsum += wi * xw[i][lane];
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[e] += wi * xa[i][e][lane];
    }
  }
  if (row_in >= rows_total) return;
  const float inv = 1.f / wsum;
  *reinterpret_cast<uint2*>(out + (size_t)row * D + c) =
      make_uint2(pack_bf16x2_hw(acc[0] * inv, acc[1] * inv), pack_bf16x2_hw(acc[2] * inv, acc[3] * inv));
  if (lse && c == 0) lse[row] = (mx + __log2f(wsum)) * kLn2;
}

// float32 path.  One workgroup = NW waves = 16 * NR query rows of one GQA group
// (token-major, as above); the waves share the rows and split the keys: wave w
// takes the 16-key tiles w, w + NW, ... of the prefix and the draft tokens and
// keeps its own online softmax; the partials meet in LDS and are merged
// in wave order, so no workspace and no second launch is needed.
//
// The products are v_mfma_f32_16x16x4_f32 (float32 operands and accumulators).
// S^T = K Q^T leaves a lane the scores of one query row and four keys, which
// are the B operands of O^T += V^T P^T as they stand.  The order of the
// contraction and of the output rows is free, so K, Q and V are read straight
// from global memory in 16-byte pieces, one per four MFMAs; nothing is staged:
// the rows of a workgroup share each key through its waves' registers, and a
// group's workgroups meet in one XCD's L2.
//
// Bound by the float32 matrix rate of the compute units that have rows, and
// the chain of a wave's tiles.  DS = 2: two workgroups take a row block, each
// the whole scores and half of the output row (no exchange between them), for
// launches that would leave half of the units idle.  B = 2, 16/8 heads, D = 128,
// 1000 + 64 keys, 64 tokens (128 row blocks) takes 25.5 us, 42 TFLOP/s, and 32.7
// with one workgroup a block; one key at a time with a shuffled dot product per
// row, as it was at first, took 771 us.  Keys and values requested a whole tile
// ahead (182 registers) took 26.7.
//
// NW = 1: a workgroup of one wave walks all the tiles of its rows, for launches
// of so many row blocks that the waves fill the units without splitting keys, or
// of so few keys that there is nothing to split: eight waves would pay a
// workgroup's barriers and LDS, one or two workgroups a unit, for a tile each.
// 4096 groups, D = 128: 1 row x 1 key 112 us with eight waves, 18 with one; 4 rows
// x 68 keys 165 and 70; 4 rows x 516 keys 529 and 387.
template <int D, int NR, int DS, int NW>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(2))) void slot_attn_f32_kernel(AttnParams32 p) {
  constexpr int RB = 16 * NR;   // query rows per workgroup
  constexpr int NKS = D / 16;   // 16-byte pieces of a K row per lane
  constexpr int DO = D / DS;    // elements of the output row taken by this workgroup
  constexpr int NC = DO / 64;   // 16-byte pieces of a V row per lane
  constexpr int NOB = DO / 16;  // 16-wide blocks of the output: block 4 * c + e holds d = 64 * c + 4 * i + e
  constexpr int OSTR = DO + 4;  // row stride of the partial outputs in LDS
  constexpr int QSTR = D + 4;   // and of the queries
  __shared__ __attribute__((aligned(16))) float part_o[NW][RB][OSTR];
  __shared__ __attribute__((aligned(16))) float qs[RB][QSTR];  // scaled queries; the padding spreads the rows over the banks
  __shared__ float part_m[NW][RB], part_l[NW][RB];

  const int n_rb = (p.G * p.T + RB - 1) / RB;
  const int w = xcd_work_index(blockIdx.x, gridDim.x >> 3, min(p.B * p.Hkv * n_rb * DS - p.item0, kAttnMaxGrid)) + p.item0;
  if (w < p.item0) return;
  const int d0 = (w % DS) * DO;  // first element taken
  const int rb = w / DS % n_rb, bg = w / (DS * n_rb);
  const int b = bg / p.Hkv;
  const int R = p.G * p.T;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n = lane & 15, q4 = lane >> 4;
  const int Pb = p.prefix_lens ? min(max(p.prefix_lens[b], 0), p.P) : p.P;

  // this lane's query rows (one per row tile) and their visible draft keys;
  // rows past the end follow the last one and are not stored
  int vis_lo[NR], vis_hi[NR];
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    const int row = min(rb * RB + 16 * r + n, R - 1);
    const int t = row / p.G, s = t / p.L;
    const int pass = p.slot_pass ? (int)p.slot_pass[b * p.S + s] : p.pass;
    vis_hi[r] = pass == 0 ? (s + 1) * p.L : t + 1;
    vis_lo[r] = p.cross ? 0 : s * p.L;
  }
  for (int x = threadIdx.x; x < RB * (D / 4); x += NW * 64) {
    const int lr = x / (D / 4), c = 4 * (x % (D / 4));
    const int row = min(rb * RB + lr, R - 1);
    const size_t qr = (size_t)bg * R + (size_t)(row % p.G) * p.T + row / p.G;
    *reinterpret_cast<f32x4*>(&qs[lr][c]) = load_f32x4(p.q + qr * D + c) * p.scale;
  }
  __syncthreads();
  const uint32_t q_addr = lds_addr(&qs[n][4 * q4]);

  // key tiles: the prefix's, then those covering the block's draft keys
  const int n_pre = (Pb + 15) / 16;
  const int t0 = rb * RB / p.G, t1 = (min(R, rb * RB + RB) - 1) / p.G;
  const int slot_lo = (p.cross ? 0 : (t0 / p.L) * p.L) & ~15;
  const int nt = n_pre + (min(p.T, (t1 / p.L + 1) * p.L) - slot_lo + 15) / 16;
  const float* kc = p.k_cache + (size_t)bg * p.C * D;
  const float* vc = p.v_cache + (size_t)bg * p.C * D + d0;
  const float* ks_ = p.k_slot + (size_t)bg * p.T * D;
  const float* vs_ = p.v_slot + (size_t)bg * p.T * D + d0;

  f32x4 oacc[NR][NOB];
  float m[NR], l[NR];
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    m[r] = -INFINITY;
    l[r] = 0.f;
#pragma unroll
    for (int ob = 0; ob < NOB; ++ob) oacc[r][ob] = f32x4{0.f, 0.f, 0.f, 0.f};
  }

  f32x4 kf[NKS];
  // K row n of tile i, clamped to the last valid key (its score is masked)
  auto load_k = [&](int i) {
    const bool pre = i < n_pre;
    const int key0 = pre ? 16 * i : slot_lo + 16 * (i - n_pre);
    const float* src = (pre ? kc : ks_) + (size_t)min(key0 + n, (pre ? Pb : p.T) - 1) * D + 4 * q4;
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) kf[ks] = load_f32x4(src + 16 * ks);
  };

  if (wave < nt) load_k(wave);
  for (int i = wave; i < nt; i += NW) {
    const bool pre = i < n_pre;
    const int key0 = pre ? 16 * i : slot_lo + 16 * (i - n_pre);
    const int last = (pre ? Pb : p.T) - 1;
    const float* vsrc = pre ? vc : vs_;
    f32x4 vf[4][NC];  // V rows 4 * q4 + v, elements 64 * c + 4 * n + e
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
      for (int c = 0; c < NC; ++c)
        vf[v][c] = load_f32x4(vsrc + (size_t)min(key0 + 4 * q4 + v, last) * D + 64 * c + 4 * n);

    f32x4 s[NR];  // scores of keys 4 * q4 + v
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      f32x4 s0{0.f, 0.f, 0.f, 0.f}, s1{0.f, 0.f, 0.f, 0.f};  // two chains
      // query fragments come from LDS for each tile (in registers they would
      // not leave room for the output and the key and value pieces in flight)
      bf16x8 qf[NKS];
      const uint32_t qa = q_addr + r * 16 * QSTR * 4;
      qf[0] = lds_read_b128<0>(qa);
      qf[1] = lds_read_b128<64>(qa);
      qf[2] = lds_read_b128<128>(qa);
      qf[3] = lds_read_b128<192>(qa);
      if constexpr (NKS == 8) {
        qf[4] = lds_read_b128<256>(qa);
        qf[5] = lds_read_b128<320>(qa);
        qf[6] = lds_read_b128<384>(qa);
        qf[7] = lds_read_b128<448>(qa);
      }
      lds_wait<0>();
#pragma unroll
      for (int ks = 0; ks < NKS; ++ks) lds_tie(qf[ks]);
#pragma unroll
      for (int ks = 0; ks < NKS; ks += 2) {
        const f32x4 qa4 = __builtin_bit_cast(f32x4, qf[ks]), qb4 = __builtin_bit_cast(f32x4, qf[ks + 1]);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          s0 = mfma16x16x4_f32(kf[ks][e], qa4[e], s0);
          s1 = mfma16x16x4_f32(kf[ks + 1][e], qb4[e], s1);
        }
      }
      s[r] = s0 + s1;
    }
    // the next tile's keys take the registers of this one's and arrive during
    // the softmax and the PV products
    __builtin_amdgcn_sched_barrier(0);
    if (i + NW < nt) load_k(i + NW);
    __builtin_amdgcn_sched_barrier(0);
    const bool masked = !pre || key0 + 16 > Pb;
    auto visible = [&](int r, int key) { return pre ? key < Pb : key >= vis_lo[r] && key < vis_hi[r]; };
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      if (masked) {
#pragma unroll
        for (int v = 0; v < 4; ++v)
          if (!visible(r, key0 + 4 * q4 + v)) s[r][v] = -INFINITY;
      }
      float mt = max3f(max3f(s[r][0], s[r][1], s[r][2]), s[r][3], s[r][3]);
      mt = fmaxf(mt, __shfl_xor(mt, 16));
      mt = fmaxf(mt, __shfl_xor(mt, 32));
      const float m_new = fmaxf(m[r], mt);
      if (__any(m_new > m[r])) {
        const float c = m[r] == -INFINITY ? 0.f : expf(m[r] - m_new);
        l[r] *= c;
#pragma unroll
        for (int ob = 0; ob < NOB; ++ob)
#pragma unroll
          for (int v = 0; v < 4; ++v) oacc[r][ob][v] *= c;
        m[r] = m_new;
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        s[r][v] = s[r][v] == -INFINITY ? 0.f : expf(s[r][v] - m_new);
        l[r] += s[r][v];
      }
    }
    // A value a row does not see must not reach it, and 0 * inf or 0 * NaN
    // would: such tiles (masked, with a value that is not finite) are summed
    // key by key over the visible keys only.
    bool bad = false;
    if (masked) {
#pragma unroll
      for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
          for (int e = 0; e < 4; ++e) bad = bad || !(fabsf(vf[v][c][e]) < INFINITY);
      bad = __any(bad);
    }
    if (!bad) {
#pragma unroll
      for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int r = 0; r < NR; ++r)
#pragma unroll
          for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int e = 0; e < 4; ++e)
              oacc[r][4 * c + e] = mfma16x16x4_f32(vf[v][c][e], s[r][v], oacc[r][4 * c + e]);
    } else {
#pragma unroll
      for (int r = 0; r < NR; ++r)
#pragma unroll 1
        for (int j = 0; j < 16; ++j) {
          const float pj = __shfl(j & 2 ? (j & 1 ? s[r][3] : s[r][2]) : (j & 1 ? s[r][1] : s[r][0]), 16 * (j >> 2) + n);
          if (!visible(r, key0 + j)) continue;
          const float* vrow = vsrc + (size_t)min(key0 + j, last) * D + 16 * q4;
#pragma unroll
          for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
              const f32x4 vv = load_f32x4(vrow + 64 * c + 4 * v);
#pragma unroll
              for (int e = 0; e < 4; ++e) oacc[r][4 * c + e][v] = fmaf(pj, vv[e], oacc[r][4 * c + e][v]);
              __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
  }

  // ---- merge of the waves' partials, in wave order
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    l[r] += __shfl_xor(l[r], 16);
    l[r] += __shfl_xor(l[r], 32);
    const int lr = 16 * r + n;
    if (q4 == 0) {
      part_m[wave][lr] = m[r];
      part_l[wave][lr] = l[r];
    }
    // oacc[4 * c + e][v] is element 64 * c + 16 * q4 + 4 * v + e of the row
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int v = 0; v < 4; ++v)
        *reinterpret_cast<f32x4*>(&part_o[wave][lr][64 * c + 16 * q4 + 4 * v]) =
            f32x4{oacc[r][4 * c][v], oacc[r][4 * c + 1][v], oacc[r][4 * c + 2][v], oacc[r][4 * c + 3][v]};
  }
  __syncthreads();
  for (int x = threadIdx.x; x < RB * (DO / 4); x += NW * 64) {
    const int lr = x / (DO / 4), c = 4 * (x % (DO / 4));
    const int row = rb * RB + lr;
    if (row >= R) break;
    float mx = part_m[0][lr];
#pragma unroll
    for (int i = 1; i < NW; ++i) mx = fmaxf(mx, part_m[i][lr]);
    float lt = 0.f;
    f32x4 o{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < NW; ++i) {
      const float pm = part_m[i][lr], pl = part_l[i][lr];
      if (pm == -INFINITY && pl == 0.f) continue;  // a wave without a visible key of this row
      const float sc = expf(pm - mx);
      lt += sc * pl;
      o += sc * *reinterpret_cast<const f32x4*>(&part_o[i][lr][c]);
    }
    const size_t grow = (size_t)bg * R + (size_t)(row % p.G) * p.T + row / p.G;
    store_f32x4(p.out + grow * D + d0 + c, o / lt);
    if (p.lse && d0 + c == 0) p.lse[grow] = mx + logf(lt);
  }
}

// ------------------------------------------------------------------ launchers

template <int D>
void launch_attn_merge(const AttnParams& p, hipStream_t stream) {
  constexpr int RPW = 64 / (D / 4);  // rows per wave
  if (p.n_split <= 8) {
    slot_attn_merge_kernel<D, 1><<<dim3((p.rows_total + 4 * RPW - 1) / (4 * RPW)), dim3(256), 0, stream>>>(
        p.part_o, p.part_lse, p.n_split, p.rows_total, 0, p.out, p.lse);
  } else {
    for (int64_t row0 = 0; row0 < p.rows_total; row0 += (int64_t)kAttnMaxGrid * RPW) {
      const int blocks = (int)std::min<int64_t>((p.rows_total - row0 + RPW - 1) / RPW, kAttnMaxGrid);
      slot_attn_merge_kernel<D, 4><<<dim3(blocks), dim3(256), 0, stream>>>(p.part_o, p.part_lse, p.n_split,
                                                                           p.rows_total, (int)row0, p.out, p.lse);
    }
  }
}

hipError_t launch_slot_attn_bf16(const AttnParams& p, int head_dim, hipStream_t stream) {
  const int grid = 8 * p.per_xcd;
  const bool wide = p.rows_per_block == kAttnWideRowsPerBlock;
  if (head_dim == 128) {
    if (wide) {
      slot_attn_bf16_kernel<128, 8><<<dim3(grid), dim3(512), 0, stream>>>(p);
    } else {
      slot_attn_bf16_kernel<128, 4><<<dim3(grid), dim3(256), 0, stream>>>(p);
    }
  } else {
    if (wide) {
      slot_attn_bf16_kernel<64, 8><<<dim3(grid), dim3(512), 0, stream>>>(p);
    } else {
      slot_attn_bf16_kernel<64, 4><<<dim3(grid), dim3(256), 0, stream>>>(p);
    }
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || p.n_split == 1) return e;
  if (head_dim == 128) {
    launch_attn_merge<128>(p, stream);
  } else {
    launch_attn_merge<64>(p, stream);
  }
  return hipGetLastError();
}

template <int D, int NR, int DS, int NW = kAttnF32Waves>
void launch_attn_f32_as(AttnParams32 p, int blocks, hipStream_t stream) {
  const int64_t items = (int64_t)DS * blocks;
  for (int64_t i = 0; i < items; i += kAttnMaxGrid) {
    p.item0 = (int)i;
    const int n = (int)std::min<int64_t>(items - i, kAttnMaxGrid);
    slot_attn_f32_kernel<D, NR, DS, NW><<<dim3(8 * ((n + 7) / 8)), dim3(NW * 64), 0, stream>>>(p);
  }
}

template <int NR>
void launch_attn_f32_rows(const AttnParams32& p, int head_dim, int n_rb, hipStream_t stream) {
  const int blocks = p.B * p.Hkv * n_rb;
  if (head_dim == 64) {
    launch_attn_f32_as<64, NR, 1>(p, blocks, stream);
  } else if (NR == 1 && attn_f32_row_parts(head_dim, 16, blocks) == 2) {
    launch_attn_f32_as<128, 1, 2>(p, blocks, stream);
  } else {
    launch_attn_f32_as<128, NR, 1>(p, blocks, stream);
  }
}

hipError_t launch_slot_attn_f32(const AttnParams32& p, int head_dim, hipStream_t stream) {
  const int R = p.G * p.T, rows = attn_f32_rows_per_block(p.B * (int64_t)p.Hkv, R, (int64_t)p.P + p.T);
  if (attn_f32_one_wave(p.B * (int64_t)p.Hkv, R, attn_f32_keys_seen(p.P, p.T, p.L, p.cross))) {
    const int blocks = p.B * p.Hkv * ((R + 15) / 16);
    if (head_dim == 64) {
      launch_attn_f32_as<64, 1, 1, 1>(p, blocks, stream);
    } else {
      launch_attn_f32_as<128, 1, 1, 1>(p, blocks, stream);
    }
  } else if (rows == 32) {
    launch_attn_f32_rows<2>(p, head_dim, (R + 31) / 32, stream);
  } else {
    launch_attn_f32_rows<1>(p, head_dim, (R + 15) / 16, stream);
  }
  return hipGetLastError();
}

}  // namespace zarya
