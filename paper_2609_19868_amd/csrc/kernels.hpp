// Kernel parameter blocks and launchers of libzarya (host <-> device contract).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace zarya {

// bf16 slot attention.  Rows of a GQA group (G heads x T tokens) are
// contiguous in q and out, so a group is addressed as one [R = G*T, D] block.
struct AttnParams {
  const uint16_t* q;        // [B, Hq, T, D]
  const uint16_t* k_cache;  // [B, Hkv, C, D]
  const uint16_t* v_cache;
  const uint16_t* k_slot;  // [B, Hkv, T, D]
  const uint16_t* v_slot;
  const uint8_t* slot_pass;    // [B, S] or null
  const int32_t* prefix_lens;  // [B] or null (then P for every row)
  uint16_t* out;               // [B, Hq, T, D]
  float* lse;                // [B, Hq, T] or null (natural log)
  float* part_o;             // [n_split, rows_total, D]  (n_split > 1)
  float* part_lse;           // [n_split, rows_total]     (n_split > 1, log2 units)
  int B, Hq, Hkv, P, C, S, L, T, G, R;
  int pass, cross;
  float scale_log2;  // softmax scale * log2(e)
  int n_split, n_rb, tiles_per_split, n_prefix_tiles;
  int per_xcd, n_items;
  int rows_total;      // B * Hq * T
  int rows_per_block;  // kAttnRowsPerBlock or kAttnWideRowsPerBlock
  // causal launch, one split, 8 | B*Hkv: every XCD holds B*Hkv/8 whole
  // groups and takes their row blocks heaviest first
  int heavy_first;
};

struct AttnParams32 {
  const float* q;
  const float* k_cache;
  const float* v_cache;
  const float* k_slot;
  const float* v_slot;
  const uint8_t* slot_pass;
  const int32_t* prefix_lens;
  float* out;
  float* lse;
  int B, Hq, Hkv, P, C, S, L, T, G;
  int pass, cross;
  float scale;
  int rows_total;
  int item0;  // first work item of this launch (set by the launcher)
};

// LM-head confidence.  Partials are per (vocab group, row): m = max logit,
// s = sum of exp(logit - m), idx = lowest id at the max.
struct ConfParams {
  const void* hidden;   // [M, H]
  const void* w_vocab;  // [V, H]
  int M, H, V;
  int n_vg;        // vocabulary groups (partials per row)
  int vg_split;    // float32 path: workgroups (and partials) per vocabulary group
  int n_rt;        // row tiles (bf16 path)
  int per_xcd, n_items;
  float* part_m;   // [M, n_vg]
  float* part_s;   // [M, n_vg]
  int* part_idx;   // [M, n_vg]
  // Gumbel-max sampling (null part_g: no sampling).  Per (row, group): best
  // perturbed score z*log2(e)/T - log2(-log2 u) and its id.  The bf16 path
  // does not track the argmax when sampling (part_idx then holds INT_MAX).
  float* part_g;
  int* part_gi;
  float c2t;  // log2(e) / temperature
  uint32_t seed_lo, seed_hi, off_lo, off_hi;
  // Row selection (null: row i of the output is hidden row i): output row i
  // is hidden row row_index[i] of hidden_rows (clamped into range here; the
  // merge marks out-of-range rows).
  const int32_t* row_index;
  int hidden_rows;
  // bf16 path: W is loaded non-temporally (the hidden rows an XCD's work
  // items re-read fit in its L2 beside the W stream; see kConfXResidentBytes)
  int w_stream;
};

// Hidden row of output row r.
__device__ __forceinline__ int conf_hidden_row(const int32_t* row_index, int hidden_rows, int r) {
  return row_index ? min(max(row_index[r], 0), hidden_rows - 1) : r;
}

struct ConfMergeParams {
  const float* part_m;
  const float* part_s;
  const int* part_idx;
  int n_vg, M, H, V;
  int bf16;
  const void* hidden;
  const void* w_vocab;
  const int32_t* target_ids;
  float* max_prob;
  int32_t* argmax_id;
  float* lse;
  float* target_prob;
  const float* part_g;  // sampling partials, or null
  const int* part_gi;
  int32_t* sample_id;
  float* sample_prob;
  const int32_t* row_index;  // as in ConfParams
  int hidden_rows;
};

struct SelectParams {
  int B, S, L;
  const float* token_conf;
  const uint8_t* slot_open;
  int conf_rule, rule;
  float threshold;
  int k;
  float* slot_conf;
  int32_t* selected;
  int32_t* n_selected;
};

struct AcceptParams {
  int B, S, L;
  const float* token_prob;
  const int32_t* selected;
  float threshold;
  int rule;
  uint8_t* accepted;
  int32_t* n_accepted;
  int32_t* n_total;
};

struct AppendParams {
  int B, Hkv, C, S, L, row_bytes;  // row_bytes = head_dim * element size, a multiple of 16
  const void* k_slot;
  const void* v_slot;
  const uint8_t* accepted;
  const int32_t* order;
  int32_t* prefix_lens;
  void* k_cache;
  void* v_cache;
};

// Mode A reveal: one workgroup per batch row sorts the row's N keys in LDS.
struct RevealParams {
  int B, N, NP;  // NP = N rounded up to a power of two (>= 2)
  int rule;      // 0 confidence, 1 leftmost, 2 random
  const float* conf;
  uint8_t* mask;
  const int32_t* k;
  uint32_t seed_lo, seed_hi, off_lo, off_hi;
  const int32_t* sample_id;
  int32_t* tokens;
  int32_t* order;
  int32_t* n_revealed;
};
constexpr int kRevealMaxN = 8192;

// Mode A mask budget on the host: fills counts (if not null) and returns the
// plan length; *n_diff_steps gets the number of diffusion steps.
int64_t mask_budget_plan(int32_t n_masked, int32_t n_steps, double alpha0, uint64_t seed, int32_t* counts,
                         int32_t* n_diff_steps);

// largest S*L the append kernel stages in LDS
constexpr int kAppendMaxTokens = 8192;

constexpr int kAttnKeysPerTile = 64;
constexpr int kAttnF32Waves = 8;            // float32 path: waves per workgroup (or one), which split the keys
// Largest grid of a launch whose workgroups grow with the rows: a grid holds
// fewer than 2^32 threads, so more workgroups than this take several launches.
constexpr int kAttnMaxGrid = 1 << 20;
constexpr int kAttnRowsPerBlock = 128;      // four waves
constexpr int kAttnWideRowsPerBlock = 256;  // eight waves: every K/V tile staged once for 256 rows
constexpr int kAttnTargetWGs = 256;         // workgroups the bf16 planner splits the prefix for: one a compute unit
// float32 path: query rows per workgroup.  32 rows read each key half as often
// as 16; 16 rows make twice as many workgroups, which pays where 32 leave
// compute units idle (16/8 heads x 64 tokens, D = 128, 16 and 32 rows: 2048 keys,
// 64 blocks of 32 rows 47 and 93 us, 128 blocks 61 and 95, 256 blocks 116 and 97;
// 128 keys, 64 blocks 9.0 and 16.3).  Up to 128 keys, one tile a wave, 32 rows are
// taken, which is not the faster side (64 + 64 keys 7.8 and 12.1 us).
constexpr int attn_f32_rows_per_block(int64_t groups, int64_t rows_per_group, int64_t keys) {
  return groups * ((rows_per_group + 31) / 32) < 256 && keys > 16 * kAttnF32Waves ? 16 : 32;
}
// Keys that a block of 16 rows (of at most 16 tokens) sees at most.
constexpr int64_t attn_f32_keys_seen(int64_t prefix, int64_t tokens, int64_t slot_len, int cross) {
  const int64_t own = cross ? tokens : 16 + 2 * slot_len;
  return prefix + (own < tokens ? own : tokens);
}
// Workgroups of one wave and 16 rows instead: 1024 blocks of 16 rows fill the
// units (4 rows x 516 keys, D = 128, eight waves and one: 1024 blocks 137 and
// 100 us, 512 blocks 70 and 65; 128 rows x 576 keys a group, 1024 blocks 69 and
// 69, but 2112 keys 197 and 217: there 32 rows share each key), or fewer with
// one or two key tiles, of which eight waves would leave most without one
// (512 blocks x 16 keys 18.5 and 14.0; 32 blocks 10.3 and 10.8).
constexpr bool attn_f32_one_wave(int64_t groups, int64_t rows_per_group, int64_t keys_seen) {
  const int64_t blocks = groups * ((rows_per_group + 15) / 16);
  return (blocks >= 1024 && keys_seen <= 512) || (blocks >= 512 && keys_seen <= 32);
}
// Workgroups per row block.  With 16 rows and at most half a workgroup per
// compute unit two share a block: each computes all of the scores and half of
// the value products, three quarters of the work on twice the units (D = 128;
// at D = 64 half a row is less than the lanes' 16-byte pieces).  1000 keys, 128
// blocks, shared and not: 26.5 and 33.4 us; 256 blocks, 64 keys 13.3 and 9.5.
constexpr int attn_f32_row_parts(int head_dim, int rows_per_block, int64_t blocks) {
  return head_dim == 128 && rows_per_block == 16 && blocks <= 128 ? 2 : 1;
}
// Tile configuration of the bf16 LM-head reduction (measured on MI355X over
// the 0.6B/1.7B/4B shapes): 8 waves over a 256 x 256 tile, 64-deep stages,
// three W and two hidden LDS buffers (160 KB), one workgroup per compute
// unit.  With few rows (a single sequence's draft tokens, the tokens a
// first-hitting step reveals) most of a 256-row tile would be padding and the
// reduction is bound by the W stream instead: 4 waves over a 256 x 64 tile,
// up to 128 rows (the measured crossover).  The vocabulary is split into
// groups until row tiles x groups reaches kConfTargetWGs (one per CU).
constexpr int kConfNW = 8, kConfBR = 256, kConfBK = 64, kConfNSW = 3, kConfNSX = 2;
constexpr int kConfSmallNW = 4, kConfSmallBR = 64, kConfSmallMaxRows = 128;
constexpr int kConfTargetWGs = 256;
// Partials of one row at most, on either path (the merge holds them all in a wave).
constexpr int kConfMaxGroups = 256;
static_assert(kConfTargetWGs <= kConfMaxGroups, "groups per row");
// Device scratch of zarya_slot_confidence_noalloc: room for the partials of
// every bf16 call up to 65536 rows (row tiles x vocabulary groups <= 256, 12
// bytes per row and group).
constexpr size_t kConfScratchBytes = (size_t)1 << 20;
// Largest hidden-row footprint per XCD (rows of the row tiles among its work
// items x H x 2 bytes) for which W is loaded non-temporally: up to this size
// the hidden tiles, re-read once per vocab tile, stay in the 4 MB L2 instead
// of being evicted by the W stream (measured on MI355X: at 2 MB the LM head's
// L2-miss traffic falls from 1.61x to 1.11x its algorithmic bytes and the
// kernel gains 2-4%; at 3 MB 1.15x and equal time; from 4 MB the hidden rows
// no longer fit either way and non-temporal W costs traffic and 1% of time).
constexpr size_t kConfXResidentBytes = (size_t)3 << 20;
constexpr int conf_tile_rows(int n_rows) { return n_rows <= kConfSmallMaxRows ? kConfSmallBR : kConfBR; }

// float32 path: tiles of 64 rows x 128 vocab ids, or of 32 rows x 256 ids where
// that is all the rows (half of a 64-row tile would be padding: 1 to 32 rows x
// 1024 against 151936 ids 172-187 us, 226-230 with 64-row tiles; 64 rows against
// 32000 ids 88 with 32-row tiles, 78 with 64).
// Ids that a workgroup's share is aimed at: the groups are split to that, rounded
// up, and the 32-id blocks are then divided evenly, so that a share may be as
// little as half of it or a little more.  64 rows x 1024, aims of 64, 128, 256 and
// 512 ids: 32000 ids 54, 79, 114, 191 us (at 128 a share is 133 ids, two tiles),
// 8000 ids 49, 48, 112, 190; with 151936 ids, 594 a share, no difference.
constexpr int kConfF32MinIds = 128;
constexpr int conf_f32_tile_rows(int n_rows) { return n_rows <= 32 ? 32 : 64; }

hipError_t launch_slot_attn_bf16(const AttnParams& p, int head_dim, hipStream_t stream);
hipError_t launch_slot_attn_f32(const AttnParams32& p, int head_dim, hipStream_t stream);
hipError_t launch_slot_conf_bf16(const ConfParams& p, hipStream_t stream);
hipError_t launch_slot_conf_f32(const ConfParams& p, hipStream_t stream);
hipError_t launch_slot_conf_merge(const ConfMergeParams& p, hipStream_t stream);
hipError_t launch_select_slots(const SelectParams& p, hipStream_t stream);
hipError_t launch_verify_accept(const AcceptParams& p, hipStream_t stream);
hipError_t launch_kv_append(const AppendParams& p, hipStream_t stream);
hipError_t launch_mdm_reveal(const RevealParams& p, hipStream_t stream);

}  // namespace zarya
