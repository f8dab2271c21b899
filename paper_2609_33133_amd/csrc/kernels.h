// Host-callable launchers of the gfx950 kernels (internal to libaugtree).
//
// Arrays of two pointers are indexed by the kind of rows or keys a tile
// covers: [0] response rows / branch keys, [1] prompt rows / prompt keys.
// A launch of up to kInlineTiles tiles carries its schedule in the kernel
// arguments (tiles == nullptr), so small launches need no schedule upload.
#pragma once

#include <hip/hip_runtime_api.h>
#include <stdint.h>

#include "tiles.h"

namespace augtree {

// (Kernel arguments are limited to 4 KB.) An uploaded schedule costs a copy
// of 5 us on the stream before the launch: the forward of 99 tiles (8 query
// heads) 75 us with it and 69 without; the longer arguments cost nothing
// measurable.
constexpr int kInlineTiles = 112;

// Division by a launch constant d on the device: q = mulhi(n, magic), one too
// large at most (fast_div in common.h corrects it). magic = ceil(2^32 / d),
// and 0 for d = 1. (A 32-bit division costs a scalar wavefront about 40
// dependent instructions; a workgroup needs five before its first load.)
inline uint32_t div_magic(int d) { return d <= 1 ? 0u : (uint32_t)((((uint64_t)1 << 32) + d - 1) / d); }

struct FwdParams {
  const QTile* tiles;         // device schedule, or nullptr: `inl`
  const uint16_t* q[2];       // [rows, hq, d]
  const uint16_t* ka;         // segment A keys/values (prompt) [*, hkv, d]
  const uint16_t* va;
  const uint16_t* kb[2];      // segment B keys/values of response / prompt rows
  const uint16_t* vb[2];
  uint16_t* o[2];             // bf16 outputs [rows, hq, d] (bf16 kernel)
  float* o32;                 // fp32 partial outputs (fp32 kernel), slot 1 at + o32_part
  int64_t o32_part;
  float* lse[2];              // [hq, lse_rows]; fp32 kernel: lse[0], slot 1 at + lse_part
  int64_t lse_rows[2];
  int64_t lse_part;
  int hq, hkv, group, head_dim;
  float scale_log2;           // softmax_scale * log2(e)
  int n_units;                // tiles x KV heads (set by the launcher, as the magic numbers)
  uint32_t hkv_magic, group_magic;
  QTile inl[kInlineTiles];
};

struct DqParams {
  const QTile* tiles;
  const uint16_t* q[2];
  const uint16_t* dout[2];
  const uint16_t* o[2];       // forward output (bf16): D = rowsum(dO * O) is formed here
  const float* lse[2];        // natural-log LSE [hq, lse_rows]
  float* dsum[2];             // D written here [hq, lse_rows] (read by the dK/dV kernel)
  int64_t lse_rows[2];
  const uint16_t* ka;
  const uint16_t* va;
  const uint16_t* kb[2];
  const uint16_t* vb[2];
  uint16_t* dq[2];            // bf16 [rows, hq, d] (nullable)
  float* dq32[2];             // fp32 (nullable)
  int hq, hkv, group, head_dim;
  float scale, scale_log2;
  int n_units;
  uint32_t hkv_magic, group_magic;
  QTile inl[kInlineTiles];
};

struct DkvParams {
  const KVTile* tiles;
  const uint16_t* k[2];       // keys/values [*, hkv, d]: [0] response, [1] prompt
  const uint16_t* v[2];
  const uint16_t* q[2];       // queries [*, hq, d]: [0] response rows, [1] prompt rows
  const uint16_t* dout[2];
  const float* lse[2];        // [hq, lse_rows]
  const float* dsum[2];
  int64_t lse_rows[2];
  uint16_t* dk[2];            // bf16 outputs [*, hkv, d] (KV_OUT_BF16)
  uint16_t* dv[2];
  float* slab;                // fp32 slab [2][slab_rows, hkv, d] (KV_OUT_SLAB; rows per tile: out_row0)
  int64_t slab_rows;
  int hq, hkv, group, head_dim;
  float scale, scale_log2;
  uint32_t hkv_magic;
  // split sweeps (n_items > 0): the launch's workgroups, the tiles whose
  // parts the combine kernel has to add (code: first slot, part 0, nparts) and
  // the fp32 scratch of the partial sums, [slots][hkv][2][128 x d]
  const KVItem* items;        // device, or nullptr: words after the inline tiles
  const KVItem* combine;      // device, or nullptr: words after those
  int n_items, n_combine;
  int n_inline;               // tiles in `inl`
  int serial;                 // any tile is KV_SERIAL
  float* part;
  KVTile inl[kInlineTiles];   // n_inline tiles, then n_items and n_combine item words

  // item (combine: tile to add) i of the kernel arguments
  __host__ __device__ KVItem inline_item(int i) const {
    const uint32_t w = reinterpret_cast<const uint32_t*>(inl + n_inline)[i];
    return KVItem{(int32_t)(w >> 24), w & 0xffffffu};
  }
  __host__ __device__ KVItem inline_combine(int i) const { return inline_item(n_items + i); }
};
static_assert(sizeof(FwdParams) <= 4096 && sizeof(DqParams) <= 4096 && sizeof(DkvParams) <= 4096, "kernel arguments");

// fp32 values of one scratch slot and KV head (dK and dV of a 128-key tile)
inline int64_t dkv_part_elems(int head_dim) { return 2 * (int64_t)kDkvBlockN * head_dim; }

hipError_t launch_attn_fwd(const FwdParams& p, int n_tiles, bool out_f32, hipStream_t stream);
hipError_t launch_attn_dq(const DqParams& p, int n_tiles, hipStream_t stream);
hipError_t launch_attn_dkv(const DkvParams& p, int n_tiles, hipStream_t stream);
// rows row0 .. row0 + rows - 1 of [total_rows]-row tensors
hipError_t launch_lse_merge(int64_t row0, int64_t rows, int64_t total_rows, int heads, int head_dim, int n_parts,
                            const float* o_parts, const float* lse_parts, uint16_t* o, float* o32, float* lse,
                            hipStream_t stream);
// out[t][row] = self[t][row] + sum over k of parts[k][t][src(k, row)] (src =
// row, or row_map[k * rows + row], skipped when negative), tensors t < n_tensors
// written to out[t] (bf16) and/or out32[t] (fp32), each [rows, row_elems]
hipError_t launch_grad_reduce(int n_tensors, int64_t rows, int64_t row_elems, const float* self, int n_parts,
                              int64_t part_rows, int64_t part_stride, const float* parts, const int32_t* row_map,
                              uint16_t* const out[2], float* const out32[2], hipStream_t stream);

inline int fwd_block_m() { return kFwdBlockM; }
inline int fwd_block_n() { return kFwdBlockN; }
inline int dq_block_m() { return kDqBlockM; }
inline int dkv_block_n() { return kDkvBlockN; }
inline int dkv_block_q() { return kDkvBlockQ; }

}  // namespace augtree
