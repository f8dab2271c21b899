// Tile descriptors shared by the host schedule builder and the kernels.
#pragma once

#include <stdint.h>

#if !defined(__host__)  // plain C++ (the host library)
#define __host__
#define __device__
#endif

namespace augtree {

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

// Tile sizes of the kernels (the host schedules are cut to them).
constexpr int kFwdBlockM = 128;   // forward: query rows per tile
constexpr int kFwdBlockN = 64;    // forward: keys per block
constexpr int kDqBlockM = 128;    // dQ: query rows per tile
constexpr int kDqBlockN = 64;     // dQ: keys per block
constexpr int kDkvBlockN = 128;   // dK/dV: keys per tile
constexpr int kDkvBlockQ = 64;    // dK/dV: query rows per block

// (row, head) pairs of a forward or dQ workgroup, 32 per wavefront. A tile is
// launched as g workgroups per KV head (g query heads each), which hold all
// its pairs only while it has at most this many rows.
constexpr int kPairsPerWorkgroup = 128;
static_assert(kFwdBlockM <= kPairsPerWorkgroup && kDqBlockM <= kPairsPerWorkgroup, "a tile's pairs fit its workgroups");

// Query tile of the forward and dQ kernels: up to BM query rows, attending to
// segment A (prompt keys, every key visible) and then segment B (causal:
// query i of the tile sits at segment position b_qpos + i and sees keys
// 0 .. b_qpos + i).
struct QTile {
  int32_t q_row0, q_len;
  int32_t a_row0, a_len;
  int32_t b_row0, b_len, b_qpos;
  int32_t flags;  // QT_*
};

// Element offset of (row, head) of a query tile from its first row at its KV
// head, in a [*, hq, D] tensor. 64 bits: 128 rows of 132,105 heads of 128 pass
// 2^31 elements.
template <int D>
__host__ __device__ inline int64_t pair_offset(int row, int head, int hq) {
  return (int64_t)row * hq * D + head * D;
}

enum : int32_t {
  // the query rows are prompt rows (Q_P, O_P, LSE_P; segment B = prompt
  // keys); otherwise response rows (Q_R, O_R, LSE_R; segment B = the
  // branch's own keys)
  QT_PROMPT_ROWS = 1,
  // fp32 partial outputs: write the second partial slot (own-branch partial)
  QT_PART1 = 2,
};

// Key tile of the dK/dV kernel: up to 128 keys of one KV head against up to
// two ranges of query rows, swept in this order:
//   X: response rows x_row0 .. x_row0 + x_len - 1 (Q_R, dO_R, LSE_R, D_R),
//      causal if KV_X_CAUSAL, otherwise every key visible;
//   Y: prompt rows kv_row0 .. kv_row0 + y_len - 1 (Q_P, ...), causal (prompt
//      keys only: prompt queries before the tile's first key cannot see it).
// In a causal range, query i sits at position kpos0 + i of its segment (the
// range starts at the tile's first key) and key j at kpos0 + j: visible iff
// j <= i. Outputs: the key rows' dK/dV in bf16 (KV_OUT_BF16, rows kv_row0 ..)
// and/or fp32 (KV_OUT_SLAB): dK of key j at row out_row0 + j of the fp32 slab,
// dV slab_rows rows further on.
struct KVTile {
  int32_t kv_row0, kv_len;
  int32_t x_row0, x_len;
  int32_t y_len;
  int32_t kpos0;
  int32_t out_row0;
  int32_t flags;  // KV_*
};

enum : int32_t {
  KV_PROMPT_KEYS = 1,  // keys K_P/V_P (outputs dK_P/dV_P); otherwise K_R/V_R
  KV_X_CAUSAL = 2,
  KV_OUT_BF16 = 4,
  KV_OUT_SLAB = 8,
  KV_SERIAL = 16,      // split tile whose parts run one after the other in one workgroup
  KV_PART_SHIFT = 8,  // flags >> KV_PART_SHIFT: blocks of a part (split tiles)
};

// One workgroup of a dK/dV launch whose long sweeps are split: part `part` of
// `nparts` of tile `tile`'s query blocks in sweep order. The parts are
// flags >> KV_PART_SHIFT blocks long, the last one takes the rest (the same
// cuts for every tile of a segment, so that parts that run together read the
// same query rows). A tile with nparts = 1 writes its outputs. The parts of a
// split tile are added in part order, in one of two ways with the same bits:
// each part is a workgroup that writes its fp32 sums to scratch slot
// slot0 + part, and a combine kernel adds them; or (KV_SERIAL) one item,
// part 0, stands for the tile, and its workgroup runs the parts one after the
// other and keeps their running sum in slot slot0. code = slot0 << 8 |
// part << 4 | (nparts - 1). A launch whose tiles and items fit the
// kernel arguments carries its items there as one word each: tile << 24 |
// code (tile < 256, slot0 < 65536).
struct KVItem {
  int32_t tile;
  uint32_t code;
};

constexpr int kMaxParts = 16;  // parts of one tile (4 bits of the code)

__host__ __device__ inline uint32_t kv_item_code(int slot, int part, int nparts) {
  return (uint32_t)slot << 8 | (uint32_t)part << 4 | (uint32_t)(nparts - 1);
}
__host__ __device__ inline int kv_item_slot(uint32_t code) { return (int)(code >> 8); }
__host__ __device__ inline int kv_item_part(uint32_t code) { return (int)(code >> 4) & 15; }
__host__ __device__ inline int kv_item_nparts(uint32_t code) { return (int)(code & 15) + 1; }

}  // namespace augtree
