// Split dK/dV sweeps without a GPU: the launchers are stand-ins that check
// every launch of the backward entry points. The items of a launch have to
// cover each tile's query blocks exactly once in consecutive parts, the
// scratch slots of the split tiles have to be distinct and inside the
// workspace, and what travels in the kernel arguments has to be what the
// schedule in the workspace would say. Prints "ok <launches with splits>".
#include <hip/hip_runtime_api.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "../../include/augtree.h"
#include "kernels.h"

using namespace augtree;

namespace {
int g_fail = 0, g_split = 0, g_inline = 0, g_max_parts = 0, g_fallback = 0;
bool g_launch_split = false;
const char* g_ws = nullptr;
size_t g_ws_bytes = 0;
std::vector<int> g_parts;  // parts per tile of the last dK/dV launch, keyed by schedule order
#define CHECK(c)                                                   \
  do {                                                             \
    if (!(c)) {                                                    \
      std::fprintf(stderr, "FAIL line %d: %s\n", __LINE__, #c);    \
      ++g_fail;                                                    \
    }                                                              \
  } while (0)
}  // namespace

extern "C" {
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) {
  std::memset(p, 0, sizeof(*p));
  std::strcpy(p->gcnArchName, "gfx950");
  return hipSuccess;
}
const char* hipGetErrorString(hipError_t) { return ""; }
hipError_t hipMemcpyAsync(void* dst, const void* src, size_t n, hipMemcpyKind, hipStream_t) {
  std::memcpy(dst, src, n);
  return hipSuccess;
}
}

namespace augtree {
hipError_t launch_attn_fwd(const FwdParams&, int, bool, hipStream_t) { return hipSuccess; }
hipError_t launch_attn_dq(const DqParams&, int, hipStream_t) { return hipSuccess; }
hipError_t launch_lse_merge(int64_t, int64_t, int64_t, int, int, int, const float*, const float*, uint16_t*, float*,
                            float*, hipStream_t) { return hipSuccess; }
hipError_t launch_grad_reduce(int, int64_t, int64_t, const float*, int, int64_t, int64_t, const float*,
                              const int32_t*, uint16_t* const[2], float* const[2], hipStream_t) { return hipSuccess; }

hipError_t launch_attn_dkv(const DkvParams& p, int n, hipStream_t) {
  const KVTile* tiles = p.tiles ? p.tiles : p.inl;
  CHECK(p.tiles || n <= kInlineTiles);
  g_parts.assign(n, 1);
  if (p.n_items == 0) {
    for (int i = 0; i < n; ++i) CHECK(tiles[i].flags >> KV_PART_SHIFT == 0);
    return hipSuccess;
  }
  ++g_split;
  g_launch_split = true;
  g_inline += !p.items;
  CHECK((p.items == nullptr) == (p.tiles == nullptr));
  CHECK(p.items || (p.n_inline == n && 4 * (p.n_items + p.n_combine) <= (int)sizeof(KVTile) * (kInlineTiles - n)));
  const size_t slot_bytes = (size_t)p.hkv * 2 * kDkvBlockN * p.head_dim * sizeof(float);
  CHECK((const char*)p.part >= g_ws && ((uintptr_t)p.part & 15) == 0);
  std::vector<std::vector<char>> seen(n);
  std::vector<char> slots;
  std::vector<uint32_t> first(n, ~0u);
  for (int i = 0; i < p.n_items; ++i) {
    const KVItem it = p.items ? p.items[i] : p.inline_item(i);
    CHECK(it.tile >= 0 && it.tile < n);
    const int np = kv_item_nparts(it.code), part = kv_item_part(it.code);
    CHECK(part < np && np <= kMaxParts);
    if (seen[it.tile].empty()) seen[it.tile].assign(np, 0);
    CHECK((int)seen[it.tile].size() == np && !seen[it.tile][part]);
    seen[it.tile][part] = 1;
    g_parts[it.tile] = np;
    g_max_parts = np > g_max_parts ? np : g_max_parts;
    const KVTile& t = tiles[it.tile];
    const int all = p.group * ((t.x_len + kDkvBlockQ - 1) / kDkvBlockQ + (t.y_len + kDkvBlockQ - 1) / kDkvBlockQ);
    const int len = t.flags >> KV_PART_SHIFT;
    if (np == 1) continue;
    CHECK(len > 0 && (np - 1) * len < all);  // every part has blocks
    const size_t slot = kv_item_slot(it.code) + part;
    CHECK((const char*)p.part + (slot + 1) * slot_bytes <= g_ws + g_ws_bytes);
    if (slot >= slots.size()) slots.resize(slot + 1, 0);
    CHECK(!slots[slot]);
    slots[slot] = 1;
    first[it.tile] = (uint32_t)kv_item_slot(it.code);
  }
  for (const auto& v : seen) {
    CHECK(!v.empty());
    for (char c : v) CHECK(c);
  }
  std::vector<char> added(n, 0);
  for (int i = 0; i < p.n_combine; ++i) {
    const KVItem it = p.combine ? p.combine[i] : p.inline_combine(i);
    CHECK(it.tile >= 0 && it.tile < n && !added[it.tile]);
    added[it.tile] = 1;
    CHECK(kv_item_nparts(it.code) == g_parts[it.tile] && (uint32_t)kv_item_slot(it.code) == first[it.tile]);
  }
  for (int i = 0; i < n; ++i) CHECK(added[i] == (g_parts[i] > 1));
  return hipSuccess;
}
}  // namespace augtree

namespace {
void* A(int i) { return reinterpret_cast<void*>((uintptr_t)0x10000000 + 0x100000u * (uintptr_t)i); }

void run(const std::vector<int>& ps, const std::vector<std::vector<int>>& rs, int hq, int hkv, int d) {
  std::vector<int32_t> cp{0}, cb{0}, cr{0};
  for (size_t g = 0; g < ps.size(); ++g) {
    cp.push_back(cp.back() + ps[g]);
    for (int r : rs[g]) cr.push_back(cr.back() + r);
    cb.push_back((int)cr.size() - 1);
  }
  const augtree_groups g{(int)ps.size(), (int)cr.size() - 1, hq, hkv, d, 0.125f, cp.data(), cb.data(), cr.data()};
  auto u = [](int i) { return static_cast<uint16_t*>(A(i)); };
  auto f = [](int i) { return static_cast<float*>(A(i)); };
  for (int which = 0; which < 4; ++which) {
    const int op = which < 2 ? AUGTREE_OP_TREE_BWD : which == 2 ? AUGTREE_OP_REPLAY_BWD : AUGTREE_OP_PREFILL_BWD;
    g_ws_bytes = augtree_workspace_size(&g, op, 3);
    void* ws = std::aligned_alloc(256, g_ws_bytes);
    g_ws = static_cast<char*>(ws);
    int st;
    if (which < 2)
      st = augtree_tree_bwd(&g, u(1), u(2), u(3), u(4), f(5), u(13), u(6), u(7), u(8), u(9), f(10), u(16), u(14),
                            u(21), u(22), which ? f(23) : nullptr, u(17), u(18), u(19), ws, g_ws_bytes, nullptr);
    else if (which == 2)
      st = augtree_replay_bwd(&g, u(6), u(7), u(8), u(2), u(3), u(9), f(10), u(16), u(17), u(18), u(19), 3, f(20), ws,
                              g_ws_bytes, nullptr);
    else
      st = augtree_prefill_bwd(&g, u(1), u(2), u(3), u(4), f(5), u(13), u(14), nullptr, f(15), ws, g_ws_bytes, nullptr);
    CHECK(st == AUGTREE_OK);
    if (which < 2 && g_launch_split) {
      // a workspace without room for the partial sums: accepted, whole sweeps
      const size_t full = g_ws_bytes;
      for (size_t less = 256; less < full; less *= 2) {
        g_ws_bytes = full - less;
        g_launch_split = false;
        st = augtree_tree_bwd(&g, u(1), u(2), u(3), u(4), f(5), u(13), u(6), u(7), u(8), u(9), f(10), u(16), u(14),
                              u(21), u(22), which ? f(23) : nullptr, u(17), u(18), u(19), ws, g_ws_bytes, nullptr);
        if (st == AUGTREE_OK) ++g_fallback;
        else CHECK(st == AUGTREE_ERR_WORKSPACE);
        if (less > 4096) CHECK(!g_launch_split);
      }
    }
    g_launch_split = false;
    std::free(ws);
  }
}
}  // namespace

int main() {
  run({384}, {{290, 411, 176, 620}}, 8, 2, 128);                                // inline schedule
  run({905, 384, 1337}, {{512, 731, 288, 1040, 196, 655}, {290, 411}, {702, 530}}, 8, 2, 128);
  run({1}, {{9000}}, 8, 1, 64);                                                 // one key, long sweep
  run({64}, {std::vector<int>(60, 1500)}, 28, 4, 128);                          // chunked and split
  run({4096}, {{1}}, 32, 8, 128);                                               // prefill only
  run({129, 4000}, {{127, 3}, {2}}, 7, 1, 64);
  uint64_t s = 88172645463325252ull;
  auto rnd = [&](int lo, int hi) {
    s ^= s << 13; s ^= s >> 7; s ^= s << 17;
    return lo + (int)(s % (uint64_t)(hi - lo + 1));
  };
  for (int r = 0; r < 60; ++r) {
    std::vector<int> ps;
    std::vector<std::vector<int>> rs;
    for (int g = rnd(1, 4); g > 0; --g) {
      ps.push_back(rnd(1, r % 2 ? 3000 : 300));
      std::vector<int> b;
      for (int i = rnd(1, 12); i > 0; --i) b.push_back(rnd(1, r % 3 ? 4000 : 100));
      rs.push_back(b);
    }
    const int hk = rnd(1, 3);
    run(ps, rs, hk * rnd(1, 8), hk, rnd(0, 1) ? 128 : 64);
  }
  if (g_fail || !g_inline || g_max_parts < 8 || g_fallback < 20) {
    std::printf("%d failures (%d inline, most parts %d, %d fallbacks)\n", g_fail, g_inline, g_max_parts, g_fallback);
    return 1;
  }
  std::printf("ok %d\n", g_split);
  return 0;
}
