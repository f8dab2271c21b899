// Split dK/dV sweeps without a GPU: the launchers are stand-ins that check
// every launch of the backward entry points. The items of a launch have to
// cover each tile's query blocks exactly once in consecutive parts, the
// scratch slots of the split tiles have to be distinct and inside the
// workspace, and what travels in the kernel arguments has to be what the
// schedule in the workspace would say. A tree's cuts have to be the same
// whether its parts are workgroups of their own or run in one, and whether it
// is alone in a batch or not. Prints "ok <launches with splits>".
#include <hip/hip_runtime_api.h>

#include <algorithm>
#include <array>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "../../include/augtree.h"
#include "kernels.h"

using namespace augtree;

namespace {
int g_fail = 0, g_split = 0, g_inline = 0, g_max_parts = 0, g_fallback = 0, g_serial = 0, g_mixed = 0;
typedef std::array<int, 7> Cut;  // a tile and how it is cut, without its place in the batch
std::vector<Cut> g_cuts;         // of the last dK/dV launch
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
  CHECK(n > (p.n_items ? 35 : 112) || (!p.tiles && !p.items));  // what augtree.h says of the kernel arguments
  g_parts.assign(n, 1);
  auto note_cuts = [&] {
    g_cuts.clear();
    for (int i = 0; i < n; ++i)
      g_cuts.push_back({tiles[i].kv_len, tiles[i].x_len, tiles[i].y_len, tiles[i].kpos0, tiles[i].flags & 3,
                        tiles[i].flags >> KV_PART_SHIFT, g_parts[i]});
    std::sort(g_cuts.begin(), g_cuts.end());
  };
  if (p.n_items == 0) {
    for (int i = 0; i < n; ++i) CHECK(tiles[i].flags >> KV_PART_SHIFT == 0 && !(tiles[i].flags & KV_SERIAL));
    CHECK(!p.serial);
    note_cuts();
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
  bool any_serial = false, any_apart = false;
  for (int i = 0; i < p.n_items; ++i) {
    const KVItem it = p.items ? p.items[i] : p.inline_item(i);
    CHECK(it.tile >= 0 && it.tile < n);
    const int np = kv_item_nparts(it.code), part = kv_item_part(it.code);
    CHECK(part < np && np <= kMaxParts);
    const bool serial = (tiles[it.tile].flags & KV_SERIAL) != 0;  // one item for all parts
    any_serial = any_serial || serial;
    any_apart = any_apart || (np > 1 && !serial);
    CHECK(!serial || (np > 1 && part == 0));
    if (seen[it.tile].empty()) seen[it.tile].assign(serial ? 1 : np, 0);
    CHECK((int)seen[it.tile].size() == (serial ? 1 : np) && !seen[it.tile][part]);
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
  for (int i = 0; i < n; ++i) CHECK(added[i] == (g_parts[i] > 1 && !(tiles[i].flags & KV_SERIAL)));
  CHECK((p.serial != 0) == any_serial);
  g_serial += any_serial && !any_apart;
  g_mixed += any_serial && any_apart;
  note_cuts();
  return hipSuccess;
}
}  // namespace augtree

namespace {
void* A(int i) { return reinterpret_cast<void*>((uintptr_t)0x10000000 + 0x100000u * (uintptr_t)i); }

int call(const augtree_groups& g, int which, size_t ws_bytes) {
  auto u = [](int i) { return static_cast<uint16_t*>(A(i)); };
  auto f = [](int i) { return static_cast<float*>(A(i)); };
  // (only the schedules at its start are written on the host)
  void* ws = std::aligned_alloc(256, std::min<size_t>((ws_bytes + 255) / 256 * 256, 4 << 20));
  g_ws = static_cast<char*>(ws);
  g_ws_bytes = ws_bytes;
  g_launch_split = false;
  int st;
  if (which < 2)
    st = augtree_tree_bwd(&g, u(1), u(2), u(3), u(4), f(5), u(13), u(6), u(7), u(8), u(9), f(10), u(16), u(14), u(21),
                          u(22), which ? f(23) : nullptr, u(17), u(18), u(19), ws, ws_bytes, nullptr);
  else if (which == 2)
    st = augtree_replay_bwd(&g, u(6), u(7), u(8), u(2), u(3), u(9), f(10), u(16), u(17), u(18), u(19), 3, f(20), ws,
                            ws_bytes, nullptr);
  else
    st = augtree_prefill_bwd(&g, u(1), u(2), u(3), u(4), f(5), u(13), u(14), nullptr, f(15), ws, ws_bytes, nullptr);
  std::free(ws);
  return st;
}

// runs the backward entry points on a batch; returns the tree backward's cuts
std::vector<Cut> run(const std::vector<int>& ps, const std::vector<std::vector<int>>& rs, int hq, int hkv, int d) {
  std::vector<int32_t> cp{0}, cb{0}, cr{0};
  for (size_t g = 0; g < ps.size(); ++g) {
    cp.push_back(cp.back() + ps[g]);
    for (int r : rs[g]) cr.push_back(cr.back() + r);
    cb.push_back((int)cr.size() - 1);
  }
  const augtree_groups g{(int)ps.size(), (int)cr.size() - 1, hq, hkv, d, 0.125f, cp.data(), cb.data(), cr.data()};
  std::vector<Cut> tree_cuts;
  for (int which = 0; which < 4; ++which) {
    const int op = which < 2 ? AUGTREE_OP_TREE_BWD : which == 2 ? AUGTREE_OP_REPLAY_BWD : AUGTREE_OP_PREFILL_BWD;
    const size_t full = augtree_workspace_size(&g, op, 3);
    CHECK(call(g, which, full) == AUGTREE_OK);
    const std::vector<Cut> cuts = g_cuts;
    if (which == 0) tree_cuts = cuts;
    if (which >= 2 || !g_launch_split) continue;
    // less room: the parts in one workgroup, with the same cuts; then whole
    // sweeps; then refused
    int level = 0;
    for (size_t less = 256; less < full; less *= 2) {
      const int st = call(g, which, full - less);
      const int now = st != AUGTREE_OK ? 2 : g_launch_split ? 0 : 1;
      CHECK(now >= level && (st == AUGTREE_OK || st == AUGTREE_ERR_WORKSPACE));
      if (now == 0) CHECK(g_cuts == cuts);
      if (now == 1)
        for (const Cut& c : g_cuts) CHECK(c[6] == 1);
      level = now;
      g_fallback += now == 1;
    }
  }
  if (ps.size() > 1) {
    std::vector<Cut> alone;
    for (size_t i = 0; i < ps.size(); ++i) {
      const std::vector<Cut> c = run({ps[i]}, {rs[i]}, hq, hkv, d);
      alone.insert(alone.end(), c.begin(), c.end());
    }
    std::sort(alone.begin(), alone.end());
    CHECK(alone == tree_cuts);
  }
  return tree_cuts;
}
}  // namespace

int main() {
  run({384}, {{290, 411, 176, 620}}, 8, 2, 128);                                // inline schedule
  run({905, 384, 1337}, {{512, 731, 288, 1040, 196, 655}, {290, 411}, {702, 530}}, 8, 2, 128);
  run({1}, {{9000}}, 8, 1, 64);                                                 // one key, long sweep
  run({64}, {std::vector<int>(60, 1500)}, 28, 4, 128);                          // chunked and split
  run({4096}, {{1}}, 32, 8, 128);                                               // prefill only
  run({129, 4000}, {{127, 3}, {2}}, 7, 1, 64);
  run(std::vector<int>(24, 400), std::vector<std::vector<int>>(24, std::vector<int>(8, 500)), 8, 2, 128);  // full chip
  std::vector<int> ps(25, 400);
  std::vector<std::vector<int>> rs(25, std::vector<int>(8, 500));
  ps[7] = 100;
  rs[7].assign(30, 2000);
  run(ps, rs, 8, 2, 128);                                                       // full chip, one long tree
  uint64_t s = 88172645463325252ull;
  auto rnd = [&](int lo, int hi) {
    s ^= s << 13; s ^= s >> 7; s ^= s << 17;
    return lo + (int)(s % (uint64_t)(hi - lo + 1));
  };
  for (int r = 0; r < 60; ++r) {
    ps.clear();
    rs.clear();
    for (int g = rnd(1, 4); g > 0; --g) {
      ps.push_back(rnd(1, r % 2 ? 3000 : 300));
      std::vector<int> b;
      for (int i = rnd(1, 12); i > 0; --i) b.push_back(rnd(1, r % 3 ? 4000 : 100));
      rs.push_back(b);
    }
    const int hk = rnd(1, 3);
    run(ps, rs, hk * rnd(1, 8), hk, rnd(0, 1) ? 128 : 64);
  }
  if (g_fail || !g_inline || g_max_parts < 8 || g_fallback < 20 || g_serial < 20 || g_mixed < 3) {
    std::printf("%d failures (%d inline, most parts %d, %d fallbacks, %d serial, %d mixed)\n", g_fail, g_inline,
                g_max_parts, g_fallback, g_serial, g_mixed);
    return 1;
  }
  std::printf("ok %d\n", g_split);
  return 0;
}
