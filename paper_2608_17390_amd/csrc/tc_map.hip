// Map maintenance kernels: column repack, pyramid build, ordered edits and
// the dirty-node pyramid update.
//
// The pyramid is the maximum-mipmap structure cited in Section 1.1,
// extended to the two solid intervals of a column: a node of level L covers
// a 2^L x 2^L block of cells and keeps the largest floor top (fmax), the
// smallest slab bottom (smin) and the largest slab top (smax) of the block.
// A ray whose height range over the node's time span stays above fmax and
// either above smax or below smin cannot meet solid in the block.
//
// Beside each node, a 64-bit occupancy mask over height (bit k: a slab of
// the block meets the band [4k, 4k + 4]) is the union of its children's,
// as the paper's occupancy pyramid takes the union of its children
// (Section 3.2); it is built and updated with the node.
//
// Window levels (one per level, used by the packet beam's box test) hold,
// per node, the combine of its 2 x 2 node neighbourhood on the same level;
// they are built after the levels and, after edits, updated for the entries
// whose neighbourhood meets an edited node.
//
// Edits follow Section 2 (a dirty rectangle with new heights and slab
// metadata) and Section 4.4 (the dig crater).  Only the nodes above the
// edited rectangles are recomputed, from the same 2x2 reduction as the full
// build, so the updated pyramid is byte-identical to a rebuild.
#include "tc_internal.h"

namespace {

constexpr int kEditSet = 1;

__device__ inline uint32_t cell_to_node(uint32_t c) {
  // packed column F | B << 8 | T << 16 -> node fmax | smin << 8 | smax << 16
  uint32_t F = c & 0xFF, B = (c >> 8) & 0xFF, T = (c >> 16) & 0xFF;
  return B ? (F | (B << 8) | (T << 16)) : (F | (255u << 8));
}

__device__ inline uint32_t node_merge(uint32_t a, uint32_t b) {
  uint32_t f = max(a & 0xFF, b & 0xFF);
  uint32_t lo = min((a >> 8) & 0xFF, (b >> 8) & 0xFF);
  uint32_t hi = max((a >> 16) & 0xFF, (b >> 16) & 0xFF);
  return f | (lo << 8) | (hi << 16);
}

// Node (i, j) of level L from its up-to-four children at level L-1.
__device__ inline uint32_t reduce_node(const tci_map& m, const uint32_t* base,
                                       int32_t L, int32_t i, int32_t j) {
  const tci_level& c = m.lv[L - 1];
  uint32_t acc = 0u | (255u << 8);  // empty: fmax 0, smin 255, smax 0
  #pragma unroll
  for (int dj = 0; dj < 2; ++dj) {
    #pragma unroll
    for (int di = 0; di < 2; ++di) {
      int32_t ci = 2 * i + di, cj = 2 * j + dj;
      if (ci < c.w && cj < c.h) {
        uint32_t v = base[tci_tile_index(c, ci, cj)];
        acc = node_merge(acc, L == 1 ? cell_to_node(v) : v);
      }
    }
  }
  return acc;
}

__global__ void repack_kernel(const uint8_t* __restrict__ planes, int32_t W,
                              int32_t H, uint32_t* __restrict__ base,
                              tci_level l0) {
  // one thread per word of the tiled level-0 array
  int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t ntiles = (int64_t)l0.tiles_x * ((H + 7) >> 3);
  if (k >= ntiles * 64) return;
  int32_t tile = (int32_t)(k >> 6), e = (int32_t)(k & 63);
  int32_t x = (tile % l0.tiles_x) * 8 + (e & 7);
  int32_t y = (tile / l0.tiles_x) * 8 + (e >> 3);
  uint32_t v = 0;
  if (x < W && y < H) {
    size_t idx = (size_t)y * W + x;
    size_t plane = (size_t)W * H;
    uint32_t F = planes[idx], B = planes[plane + idx], T = planes[2 * plane + idx];
    v = F | (B << 8) | (T << 16);
  }
  base[l0.off + k] = v;
}

// Occupancy bands of one column's slab [B, T]: bits (B + 3) / 4 - 1 ..
// T / 4, the bands [4k, 4k + 4] that meet it (none without a slab).
__device__ inline uint64_t cell_mask(uint32_t c) {
  const uint32_t B = (c >> 8) & 0xFF, T = (c >> 16) & 0xFF;
  if (!B) return 0;
  const uint32_t lo = (B + 3) / 4 - 1, hi = T / 4;
  return (~0ull >> (63 - hi)) & (~0ull << lo);
}

// Occupancy mask of node (i, j) of level L: the union of its children's.
__device__ inline uint64_t reduce_mask(const tci_map& m, const uint32_t* base,
                                       int32_t L, int32_t i, int32_t j) {
  const tci_level& c = m.lv[L - 1];
  uint64_t acc = 0;
  #pragma unroll
  for (int dj = 0; dj < 2; ++dj) {
    #pragma unroll
    for (int di = 0; di < 2; ++di) {
      int32_t ci = 2 * i + di, cj = 2 * j + dj;
      if (ci < c.w && cj < c.h) {
        if (L == 1) {
          acc |= cell_mask(base[tci_tile_index(c, ci, cj)]);
        } else {
          const uint32_t k = tci_mask_index(m.mk[L - 1], ci, cj);
          acc |= (uint64_t)base[k] | ((uint64_t)base[k + 1] << 32);
        }
      }
    }
  }
  return acc;
}

__device__ inline void store_mask(const tci_map& m, uint32_t* base, int32_t L,
                                  int32_t i, int32_t j, uint64_t v) {
  const uint32_t k = tci_mask_index(m.mk[L], i, j);
  base[k] = (uint32_t)v;
  base[k + 1] = (uint32_t)(v >> 32);
}

__global__ void build_level_kernel(tci_map m, uint32_t* __restrict__ base,
                                   int32_t L) {
  const tci_level& l = m.lv[L];
  int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t total = (int64_t)l.tiles_x * ((l.h + 7) >> 3) * 64;
  if (k >= total) return;
  int32_t tile = (int32_t)(k >> 6), e = (int32_t)(k & 63);
  int32_t i = (tile % l.tiles_x) * 8 + (e & 7);
  int32_t j = (tile / l.tiles_x) * 8 + (e >> 3);
  uint32_t v = 0;
  uint64_t mask = 0;
  if (i < l.w && j < l.h) {
    v = reduce_node(m, base, L, i, j);
    mask = reduce_mask(m, base, L, i, j);
  }
  base[l.off + k] = v;
  store_mask(m, base, L, i, j, mask);
}

__device__ inline bool covers(const tci_edit& e, int32_t x, int32_t y) {
  return x >= e.x0 && x < e.x0 + e.w && y >= e.y0 && y < e.y0 + e.h;
}

// Apply edit e to a packed column at cell (x, y) inside e's rectangle.
__device__ inline uint32_t apply_one(const tci_edit& e,
                                     const uint8_t* __restrict__ patch,
                                     uint32_t col, int32_t x, int32_t y) {
  int32_t i = x - e.x0, j = y - e.y0;
  if (e.kind == kEditSet) {
    int64_t n = (int64_t)e.w * e.h;
    int64_t o = e.data_off + (int64_t)j * e.w + i;
    uint32_t F = patch[o], B = patch[o + n], T = patch[o + 2 * n];
    return F | (B << 8) | (T << 16);
  }
  // crater of size s = w = h <= 4096 and depth <= 255: r2 < 2^25 and
  // depth (R2 - r2) < 2^32, so 32-bit arithmetic is exact
  const int32_t s = e.w;
  const int32_t a = 2 * i + 1 - s, b = 2 * j + 1 - s;
  const uint32_t r2 = (uint32_t)(a * a) + (uint32_t)(b * b), R2 = (uint32_t)(s * s);
  if (r2 >= R2) return col;
  const uint32_t drop = ((uint32_t)e.depth * (R2 - r2)) / R2;
  const uint32_t F = col & 0xFF;
  return F > drop ? F - drop : 0u;  // slab removed: B = T = 0
}

// grid.x = edit index; threads stride over that edit's clipped rectangle.
// A cell is owned by the first edit that covers it; the owner applies all
// covering edits in list order, so the result is the sequential one and no
// two threads write the same cell.  Only the edits whose rectangles meet
// this edit's can cover its cells: olap lists them (start[n + 1], then the
// ascending lists), or with `all` every edit is tested.
__global__ void edits_kernel(const tci_edit* __restrict__ edits, int32_t n,
                             const int32_t* __restrict__ olap, int32_t all,
                             const uint8_t* __restrict__ patch,
                             uint32_t* __restrict__ base, tci_level l0,
                             int32_t W, int32_t H) {
  const int32_t ei = blockIdx.x;
  const tci_edit e = edits[ei];
  const int32_t x0 = max(e.x0, 0), y0 = max(e.y0, 0);
  const int32_t x1 = min(e.x0 + e.w, W), y1 = min(e.y0 + e.h, H);
  if (x0 >= x1 || y0 >= y1) return;
  const int32_t lb = all ? 0 : olap[ei], lc = all ? n : olap[ei + 1] - lb;
  const int32_t* lst = olap + n + 1 + lb;
  // (a clipped rectangle holds at most 2^28 cells)
  const int32_t cw = x1 - x0, cells = cw * (y1 - y0);
  for (int32_t k = blockIdx.y * blockDim.x + threadIdx.x; k < cells;
       k += gridDim.y * blockDim.x) {
    const int32_t x = x0 + k % cw, y = y0 + k / cw;
    bool owned = true;
    for (int32_t t = 0; t < lc; ++t) {
      const int32_t p = all ? t : lst[t];
      if (p >= ei) break;
      if (covers(edits[p], x, y)) {
        owned = false;
        break;
      }
    }
    if (!owned) continue;
    const uint32_t idx = tci_tile_index(l0, x, y);
    uint32_t col = apply_one(e, patch, base[idx], x, y);
    for (int32_t t = 0; t < lc; ++t) {
      const int32_t q = all ? t : lst[t];
      if (q > ei && covers(edits[q], x, y)) col = apply_one(edits[q], patch, col, x, y);
    }
    base[idx] = col;
  }
}

// Edits and the six pyramid levels over them in one launch, for lists of at
// most tci::kTileEdits edits.  A block takes a block of 64 x 64 cells that an
// edit's rectangle touches, a wave 16 x 16 of them, a lane 2 x 2: it applies
// every edit that covers its cells, in list order, and has the node and mask
// of level 1 at hand; those of levels 2..4 fold together by cross-lane
// exchanges, and the first wave folds the block's 16 level-4 nodes into those
// of levels 5 and 6.  A block of cells belongs to the first edit that touches
// it (64 edits are compared at a time, one per lane), so no two blocks write
// the same word; cells and nodes no edit touches come out as they were.
// grid.x = edit; grid.y blocks stride over its blocks of cells.  Every launch
// of an edit's chain is bound by latency: a few microseconds however little
// it does, of which one round of loads and the first fetch of its own code
// are most.  So it pays to have fewer of them, each with one round of loads
// and little code: the chain of a 96-cell crater on a 2048 x 16384 map was six
// launches (one for the cells, five for the levels) of 25 us together and is
// two of 17 (7 this one).  Longer lists than kTileEdits compare too many
// edits per block of cells and keep the launch per cells and per level group.
// Where many edits meet one block, what bounds it is the way through them, one
// after the other: their records are held in LDS, the next one's read while
// one is applied, a wave goes through those that touch its own cells, and
// nothing of a cell's column is touched on the way.  The last patch over a cell
// is read at the end, and craters add up: max(max(F - a, 0) - b, 0) is
// max(F - (a + b), 0).  A frame of 200 craters of 16 cells in 24 x 24: 101 us; with a
// record read from memory and applied to the column at a time 299, and with the
// launch per cells 101.  512 of 96 cells in 200 x 200: 305, 604 and 490.
constexpr int32_t kTileThreads = 1024;

// The levels' records in LDS: a kernel that goes through the levels in turn
// then waits for the kernel's arguments once.
struct levels_t {
  tci_level lv[TCI_MAX_LEVELS], mk[TCI_MAX_LEVELS], wl[TCI_MAX_LEVELS];
};
__device__ inline void load_levels_lds(const tci_map& m, levels_t& t) {
  const int32_t k = threadIdx.x >> 6, L = threadIdx.x & 63;
  if (L < TCI_MAX_LEVELS) {
    if (k == 0) t.lv[L] = m.lv[L];
    else if (k == 1) t.mk[L] = m.mk[L];
    else if (k == 2) t.wl[L] = m.wl[L];
  }
  __syncthreads();
}

// An edit's rectangle clipped to the map: cells x0..x1, y0..y1, empty if
// x0 > x1 or y0 > y1.
struct clip_t {
  int32_t x0, y0, x1, y1;
};
__device__ inline clip_t clip(const int4& e, int32_t W, int32_t H) {
  return clip_t{max(e.x, 0), max(e.y, 0), min(e.x + e.z, W) - 1, min(e.y + e.w, H) - 1};
}
// Does it touch block (bx, by) of 2^sh x 2^sh cells?
__device__ inline bool touches(const clip_t& r, int32_t bx, int32_t by, int32_t sh) {
  return (r.x0 <= r.x1) & (r.y0 <= r.y1) & ((r.x0 >> sh) <= bx) & (bx <= (r.x1 >> sh)) &
         ((r.y0 >> sh) <= by) & (by <= (r.y1 >> sh));
}

// Lane ^ o's word, without the LDS round trip of a general exchange where
// the hardware moves lanes itself (o = 1, 2: within four lanes; 8: half a
// turn of 16).
template <int o>
__device__ inline uint32_t from_lane_xor(uint32_t v) {
  if constexpr (o == 1) return __builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xF, 0xF, true);
  else if constexpr (o == 2) return __builtin_amdgcn_mov_dpp((int)v, 0x4E, 0xF, 0xF, true);
  else if constexpr (o == 8) return __builtin_amdgcn_mov_dpp((int)v, 0x128, 0xF, 0xF, true);
  else return (uint32_t)__shfl_xor((int)v, o);
}

template <int o>
__device__ inline void fold_step(uint32_t& v, uint64_t& mk) {
  v = node_merge(v, from_lane_xor<o>(v));
  const uint32_t lo = from_lane_xor<o>((uint32_t)mk);
  const uint32_t hi = from_lane_xor<o>((uint32_t)(mk >> 32));
  mk |= (uint64_t)lo | ((uint64_t)hi << 32);
}

// The nodes and masks of levels L0 + 1 .. L0 + n (n <= 3) over 8 x 8
// level-L0 nodes (v, mk) held one per lane: that of lane k at (x, y), its
// place in the block (k & 7, k >> 3), in: inside the level.  The lane of each
// node's first level-L0 node stores it and hands it to put(level, x, y,
// node, mask); v and mk end as the level L0 + 3 node's.
template <class Put>
__device__ inline void fold_levels(const levels_t& t, int32_t top, uint32_t* base, int32_t L0,
                                   int32_t n, int32_t x, int32_t y, bool in, int32_t lane,
                                   uint32_t& v, uint64_t& mk, Put put) {
  auto store = [&](int32_t k) {
    if (L0 + k > top || k > n || !in || (((lane & 7) | (lane >> 3)) & ((1 << k) - 1)) != 0) return;
    const int32_t i = x >> k, j = y >> k;
    base[tci_tile_index(t.lv[L0 + k], i, j)] = v;
    *reinterpret_cast<uint2*>(base + tci_mask_index(t.mk[L0 + k], i, j)) =
        make_uint2((uint32_t)mk, (uint32_t)(mk >> 32));
    put(L0 + k, i, j, v, mk);
  };
  fold_step<1>(v, mk);
  fold_step<8>(v, mk);
  store(1);
  fold_step<2>(v, mk);
  fold_step<16>(v, mk);
  store(2);
  fold_step<4>(v, mk);
  fold_step<32>(v, mk);
  store(3);
}

__global__ __launch_bounds__(kTileThreads) void edit_tiles_kernel(
    tci_map m, const tci_edit* __restrict__ edits, int32_t n, const uint8_t* __restrict__ patch,
    uint32_t* __restrict__ base) {
  __shared__ levels_t tab;
  __shared__ uint32_t node4[16], lo4[16], hi4[16];
  // the edits' rectangles (x0, y0, w, h), and what else they are: for a patch
  // -1 and its bytes' offset, for a crater its depth and 1 / w^2, a little less
  __shared__ int4 rect[tci::kTileEdits], rest[tci::kTileEdits];
  const int32_t ei = blockIdx.x, lane = threadIdx.x & 63;
  const int32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  auto rect_of = [](const tci_edit& e) { return make_int4(e.x0, e.y0, e.w, e.h); };
  const clip_t r = clip(rect_of(edits[ei]), m.W, m.H);
  if (r.x0 > r.x1 || r.y0 > r.y1) return;
  const int32_t bx0 = r.x0 >> 6, by0 = r.y0 >> 6;
  const int32_t nbx = (r.x1 >> 6) - bx0 + 1, nb = nbx * ((r.y1 >> 6) - by0 + 1);
  if ((int32_t)blockIdx.y >= nb) return;
  if ((int32_t)threadIdx.x < n) {
    const tci_edit e = edits[threadIdx.x];
    rect[threadIdx.x] = rect_of(e);
    rest[threadIdx.x] = e.kind == kEditSet
        ? make_int4(-1, 0, (int32_t)e.data_off, (int32_t)(e.data_off >> 32))
        : make_int4(e.depth, __float_as_int(0x1.fffff8p-1f / (float)(e.w * e.w)), 0, 0);
  }
  load_levels_lds(m, tab);
  // which of edits c .. c + 63 touch block (bx, by) of 2^sh x 2^sh cells (all
  // lanes take part)
  auto who = [&](int32_t c, int32_t bx, int32_t by, int32_t sh) {
    return (uint64_t)__ballot(c + lane < n &&
                              touches(clip(rect[min(c + lane, n - 1)], m.W, m.H), bx, by, sh));
  };
  // (every wave of the block runs the same rounds: the barriers are reached
  // by all of them)
  for (int32_t b = blockIdx.y; b < nb; b += gridDim.y) {
    const int32_t bx = bx0 + b % nbx, by = by0 + b / nbx;
    // the lane's four cells: two pairs in memory (tiles are whole, so the
    // cells of a lane whose first is in the map can be read)
    const int32_t x1 = bx * 32 + (wave & 3) * 8 + (lane & 7), y1 = by * 32 + (wave >> 2) * 8 + (lane >> 3);
    const int32_t x = 2 * x1, y = 2 * y1;
    const bool in = x < m.W && y < m.H;
    uint32_t* c0 = base + (in ? tci_tile_index(tab.lv[0], x, y) : 0u);
    uint2 p[2] = {make_uint2(0u, 0u), make_uint2(0u, 0u)};
    if (in) {
      p[0] = *reinterpret_cast<const uint2*>(c0);
      p[1] = *reinterpret_cast<const uint2*>(c0 + 8);
    }
    bool owned = true;
    for (int32_t c = 0; c <= ei && owned; c += 64)
      owned = (who(c, bx, by, 6) & (ei - c < 64 ? (1ull << (ei - c)) - 1 : ~0ull)) == 0;
    if (!owned) continue;
    // per cell: the last patch over it, and of the craters after that what
    // they take off and whether one is over it (dig > 0)
    int32_t set[4] = {-1, -1, -1, -1}, dig[4] = {0, 0, 0, 0};
    uint32_t drop[4] = {0u, 0u, 0u, 0u};
    for (int32_t c = ei & ~63; c < n; c += 64) {
      uint64_t mask = who(c, bx * 4 + (wave & 3), by * 4 + (wave >> 2), 4);
      if (!mask) continue;
      int32_t k = c + __ffsll((unsigned long long)mask) - 1;
      int4 e = rect[k], q = rest[k];
      while (mask) {
        mask &= mask - 1;
        const int32_t next = mask ? c + __ffsll((unsigned long long)mask) - 1 : k;
        const int4 en = rect[next], qn = rest[next];
        const int32_t i = x - e.x, j = y - e.y;
        if (__builtin_amdgcn_readfirstlane(q.x) < 0) {
          const bool ci[2] = {(uint32_t)i < (uint32_t)e.z, (uint32_t)(i + 1) < (uint32_t)e.z};
          const bool cj[2] = {(uint32_t)j < (uint32_t)e.w, (uint32_t)(j + 1) < (uint32_t)e.w};
#pragma unroll
          for (int32_t d = 0; d < 4; ++d) {
            const bool over = ci[d & 1] & cj[d >> 1];
            set[d] = over ? k : set[d];
            drop[d] = over ? 0u : drop[d];
            dig[d] = over ? 0 : dig[d];
          }
        } else {
          // A cell is in the crater if R2 - r2 > 0 (its rectangle, of side s <=
          // 4096, touches the wave's cells, so |a| < 2^14).  That is below 2^24,
          // and times a depth below 2^32; the quotient of it by R2 comes from
          // the lowered reciprocal, so it is right or one too small.
          const int32_t a = 2 * i + 1 - e.z, g = 2 * j + 1 - e.z, R2 = __mul24(e.z, e.z);
          const int32_t aa[2] = {__mul24(a, a), __mul24(a + 2, a + 2)};
          const int32_t gg[2] = {R2 - __mul24(g, g), R2 - __mul24(g + 2, g + 2)};
          const float inv = __int_as_float(q.y);
#pragma unroll
          for (int32_t d = 0; d < 4; ++d) {
            const int32_t in2 = gg[d >> 1] - aa[d & 1];
            dig[d] = max(dig[d], in2);
            const uint32_t num = __umul24((uint32_t)q.x, (uint32_t)max(in2, 0));
            const uint32_t t = (uint32_t)((float)num * inv);
            const uint32_t left = num - __umul24(__umul24(t, (uint32_t)e.z), (uint32_t)e.z);
            drop[d] += t + (left >= (uint32_t)R2 ? 1u : 0u);
          }
        }
        k = next;
        e = en;
        q = qn;
      }
    }
#pragma unroll
    for (int32_t d = 0; d < 4; ++d) {
      const int32_t cx = x + (d & 1), cy = y + (d >> 1);
      uint32_t& col = d & 1 ? p[d >> 1].y : p[d >> 1].x;
      if (cx < m.W && cy < m.H) {
        if (set[d] >= 0) {
          const int4 e = rect[set[d]], q = rest[set[d]];
          const int64_t off = (int64_t)(((uint64_t)(uint32_t)q.w << 32) | (uint32_t)q.z);
          const int64_t size = (int64_t)e.z * e.w, o = off + (int64_t)(cy - e.y) * e.z + (cx - e.x);
          col = (uint32_t)patch[o] | (uint32_t)patch[o + size] << 8 | (uint32_t)patch[o + 2 * size] << 16;
        }
        const uint32_t F = col & 0xFF;
        if (dig[d] > 0) col = F > drop[d] ? F - drop[d] : 0u;   // slab removed: B = T = 0
      }
    }
    if (in) {
      *reinterpret_cast<uint2*>(c0) = p[0];
      *reinterpret_cast<uint2*>(c0 + 8) = p[1];
    }
    // the level-1 node; a cell beside the map counts as empty (fmax 0, smin
    // 255, smax 0), as the zero word there does
    uint32_t v = node_merge(node_merge(cell_to_node(p[0].x), cell_to_node(p[0].y)),
                            node_merge(cell_to_node(p[1].x), cell_to_node(p[1].y)));
    uint64_t mk = cell_mask(p[0].x) | cell_mask(p[0].y) | cell_mask(p[1].x) | cell_mask(p[1].y);
    if (in && m.top > 0) {
      base[tci_tile_index(tab.lv[1], x1, y1)] = v;
      *reinterpret_cast<uint2*>(base + tci_mask_index(tab.mk[1], x1, y1)) =
          make_uint2((uint32_t)mk, (uint32_t)(mk >> 32));
    }
    auto none = [](int32_t, int32_t, int32_t, uint32_t, uint64_t) {};
    fold_levels(tab, m.top, base, 1, 3, x1, y1, in, lane, v, mk, none);
    if (lane == 0) {
      node4[wave] = v;
      lo4[wave] = (uint32_t)mk;
      hi4[wave] = (uint32_t)(mk >> 32);
    }
    __syncthreads();
    if (wave == 0 && m.top > 4) {
      // the 4 x 4 level-4 nodes in the first corner of 8 x 8 lanes
      const bool here = (lane & 7) < 4 && lane < 32;
      const int32_t q = (lane & 3) + ((lane >> 3) & 3) * 4;
      const int32_t x4 = bx * 4 + (lane & 7), y4 = by * 4 + (lane >> 3);
      uint32_t v4 = here ? node4[q] : 255u << 8;
      uint64_t k4 = here ? (uint64_t)lo4[q] | ((uint64_t)hi4[q] << 32) : 0;
      fold_levels(tab, m.top, base, 4, 2, x4, y4, here && x4 * 16 < m.W && y4 * 16 < m.H, lane, v4,
                  k4, none);
    }
    __syncthreads();
  }
}

// Window entry (i, j) of level L: the combine of level-L nodes (i..i+1,
// j..j+1) that exist (level 0: the cells, as nodes).
__device__ inline uint32_t window_entry(const tci_map& m, const uint32_t* base, int32_t L,
                                        int32_t i, int32_t j) {
  const tci_level& l = m.lv[L];
  uint32_t acc = 0u | (255u << 8);  // empty: fmax 0, smin 255, smax 0
  #pragma unroll
  for (int dj = 0; dj < 2; ++dj) {
    #pragma unroll
    for (int di = 0; di < 2; ++di) {
      const int32_t ni = i + di, nj = j + dj;
      if (ni < l.w && nj < l.h) {
        const uint32_t v = base[tci_tile_index(l, ni, nj)];
        acc = node_merge(acc, L == 0 ? cell_to_node(v) : v);
      }
    }
  }
  return acc;
}

__global__ void build_window_kernel(tci_map m, uint32_t* __restrict__ base, int32_t L) {
  const tci_level& w = m.wl[L];
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t total = (int64_t)w.tiles_x * ((w.h + 7) >> 3) * 64;
  if (k >= total) return;
  const int32_t tile = (int32_t)(k >> 6), e = (int32_t)(k & 63);
  const int32_t i = (tile % w.tiles_x) * 8 + (e & 7);
  const int32_t j = (tile / w.tiles_x) * 8 + (e >> 3);
  base[w.off + k] = (i < w.w && j < w.h) ? window_entry(m, base, L, i, j) : 0u;
}

// grid.x = rectangle index: entries x0 - 1 .. x1, y0 - 1 .. y1 (clipped to
// the level) of the level-L rectangle, the entries whose 2 x 2 node block
// meets it.  The first block also clears zero[0 .. nzero) (a captured
// frame's render counters: one launch fewer in the frame).
__global__ void update_window_kernel(tci_map m, uint32_t* __restrict__ base, int32_t L,
                                     const int32_t* __restrict__ rects, uint64_t* zero,
                                     int32_t nzero) {
  if (blockIdx.x == 0 && blockIdx.y == 0 && (int32_t)threadIdx.x < nzero) zero[threadIdx.x] = 0;
  const int32_t* r = rects + 4 * blockIdx.x;
  const tci_level& w = m.wl[L];
  const int32_t x0 = max(r[0] - 1, 0), y0 = max(r[1] - 1, 0);
  const int32_t x1 = min(r[2], w.w - 1), y1 = min(r[3], w.h - 1);
  if (x0 > x1 || y0 > y1) return;
  const int32_t rw = x1 - x0 + 1;
  const int64_t n = (int64_t)rw * (y1 - y0 + 1);
  for (int64_t k = (int64_t)blockIdx.y * blockDim.x + threadIdx.x; k < n;
       k += (int64_t)gridDim.y * blockDim.x) {
    const int32_t i = x0 + (int32_t)(k % rw), j = y0 + (int32_t)(k / rw);
    base[tci_tile_index(w, i, j)] = window_entry(m, base, L, i, j);
  }
}

// One row of a block of level-s nodes: the combine (fmax, smin, smax) of
// nodes x0 <= x < x0 + S of row y, clipped to the level (level 0: the
// cells, as nodes), and with kMask the union of their occupancy masks; an
// empty combine if the row lies outside the block (in false).  The S loads
// are unrolled so that they are in flight together.
template <int S, bool kMask>
__device__ inline uint32_t reduce_row(const tci_map& m, const uint32_t* base, int32_t s,
                                      int32_t x0, int32_t y, bool in, uint64_t& mk) {
  const tci_level& c = m.lv[s];
  const int32_t nx = in ? min(S, c.w - x0) : 0;
  uint32_t v[S];
  uint2 mw[kMask ? S : 1];
#pragma unroll
  for (int dx = 0; dx < S; ++dx) {
    v[dx] = dx < nx ? base[tci_tile_index(c, x0 + dx, y)] : 0u;
    if constexpr (kMask) {
      mw[dx] = ((dx < nx) & (s > 0)) ? *reinterpret_cast<const uint2*>(
                                           base + tci_mask_index(m.mk[s], x0 + dx, y))
                                     : make_uint2(0u, 0u);
    }
  }
  uint32_t acc = 0u | (255u << 8);  // empty: fmax 0, smin 255, smax 0
  mk = 0;
#pragma unroll
  for (int dx = 0; dx < S; ++dx) {
    if (dx >= nx) continue;
    if (s == 0) {
      acc = node_merge(acc, cell_to_node(v[dx]));
      if constexpr (kMask) mk |= cell_mask(v[dx]);
    } else {
      acc = node_merge(acc, v[dx]);
      if constexpr (kMask) mk |= (uint64_t)mw[dx].x | ((uint64_t)mw[dx].y << 32);
    }
  }
  return acc;
}

// The items (nodes, or window entries) x0..x1, y0..y1 of one rectangle job
// of level L = s + k, each the combine of its S x S block of level-s nodes
// (S = 2^k for a node, 2^(k + 1) for a window entry's 2 x 2 node block).
// Both combines are associative, so an item of any level above s is the
// combine over its block of level-s nodes.  S consecutive lanes take one
// item, one block row each, and fold their rows together with cross-lane
// exchanges, so an item waits on one round of loads.
template <int S, bool kNode>
__device__ inline void group_job(const tci_map& m, uint32_t* base, int32_t s, int32_t L,
                                 int32_t x0, int32_t y0, int32_t x1, int32_t y1) {
  const int32_t k = L - s, rw = x1 - x0 + 1;
  const int64_t n = (int64_t)rw * (y1 - y0 + 1) * S;
  const tci_level& src = m.lv[s];
  // (blockDim.x is a multiple of S, so the S lanes of an item are aligned
  // and leave or stay in the loop together)
  for (int64_t q = (int64_t)blockIdx.y * blockDim.x + threadIdx.x; q < n;
       q += (int64_t)gridDim.y * blockDim.x) {
    const int64_t item = q / S;
    const int32_t row = (int32_t)(q % S);
    const int32_t i = x0 + (int32_t)(item % rw), j = y0 + (int32_t)(item / rw);
    const int32_t bx = i << k, by = (j << k) + row;
    uint64_t mk;
    uint32_t acc = reduce_row<S, kNode>(m, base, s, bx, by, by < src.h, mk);
#pragma unroll
    for (int o = 1; o < S; o <<= 1) {
      acc = node_merge(acc, (uint32_t)__shfl_xor((int)acc, o, S));
      if constexpr (kNode) {
        const uint32_t lo = (uint32_t)__shfl_xor((int)(uint32_t)mk, o, S);
        const uint32_t hi = (uint32_t)__shfl_xor((int)(uint32_t)(mk >> 32), o, S);
        mk |= (uint64_t)lo | ((uint64_t)hi << 32);
      }
    }
    if (row == 0) {
      if constexpr (kNode) {
        base[tci_tile_index(m.lv[L], i, j)] = acc;
        store_mask(m, base, L, i, j, mk);
      } else {
        base[tci_tile_index(m.wl[L], i, j)] = acc;
      }
    }
  }
}

// One launch per group of levels after edits, reading only level s, which
// the launch before finished (level 0, the cells, for the first group), and
// for window levels w0 .. s - 1 those levels themselves (finished as well):
// blocks [0, (e - s) nr) recompute the dirty nodes and masks of levels
// s + 1 .. e; the blocks after them the dirty window entries of levels
// w0 .. e - 1, and with wtop of level e too (the top group).  Job j of either
// kind is level (first level) + j / nr, rectangle j % nr; the rectangles of
// level L (x0, y0, x1, y1 inclusive, in level-L node coordinates) are at
// rects + 4 (L stride + r).  Every output depends on level s alone, so no
// job waits for another, and a level's rectangles may overlap (two threads
// then write the same value).  Groups of at most 3 levels keep blocks at
// most 8 x 8 nodes for a node (k <= 3) and 16 x 16 for a window entry.  The
// first block also clears zero[0 .. nzero) (a captured frame's render
// counters, in the top group).
__global__ void update_group_kernel(tci_map m, uint32_t* __restrict__ base, int32_t s,
                                    int32_t e, int32_t w0, int32_t wtop,
                                    const int32_t* __restrict__ rects, int32_t stride,
                                    int32_t nr, uint64_t* zero, int32_t nzero) {
  if (blockIdx.x == 0 && blockIdx.y == 0 && (int32_t)threadIdx.x < nzero) zero[threadIdx.x] = 0;
  const int32_t nl = (e - s) * nr;
  const bool node_job = (int32_t)blockIdx.x < nl;
  const int32_t job = node_job ? (int32_t)blockIdx.x : (int32_t)blockIdx.x - nl;
  const int32_t L = (node_job ? s + 1 : w0) + job / nr;
  const int32_t* r = rects + 4 * ((size_t)L * stride + job % nr);
  const int32_t k = L - s;
  int32_t x0 = r[0], y0 = r[1], x1 = r[2], y1 = r[3];
  if (node_job) {
    if (k == 1) group_job<2, true>(m, base, s, L, x0, y0, x1, y1);
    else if (k == 2) group_job<4, true>(m, base, s, L, x0, y0, x1, y1);
    else group_job<8, true>(m, base, s, L, x0, y0, x1, y1);
    return;
  }
  // entries x0 - 1 .. x1, y0 - 1 .. y1: those whose node block meets the
  // rectangle
  const tci_level& w = m.wl[L];
  x0 = max(x0 - 1, 0);
  y0 = max(y0 - 1, 0);
  x1 = min(x1, w.w - 1);
  y1 = min(y1, w.h - 1);
  if (x0 > x1 || y0 > y1) return;
  if (k <= 0) group_job<2, false>(m, base, L, L, x0, y0, x1, y1);
  else if (k == 1) group_job<4, false>(m, base, s, L, x0, y0, x1, y1);
  else if (k == 2) group_job<8, false>(m, base, s, L, x0, y0, x1, y1);
  else group_job<16, false>(m, base, s, L, x0, y0, x1, y1);
}

// The last launch after edits: all of the levels above s, where they hold
// few nodes (at most kTopNodes together), whatever the edits touched.  Block
// 0 computes them: a wave takes 8 x 8 nodes of level s + 1 from level s,
// which the launch before finished, and folds them into three levels more;
// the top of those is folded again from LDS, three levels to a barrier, up to
// the last; then the window entries of all of them come from LDS.  10 us on
// a 2048 x 16384 map (a barrier per level, with its stores between, took 20:
// the waits for stores and for loads behind branches were most).  The other blocks compute
// the dirty window entries of levels w0 .. s (job j of them level w0 + j / nr,
// rectangle j % nr, as in update_group_kernel), from those levels.  The first
// block also clears zero[0 .. nzero).
constexpr int32_t kTopNodes = 5461;      // 4096 + 1024 + ... + 1
constexpr int32_t kTopThreads = 1024;

__global__ __launch_bounds__(kTopThreads) void update_top_kernel(tci_map m,
                                                                 uint32_t* __restrict__ base,
                                                                 int32_t s, int32_t w0,
                                                                 const int32_t* __restrict__ rects,
                                                                 int32_t stride, int32_t nr,
                                                                 uint64_t* zero, int32_t nzero) {
  __shared__ uint32_t node[kTopNodes];
  __shared__ uint32_t mlo[kTopNodes], mhi[kTopNodes];
  __shared__ int32_t first[TCI_MAX_LEVELS];    // each level's first node in them
  __shared__ levels_t tab;
  if (blockIdx.x > 0) {
    const int32_t job = (int32_t)blockIdx.x - 1, L = w0 + job / nr;
    const int32_t* r = rects + 4 * ((size_t)L * stride + job % nr);
    const tci_level& w = m.wl[L];
    const int32_t x0 = max(r[0] - 1, 0), y0 = max(r[1] - 1, 0);
    const int32_t x1 = min(r[2], w.w - 1), y1 = min(r[3], w.h - 1);
    if (x0 <= x1 && y0 <= y1) group_job<2, false>(m, base, L, L, x0, y0, x1, y1);
    return;
  }
  if (blockIdx.y > 0) return;
  if ((int32_t)threadIdx.x < nzero) zero[threadIdx.x] = 0;
  const int32_t lane = threadIdx.x & 63;
  const int32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  load_levels_lds(m, tab);
  if (threadIdx.x < TCI_MAX_LEVELS) {
    int32_t at = 0;
    for (int32_t L = s + 1; L < (int32_t)threadIdx.x; ++L) at += tab.lv[L].w * tab.lv[L].h;
    first[threadIdx.x] = at;
  }
  __syncthreads();
  auto put = [&](int32_t L, int32_t i, int32_t j, uint32_t v, uint64_t mk) {
    const int32_t q = first[L] + j * tab.lv[L].w + i;
    node[q] = v;
    mlo[q] = (uint32_t)mk;
    mhi[q] = (uint32_t)(mk >> 32);
  };
  for (int32_t L = s + 1;; L += 3) {
    // 8 x 8 blocks of level L: from level s, or from LDS
    const tci_level l = tab.lv[L];
    const int32_t tw = (l.w + 7) >> 3, nt = tw * ((l.h + 7) >> 3);
    for (int32_t t = wave; t < nt; t += kTopThreads / 64) {
      const int32_t x = (t % tw) * 8 + (lane & 7), y = (t / tw) * 8 + (lane >> 3);
      const bool in = x < l.w && y < l.h;
      uint32_t v = 255u << 8;   // (empty: fmax 0, smin 255, smax 0)
      uint64_t mk = 0;
      if (L == s + 1) {
        // a child beside its level stands for its neighbour inside it,
        // which changes no combine: no branch stands between the loads
        const tci_level c = tab.lv[s], cm = tab.mk[s];
        uint32_t cv[4];
        uint2 ck[4];
#pragma unroll
        for (int32_t d = 0; d < 4; ++d) {
          const int32_t i = min(2 * x + (d & 1), c.w - 1), j = min(2 * y + (d >> 1), c.h - 1);
          cv[d] = base[tci_tile_index(c, i, j)];
          ck[d] = *reinterpret_cast<const uint2*>(base + tci_mask_index(cm, i, j));
        }
        if (in) {
          v = node_merge(node_merge(cv[0], cv[1]), node_merge(cv[2], cv[3]));
          mk = (uint64_t)(ck[0].x | ck[1].x | ck[2].x | ck[3].x) |
               ((uint64_t)(ck[0].y | ck[1].y | ck[2].y | ck[3].y) << 32);
          base[tci_tile_index(l, x, y)] = v;
          *reinterpret_cast<uint2*>(base + tci_mask_index(tab.mk[L], x, y)) =
              make_uint2((uint32_t)mk, (uint32_t)(mk >> 32));
          put(L, x, y, v, mk);
        }
      } else if (in) {
        const int32_t q = first[L] + y * l.w + x;
        v = node[q];
        mk = (uint64_t)mlo[q] | ((uint64_t)mhi[q] << 32);
      }
      fold_levels(tab, m.top, base, L, 3, x, y, in, lane, v, mk, put);
    }
    if (L + 3 >= m.top) break;
    __syncthreads();
  }
  __syncthreads();
  for (int32_t L = s + 1; L <= m.top; ++L) {
    const tci_level l = tab.lv[L];
    const int32_t at = first[L];
    const float inv = 1.0f / (float)l.w;
    for (int32_t k = threadIdx.x; k < l.w * l.h; k += kTopThreads) {
      // (k < 2^13: half a unit over is far more than the product's rounding)
      const int32_t j = (int32_t)(((float)k + 0.5f) * inv), i = k - j * l.w;
      const int32_t dx = i + 1 < l.w ? 1 : 0, dy = j + 1 < l.h ? l.w : 0;
      base[tci_tile_index(tab.wl[L], i, j)] =
          node_merge(node_merge(node[at + k], node[at + k + dx]),
                     node_merge(node[at + k + dy], node[at + k + dx + dy]));
    }
  }
}

__global__ void zero_u64_kernel(uint64_t* p, int32_t n) {
  int32_t k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k < n) p[k] = 0;
}

inline int32_t blocks_for(int64_t items, int32_t per, int32_t cap) {
  int64_t b = (items + per - 1) / per;
  if (b < 1) b = 1;
  return (int32_t)(b > cap ? cap : b);
}

}  // namespace

hipError_t tci_launch_repack(const uint8_t* planes, int32_t W, int32_t H,
                             uint32_t* base, tci_level l0, hipStream_t s) {
  int64_t words = (int64_t)l0.tiles_x * ((H + 7) >> 3) * 64;
  int32_t blocks = blocks_for(words, 256, 1 << 30);
  hipLaunchKernelGGL(repack_kernel, dim3(blocks), dim3(256), 0, s, planes, W,
                     H, base, l0);
  return hipGetLastError();
}

hipError_t tci_launch_build_level(const tci_map& m, uint32_t* base, int32_t L,
                                  hipStream_t s) {
  const tci_level& l = m.lv[L];
  int64_t words = (int64_t)l.tiles_x * ((l.h + 7) >> 3) * 64;
  int32_t blocks = blocks_for(words, 256, 1 << 30);
  hipLaunchKernelGGL(build_level_kernel, dim3(blocks), dim3(256), 0, s, m,
                     base, L);
  return hipGetLastError();
}

hipError_t tci_launch_edits(const tci_edit* edits, int32_t n, const int32_t* olap,
                            bool olap_all, const uint8_t* patch, uint32_t* base,
                            tci_level l0, int32_t W, int32_t H,
                            int32_t max_w, int32_t max_h, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  int32_t gy = blocks_for((int64_t)max_w * max_h, 256, 64);
  hipLaunchKernelGGL(edits_kernel, dim3(n, gy), dim3(256), 0, s, edits, n, olap,
                     (int32_t)olap_all, patch, base, l0, W, H);
  return hipGetLastError();
}

hipError_t tci_launch_build_window(const tci_map& m, uint32_t* base, int32_t L,
                                   hipStream_t s) {
  const tci_level& w = m.wl[L];
  const int64_t words = (int64_t)w.tiles_x * ((w.h + 7) >> 3) * 64;
  const int32_t blocks = blocks_for(words, 256, 1 << 30);
  hipLaunchKernelGGL(build_window_kernel, dim3(blocks), dim3(256), 0, s, m, base, L);
  return hipGetLastError();
}

hipError_t tci_launch_update_window(const tci_map& m, uint32_t* base, int32_t L,
                                    const int32_t* rects, int32_t nrect, int32_t max_w,
                                    int32_t max_h, hipStream_t s, uint64_t* zero,
                                    int32_t nzero) {
  if (nrect <= 0) return nzero > 0 ? tci_launch_zero_u64(zero, nzero, s) : hipSuccess;
  const int32_t gy = blocks_for((int64_t)max_w * max_h, 256, 64);
  hipLaunchKernelGGL(update_window_kernel, dim3(nrect, gy), dim3(256), 0, s, m, base, L, rects,
                     zero, nzero);
  return hipGetLastError();
}

bool tci_edit_tiles(int32_t n) { return n <= tci::kTileEdits; }

hipError_t tci_launch_edit_tiles(const tci_map& m, const tci_edit* edits, int32_t n,
                                 const uint8_t* patch, uint32_t* base, int32_t max_w,
                                 int32_t max_h, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  // a rectangle touches at most one block of cells more per axis than it
  // fills; a short list may have rectangles of any size
  const int64_t blocks = (int64_t)((max_w + 63) / 64 + 1) * ((max_h + 63) / 64 + 1);
  const int32_t gy = blocks_for(blocks, 1, n < 64 ? 4096 / n : 64);
  hipLaunchKernelGGL(edit_tiles_kernel, dim3(n, gy), dim3(kTileThreads), 0, s, m, edits, n, patch,
                     base);
  return hipGetLastError();
}

bool tci_update_top(const tci_map& m, int32_t s) {
  int64_t nodes = 0;
  for (int32_t L = s + 1; L <= m.top; ++L) nodes += (int64_t)m.lv[L].w * m.lv[L].h;
  return s >= 1 && s < m.top && nodes <= kTopNodes;
}

hipError_t tci_launch_update_top(const tci_map& m, uint32_t* base, int32_t s, int32_t w0,
                                 const int32_t* rects, int32_t stride, int32_t nr,
                                 int64_t max_lanes, hipStream_t st, uint64_t* zero,
                                 int32_t nzero) {
  if (nr <= 0) return nzero > 0 ? tci_launch_zero_u64(zero, nzero, st) : hipSuccess;
  const int32_t gy = blocks_for(max_lanes, kTopThreads, 64);
  hipLaunchKernelGGL(update_top_kernel, dim3(1 + (s - w0 + 1) * nr, gy), dim3(kTopThreads), 0, st,
                     m, base, s, w0, rects, stride, nr, zero, nzero);
  return hipGetLastError();
}

hipError_t tci_launch_update_group(const tci_map& m, uint32_t* base, int32_t s, int32_t e,
                                   int32_t w0, bool wtop, const int32_t* rects, int32_t stride,
                                   int32_t nr, int64_t max_lanes, hipStream_t st, uint64_t* zero,
                                   int32_t nzero) {
  const int32_t levels = (e - s) + (e - w0) + (wtop ? 1 : 0);
  if (nr <= 0 || levels <= 0) return nzero > 0 ? tci_launch_zero_u64(zero, nzero, st) : hipSuccess;
  const int32_t gy = blocks_for(max_lanes, 256, 64);
  hipLaunchKernelGGL(update_group_kernel, dim3(levels * nr, gy), dim3(256), 0, st, m, base, s, e,
                     w0, (int32_t)wtop, rects, stride, nr, zero, nzero);
  return hipGetLastError();
}

hipError_t tci_launch_zero_u64(uint64_t* p, int32_t n, hipStream_t s) {
  hipLaunchKernelGGL(zero_u64_kernel, dim3((n + 255) / 256), dim3(256), 0, s,
                     p, n);
  return hipGetLastError();
}
