// The walk in single precision: the same cells as the exact walk of
// tc_walk.h, at about half its instructions per step.
//
// What bounds it: the issue of vector instructions.  A wave64 instruction
// takes 2 cycles of a SIMD (single-precision multiply, add and multiply-add,
// add, and/xor, right shift, on vector registers only) or 4 (conversions,
// compares, min/max, selects, three-operand and 24-bit integer ones, and any
// with a scalar operand), and a frame's waves keep the SIMDs issuing nearly
// all the time.  Measured, the render of the exact walk before and of this
// one after (MI355X): 64 mixed views and 8 shadow passes 4.69 -> 3.72 ms,
// twelve 1280x800 views 417 -> 346 us, a 1920x1080 horizon view 210 -> 173
// us, when it came in; 4.62 -> 3.35 ms, 398 -> 316 us and 101 -> 74 us (another
// such view) as it stands.
//
// A step of the exact walk spends most of its instructions on 48-bit
// products: two crossing keys, an exit height and three scaled heights to
// compare it with.  Here a crossing's time is one single-precision product,
// t = d / D (d the distance to the face from the ray's origin, D the
// direction's component), and a height one multiply-add, z = Oz + t Dz.
// Nothing is decided on a rounded value:
//   * which cell a step enters is taken from q = O + te D, the position on
//     the other axis at the crossing.  d is a whole number of cells minus
//     the origin's 16-bit fraction (one rounding), 1 / D is the hardware's
//     reciprocal (1 ulp), so te D and q are off by at most 2^-22 of te D
//     plus one rounding.  A q farther than that from a cell line has the
//     right cell (and then the face it leaves through is right as well: were
//     the other face crossed first, q would lie outside the node).  A q
//     closer to a line than 2^-21 |q| + 2^-20 is decided by the exact order
//     of the two crossings (corner_step);
//   * a node is skipped only if the ray's heights over it, widened by a
//     margin, meet no solid.  A height is off by what its time is, 2^-22 of
//     the ray's rise or fall so far, so the margin is 2^-20 of that (and what
//     the origin's own height is off by: skim_margin), as a direction raised
//     and one lowered by that part: a level ray and a ray near its origin are
//     compared almost exactly.  The rounding of the sum needs no margin, as a
//     height not above a whole number doesn't round to one above it.  (With
//     one margin for all heights, 2^-20 (|Oz| + 512), a ray a unit above a
//     plateau left every cell of it open: 1,800 cells took 3,230 us, now
//     24, and a 1280x800 view shaded under a level light 298 us, now 86);
//   * a cell that may hold the hit is tested in whole numbers
//     (skim_exact_cell); a ray it does not stop walks on.
// So hit records are those of the exact walk, bit for bit.
//
// The state is the cell the ray enters its node through and the level: a
// node is the cell's coordinates shifted down, a descent or a climb changes
// the level alone, where the exact walk's node coordinates need the middle
// crossings' keys to descend.
#pragma once

#include "tc_corner.h"
#include "tc_walk.h"

namespace {

// Ray constants, in cells: the origin's cell and its fractions in it, the
// direction's components and their reciprocals (infinite for a zero
// component, which counts as forward: its far face is never reached; the
// fraction is then 1/2 whatever it is, as the ray stays in the origin's cell
// on that axis and a place on the cell's line would leave every crossing
// open: 1023x1023 axis-aligned rays on lines took 183 to 236 us where those
// beside them took 93 to 110, now the same), the origin's height, and the direction's vertical component lowered (dzl) and
// raised (dzh) by the margin (both have its sign).
struct skim_ray {
  int32_t cx, cy;
  float fx, fy, rx, ry, dx, dy, oz, dzl, dzh;
};

struct skim_t {
  int32_t x, y;   // the cell the ray is in on entering the current node
  int32_t L;
  float zin;      // its height there, moved by the margin to the safe side
                  // (up for a descending ray, down for the others)
};

// The margin of a ray's heights, as a part of its rise or fall since the
// origin: four times its times' rounding.  An origin's height from 256 on is
// itself rounded, by up to 2^-24 of it: the ray has come |oz| - 255 by the
// time that its height is of any interest.
__device__ __forceinline__ float skim_margin(float oz) {
  const float a = fabsf(oz);
  return 0x1p-20f + (a >= 256.0f ? a * 0x1p-24f * __builtin_amdgcn_rcpf(a - 255.0f) : 0.0f);
}
// How far a height z (moved to one side) may lie from the true one on the
// other, with the roundings of z and of what is compared.
__device__ __forceinline__ float skim_width(float z, float oz, float margin) {
  return fmaf(fabsf(z - oz), 2.5f * margin, fabsf(z) * 0x1p-22f);
}

__device__ __forceinline__ void skim_init(const ray_t& r, skim_ray& f) {
  f.cx = (int32_t)r.Ox >> 16;
  f.cy = (int32_t)r.Oy >> 16;
  f.fx = r.Dx == 0 ? 0.5f : (float)((uint32_t)r.Ox & 0xFFFF) * 0x1p-16f;
  f.fy = r.Dy == 0 ? 0.5f : (float)((uint32_t)r.Oy & 0xFFFF) * 0x1p-16f;
  f.dx = (float)r.Dx;
  f.dy = (float)r.Dy;
  f.rx = __builtin_amdgcn_rcpf(f.dx);
  f.ry = __builtin_amdgcn_rcpf(f.dy);
  f.oz = (float)(int32_t)r.Oz * 0x1p-16f;
  const float dz = (float)r.Dz, m = fabsf(dz) * skim_margin(f.oz);
  f.dzl = dz - m;
  f.dzh = dz + m;
}

// The ray's height at time t, lowered or raised by the margin: the side on
// which an entry into a node counts (up for a descending ray, down for the
// others), and the other, for an exit.
__device__ __forceinline__ float skim_zin(const skim_ray& f, float t, bool desc) {
  return fmaf(t, desc ? f.dzh : f.dzl, f.oz);
}
__device__ __forceinline__ float skim_zout(const skim_ray& f, float t, bool desc) {
  return fmaf(t, desc ? f.dzl : f.dzh, f.oz);
}

// On which side of every line is q surely?  False if a line is too close.
__device__ __forceinline__ bool skim_sure(float q) {
  const float fr = __builtin_amdgcn_fractf(q);
  return fabsf(fr - 0.5f) < fmaf(fabsf(q), -0x1p-21f, 0.5f - 0x1p-20f);
}
// Start at parameter t (in cells per direction unit; no solid lies on the
// ray before it): in the ray's cell at t, on level 0, or at a slightly
// earlier t if that cell is not sure, or at the origin on level L0.
__device__ __forceinline__ void skim_start(const skim_ray& f, float t, int32_t L0, skim_t& s) {
  float qx = fmaf(t, f.dx, f.fx), qy = fmaf(t, f.dy, f.fy);
  if (!(skim_sure(qx) & skim_sure(qy))) {
    t *= 0.984375f;
    qx = fmaf(t, f.dx, f.fx);
    qy = fmaf(t, f.dy, f.fy);
  }
  const bool at = (t > 0.0f) & skim_sure(qx) & skim_sure(qy);
  t = at ? t : 0.0f;
  s.x = f.cx + (at ? floor_int(qx) : 0);
  s.y = f.cy + (at ? floor_int(qy) : 0);
  s.L = at ? 0 : L0;
  s.zin = skim_zin(f, t, f.dzl < 0.0f);
}

// A ray's integers, as the whole-number steps take them.
struct skim_int {
  int32_t Ox, Oy, Oz, Dx, Dy, Dz;
};

__device__ __forceinline__ ray_t skim_whole(const skim_int& q) {
  ray_t r;
  r.Ox = q.Ox;
  r.Oy = q.Oy;
  r.Oz = q.Oz;
  r.Dx = q.Dx;
  r.Dy = q.Dy;
  r.Dz = q.Dz;
  r.ax = (uint32_t)(r.Dx < 0 ? -r.Dx : r.Dx);
  r.ay = (uint32_t)(r.Dy < 0 ? -r.Dy : r.Dy);
  return r;
}

// Does the ray stop in cell (x, y) of its walk (packed column v)?  Then its
// hit record (word, and depth's bits).  The crossing it enters the cell
// through is the later of the cell's near x and y crossings (y on a tie,
// since x steps first), if any.  Rare, but inlined: as a call it spilled the
// walk's registers around it.
struct skim_cell {
  int32_t hit;
  uint32_t word, depth;
};
__device__ __forceinline__ skim_cell skim_exact_cell(skim_int q, int32_t x, int32_t y,
                                                               uint32_t v, int32_t W) {
  ray_t r = skim_whole(q);
  walk_idx_t k;
  walk_origin(r, k);
  const bool fx = r.Dx > 0, fy = r.Dy > 0, desc = r.Dz < 0;
  // crossing numbers of the far faces; the near ones are one less
  const int32_t ix = far_index(x, 0, fx ? 1 : 0, fx ? 1 : -1, k.offx);
  const int32_t iy = far_index(y, 0, fy ? 1 : 0, fy ? 1 : -1, k.offy);
  const int64_t KXe = add_mul48(k.KX0, (uint32_t)ix, r.ay);
  const int64_t KYe = add_mul48(k.KY0, (uint32_t)iy, r.ax);
  const bool ex = KXe <= KYe;
  const int64_t Ze = add_smul48(ex ? k.ZX0 : k.ZY0, ex ? ix : iy, r.Dz);
  const uint32_t De = ex ? r.ax : r.ay, re = ex ? r.rx : r.ry;
  const bool ny = iy > 0 && (ix <= 0 || KYe - (int64_t)r.ax >= KXe - (int64_t)r.ay);
  int64_t zin = r.Oz >> 16;
  uint32_t din = 1, rin = (r.Oz & 0xFFFF) != 0;
  int32_t entry = kInside;
  if (ix > 0 || iy > 0) {
    zin = add_smul48(ny ? k.ZY0 : k.ZX0, (ny ? iy : ix) - 1, r.Dz);
    din = ny ? r.ay : r.ax;
    rin = ny ? r.ry : r.rx;
    entry = ny ? (fy ? kWmy : kWpy) : (fx ? kWmx : kWpx);
  }
  const int64_t lo = (desc ? Ze : zin) + (int64_t)(desc ? re : rin);
  const uint32_t Dlo = desc ? De : din;
  const int64_t hi = desc ? zin : Ze;
  const uint32_t Dhi = desc ? din : De;
  const uint32_t a = v & 0xFF, b = (v >> 8) & 0xFF, c = (v >> 16) & 0xFF;
  uint32_t word = 0;
  float depth = 0.0f;
  const bool hit = (lo <= hmul(a, Dlo)) | ((lo <= hmul(c, Dlo)) & (hi >= hmul(b, Dhi)));
  if (hit) resolve_hit(r, x, y, entry, zin, din, rin, W, v, word, depth);
  return skim_cell{hit ? 1 : 0, word, __float_as_uint(depth)};
}

// Does voxel column (X, Y) of level k of the voxel occupancy pyramid hold a
// set bit over heights [zl, zh]?  The heights are the ray's range over the
// column, already widened to cover their rounding; both ends are clipped into the pyramid's heights, so a range
// partly or wholly below height 0 tests the first voxel, which every
// in-map column's floor (unbounded below) sets, and a range wholly above
// the top (z > 256) holds nothing.
// Per 8-voxel tile in z, the column's eight bits sit in four words (two
// 64-bit loads): in-tile Morton index x0 y0 z0 x1 y1 | z1 x2 y2 z2 puts
// z0 in the bit and z1, z2 in the word.  `reads` counts the loads.
// `l` is the level's record (load_voxel_levels).
__device__ __forceinline__ bool voxel_range(const uint32_t* base, const uint4 l, int32_t vz_log2,
                                            int32_t X, int32_t Y, float zl, float zh,
                                            int32_t& reads) {
  const float inv = __builtin_amdgcn_ldexpf(1.0f, -vz_log2);
  const int32_t z0 = (int32_t)floorf(fmaxf(zl * inv, 0.0f));
  const int32_t z1 = min((int32_t)floorf(__builtin_amdgcn_fmed3f(zh * inv, 0.0f, 1024.0f)),
                         (int32_t)l.w - 1);
  if (z0 > z1) return false;
  const uint32_t x = (uint32_t)X & 7, y = (uint32_t)Y & 7;
  const uint32_t sh = (x & 1) | ((y & 1) << 1) | ((x & 2) << 2) | ((y & 2) << 3);
  const uint32_t col = l.x + (((uint32_t)(Y >> 3) * l.y + (uint32_t)(X >> 3)) << 4) +
                       (((x >> 2) << 1) | (y & 4));
  for (int32_t tz = z0 >> 3; tz <= (z1 >> 3); ++tz) {
    const uint32_t* t = base + col + (uint32_t)tz * l.z;
    const uint2 a = *reinterpret_cast<const uint2*>(t);
    const uint2 b = *reinterpret_cast<const uint2*>(t + 8);
    reads += 2;
    // two bits of each word: z0 in bits 0 and 4 above sh
    auto two = [&](uint32_t w) {
      const uint32_t c = w >> sh;
      return (c | (c >> 3)) & 3u;
    };
    const uint32_t bits = two(a.x) | (two(a.y) << 2) | (two(b.x) << 4) | (two(b.y) << 6);
    const int32_t lo = max(z0 - tz * 8, 0), hi = min(z1 - tz * 8, 7);
    const uint32_t want = ((2u << hi) - 1u) & ~((1u << lo) - 1u);
    if (bits & want) return true;
  }
  return false;
}

// The voxel levels' records in LDS, one 16-byte read a step: the level's
// offset, tiles per row, words from a tile to the one above, and voxels in
// height.
__device__ __forceinline__ void load_voxel_levels(const tci_voxels& vx, uint4* rec) {
  if (threadIdx.x < TCI_MAX_LEVELS) {
    const tci_vlevel& l = vx.lv[threadIdx.x];
    rec[threadIdx.x] = make_uint4(l.off, (uint32_t)l.tiles_x,
                                  (uint32_t)(l.tiles_y * l.tiles_x) << 4, (uint32_t)l.nz);
  }
  __syncthreads();
}

// Walk until a cell that may hold the hit (kHitCell, its column in col), a
// certain miss (kMissed), or `budget` steps (kWalking).  ze is the height at which the ray leaves that
// cell, moved by the margin to the other side than zin.
// kDir: 1 Dz < 0, 2 otherwise.
// kTest: what a node above the cells is tested against.  kMinMax: its
// min/max pyramid node.  kMasks: a node that only the slab test keeps, also
// its occupancy mask (t.moff: the mask levels' word offsets): the ray's
// heights over the node must meet an occupied band, or the ray passes between
// the node's slabs.  kVoxels: the voxel occupancy pyramid *t.vx (Section
// 3.2) instead: a node of level L >= the voxels' footprint level Lv is voxel
// column (ni, nj) of voxel level L - Lv; nodes below Lv are always descended
// (the leaf voxel's cells are then tested one by one), and a climb from below
// Lv goes straight to Lv, when the step entered a new parent of the leaf
// voxel: its up to three siblings under the same parent are walked on cells.
enum { kMinMax = 0, kMasks = 1, kVoxels = 2 };
struct skim_test {
  const uint32_t* moff;
  const tci_voxels* vx;
  const uint4* vrec;       // the voxel levels' records, in LDS
};
// With kSeg the walk also ends (kSegEnd) once it enters a cell at or beyond
// line seg_end of axis seg_x (x or y), in the ray's direction.
template <int kDir, int kTest = kMinMax, bool kSeg = false>
__device__ __forceinline__ int32_t skim_steps(const tci_map& m, const lvl_t* lv,
                                              const skim_ray& f, skim_t& s, int32_t max_level,
                                              int32_t budget, uint32_t& col, float& ze_out,
                                              int32_t& reads, bool count,
                                              const skim_test& t = skim_test{},
                                              bool seg_x = false, int32_t seg_end = 0) {
  const bool desc = kDir == 1;
  const bool fx = f.dx >= 0.0f, fy = f.dy >= 0.0f;
  const int32_t nx1 = fx ? 1 : 0, ny1 = fy ? 1 : 0;
  const __amdgpu_buffer_rsrc_t buf = map_buffer(m);
  int32_t st = kWalking;
  uint32_t v = 0;
  float ze = 0.0f;
  for (int32_t it = 0; it < budget; ++it) {
    if constexpr (kSeg) {
      const int32_t c = seg_x ? s.x : s.y;
      if ((seg_x ? fx : fy) ? c >= seg_end : c <= seg_end) {
        st = kSegEnd;
        break;
      }
    }
    const int32_t L = s.L;
    const uint4 lq = *reinterpret_cast<const uint4*>(&lv[L]);
    const int32_t w1 = (int32_t)lq.y, h1 = (int32_t)lq.z;
    const int32_t ni = s.x >> L, nj = s.y >> L;
    const bool inmap = ((uint32_t)ni <= (uint32_t)w1) & ((uint32_t)nj <= (uint32_t)h1);
    const bool node = kTest != kVoxels || L == 0;   // tested against its word
    if (count) reads += (inmap & node) ? 1 : 0;
    const uint32_t at = tiled_at((uint32_t)ni, (uint32_t)nj, lq.w);
    v = buffer_word(buf, lq.x + at);
    // times of the crossings through the far faces
    const int32_t gx = (ni + nx1) << L, gy = (nj + ny1) << L;
    const float tx = ((float)(gx - f.cx) - f.fx) * f.rx;
    const float ty = ((float)(gy - f.cy) - f.fy) * f.ry;
    const bool ex = tx <= ty;
    const float te = fminf(tx, ty);
    ze = skim_zout(f, te, desc);
    const float lo = desc ? ze : s.zin, hi = desc ? s.zin : ze;
    bool occ = inmap & ((lo <= (float)(v & 0xFF)) |
                        ((lo <= (float)((v >> 16) & 0xFF)) & (hi >= (float)((v >> 8) & 0xFF))));
    if constexpr (kTest == kMasks) {
      if (occ && L > 0 && !(lo <= (float)(v & 0xFF))) {
        const uint2 mw = *reinterpret_cast<const uint2*>(m.base + t.moff[L] + 2 * at);
        if (count) reads += 2;
        const uint64_t mask = (uint64_t)mw.x | ((uint64_t)mw.y << 32);
        const int32_t kl = min(max((int32_t)floorf(lo * 0.25f), 0), 63);
        const int32_t kh = min(max((int32_t)floorf(hi * 0.25f), 0), 63);
        occ = (mask & (~0ull >> (63 - kh)) & (~0ull << kl)) != 0;
      }
    }
    if constexpr (kTest == kVoxels) {
      if (L > 0) {
        const int32_t Lv = t.vx->v_log2;
        occ = inmap;
        if (inmap && L >= Lv) {
          int32_t vr = 0;
          occ = voxel_range(t.vx->base, t.vrec[L - Lv], t.vx->vz_log2 + L - Lv, ni, nj, lo, hi, vr);
          if (count) reads += vr;
        }
      }
    }
    if (occ) {
      st = L == 0 ? kHitCell : kWalking;
      s.L = L - 1;
    } else {
      float zn = skim_zin(f, te, desc);
      // beside the map and moving away, or above all solid for good
      bool gone = !desc & (zn > 255.0f);
      if (!inmap) {
        gone |= ((ni < 0) & (f.dx <= 0.0f)) | ((ni > w1) & fx) |
                ((nj < 0) & (f.dy <= 0.0f)) | ((nj > h1) & fy);
      }
      st = gone ? kMissed : kWalking;
      const float q = fmaf(te, ex ? f.dy : f.dx, ex ? f.fy : f.fx);
      const int32_t o = floor_int(q) + (ex ? f.cy : f.cx);
      int32_t x = ex ? gx + nx1 - 1 : o, y = ex ? o : gy + ny1 - 1;
      if (__builtin_expect(!skim_sure(q) & !gone, 0)) {
        const skim_next n = corner_step(f.cx, f.cy, f.fx, f.fy, f.dx, f.dy, gx, gy, ex, q);
        x = n.x;
        y = n.y;
        zn = skim_zin(f, n.ex ? tx : ty, desc);
      }
      // go up one level when the step entered a new parent node
      int32_t up = 1;
      if constexpr (kTest == kVoxels) up = max(min(t.vx->v_log2, max_level) - L, 1);
      // (over voxels only with a new parent of that: their columns are mostly
      // occupied near the terrain, and a climb that must descend again costs
      // two steps; two cave views 164 -> 143, 256 -> 237, 253 -> 228 us, where
      // the same rule made the pyramid's 64 mixed views 4 % slower)
      const int32_t later = kTest == kVoxels ? 1 : 0;
      s.L = L + (((L < max_level) & (((uint32_t)((s.x ^ x) | (s.y ^ y)) >> (L + up - 1 + later)) > 1u)) ? up : 0);
      s.x = x;
      s.y = y;
      s.zin = zn;
    }
    // (the one place a lane leaves a step through, against a return in each
    // branch: 64 mixed views and 8 shadow passes 3.55 -> 3.42 ms, twelve 1280x800
    // views 336 -> 327 us, a 320x240 view 33.6 -> 31.5, a 1280x800 view shaded
    // 121.5 -> 115.2, two cave views 142 -> 131; a headline wave issues 601
    // scalar instructions then, 714 before, and 12 vector ones more)
    if (st != kWalking) break;
  }
  if (st == kHitCell) s.L = 0;
  col = v;
  ze_out = ze;
  return st;
}

// The hit record of a candidate cell (skim_steps), if the single-precision
// values alone settle it: the ray's heights at the cell's entry and exit lie
// farther than their width from every height they are compared with, and
// where the hit is on the face it enters through, the two near crossings'
// times differ by more than their rounding.  The record is formed from the
// ray's integers as resolve_hit forms it: the distance to the hit's plane,
// in whole units, over the direction's component.  False: not settled (the
// cell is then tested in whole numbers).  ray() gives the ray again.
template <class RayFn>
__device__ __forceinline__ bool skim_sure_hit(const skim_ray& fr, const skim_t& s, uint32_t v,
                                              float ze, int32_t W, RayFn ray, uint32_t& word,
                                              float& depth) {
  // (what depends on the ray alone is not to be computed ahead of the walk
  // and held through it)
  skim_ray f = fr;
  asm volatile("" : "+v"(f.dx), "+v"(f.dy), "+v"(f.dzl), "+v"(f.oz));
  const bool down = f.dzl < 0.0f;
  const float mg = skim_margin(f.oz), wi = skim_width(s.zin, f.oz, mg), we = skim_width(ze, f.oz, mg);
  const float zil = s.zin - wi, zih = s.zin + wi, zel = ze - we, zeh = ze + we;
  const float F = (float)(v & 0xFF), B = (float)((v >> 8) & 0xFF), T = (float)((v >> 16) & 0xFF);
  const bool two = (v & 0xFF00) != 0;
  const bool in_floor = zih <= F;
  const bool in_slab = two & (zil >= B) & (zih <= T);
  const bool below = zih < B, above = two & (zil > T);
  const bool out = (zil > F) & (!two | below | above);
  const bool plane = out & (down ? zeh <= (above ? T : F) : (two & below & (zel >= B)));
  const bool entry = in_floor | in_slab;
  // the face entered through: the later of the near crossings
  const bool fx = f.dx >= 0.0f, fy = f.dy >= 0.0f;
  const int32_t X = s.x + (fx ? 0 : 1), Y = s.y + (fy ? 0 : 1);
  const float tx = ((float)(X - f.cx) - f.fx) * f.rx;
  const float ty = ((float)(Y - f.cy) - f.fy) * f.ry;
  const bool ax = tx > ty;
  const bool axis_sure = fabsf(tx - ty) > fmaxf(tx, ty) * 0x1p-20f & fmaxf(tx, ty) > 0.0f;
  if (!(plane | (entry & axis_sure))) return false;
  const int32_t h = down ? (int32_t)(above ? (v >> 16) & 0xFF : v & 0xFF)
                         : (int32_t)((v >> 8) & 0xFF);
  // origin (cells and fraction, or the height) and plane of the hit's axis
  const int32_t oc = ax ? f.cx : f.cy;
  const float of = ax ? f.fx : f.fy;
  const skim_int q = ray();
  const int32_t O = entry ? (int32_t)((uint32_t)oc << 16) + (int32_t)(of * 65536.0f) : q.Oz;
  const int32_t P = entry ? (ax ? X : Y) : h;
  const float dz = (float)q.Dz, D = entry ? (ax ? f.dx : f.dy) : dz;
  const int32_t face = entry ? (ax ? (fx ? kWmx : kWpx) : (fy ? kWmy : kWpy))
                             : (down ? kTop : kUnder);
  const bool slab = entry ? !in_floor : (above | !down);
  word = (uint32_t)(s.y * W + s.x) | ((uint32_t)face << 27) | (slab ? 1u << 30 : 0u);
  depth = hit_depth(fma((double)P, 65536.0, -(double)O), fabs((double)D), f.dx, f.dy, dz);
  return true;
}

// The step out of the current cell (level 0).
__device__ __forceinline__ void skim_step(const skim_ray& f, skim_t& s) {
  const bool fx = f.dx >= 0.0f, fy = f.dy >= 0.0f;
  const int32_t gx = s.x + (fx ? 1 : 0), gy = s.y + (fy ? 1 : 0);
  const float tx = ((float)(gx - f.cx) - f.fx) * f.rx, ty = ((float)(gy - f.cy) - f.fy) * f.ry;
  const bool ex = tx <= ty;
  const float q = fmaf(fminf(tx, ty), ex ? f.dy : f.dx, ex ? f.fy : f.fx);
  const int32_t o = floor_int(q) + (ex ? f.cy : f.cx);
  skim_next n{ex ? gx + (fx ? 0 : -1) : o, ex ? o : gy + (fy ? 0 : -1), ex ? 1 : 0};
  if (__builtin_expect(!skim_sure(q), 0))
    n = corner_step(f.cx, f.cy, f.fx, f.fy, f.dx, f.dy, gx, gy, ex, q);
  s.x = n.x;
  s.y = n.y;
  s.zin = skim_zin(f, n.ex ? tx : ty, f.dzl < 0.0f);
}

// The whole walk: its state (kHitCell with the record in word and depth,
// kMissed, or kWalking when the budget ran out).  The steps a ray took before it
// passed a cell within the margin of its solid are not counted: a split pass's
// budget is halved there, until nothing is left of it.  With kBoost a wave
// raises its issue priority after boost, 2 boost and 4 boost steps of its walk,
// of which it has taken `done` before (an instance of its own: the stops cost
// the walk 1.4 %).
template <bool kBoost, int kTest, class RayFn>
__device__ __forceinline__ int32_t skim_walk(const tci_map& m, const lvl_t* lv,
                                             const skim_ray& f, skim_t& s, int32_t max_level,
                                             int32_t budget, int32_t done, int32_t boost,
                                             int32_t& reads, bool count, RayFn ray,
                                             uint32_t& word, float& depth, const skim_test& t) {
  uint32_t col = 0;
  float ze = 0.0f;
  const bool down = f.dzl < 0.0f;
  int32_t used = done;
  int32_t end = done + budget;
  for (;;) {
    int32_t stop = end - used, st;
    if (kBoost && used < 4 * boost)
      stop = min(stop, (used < boost ? boost : used < 2 * boost ? 2 * boost : 4 * boost) - used);
    if (down)
      st = skim_steps<1, kTest>(m, lv, f, s, max_level, stop, col, ze, reads, count, t);
    else
      st = skim_steps<2, kTest>(m, lv, f, s, max_level, stop, col, ze, reads, count, t);
    if (kBoost && st == kWalking) {
      used += stop;
      if (used == boost) __builtin_amdgcn_s_setprio(1);
      else if (used == 2 * boost) __builtin_amdgcn_s_setprio(2);
      else if (used == 4 * boost) __builtin_amdgcn_s_setprio(3);
      if (used < end) continue;
    }
    if (st != kHitCell) return st;
    if (__builtin_expect(skim_sure_hit(f, s, col, ze, m.W, ray, word, depth), 1)) return kHitCell;
    const skim_cell c = skim_exact_cell(ray(), s.x, s.y, col, m.W);
    if (c.hit) {
      word = c.word;
      depth = __uint_as_float(c.depth);
      return kHitCell;
    }
    // within the margin of solid, but not in it: on to the next cell
    skim_step(f, s);
    if (budget <= kIterCap) {
      end -= (end - used + 1) >> 1;
      if (end == used) return kWalking;
    }
  }
}

// Does the ray (its integers in q) meet any solid?  Its origin usually lies
// a unit off a surface, so in the origin's cell the entry is compared in whole
// numbers and the exit alone with the margin; the walk proper begins in the
// next cell.  A walk that uses up its bound
// (never expected) counts as a hit.
template <int kDir, bool kCount>
__device__ __forceinline__ bool skim_blocked(const tci_map& m, const lvl_t* lv, const skim_int& q,
                                             int32_t max_level, int32_t& reads) {
  constexpr bool desc = kDir == 1;
  skim_ray f;
  skim_t s;
  skim_init(skim_whole(q), f);
  const float mg = skim_margin(f.oz);
  {
    const lvl_t l = lv[0];
    const int32_t x = f.cx, y = f.cy;
    const bool fx = f.dx >= 0.0f, fy = f.dy >= 0.0f;
    const bool inmap = ((uint32_t)x <= (uint32_t)l.w1) & ((uint32_t)y <= (uint32_t)l.h1);
    const uint32_t ci = (uint32_t)clamp0(x, l.w1), cj = (uint32_t)clamp0(y, l.h1);
    const uint32_t v = map_word(m.base, l.off + ((umul24(cj >> 3, (uint32_t)l.tiles_x) + (ci >> 3)) << 6) +
                                            ((cj & 7) << 3) + (ci & 7));
    if (kCount) reads += inmap ? 1 : 0;
    const float tx = ((fx ? 1.0f : 0.0f) - f.fx) * f.rx, ty = ((fy ? 1.0f : 0.0f) - f.fy) * f.ry;
    const bool ex = tx <= ty;
    const float te = fminf(tx, ty);
    const float zl = fmaf(te, f.dzl, f.oz), zh = fmaf(te, f.dzh, f.oz);
    const float r = fabsf(zl) * 0x1p-22f;   // (what the two may be rounded by)
    const float F = (float)(v & 0xFF), B = (float)((v >> 8) & 0xFF), T = (float)((v >> 16) & 0xFF);
    const int32_t F16 = (int32_t)(v & 0xFF) << 16, B16 = (int32_t)(v & 0xFF00) << 8,
                  T16 = (int32_t)(v & 0xFF0000);
    const bool two = (v & 0xFF00) != 0;
    const bool in = (q.Oz <= F16) | (two & (q.Oz >= B16) & (q.Oz <= T16));
    bool maybe, sure;
    if (desc) {
      const bool over = two & (q.Oz > T16);
      maybe = (zl <= F) | (over & (zl <= T));
      sure = (zh + r <= F) | (over & (zh + r <= T));
    } else {
      const bool under = two & (q.Oz < B16);
      maybe = under & (zh >= B);
      sure = under & (zl - r >= B);
    }
    if (inmap & (in | sure)) return true;
    if (__builtin_expect(inmap & maybe, 0))
      if (skim_exact_cell(q, x, y, v, m.W).hit) return true;
    const bool away = ((x < 0) & (f.dx <= 0.0f)) | ((x > l.w1) & fx) |
                      ((y < 0) & (f.dy <= 0.0f)) | ((y > l.h1) & fy);
    if (away) return false;
    s.L = 0;
    s.x = x;
    s.y = y;
    skim_step(f, s);
  }
  for (;;) {
    uint32_t v = 0;
    float ze = 0.0f;
    const int32_t st = skim_steps<kDir>(m, lv, f, s, max_level, kIterCap + 1, v, ze, reads, kCount);
    if (st != kHitCell) return st != kMissed;
    // surely in solid, also with the heights moved the other way; or else
    // tested in whole numbers
    const float zl = desc ? ze : s.zin, zh = desc ? s.zin : ze;
    const float lo = zl + skim_width(zl, f.oz, mg), hi = zh - skim_width(zh, f.oz, mg);
    const float F = (float)(v & 0xFF), B = (float)((v >> 8) & 0xFF), T = (float)((v >> 16) & 0xFF);
    if (__builtin_expect((lo <= F) | (((v & 0xFF00) != 0) & (lo <= T) & (hi >= B)), 1)) return true;
    if (skim_exact_cell(q, s.x, s.y, v, m.W).hit) return true;
    skim_step(f, s);
  }
}

}  // namespace
