// Ray casting kernels: one thread per pixel over 8x8 pixel packets, the
// split pass for the longest walks, and persistent packet-queue waves.  The
// walk is the exact cell sequence of a 2D digital differential analyser over
// the map, accelerated by the per-layer min/max pyramid (Section 3.1 SOLID and
// RAYMARCH, Section 3.2 skip-to-exit): in single precision with exact decisions
// (tc_skim.h), and in whole numbers throughout (tc_walk.h) in the flat and
// persistent modes and the split pass's short queues.
#include <hip/hip_ext.h>

#include "tc_beam.h"
#include "tc_packet.h"
#include "tc_skim.h"

namespace {

// 8x8 pixel packets (waves) per block of the one-thread-per-pixel kernels.
// Measured on the headline view: two give 1.8 % faster frames than four,
// one 0.4 %.
constexpr int32_t kPackets = 2;

// This lane's index in its wave, from the hardware (two VALU instructions)
// rather than from a register kept live (nor is what is computed from it
// moved ahead of a loop that uses it).
__device__ __forceinline__ int32_t lane_now() {
  int32_t l = (int32_t)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
  asm volatile("" : "+v"(l));
  return l;
}

// One thread per pixel; a wave casts one packet of 64 pixels.
// kOcc: node tests also consult the occupancy masks (render mode 4).
// kVox: nodes above the cells are tested against the voxel occupancy
// pyramid *vx instead (render mode 5, the voxel-accelerated march).
// kCount: the launch counts the nodes and cells its rays read (o.count);
// the production instance keeps no counter through the walk.
// kBoost: the launch may have a priority boost (o.boost; the hierarchical
// mode's walk is instantiated without).
template <bool kFlat, bool kOcc, bool kCount, bool kVox = false, bool kBoost = false>
__device__ __forceinline__ void render_body(
    const tci_map& m, const tci_view* __restrict__ views, int32_t nviews,
    const int64_t* __restrict__ pkt_prefix, const int32_t* __restrict__ rows, int64_t npkt,
    void* out, const tci_render_opts& o, const tci_voxels* vx = nullptr) {
  __shared__ lvl_t lv[TCI_MAX_LEVELS];
  __shared__ uint32_t woff[TCI_MAX_LEVELS];
  __shared__ uint32_t moff[kOcc ? TCI_MAX_LEVELS : 1];
  __shared__ uint4 vrec[kVox ? TCI_MAX_LEVELS : 1];
  if constexpr (kVox) load_voxel_levels(*vx, vrec);
  load_levels_beam(m, lv, woff, kOcc ? moff : nullptr);
  // clear the queue counter the next render of this ring slot will use
  // (its last user finished before this launch)
  if (o.qzero && blockIdx.x == 0 && threadIdx.x == 0) *o.qzero = 0u;
  // XCD-aware order: hand each XCD a contiguous range of packets to share
  // its L2
  const int64_t b = tcp::xcd_block(blockIdx.x, gridDim.x, o.xcd_remap);
  // the packet is the wave's: keep its index, view and tile in scalar
  // registers
  const int32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int64_t p = b * kPackets + wave;
  if (p >= npkt) return;
  const int32_t vi = __builtin_amdgcn_readfirstlane(tcp::find_view(pkt_prefix, nviews, p));
  const tci_view& v = views[vi];
  int32_t tx, ty;
  tcp::packet_tile(v, p - v.pkt_base, o.tile_order, rows, tx, ty);
  tx = __builtin_amdgcn_readfirstlane(tx);
  ty = __builtin_amdgcn_readfirstlane(ty);
  const int32_t pw = v.pw_log2;
  const int32_t px = (tx << pw) + (lane & ((1 << pw) - 1)), py = (ty << (6 - pw)) + (lane >> pw);
  // the packet's common start (all 64 lanes take part)
  float t_start = 0.0f;
  int32_t beam_reads = 0;
  if (!kFlat && o.beam_passes > 0)
    t_start = beam_start(m, lv, woff, v, tx, ty, o.beam_passes, lane, beam_reads);
  if (px >= v.w || py >= v.h) {
    if (kCount && beam_reads) atomicAdd(o.count, (unsigned long long)beam_reads);
    return;
  }
  ray_t r;
  packet_ray(v, tx, ty, lane, r);
  uint32_t word;
  float depth;
  if (r.Dx == 0 && r.Dy == 0) {
    trace_vertical(m, lv, r, word, depth);
    if (kCount && beam_reads) atomicAdd(o.count, (unsigned long long)beam_reads);
  } else if constexpr (kFlat) {
    walk_t s;
    walk_idx_t k;
    walk_origin(r, k);
    walk_at_origin(r, 0, s);
    uint32_t col = 0;
    const int32_t boost = __builtin_amdgcn_readfirstlane(o.boost);
    // the walk runs a loop specialised to the sign of the ray's vertical
    // direction (a packet's rays mostly share it; a wave holding both signs
    // runs the two loops one after the other)
    int32_t st;
    if (r.Dz < 0)
      st = walk_steps<false, 1>(m, lv, r, k, s, 0, kIterCap + 1, col, boost, kCount);
    else
      st = walk_steps<false, 2>(m, lv, r, k, s, 0, kIterCap + 1, col, boost, kCount);
    if (st == kWalking) st = kCapped;   // the whole budget ran out (never expected)
    // the origin is needed again only here: recompute it from the view
    // rather than keep it in registers through the walk (the lane index is
    // read again from the hardware, so no register holds it either)
    packet_ray<false>(v, tx, ty, lane_now(), r);
    finish(r, s, m.W, st, col, word, depth);
    if (kCount) atomicAdd(o.count, (unsigned long long)s.reads);
  } else {
    constexpr int kTest = kOcc ? kMasks : kVox ? kVoxels : kMinMax;
    const int32_t Lmax = clamp_level(o.max_level, m.top);
    const int32_t boost = __builtin_amdgcn_readfirstlane(o.boost);
    // the budget bounds the walk: at most the split budget, or without a
    // split pass kIterCap + 1 steps
    bool split = o.split_budget > 0 && o.qcap > 0;
    skim_ray f;
    skim_init(r, f);
    skim_t s;
    const float t0 = t_start * 0x1p-16f;
    const int32_t L0 = clamp_level(o.start_level, m.top);
    skim_start(f, t0, L0, s);
    // no register holds the ray's integers through the walk: the few places
    // that need them recompute them from the view
    auto ray = [&]() {
      ray_t q;
      packet_ray(v, tx, ty, lane_now(), q);
      return skim_int{(int32_t)q.Ox, (int32_t)q.Oy, (int32_t)q.Oz, q.Dx, q.Dy, q.Dz};
    };
    int32_t reads = beam_reads, st, done = 0;
    for (;;) {
      const int32_t budget = split ? o.split_budget : kIterCap + 1;
      st = skim_walk<kBoost, kTest>(m, lv, f, s, Lmax, budget, done, boost, reads, kCount, ray, word,
                                     depth, skim_test{moff, vx, vrec});
      if (!split) break;
      split = false;
      done = budget;
      // long walks go to the split pass, as many as the queue holds
      const uint64_t want = __ballot(st == kWalking);
      if (!want) break;
      const uint64_t act = __ballot(1);
      const int32_t leader = __ffsll((unsigned long long)act) - 1;
      uint32_t base = 0;
      const int32_t ln = lane_now();
      if (ln == leader) base = atomicAdd(o.qcount, (uint32_t)__popcll(want));
      base = __shfl(base, leader);
      if (st != kWalking) break;
      const uint32_t rank = __builtin_amdgcn_mbcnt_hi(
          (uint32_t)(want >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)want, 0));
      if (base + rank < o.qcap) {
        // the second pass need only split the path from the current cell's
        // line on the dominant axis
        const int32_t from = fabsf(f.dx) >= fabsf(f.dy) ? s.x : s.y;
        const int32_t qp = ((ty << (6 - pw)) + (ln >> pw)) * v.w + (tx << pw) + (ln & ((1 << pw) - 1));
        o.queue[base + rank] = make_uint4((uint32_t)vi, (uint32_t)qp, (uint32_t)from, 0u);
        if (kCount) atomicAdd(o.count, (unsigned long long)reads);
        return;
      }
    }
    if (st != kHitCell) {
      word = st == kMissed ? kMiss : kStuck;   // (kStuck: never expected)
      depth = st == kMissed ? __builtin_inff() : __builtin_nanf("");
    }
    if (kCount) atomicAdd(o.count, (unsigned long long)reads);
  }
  const int32_t ql = lane_now(), qw = v.pw_log2;
  tcp::store_hit(out, v.out_base + (int64_t)((ty << (6 - qw)) + (ql >> qw)) * v.w + (tx << qw) +
                          (ql & ((1 << qw) - 1)),
                 word, depth);
}

// The one-thread-per-pixel kernels, each with and without read counting.
// The hierarchical one runs 8 waves per SIMD (64 VGPRs, which its walk fits
// without spilling vector registers): 64 mixed views and 8 shadow passes take
// 3.56 ms with 8, 3.64 with 7 and 3.90 with 6, twelve 1280x800 views 335, 338
// and 355 us.  A call whose tables come in the kernel's arguments has few
// views and ends with its longest walks, which the 28 scalar registers that
// 8 waves spill make longer (a 320x240 view 34.3 against 33.2 us): 7 there.
template <bool kCount, bool kBoost>
__global__ __launch_bounds__(64 * kPackets) __attribute__((amdgpu_waves_per_eu(8, 8)))
void render_hier_kernel(tci_map m, const tci_view* __restrict__ views, int32_t nviews,
                        const int64_t* __restrict__ pkt_prefix, int64_t npkt, void* out,
                        tci_render_opts o) {
  render_body<false, false, kCount, false, kBoost>(m, views, nviews, pkt_prefix, o.rows, npkt, out,
                                                   o);
}

// The same, with the call's view records, packet prefix and tile-row table
// passed in the kernel's arguments instead of a device table (a small call
// then needs no upload before its render).
template <bool kBoost>
__global__ __launch_bounds__(64 * kPackets) __attribute__((amdgpu_waves_per_eu(7, 8)))
void render_hier_inline_kernel(tci_map m, int32_t nviews, int64_t npkt, void* out,
                               tci_render_opts o, tci_inline t) {
  const char* b = (const char*)t.words;
  render_body<false, false, false, false, kBoost>(m, (const tci_view*)b, nviews,
                                                  (const int64_t*)(b + t.off_prefix),
                                                  (const int32_t*)(b + t.off_rows), npkt, out, o);
}

template <bool kCount>
__global__ __launch_bounds__(64 * kPackets)
void render_flat_kernel(tci_map m, const tci_view* __restrict__ views, int32_t nviews,
                        const int64_t* __restrict__ pkt_prefix, int64_t npkt, void* out,
                        tci_render_opts o) {
  render_body<true, false, kCount>(m, views, nviews, pkt_prefix, o.rows, npkt, out, o);
}

template <bool kCount>
__global__ __launch_bounds__(64 * kPackets)
void render_occ_kernel(tci_map m, const tci_view* __restrict__ views, int32_t nviews,
                       const int64_t* __restrict__ pkt_prefix, int64_t npkt, void* out,
                       tci_render_opts o) {
  render_body<false, true, kCount, false, true>(m, views, nviews, pkt_prefix, o.rows, npkt, out, o);
}

template <bool kCount>
__global__ __launch_bounds__(64 * kPackets)
void render_vox_kernel(tci_map m, const tci_view* __restrict__ views, int32_t nviews,
                       const int64_t* __restrict__ pkt_prefix, int64_t npkt, void* out,
                       tci_render_opts o, tci_voxels vx) {
  render_body<false, false, kCount, true, true>(m, views, nviews, pkt_prefix, o.rows, npkt, out,
                                                o, &vx);
}

// Dominant-axis cell line where the ray leaves the map's columns, or rises
// above every height, estimated in double precision (only the sizes of the
// split segments depend on it).
__device__ __forceinline__ int32_t exit_line(const ray_t& r, const tci_map& m,
                                             int32_t axis) {
  const double S = 65536.0;
  double t = 1e300;
  if (r.Dx > 0) t = fmin(t, ((double)m.W * S - (double)r.Ox) / r.Dx);
  if (r.Dx < 0) t = fmin(t, (double)r.Ox / -(double)r.Dx);
  if (r.Dy > 0) t = fmin(t, ((double)m.H * S - (double)r.Oy) / r.Dy);
  if (r.Dy < 0) t = fmin(t, (double)r.Oy / -(double)r.Dy);
  if (r.Dz > 0) t = fmin(t, (256.0 * S - (double)r.Oz) / r.Dz);
  t = fmax(t, 0.0);
  const double c = axis == 0 ? ((double)r.Ox + t * r.Dx) / S : ((double)r.Oy + t * r.Dy) / S;
  const double lim = axis == 0 ? (double)m.W : (double)m.H;
  return (int32_t)floor(fmin(fmax(c, -1.0), lim));
}

// Rays up to which the split pass gives each ray its whole waves and cells
// (below); with more, each gets some lanes of a wave and the pyramid
// (split_runs).  On full-HD views: 300 rays 8.0 us with whole waves and 12.9
// with a share of lanes, 1,000 to 2,000 rays about 10 either way, 5,000 rays
// 42 and 22, 25,000 rays 370 and 73.
constexpr uint32_t kFlatRays = 1024;

// The split pass for a long queue: G = 8, 16, 32 or 64 lanes of a wave per
// ray.  The remaining path is cut into G runs whose lengths grow with the
// distance (boundary j at (j / G)^3 of the lines: most of these rays end
// soon), lane j walks run j in single precision with the pyramid
// (skim_steps), in chunks of 16 steps; the earliest run with a hit gives the
// record, the runs after it stop.
__device__ __forceinline__ void split_runs(const tci_map& m, const lvl_t* lv,
                                           const tci_view* __restrict__ views, void* out,
                                           const tci_render_opts& o, uint32_t n, int32_t lgG) {
  const int32_t lane = threadIdx.x & 63, G = 1 << lgG;
  const uint32_t per = 64u >> lgG;                       // rays of a wave
  const int32_t j = lane & (G - 1);
  const uint64_t group = (G == 64 ? ~0ull : (1ull << G) - 1) << (lane & ~(G - 1));
  const int32_t Lmax = clamp_level(o.max_level, m.top);
  const uint32_t waves = gridDim.x * 4;
  for (uint32_t w = blockIdx.x * 4 + (threadIdx.x >> 6); w * per < n; w += waves) {
    const uint32_t e = w * per + ((uint32_t)lane >> lgG);
    int32_t st = kSegEnd;
    uint32_t word = kMiss;
    float depth = __builtin_inff();
    const uint4 q = o.queue[min(e, n - 1)];
    const tci_view& v = views[q.x];
    const int32_t px = (int32_t)(q.y % (uint32_t)v.w), py = (int32_t)(q.y / (uint32_t)v.w);
    ray_t r;
    pixel_ray(v, px, py, r);
    skim_ray f;
    skim_init(r, f);
    skim_t s;
    const bool ax = r.ax >= r.ay;
    const bool fwd = (ax ? r.Dx : r.Dy) > 0;
    const int32_t c0 = (int32_t)q.z, dir = fwd ? 1 : -1;
    const int32_t N = max(1, (exit_line(r, m, ax ? 0 : 1) - c0) * dir + 1);
    auto bound = [&](int32_t k) {
      const float u = (float)k / (float)G;
      return c0 + dir * min(N, max(k, (int32_t)((float)N * (u * u * u))));
    };
    const int32_t b0 = bound(j), b1 = j == G - 1 ? (fwd ? INT32_MAX : INT32_MIN) : bound(j + 1);
    auto ray = [&]() {
      return skim_int{(int32_t)r.Ox, (int32_t)r.Oy, (int32_t)r.Oz, r.Dx, r.Dy, r.Dz};
    };
    if (e < n && b0 != b1) {
      st = kWalking;
      // the cell the ray enters line b0 in (the origin's cell, if that is
      // on it or beyond)
      const int32_t oc = ax ? f.cx : f.cy;
      s.L = 0;
      if ((b0 - oc) * dir <= 0) {
        s.x = f.cx;
        s.y = f.cy;
        s.zin = f.oz;
      } else {
        const float t = ((float)(b0 + (fwd ? 0 : 1) - oc) - (ax ? f.fx : f.fy)) * (ax ? f.rx : f.ry);
        const float p = fmaf(t, ax ? f.dy : f.dx, ax ? f.fy : f.fx);
        int32_t c = floor_int(p) + (ax ? f.cy : f.cx);
        if (__builtin_expect(!skim_sure(p), 0)) {
          ray_t r2 = r;
          walk_idx_t k;
          walk_t wk;
          walk_origin(r2, k);
          walk_at_line(r2, k, wk, ax ? 0 : 1, b0);
          c = ax ? wk.nj : wk.ni;
        }
        s.x = ax ? b0 : c;
        s.y = ax ? c : b0;
        s.zin = skim_zin(f, t, r.Dz < 0);
      }
    }
    int32_t reads = 0;
    uint32_t col = 0;
    float ze = 0.0f;
    for (int32_t round = 0;; ++round) {
      const uint64_t hit = __ballot(st == kHitCell) & group;
      if (st == kWalking && hit && lane > __ffsll((unsigned long long)hit) - 1) st = kSegEnd;
      if (!__ballot(st == kWalking)) break;
      if (st != kWalking) continue;
      if (r.Dz < 0)
        st = skim_steps<1, kMinMax, true>(m, lv, f, s, Lmax, 16, col, ze, reads,
                                          o.count != nullptr, skim_test{}, ax, b1);
      else
        st = skim_steps<2, kMinMax, true>(m, lv, f, s, Lmax, 16, col, ze, reads,
                                          o.count != nullptr, skim_test{}, ax, b1);
      if (st == kHitCell && !skim_sure_hit(f, s, col, ze, m.W, ray, word, depth)) {
        const skim_cell c = skim_exact_cell(ray(), s.x, s.y, col, m.W);
        if (c.hit) {
          word = c.word;
          depth = __uint_as_float(c.depth);
        } else {
          skim_step(f, s);
          st = kWalking;
        }
      }
      if (st == kWalking && round > kIterCap) {   // (never expected)
        st = kHitCell;
        word = kStuck;
        depth = __builtin_nanf("");
      }
    }
    if (o.count) atomicAdd(o.count, (unsigned long long)reads);
    const uint64_t hit = __ballot(st == kHitCell) & group;
    const int32_t first = hit ? __ffsll((unsigned long long)hit) - 1 : (lane & ~(G - 1));
    if (e < n && lane == first) tcp::store_hit(out, v.out_base + q.y, word, depth);
  }
}

// Split pass: G = split_waves (1, 2 or 4) waves of one block per queued
// ray, 4 / G rays per block.  The ray's remaining dominant-axis cell lines
// are cut into 64 G runs (the last one open-ended); lane k of the ray's
// wave g walks run 64 g + k from the exact state in which the flat walk
// enters it.  The earliest run with a hit holds the ray's first hit: inside
// a wave the first lane with a hit wins and the lanes after it stop; across
// the ray's waves, each wave with a hit lowers the ray's best run index in
// LDS and leaves its record there, a wave stops once an earlier wave has a
// hit, and after a barrier the ray's first wave writes the winner (or a
// miss).  Blocks stride over the queue; every wave of a block runs the
// same number of rounds, so the barriers are reached by all of them.
__device__ __forceinline__ void split_body(const tci_map& m,
                                           const tci_view* __restrict__ views, void* out,
                                           const tci_render_opts& o) {
  __shared__ lvl_t lv[TCI_MAX_LEVELS];
  __shared__ uint32_t best[4];      // per ray of the block: lowest run with a hit
  __shared__ uint2 cand[4];         // per wave: its first hit's record
  load_levels(m, lv);
  // every lane of a wave walks the same queued ray: the ray, its exit line
  // and its index-form constants are wave-uniform and stay in scalar
  // registers; only the runs' walk states are per lane
  const int32_t lane = threadIdx.x & 63;
  const int32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t G = (uint32_t)o.split_waves, per = 4 / G;
  const uint32_t grp = (uint32_t)wave / G, g = (uint32_t)wave - grp * G;
  const int32_t lgR = 6 + (G == 4 ? 2 : (G == 2 ? 1 : 0));   // 64 G runs per ray
  const uint32_t n = min(*o.qcount, o.qcap);
  if (n > kFlatRays) {
    // as many lanes per ray as about 2^18 in flight allow
    split_runs(m, lv, views, out, o, n, n <= 4096 ? 6 : n <= 8192 ? 5 : n <= 16384 ? 4 : 3);
    return;
  }
  const lvl_t l0 = lv[0];
  for (uint32_t e0 = blockIdx.x * per; e0 < n; e0 += gridDim.x * per) {
    const uint32_t e = e0 + grp;
    if (threadIdx.x < 4) best[threadIdx.x] = 0xFFFFFFFFu;
    __syncthreads();
    uint32_t qv = 0, qp = 0;
    if (e < n) {
      const uint4 q = o.queue[e];
      qv = __builtin_amdgcn_readfirstlane(q.x);
      qp = __builtin_amdgcn_readfirstlane(q.y);
      const tci_view& v = views[qv];
      const int32_t px = (int32_t)(qp % (uint32_t)v.w), py = (int32_t)(qp / (uint32_t)v.w);
      ray_t r;
      pixel_ray(v, px, py, r);
      const int32_t axis = r.ax >= r.ay ? 0 : 1;
      const int32_t c0 = (int32_t)__builtin_amdgcn_readfirstlane(q.z);  // first line still to walk
      const int32_t dir = (axis == 0 ? r.Dx : r.Dy) > 0 ? 1 : -1;
      const int32_t last = __builtin_amdgcn_readfirstlane(exit_line(r, m, axis));
      // lines still to walk (below 2^17), cut into 2^lgR runs
      const int32_t N = max(1, (last - c0) * dir + 1);
      const int32_t j = 64 * (int32_t)g + lane;          // this lane's run
      const int32_t b0 = c0 + dir * ((j * N) >> lgR);
      const int32_t b1 = c0 + dir * (((j + 1) * N) >> lgR);
      const bool open = j == (1 << lgR) - 1;
      int32_t lo = INT32_MIN, hi = INT32_MAX;
      if (!open) {
        if (dir > 0) hi = b1 - 1; else lo = b1 + 1;
      }
      walk_idx_t k;
      walk_origin(r, k);
      k.KX0 = rfl64(k.KX0);
      k.KY0 = rfl64(k.KY0);
      k.ZX0 = rfl64(k.ZX0);
      k.ZY0 = rfl64(k.ZY0);
      k.offx = __builtin_amdgcn_readfirstlane(k.offx);
      k.offy = __builtin_amdgcn_readfirstlane(k.offy);
      r.rx = __builtin_amdgcn_readfirstlane(r.rx);
      r.ry = __builtin_amdgcn_readfirstlane(r.ry);
      walk_t s;
      uint32_t col = 0;
      int32_t st = kSegEnd;
      if (open || b0 != b1) {
        // a run spans a few cell lines close to the terrain, where coarse
        // nodes would only be descended again: it walks the cells
        if (!walk_at_line(r, k, s, axis, b0)) walk_at_origin(r, 0, s);
        st = kWalking;
      }
      // walk in chunks of 10 cells, each chunk's columns loaded together
      // before it is tested; once some run holds a hit, the runs after it
      // cannot matter and stop.  The ray's vertical direction is the
      // wave's, so the loop is specialised to its sign.
      const bool down = r.Dz < 0;
      for (;;) {
        const uint64_t hit_now = __ballot(st == kHitCell || st == kCapped);
        const int32_t first = hit_now ? __ffsll((unsigned long long)hit_now) - 1 : 64;
        if (st == kWalking && (lane > first || *(volatile uint32_t*)&best[grp] < 64 * g))
          st = kSegEnd;
        if (!__ballot(st == kWalking)) break;
        if (st == kWalking) {
          if (down)
            st = walk_flat<1, 10>(m, l0, r, k, s, col, axis, lo, hi, o.count != nullptr);
          else
            st = walk_flat<2, 10>(m, l0, r, k, s, col, axis, lo, hi, o.count != nullptr);
        }
      }
      if (o.count && (open || b0 != b1)) atomicAdd(o.count, (unsigned long long)s.reads);
      const uint64_t hits = __ballot(st == kHitCell || st == kCapped);
      if (hits && lane == __ffsll((unsigned long long)hits) - 1) {
        uint32_t word;
        float depth;
        finish(r, s, m.W, st, col, word, depth);
        cand[wave] = make_uint2(word, __float_as_uint(depth));
        atomicMin(&best[grp], 64 * g + (uint32_t)lane);
      }
    }
    __syncthreads();
    if (e < n && g == 0 && lane == 0) {
      const uint32_t b = best[grp];
      const int64_t idx = views[qv].out_base + qp;
      if (b == 0xFFFFFFFFu) {
        tcp::store_hit(out, idx, kMiss, __builtin_inff());
      } else {
        const uint2 c = cand[grp * G + (b >> 6)];
        tcp::store_hit(out, idx, c.x, __uint_as_float(c.y));
      }
    }
    __syncthreads();
  }
}

// (at most 128 VGPRs: four waves per SIMD)
__global__ __launch_bounds__(256, 4) void split_kernel(tci_map m,
                                                       const tci_view* __restrict__ views,
                                                       void* out, tci_render_opts o) {
  split_body(m, views, out, o);
}
// The split pass of a render whose tables came in the kernel's arguments.
__global__ __launch_bounds__(256, 4) void split_inline_kernel(tci_map m, void* out,
                                                              tci_render_opts o, tci_inline t) {
  split_body(m, (const tci_view*)(const char*)t.words, out, o);
}

// Persistent waves.  Each wave keeps 64 rays in flight; when at least
// refill_min lanes are idle it hands them the next rays of its current
// 8x8 packet and, when that runs out, pops a new packet from the global
// queue counter.  Every wave leaves the loop once the queue is drained and
// all its lanes are idle.
__global__ __launch_bounds__(256) void render_persistent_kernel(
    tci_map m, const tci_view* __restrict__ views, int32_t nviews,
    const int64_t* __restrict__ pkt_prefix, int64_t npkt, void* out,
    uint64_t* __restrict__ counter, tci_render_opts o) {
  __shared__ lvl_t lv[TCI_MAX_LEVELS];
  load_levels(m, lv);
  const int32_t lane = threadIdx.x & 63;
  const int32_t top = m.top;
  const int32_t L0 = clamp_level(o.start_level, top);
  const int32_t Lmax = clamp_level(o.max_level, top);
  const int32_t refill_min = o.refill_min < 1 ? 1 : (o.refill_min > 64 ? 64 : o.refill_min);
  const int32_t iters = o.refill_iters < 1 ? 1 : o.refill_iters;

  int64_t pkt = -1;      // current packet (wave-uniform)
  int32_t taken = 64;    // rays of the current packet already handed out
  bool drained = false;  // queue exhausted (wave-uniform)
  bool active = false;
  ray_t r;
  walk_t s;
  walk_idx_t k;
  int64_t out_idx = 0;
  for (;;) {
    const uint64_t idle = __ballot(!active);
    const int32_t nidle = __popcll(idle);
    if (!drained && (nidle >= refill_min)) {
      const int32_t rank = __builtin_amdgcn_mbcnt_hi(
          (uint32_t)(idle >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)idle, 0));
      const int32_t remaining = 64 - taken;
      int64_t next = -1;
      if (nidle > remaining) {
        uint64_t q = 0;
        if (lane == 0) q = atomicAdd((unsigned long long*)counter, 1ull);
        next = (int64_t)__shfl(q, 0);
        if (next >= npkt) drained = true;
      }
      if (!active) {
        int64_t mypkt;
        int32_t myray;
        if (rank < remaining) { mypkt = pkt; myray = taken + rank; }
        else { mypkt = next; myray = rank - remaining; }
        if (mypkt >= 0 && mypkt < npkt && myray < 64) {
          const int32_t vi = tcp::find_view(pkt_prefix, nviews, mypkt);
          const tci_view& v = views[vi];
          int32_t px, py;
          tcp::packet_pixel(v, mypkt - v.pkt_base, myray, o.tile_order, o.rows, px, py);
          if (px < v.w && py < v.h) {
            pixel_ray(v, px, py, r);
            out_idx = v.out_base + (int64_t)py * v.w + px;
            if (r.Dx == 0 && r.Dy == 0) {
              uint32_t word;
              float depth;
              trace_vertical(m, lv, r, word, depth);
              tcp::store_hit(out, out_idx, word, depth);
            } else {
              walk_origin(r, k);
              walk_at_origin(r, L0, s);
              active = true;
            }
          }
        }
      }
      if (nidle > remaining) {
        if (next >= 0 && next < npkt) { pkt = next; taken = nidle - remaining; }
        else { taken = 64; }
      } else {
        taken += nidle;
      }
    }
    if (drained && __ballot(active) == 0) break;
    int32_t st = kWalking;
    uint32_t col = 0;
    if (active) st = walk_steps<>(m, lv, r, k, s, Lmax, iters, col);
    if (st != kWalking) {
      uint32_t word;
      float depth;
      finish(r, s, m.W, st, col, word, depth);
      tcp::store_hit(out, out_idx, word, depth);
      if (o.count) atomicAdd(o.count, (unsigned long long)s.reads);
      active = false;
    }
  }
}

}  // namespace

hipError_t tci_launch_render(const tci_map& m, const tci_view* views,
                             int32_t nviews, const int64_t* pkt_prefix,
                             int64_t npkt, void* out, int32_t flat,
                             const tci_render_opts& o, hipStream_t s,
                             const tci_voxels* vx) {
  int64_t blocks = (npkt + kPackets - 1) / kPackets;
  if (blocks < 1) return hipSuccess;
  const bool c = o.count != nullptr;
  if (flat == 3) {
    if (!vx) return hipErrorInvalidValue;
    hipLaunchKernelGGL(c ? render_vox_kernel<true> : render_vox_kernel<false>,
                       dim3((uint32_t)blocks), dim3(64 * kPackets), 0, s, m, views, nviews,
                       pkt_prefix, npkt, out, o, *vx);
    return hipGetLastError();
  }
  auto kern = flat == 1 ? (c ? render_flat_kernel<true> : render_flat_kernel<false>)
            : flat == 2 ? (c ? render_occ_kernel<true> : render_occ_kernel<false>)
            : o.boost > 0 ? (c ? render_hier_kernel<true, true> : render_hier_kernel<false, true>)
                          : (c ? render_hier_kernel<true, false> : render_hier_kernel<false, false>);
  hipLaunchKernelGGL(kern, dim3((uint32_t)blocks), dim3(64 * kPackets), 0, s, m, views, nviews,
                     pkt_prefix, npkt, out, o);
  return hipGetLastError();
}

hipError_t tci_launch_split(const tci_map& m, const tci_view* views,
                            const tci_render_opts& o, void* out, int32_t nblocks,
                            hipStream_t s, const tci_inline* t, hipEvent_t ev_start,
                            hipEvent_t ev_stop) {
  if (t && (ev_start || ev_stop))
    hipExtLaunchKernelGGL(split_inline_kernel, dim3(nblocks), dim3(256), 0, s, ev_start, ev_stop,
                          0, m, out, o, *t);
  else if (t)
    hipLaunchKernelGGL(split_inline_kernel, dim3(nblocks), dim3(256), 0, s, m, out, o, *t);
  else
    hipLaunchKernelGGL(split_kernel, dim3(nblocks), dim3(256), 0, s, m, views, out, o);
  return hipGetLastError();
}

hipError_t tci_launch_render_inline(const tci_map& m, int32_t nviews, int64_t npkt, void* out,
                                    const tci_render_opts& o, const tci_inline& t,
                                    hipStream_t s, hipEvent_t ev_start, hipEvent_t ev_stop) {
  const int64_t blocks = (npkt + kPackets - 1) / kPackets;
  if (blocks < 1) return hipSuccess;
  auto kern = o.boost > 0 ? render_hier_inline_kernel<true> : render_hier_inline_kernel<false>;
  if (ev_start || ev_stop)
    hipExtLaunchKernelGGL(kern, dim3((uint32_t)blocks), dim3(64 * kPackets), 0, s, ev_start,
                          ev_stop, 0, m, nviews, npkt, out, o, t);
  else
    hipLaunchKernelGGL(kern, dim3((uint32_t)blocks), dim3(64 * kPackets), 0, s, m, nviews, npkt,
                       out, o, t);
  return hipGetLastError();
}

hipError_t tci_launch_render_persistent(const tci_map& m,
                                        const tci_view* views, int32_t nviews,
                                        const int64_t* pkt_prefix,
                                        int64_t npkt, void* out,
                                        uint64_t* counter, int32_t nblocks,
                                        const tci_render_opts& o,
                                        hipStream_t s) {
  if (npkt < 1) return hipSuccess;
  hipLaunchKernelGGL(render_persistent_kernel, dim3(nblocks), dim3(256), 0, s,
                     m, views, nviews, pkt_prefix, npkt, out, counter, o);
  return hipGetLastError();
}
