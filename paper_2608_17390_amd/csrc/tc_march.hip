// Sampled height-field march: the paper's RAYMARCH (Section 3.1) as a
// render mode beside the exact walk, on the same tiled columns.
//
// Per pixel: the segment from the eye runs to the far limit (a distance
// along the ray) or to the plane z = 0, whichever comes first; `steps`
// interior points spaced uniformly over it are tested in order with the
// SOLID predicate (z <= F, or B <= z <= T on a column with an upper slab);
// the first solid sample and the sample before it (or the eye) bracket the
// crossing, and `bisect` halvings keep the solid end.  The segment's end
// point is never tested: a ray that meets no solid sample is a miss.
//
// Every quantity is an IEEE single computed one operation at a time (this
// file is compiled without floating-point contraction; division and square
// root are correctly rounded):
//   o = (float)O * 2^-16, d = (float)D, len = sqrt((dx*dx + dy*dy) + dz*dz)
//   t_end = far / len, and min(t_end, -oz / dz) when dz < 0
//   dt = t_end / (steps + 1), sample i at t = (float)i * dt
//   point(t) = o + t * d per component, midpoint (ta + tb) * 0.5
//   depth = tb * len
// so the solid/empty decision of every sample, and with it the hit word and
// depth, is reproducible bit for bit by any IEEE single implementation.
//
// MI355X mapping: one thread per pixel in 8x8 packets, as the exact walk.
// What bounds it is the issue of vector instructions (a sample takes some 25
// and a gather), and most samples of a view are in the air above anything
// near: the packet's rays first find their common start with the packet beam
// (tc_beam.h), and the samples before it are skipped.  A sample lies within
// 2^-7 of a cell of its ray (coordinates below 2^16 in single precision),
// the beam clears a sixteenth of a cell around it, so no skipped sample is
// solid.  Sample positions do not depend on earlier loads: each lane issues
// the column loads of kGroup samples before testing any of them (the test
// runs in order, so the first solid sample wins exactly as in a one-by-one
// march); the tiled layout keeps a packet's samples in few 256-byte tiles.
// Twelve 1280x800 views, 128 samples: 560 us without the start, 320 with it
// and groups of 8, 300 with 4 (288 against 283 for 2 and 4 on the final
// loads), 270 with 32-bit load offsets and the packet's scalar ray set-up,
// 250 with the cell as an integer (its in-map test is two unsigned compares
// for four of floats) and loads through the map's buffer (no clamps).
// Skipping runs of samples by a box test per ray as well was slower (316-332
// against 300): the lanes of a wave part over which of them to test.
// Two exits skip samples that cannot be solid: a point left of, right of,
// before or behind the map while the ray moves away from it, and a point
// above height 255 while the ray does not descend -- rounding is monotone,
// so every later sample stays there.
// The read counting instance tests every sample: its count is the method's.
#include "tc_beam.h"
#include "tc_packet.h"

namespace {

// 8x8 pixel packets (waves) per block: two (the same march time as four, as the render kernels use)
constexpr int32_t kPackets = 2;

constexpr int32_t kGroup = 4;    // samples tested together
// Passes of the packet beam, by the march's samples: one costs about as much
// as three or four samples, and the first finds most of the way.  Eight
// 1280x800 views at eye level with 8, 16, 32, 64 and 128 samples take 107, 121,
// 144, 189 and 270 us without it, 129, 144, 164, 200 and 262 with one pass, 138,
// 151, 165, 192 and 240 with two, 152, 162, 174, 193 and 222 with six; a view
// from above 34, 40, 52, 75 and 119, 34, 36, 40, 46 and 59, 35, 35, 38, 41 and 49,
// and 37, 38, 39, 43 and 49.
// The last is an instance of its own, kLong: with a number of passes that is
// known its passes are unrolled, which is 1 to 2 % of its time.
constexpr int32_t kLongSteps = 96, kBeam = 6;
__device__ __forceinline__ int32_t beam_passes(int32_t steps) {
  return steps < 12 ? 0 : steps < 32 ? 1 : 2;
}

// SOLID on a packed column word (F | B << 8 | T << 16): 0 empty, 1 floor,
// 2 slab.
__device__ __forceinline__ int32_t solid(uint32_t col, float z) {
  const uint32_t F = col & 0xFFu, B = (col >> 8) & 0xFFu, T = (col >> 16) & 0xFFu;
  if (z <= (float)F) return 1;
  if (B > 0 && z >= (float)B && z <= (float)T) return 2;
  return 0;
}

struct fray {
  float ox, oy, oz, dx, dy, dz;
};

__device__ __forceinline__ void at(const fray& r, float t, float& x, float& y, float& z) {
  x = r.ox + t * r.dx;
  y = r.oy + t * r.dy;
  z = r.oz + t * r.dz;
}

template <bool kCount, bool kLong>
__global__ __launch_bounds__(64 * kPackets) void march_kernel(
    tci_map m, const tci_view* __restrict__ views, int32_t nviews,
    const int64_t* __restrict__ pkt_prefix, int64_t npkt, void* out,
    tci_render_opts o) {
  __shared__ lvl_t lv[TCI_MAX_LEVELS];
  __shared__ uint32_t woff[TCI_MAX_LEVELS];
  load_levels_beam(m, lv, woff, nullptr);
  const int64_t b = tcp::xcd_block(blockIdx.x, gridDim.x, o.xcd_remap);
  const int32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int64_t p = b * kPackets + wave;
  if (p >= npkt) return;
  const int32_t vi = __builtin_amdgcn_readfirstlane(tcp::find_view(pkt_prefix, nviews, p));
  const tci_view& v = views[vi];
  int32_t tx, ty;
  tcp::packet_tile(v, p - v.pkt_base, o.tile_order, o.rows, tx, ty);
  tx = __builtin_amdgcn_readfirstlane(tx);
  ty = __builtin_amdgcn_readfirstlane(ty);
  // the packet's common start (all 64 lanes take part)
  float t_start = 0.0f;
  int32_t unused = 0;
  if constexpr (!kCount && kLong) {
    t_start = beam_start<kBeam>(m, lv, woff, v, tx, ty, kBeam, lane, unused) * 0x1p-16f;
  } else if constexpr (!kCount) {
    const int32_t passes = beam_passes(o.march_steps);
    if (passes > 0) t_start = beam_start(m, lv, woff, v, tx, ty, passes, lane, unused) * 0x1p-16f;
  }
  const int32_t pw = v.pw_log2;
  const int32_t px = (tx << pw) + (lane & ((1 << pw) - 1)), py = (ty << (6 - pw)) + (lane >> pw);
  if (px >= v.w || py >= v.h) return;

  ray_t q;
  packet_ray(v, tx, ty, lane, q);
  uint32_t word = kMiss;
  float depth = __builtin_inff();
  int32_t reads = 0;
  const int32_t steps = o.march_steps;
  if ((q.Dx | q.Dy | q.Dz) != 0) {
    fray r;
    r.ox = (float)(int32_t)q.Ox * 0x1p-16f;
    r.oy = (float)(int32_t)q.Oy * 0x1p-16f;
    r.oz = (float)(int32_t)q.Oz * 0x1p-16f;
    r.dx = (float)q.Dx;
    r.dy = (float)q.Dy;
    r.dz = (float)q.Dz;
    const float len = sqrtf((r.dx * r.dx + r.dy * r.dy) + r.dz * r.dz);
    float t_end = o.march_far / len;
    if (r.dz < 0.0f) {
      const float t0 = -r.oz / r.dz;
      if (t0 < t_end) t_end = t0;
    }
    if (t_end > 0.0f) {
      const float dt = t_end / (float)(steps + 1);
      const float Wf = (float)m.W, Hf = (float)m.H;
      const tci_level l0 = m.lv[0];
      const __amdgpu_buffer_rsrc_t buf = map_buffer(m);
      // the cell under a point (a conversion saturates), whether it is in the
      // map, and its column (anything beside the map: the buffer's range
      // keeps the load valid)
      auto in_map = [&](int32_t i, int32_t j) {
        return ((uint32_t)i < (uint32_t)m.W) & ((uint32_t)j < (uint32_t)m.H);
      };
      auto cell_at = [&](int32_t i, int32_t j) {
        return buffer_word(buf, l0.off + tiled_at((uint32_t)i, (uint32_t)j, (uint32_t)l0.tiles_x));
      };
      // no later sample can be solid
      auto gone = [&](float x, float y, float z) {
        return ((x < 0.0f) & (r.dx <= 0.0f)) | ((x >= Wf) & (r.dx >= 0.0f)) |
               ((y < 0.0f) & (r.dy <= 0.0f)) | ((y >= Hf) & (r.dy >= 0.0f)) |
               ((z > 255.0f) & (r.dz >= 0.0f));
      };
      int32_t hit_i = 0;
      // no ray of the packet meets solid up to t_start, nor within a
      // sixteenth of a cell of it (a sample is off its ray by less): the
      // samples before it are empty (the estimate of their number is off by
      // less than the one sample it stays behind)
      int32_t i0 = 1;
      if (!kCount)
        i0 = max(1, (int32_t)fminf(t_start * __builtin_amdgcn_rcpf(dt), (float)steps + 1.0f));
      while (i0 <= steps) {
        float x = 0.0f, y = 0.0f, z = 0.0f;
        uint32_t col[kGroup];
        float zs[kGroup];
        bool in[kGroup];
#pragma unroll
        for (int32_t u = 0; u < kGroup; ++u) {
          const float t = (float)(i0 + u) * dt;
          at(r, t, x, y, z);
          zs[u] = z;
          const int32_t i = floor_int(x), j = floor_int(y);
          in[u] = (i0 + u <= steps) & in_map(i, j);
          col[u] = cell_at(i, j);
        }
        int32_t found = 0, tested = 0;
#pragma unroll
        for (int32_t u = 0; u < kGroup; ++u) {
          if (!found) {
            tested += in[u];
            if (in[u] && solid(col[u], zs[u])) found = i0 + u;
          }
        }
        if (kCount) reads += tested;
        if (found) {
          hit_i = found;
          break;
        }
        i0 += kGroup;
        // (x, y, z) is the group's last sample
        if (gone(x, y, z)) break;
      }
      if (hit_i) {
        float ta = (float)(hit_i - 1) * dt, tb = (float)hit_i * dt;
        float x, y, z;
        at(r, tb, x, y, z);
        int32_t cx = floor_int(x), cy = floor_int(y);
        int32_t layer = solid(cell_at(cx, cy), z);
        for (int32_t k = 0; k < o.march_bisect; ++k) {
          const float tm = (ta + tb) * 0.5f;
          at(r, tm, x, y, z);
          const int32_t i = floor_int(x), j = floor_int(y);
          const bool inm = in_map(i, j);
          if (kCount) reads += inm;
          const uint32_t c = cell_at(i, j);
          const int32_t s = inm ? solid(c, z) : 0;
          if (s) {
            tb = tm;
            cx = i;
            cy = j;
            layer = s;
          } else {
            ta = tm;
          }
        }
        word = (uint32_t)(cy * m.W + cx) | ((uint32_t)(layer == 2) << 30);
        depth = tb * len;
      }
    }
  }
  if (kCount) atomicAdd(o.count, (unsigned long long)reads);
  tcp::store_hit(out, v.out_base + (int64_t)py * v.w + px, word, depth);
}

}  // namespace

hipError_t tci_launch_march(const tci_map& m, const tci_view* views,
                            int32_t nviews, const int64_t* pkt_prefix,
                            int64_t npkt, void* out, const tci_render_opts& o,
                            hipStream_t s) {
  int64_t blocks = (npkt + kPackets - 1) / kPackets;
  if (blocks < 1) return hipSuccess;
  auto kern = o.count                         ? march_kernel<true, true>
              : o.march_steps >= kLongSteps   ? march_kernel<false, true>
                                              : march_kernel<false, false>;
  hipLaunchKernelGGL(kern, dim3((uint32_t)blocks), dim3(64 * kPackets), 0, s, m,
                     views, nviews, pkt_prefix, npkt, out, o);
  return hipGetLastError();
}
