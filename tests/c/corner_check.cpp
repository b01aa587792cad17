// The single-precision step of tc_skim.h and its exact resolution at cell
// lines (tc_corner.h) against a walk from cell to cell in 128-bit whole
// numbers, over directions of small ratios and next to them, origins on
// lines, in corners and anywhere, near and far, and nodes of every size; the
// reciprocal off by up to one unit in the last place either way.
//
// Usage: corner_check [rays] [seed]
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>

#define __device__
#define __forceinline__ inline
#include "tc_corner.h"

namespace {

typedef __int128 wide;
uint64_t g_s;
uint64_t rnd() {
  uint64_t z = (g_s += 0x9E3779B97F4A7C15ull);
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}
int64_t in(int64_t lo, int64_t hi) { return lo + (int64_t)(rnd() % (uint64_t)(hi - lo + 1)); }

struct Walk {
  int64_t O[2], D[2], n[2];   // n: units to the next line of each axis
  int64_t c[2];
  void start() {
    for (int a = 0; a < 2; ++a) {
      c[a] = O[a] >> 16;
      const int64_t f = O[a] & 0xFFFF;
      n[a] = D[a] > 0 ? 65536 - f : f;
    }
  }
  int step() {   // the axis of the next crossing, taken
    const int64_t ax = std::llabs(D[0]), ay = std::llabs(D[1]);
    const int a = ax == 0 ? 1 : ay == 0 ? 0 : (wide)n[0] * ay <= (wide)n[1] * ax ? 0 : 1;
    c[a] += D[a] > 0 ? 1 : -1;
    n[a] += 65536;
    return a;
  }
};

// tc_skim.h's test that q is surely on its side of every line
bool sure(float q) {
  float fr = q - floorf(q);
  if (fr >= 1.0f) fr = 0x1.fffffep-1f;
  return fabsf(fr - 0.5f) < fmaf(fabsf(q), -0x1p-21f, 0.5f - 0x1p-20f);
}

float recip(float d) {   // within a unit in the last place
  if (d == 0.0f) return INFINITY;
  const float r = 1.0f / d;
  const int64_t w = in(0, 2);
  return w == 0 ? r : nextafterf(r, w == 1 ? 4.0f * r : 0.0f);
}

}  // namespace

int main(int argc, char** argv) {
  const long rays = argc > 1 ? atol(argv[1]) : 100000;
  g_s = argc > 2 ? strtoull(argv[2], nullptr, 10) : 1;
  long fails = 0, fast = 0, open = 0;
  for (long i = 0; i < rays; ++i) {
    Walk w;
    const int64_t big = in(0, 3) == 0 ? 32000 : in(0, 1) ? 2000 : 40;
    const int64_t unit = in(0, 1) ? 1 : in(1, 1 << 20);
    for (int a = 0; a < 2; ++a) {
      const int kind = (int)in(0, 3);
      w.O[a] = kind == 0 ? in(-big, big) * 65536 : kind == 1 ? in(-2 * big, 2 * big) * 32768
             : kind == 2 ? in(-big, big) * 65536 + in(-1, 1) : in(-big * 65536, big * 65536);
      w.D[a] = in(0, 9) == 0 ? in(-8388607, 8388607) : in(-7, 7) * unit + (in(0, 2) ? 0 : in(-1, 1));
    }
    if (w.D[0] == 0 && w.D[1] == 0) w.D[0] = unit;
    w.start();
    const int32_t cx = (int32_t)w.c[0], cy = (int32_t)w.c[1];
    const float fx = w.D[0] == 0 ? 0.5f : (float)(w.O[0] & 0xFFFF) * 0x1p-16f;
    const float fy = w.D[1] == 0 ? 0.5f : (float)(w.O[1] & 0xFFFF) * 0x1p-16f;
    const float dx = (float)w.D[0], dy = (float)w.D[1], rx = recip(dx), ry = recip(dy);
    for (int s = (int)in(1, 60); s > 0 && llabs(w.c[0]) < 40000 && llabs(w.c[1]) < 40000; --s) {
      const int L = in(0, 1) ? 0 : (int)in(0, 9);
      const int64_t ni = w.c[0] >> L, nj = w.c[1] >> L;
      const bool px = dx >= 0.0f, py = dy >= 0.0f;
      const int32_t gx = (int32_t)((ni + (px ? 1 : 0)) * (1ll << L));
      const int32_t gy = (int32_t)((nj + (py ? 1 : 0)) * (1ll << L));
      const float tx = ((float)(gx - cx) - fx) * rx, ty = ((float)(gy - cy) - fy) * ry;
      const bool ex = tx <= ty;
      const float te = fminf(tx, ty);
      const float q = fmaf(te, ex ? dy : dx, ex ? fy : fx);
      skim_next got;
      if (sure(q)) {
        const int32_t o = (int32_t)floorf(q) + (ex ? cy : cx);
        got = skim_next{ex ? gx + (px ? 1 : 0) - 1 : o, ex ? o : gy + (py ? 1 : 0) - 1, ex ? 1 : 0};
        ++fast;
      } else {
        got = corner_step(cx, cy, fx, fy, dx, dy, gx, gy, ex, q);
        ++open;
      }
      int a = 0;
      while ((w.c[0] >> L) == ni && (w.c[1] >> L) == nj) a = w.step();
      if (got.x != w.c[0] || got.y != w.c[1] || got.ex != (a == 0)) {
        if (++fails < 10)
          std::printf("O %lld %lld D %lld %lld L %d q %.9g: (%d, %d) x %d, not (%lld, %lld) x %d\n",
                      (long long)w.O[0], (long long)w.O[1], (long long)w.D[0], (long long)w.D[1], L,
                      q, got.x, got.y, got.ex, (long long)w.c[0], (long long)w.c[1], a == 0);
        break;
      }
    }
  }
  std::printf("%ld rays, %ld fast steps, %ld open ones, %ld failures\n", rays, fast, open, fails);
  return fails != 0 || open < rays / 10;
}
