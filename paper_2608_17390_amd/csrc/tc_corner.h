// The step of the single-precision walk (tc_skim.h) that rounding leaves
// open: the ray leaves its node so close to a cell line of the other axis that
// the rounded place says nothing of the line's side, nor, where that line is
// the node's own far face, of which face it leaves through.
//
// Both follow from the order of two crossings, that through the face found
// (distance dE on axis e) and that of the line (dK on the other axis, o):
//   tE - tK = dE / De - dK / Do = (dE Do - dK De) / (De Do).
// Distances are whole cells and a 16-bit fraction (33 bits) and components
// whole numbers below 2^23, so a product does not fit a double, but the
// difference does: with p = dE Do rounded, fma gives p's error exactly, and
// p - dK De too, as the two times differ by under 2^-20 of themselves.
// A crossing at the same time counts as later if it is of y (x steps first).
//
// Rays that meet lattice corners again and again (diagonal directions over
// whole cells) take this step at nearly every crossing, so it uses the walk's
// own floats alone.  1023x1023 diagonal rays through corners take 214 us, those
// beside the corners 147; with a step in the whole numbers of tc_walk.h, which
// rebuilds the ray and its crossings' keys for it, they took 398.
#pragma once

#include <cmath>
#include <cstdint>

namespace {

struct skim_next {
  int32_t x, y;   // the cell entered
  int32_t ex;     // through an x face?
};

// The ray: its origin's cell (cx, cy) and fractions (fx, fy) in it, its
// direction (dx, dy), neither zero.  gx, gy: the lines of the node's far
// faces; ex: the face found is that in x; q: the place of that crossing on
// the other axis, in cells from the origin's cell, next to a line.
__device__ __forceinline__ skim_next corner_step(int32_t cx, int32_t cy, float fx, float fy,
                                                 float dx, float dy, int32_t gx, int32_t gy,
                                                 bool ex, float q) {
  const float kf = rintf(q);
  const double De = ex ? dx : dy, Do = ex ? dy : dx;
  const double dE = (double)(float)(ex ? gx - cx : gy - cy) - (double)(ex ? fx : fy);
  const double dK = (double)kf - (double)(ex ? fy : fx);
  const double p = dE * Do;
  const double diff = fma(-dK, De, p) + fma(dE, Do, -p);
  const bool fe = De > 0.0, fo = Do > 0.0;
  // has the ray crossed the line by then?  (A line it starts on and leaves
  // forwards lies behind it: the origin's cell is the one above the line.)
  const bool crossed = diff == 0.0 ? !ex | (fo & (dK == 0.0)) : (diff > 0.0) == (fe == fo);
  const int32_t k = (int32_t)kf + (ex ? cy : cx);
  // through the other axis's face instead, if the line is that face's
  const bool other = crossed & (k == (ex ? gy : gx));
  const int32_t o = k - (crossed == fo ? 0 : 1);
  const int32_t e = (ex ? gx : gy) - (other == fe ? 1 : 0);
  return skim_next{ex ? e : o, ex ? o : e, ex != other ? 1 : 0};
}

}  // namespace
