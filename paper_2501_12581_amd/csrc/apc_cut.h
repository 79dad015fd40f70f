// Cutting a ray's chords at the sampling lattice (device code; host tests compile it too).
#pragma once

#include "apc_mboit.h"

namespace apc {

#define APC_CUT __attribute__((always_inline)) APC_HD

// Cuts the chords of one ray at the sampling lattice t_near + k*step.  The
// chords of a segment meet end to start, so only a chord's end is handed over
// (to) and the next lattice point carries on from chord to chord, by its
// number: a point formed by adding steps would drift by a rounding a step (one
// instruction a piece less: stage one 12.0 ms against 12.2 at 2560^2, m = 8, on
// 12.6M tets).  The cut points and mid depths are FP64 (depths are absolute
// positions along the ray); lengths and scalars are FP32.  F: FrameDev.
struct Cutter {
  double u = 0.0, t1 = 0.0, k = 0.0;  // cut so far, chord end, the next lattice point's number
  float s1 = 0.0f, slope = 0.0f;      // scalar at the chord's end and along it

  APC_CUT bool cutting() const { return u < t1; }
  // the first lattice point after depth t
  template <class F>
  APC_CUT void align(const F& f, double t) {
    k = __builtin_floor((t - f.t_near) * f.inv_step) + 1.0;
    if (!(__builtin_fma(k, f.step, f.t_near) > t)) k += 1.0;  // the rounded floor can fall one short
  }
  // a segment begins at depth t with scalar s
  template <class F>
  APC_CUT void start(const F& f, double t, float s) {
    u = t1 = t;
    s1 = s;
    align(f, t);
  }
  // the next chord ends at depth t with scalar s
  template <class F>
  APC_CUT void to(const F& f, double t, float s) {
    const double len = t - t1;
    slope = (s - s1) * apcm::m_rcp(float(len));
    if (f.long_chords) {
      if (!(len <= f.max_chord))
        k = HUGE_VAL;  // never that many pieces: the chord is one
      else if (k == HUGE_VAL)
        align(f, t1);  // the chord after such a one
    }
    t1 = t;
    s1 = s;
  }
  // the next piece of the chord: its mid depth from the eye (over the range's geometric mean), length and scalar
  template <class F>
  APC_CUT void piece(const F& f, float& wt, float& len, float& s) {
    const double nxt = __builtin_fma(k, f.step, f.t_near);
    const bool lat = nxt <= t1;
    const double v = lat ? nxt : t1, sum = u + v;
    wt = float(__builtin_fma(sum, f.w_scale, f.w_off));
    len = float(v - u);
    s = __builtin_fmaf(slope, float(__builtin_fma(0.5, sum, -t1)), s1);
    k = lat ? k + 1.0 : k;
    u = v;
  }
};

#undef APC_CUT

}  // namespace apc
