// Host build of the library's chord cutter, for CPU tests.  Test infrastructure only.
#include "../paper_2501_12581_amd/csrc/apc_cut.h"

struct Frame {
  double t_near, step, inv_step, max_chord, w_scale, w_off;
  int long_chords;
};

// The chords of one segment, from `at[0]` over at[1], ... at[n]: how many pieces each has, and the last `keep` cut
// points (piece ends) of the segment in ends[].
extern "C" long long shim_cut(double t_near, double step, double max_chord, const double* at, int n,
                              long long* pieces, double* ends, int keep) {
  const Frame f = {t_near, step, 1.0 / step, max_chord, 1.0, 0.0, at[n] - at[0] > max_chord};
  apc::Cutter c;
  c.start(f, at[0], 0.0f);
  long long all = 0;
  for (int i = 0; i < n; ++i) {
    c.to(f, at[i + 1], float(i + 1));
    pieces[i] = 0;
    while (c.cutting()) {
      float wt, len, s;
      c.piece(f, wt, len, s);
      ends[all % keep] = c.u;
      ++pieces[i];
      ++all;
    }
  }
  return all;
}
