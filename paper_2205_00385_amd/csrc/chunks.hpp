// Chunk lengths of the kernels that march along z (host only).
#pragma once

namespace aarmr {

// f(t) for every length t = ceil(planes / n), n = 1, 2, ..., from the longest
// down to `least`, each once: at most 2 sqrt(planes) of them.  The launches
// choose their chunk among these on every call; a loop over every n took as
// long as the kernel on long thin grids (fine product: 4x4x2048 23.6 -> 9.4 us a
// call, 16x16x8192 69 -> 53 us).
template <typename F>
inline void for_chunk_lengths(int planes, int least, F f) {
  for (int t = planes; t >= least && t > 0;) {
    f(t);
    if (t == 1) break;
    const int n = (planes + t - 2) / (t - 1);  // the fewest chunks shorter than t
    t = (planes + n - 1) / n;
  }
}

}  // namespace aarmr
