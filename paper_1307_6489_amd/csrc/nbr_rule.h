// Which form the neighbour peak takes in the fused kernel: windows of the pixels
// that can enter the image (bounds of all pixels first, then the asked pixels'
// neighbourhoods staged), or a scan of every pixel.  Both give the same bits.
//
// The windows cost a pass over the trace and then some 12 us per stage of
// slices that fit, whatever the camera; the scan costs by pixels times slices.
// Times in us of the windows and of the scan, telescopes of one camera at 0.1
// p.e. per sample and levels of 10 / 5 p.e.:
//   1500-3000 telescopes  2048 x 25  105, 193   2048 x 128  190, 303   2048 x 255  366, 459
//                         1300 x 25   97, 140   1300 x 128  317, 360   1300 x 255  339, 317
//                          900 x 25   91, 106    900 x 128  287, 253    900 x 255  302, 228
//                          600 x 25   86,  91    600 x 128  250, 209    600 x 255  503, 345
//   100 telescopes        2048 x 25   32,  32   2048 x 128   67,  78   2048 x 255  113, 125
//                          900 x 25   31,  26    900 x 128   67,  53    900 x 255  106,  82
// so cameras of fewer than 900 + 3 T pixels are scanned: above, bulk batches gain
// a quarter and more, below, they gain little or lose, and small batches lose.
//
// It is the other way where an image or the night sky asks for many pixels: 3000
// telescopes of 2048 x 128 at 5 / 2.5 p.e. (some 200 traces) take 560 us in both
// forms, at 0.2 p.e. per sample (700 traces) 911 by windows, 778 by bounds and
// scan and 576 by the scan alone.  Hence two limits.  Past `most` traces an event
// is scanned although its bounds are known (100 telescopes of 2048 x 128: limits
// of 256, 300, 400 and 600 give 99, 101, 111 and 129; 4000 of 1855 x 40: 337, 313,
// 282 and 285).  And the bounds are given up after one chunk of slices where the
// share of pixels at the boundary level says that the noise alone will ask for too
// many (3000 telescopes at 0.2 p.e. per sample so 602).  That look is a barrier in
// a telescope's chain, 1 to 2 us of 30 to 65, so it is left out for up to two
// telescopes per compute unit, where even bounds and scan together are below the
// former full scan (100 telescopes 97, 106).  With both, batches under a sky of 0.1
// to 1.6 p.e. per sample at levels from 4 / 2 to 10 / 5 p.e. take 0.4 to 1.07
// times the former full scan's time, 1.12 at most for cameras just above the line.
#pragma once
#include <algorithm>
#include <cmath>

namespace rta {

constexpr int kNbrLookTels = 2;  // telescopes per compute unit

struct NbrRule {
  int most;     // most traces staged; 0: every pixel of the camera is scanned
  float noise;  // rate of windows at the boundary level above which the event is scanned (1 or more: not looked at)
};

inline NbrRule nbr_rule(int n_pix, int n_samp, float t_pic, float t_bnd) {
  NbrRule r{0, 1.f};
  if (n_pix < 900 + 3 * n_samp || !(t_bnd > 0.f)) return r;
  r.most = (n_samp > 64 ? 300 : 400) * n_pix / 2048;
  if (n_samp < 16) return r;  // the bounds are nearly read
  // Window sums of noise taken as normal, those above the picture level in runs
  // of two.  A noise pixel at the picture level brings some 20 traces (its
  // neighbours, theirs at the boundary level, and the ring around); the
  // windows are worth it up to 22000 / T of them, and 350, at 2048 pixels.
  auto above = [](double u) { return 0.5 * std::erfc(u / std::sqrt(2.0)); };
  const double size = n_pix / 2048.0, pixels = std::min(350.0, 22000.0 / n_samp) * size * size / 20.0;
  const double at_pic = std::min(0.5, 2.0 * pixels / ((double)n_pix * (n_samp - 3)));  // one window
  double lo = 0.0, hi = 40.0;
  for (int k = 0; k < 100; ++k) {
    const double u = 0.5 * (lo + hi);
    (above(u) > at_pic ? lo : hi) = u;
  }
  r.noise = (float)above(lo * (double)t_bnd / (double)t_pic);
  return r;
}

// Share of pixels with a window at a level after the given slices, at a rate of
// its windows (of four samples, in runs of two and a half).
constexpr float nbr_share(float rate, int slices) {
  const float s = rate * (1.f + (float)(slices - 4) / 2.5f);
  return s < 0.95f ? s : 0.95f;
}

}  // namespace rta
