// Where a wavefront's run of flagged pixels lies in the workgroup's list.
//
// A workgroup of nt threads extracts a camera in passes of nt * ppl
// consecutive pixels, thread t the ppl pixels from t * ppl of each pass on.
// A run holds every pixel of its wavefront; where one pass covers more than
// the largest camera (8 pixels per lane, 8 wavefronts) the last wavefronts
// extract none and the runs of the others fill the list.
#pragma once

namespace rta {

constexpr int kRunWave = 64;

// Pixels that a wavefront extracts at most.
constexpr int run_length(int max_pix, int nt, int ppl) {
  return kRunWave * ppl * ((max_pix + nt * ppl - 1) / (nt * ppl));
}

// First entry of a wavefront's run (of one without pixels: any inside the list).
constexpr int run_begin(int max_pix, int nt, int ppl, int wave) {
  const int len = run_length(max_pix, nt, ppl);
  return wave * len < max_pix ? wave * len : 0;
}

}  // namespace rta
