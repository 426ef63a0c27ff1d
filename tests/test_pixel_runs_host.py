"""The runs of flagged pixels in a workgroup's list (``csrc/pixel_runs.h``),
compiled with g++ into a small driver: for every compiled shape (pixels per
lane, wavefronts) and camera size, the entries that a wavefront may write, one
per pixel that it extracts, lie inside the list and apart from every other
wavefront's.  CPU only."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1307_6489_amd", "csrc")
MAX_PIX = 2048

DRIVER = r"""
#include <cstdio>
#include <cstdlib>
#include "pixel_runs.h"
int main(int argc, char** argv) {
  const int max_pix = std::atoi(argv[1]), nt = std::atoi(argv[2]), ppl = std::atoi(argv[3]);
  for (int w = 0; w < nt / 64; ++w) std::printf("%d\n", rta::run_begin(max_pix, nt, ppl, w));
  return 0;
}
"""


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    d = tmp_path_factory.mktemp("runs")
    src = d / "drv.cpp"
    src.write_text(DRIVER)
    exe = d / "drv"
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    return str(exe)


def pixels_of(n_pix, nt, ppl, wave):
    """Pixels (padding of the last group of eight included) that a wavefront extracts."""
    n_pad = (n_pix + 7) // 8 * 8
    return [i for i in range(n_pad) if (i // ppl) % nt // 64 == wave]


@pytest.mark.parametrize("ppl", [2, 4, 8])
@pytest.mark.parametrize("waves", [4, 8])
def test_runs_hold_every_pixel_of_a_wavefront(driver, waves, ppl):
    nt = 64 * waves
    out = subprocess.run([driver, str(MAX_PIX), str(nt), str(ppl)], check=True, capture_output=True, text=True)
    begin = [int(v) for v in out.stdout.split()]
    for n_pix in (1, 7, 64, 511, 513, 1024, 1025, 1764, 1855, 2041, 2048):
        owner = [None] * MAX_PIX
        for w in range(waves):
            for k in range(len(pixels_of(n_pix, nt, ppl, w))):
                at = begin[w] + k
                assert 0 <= at < MAX_PIX, (n_pix, w, at)
                assert owner[at] is None, "wavefronts %d and %d share entry %d of %d pixels" % (owner[at], w, at, n_pix)
                owner[at] = w
    assert all(0 <= b < MAX_PIX for b in begin)
