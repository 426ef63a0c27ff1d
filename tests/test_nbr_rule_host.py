"""The rule between the neighbour peak's two forms (``csrc/nbr_rule.h``),
compiled with g++ into a small driver: its lines, its limits, and the noise rate
against the same estimate in numpy / scipy.  CPU only."""
import os
import subprocess

import pytest
from scipy.stats import norm

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1307_6489_amd", "csrc")

DRIVER = r"""
#include <cstdio>
#include <cstdlib>
#include "nbr_rule.h"
int main(int argc, char** argv) {
  const rta::NbrRule r = rta::nbr_rule(std::atoi(argv[1]), std::atoi(argv[2]), std::atof(argv[3]), std::atof(argv[4]));
  std::printf("%d %.9g %.9g %.9g\n", r.most, r.noise, rta::nbr_share(r.noise, 8), rta::nbr_share(r.noise, 16));
  return 0;
}
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    d = tmp_path_factory.mktemp("nbr")
    src, exe = d / "drv.cpp", d / "drv"
    src.write_text(DRIVER)
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)], check=True)

    def run(n_pix, n_samp, t_pic=10.0, t_bnd=5.0):
        out = subprocess.run([str(exe), str(n_pix), str(n_samp), repr(t_pic), repr(t_bnd)], check=True,
                             capture_output=True, text=True).stdout.split()
        return int(out[0]), float(out[1]), float(out[2]), float(out[3])
    return run


@pytest.mark.parametrize("n_samp", [4, 25, 64, 65, 255])
def test_small_cameras_are_scanned(rule, n_samp):
    line = 900 + 3 * n_samp
    assert rule(line - 1, n_samp)[0] == 0
    assert rule(line, n_samp)[0] == (400 if n_samp <= 64 else 300) * line // 2048
    assert rule(2048, n_samp)[0] == (400 if n_samp <= 64 else 300) <= 600  # what the stage holds


def test_levels_at_or_below_zero_are_scanned(rule):
    assert rule(2048, 128, 10.0, 0.0)[0] == rule(2048, 128, 1.0, -1.0)[0] == rule(2048, 128, -1.0, -2.0)[0] == 0


@pytest.mark.parametrize("n_pix,n_samp", [(2048, 16), (1764, 25), (1855, 40), (2048, 128), (2048, 255)])
@pytest.mark.parametrize("levels", [(10.0, 5.0), (5.0, 2.5), (10.0, 9.0), (6.0, 6.0), (8.0, 1.0)])
def test_noise_rate(rule, n_pix, n_samp, levels):
    _, rate, s8, s16 = rule(n_pix, n_samp, *levels)
    pixels = min(350.0, 22000.0 / n_samp) * (n_pix / 2048.0) ** 2 / 20.0
    want = norm.sf(norm.isf(2.0 * pixels / (n_pix * (n_samp - 3.0))) * levels[1] / levels[0])
    assert abs(rate - want) <= 1e-5 * want
    assert abs(s8 - min(0.95, 2.6 * rate)) < 1e-5 and abs(s16 - min(0.95, 5.8 * rate)) < 1e-5


def test_short_traces_are_not_looked_at(rule):
    assert rule(2048, 15)[1] == 1.0 and rule(2048, 16)[1] < 0.5
