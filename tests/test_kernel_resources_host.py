"""Registers of the compiled reconstruction kernels, from the metadata of the
built library: every schedule that can be chosen keeps the wavefronts that its
speed rests on.  CPU only."""
import os
import re
import shutil
import subprocess

import pytest

import paper_1307_6489_amd as rta

LLVM = "/opt/rocm/llvm/bin"
LIB = os.path.join(os.path.dirname(os.path.abspath(rta.__file__)), "librta.so")
EXTRACTORS = {"sliding": 0, "fixed": 1, "global": 2, "neighbour": 3}


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{(kernel, extractor, pixels per lane, chunk, threads): (registers, scratch bytes)}"""
    if not os.path.exists(LIB) or not os.path.exists(os.path.join(LLVM, "llvm-objdump")):
        pytest.skip("no built library or no tools to read it")
    d = tmp_path_factory.mktemp("resources")
    lib = shutil.copy(LIB, d)
    subprocess.run([os.path.join(LLVM, "llvm-objdump"), "--offloading", lib], check=True, stdout=subprocess.DEVNULL)
    out = {}
    for f in sorted(os.listdir(d)):
        if not f.endswith("gfx950"):
            continue
        notes = subprocess.run([os.path.join(LLVM, "llvm-readelf"), "--notes", os.path.join(d, f)], check=True,
                               capture_output=True, text=True).stdout
        for m in re.finditer(r"\.name: +\S*?(k_fused(?:_grid)?)ILi(\d)ELi(\d)ELi4ELi(\d+)ELi(\d+)E.*?"
                             r"\.private_segment_fixed_size: (\d+).*?\.vgpr_count: +(\d+)", notes, re.S):
            out[(m[1],) + tuple(int(v) for v in m.groups()[1:5])] = int(m[7]), int(m[6])
    assert len([k for k in out if k[0] == "k_fused_grid"]) == 48 and len([k for k in out if k[0] == "k_fused"]) == 12
    return out


def test_two_wavefronts_per_simd(kernels):
    """A SIMD has 512 registers per lane: more than 256 leave one wavefront to
    hide the trace loads of the next (sliding, 8 pixels per lane, chunk 16, 4
    wavefronts, 260 registers: 600 us for 8000 events of the mix, 457 with
    256)."""
    assert not {k: v for k, v in kernels.items() if v[0] > 256}


def test_neighbour_peak_keeps_its_registers(kernels):
    """The neighbour peak is held to four wavefronts per SIMD, 128 registers:
    what does not fit goes to scratch memory (8 pixels per lane, chunks of 16,
    316 bytes: 1172 us for 8000 events of the mix, 596 with none)."""
    assert not {k: v for k, v in kernels.items() if k[1] == EXTRACTORS["neighbour"] and (v[1] > 0 or v[0] > 128)}
