"""FP64 links and corners on lattices whose slabs pass 4 GiB: the stores of the setup kernels,
compiled for the host, address every slab with 64 bits, as the plaquette, the corner products and
the 12-real links' readers do.  (With 32-bit slab offsets, entry (2, 2) of a link on 64^3 x 128 went
over entry (0, 0) of another site.)"""
import os
import subprocess

import pytest

from paper_1312_3265_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


def test_fp64_matrices_beyond_32_bit_offsets(tmp_path):
    try:
        hipcc = build.hipcc()
    except RuntimeError:
        pytest.skip("needs hipcc for the HIP headers")
    exe = str(tmp_path / "large_lattice_check")
    subprocess.run([hipcc, "-x", "hip", "--offload-host-only", "-O1", "-std=c++17",
                    os.path.join(HERE, "large_lattice_check.cpp"), "-o", exe], check=True)
    out = subprocess.run([exe], capture_output=True, text=True, check=True).stdout.split("\n")
    assert out[:2] == ["links ok", "corners ok"]
