"""The last chunk of the short matrix-core kernels may be a part of one: its loads and
stores beyond the batch are left out by the buffer descriptor's bound.  That bound is
compared with the lane's offset and the instruction's constant; a scalar offset is not a
part of the comparison (or is subtracted from the bound, below zero).  So no access of
these kernels may have one: seen in the assembly of one kernel of each kind."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
KERNELS = """
#include "wave.hpp"
using namespace nttmi;
typedef const uint32_t* In;
template __global__ void nttmi::k_conv_tiny<6, false>(In, In, uint32_t*, uint64_t, int, I8Plan);
template __global__ void nttmi::k_div_tiny<6, false>(In, In, uint32_t*, uint64_t, int, I8Plan, Quotient);
template __global__ void nttmi::k_crt_tiny<6>(In, In, uint64_t, int, I8Plan, Combine);
template __global__ void nttmi::k_ntt_tiny<6, false>(In, uint32_t*, uint64_t, I8Plan);
template __global__ void nttmi::k_conv_mid<9, false>(In, In, uint32_t*, uint64_t, I8Plan);
template __global__ void nttmi::k_conv_mid<12, false>(In, In, uint32_t*, uint64_t, I8Plan);
template __global__ void nttmi::k_div_mid<10, false>(In, In, uint32_t*, uint64_t, I8Plan, Quotient);
template __global__ void nttmi::k_crt_mid<11>(In, In, uint64_t, I8Plan, Combine);
template __global__ void nttmi::k_ntt_mid<9, false>(In, uint32_t*, uint64_t, I8Plan);
template __global__ void nttmi::k_ntt_mid<12, true>(In, uint32_t*, uint64_t, I8Plan);
"""
# buffer_{load,store}_<type> data, offset, s[a:b], <scalar offset> ...
ACCESS = re.compile(r"^\s*(buffer_(?:load|store)\S*)\s.*s\[\d+:\d+\],\s*([^\s,]+)", re.M)


@pytest.mark.skipif(not shutil.which(HIPCC), reason="no hipcc")
def test_no_scalar_offset_in_kernels_with_partial_chunks(tmp_path):
    src, out = tmp_path / "kernels.hip", tmp_path / "kernels.s"
    src.write_text(KERNELS)
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "-S", "--cuda-device-only", "-Xclang",
                    "-target-feature", "-Xclang", "-packed-fp32-ops",
                    "-I" + os.path.join(ROOT, "paper_1005_1497_amd", "csrc"), str(src), "-o", str(out)],
                   check=True, capture_output=True)
    bodies = re.findall(r"^(_ZN5nttmi\S+):.*?\n(.*?)\.section", out.read_text(), re.S | re.M)
    assert len(bodies) == KERNELS.count("template __global__")
    for name, body in bodies:
        found = ACCESS.findall(body)
        assert len(found) >= 20, name
        assert {offset for _, offset in found} == {"0"}, name
