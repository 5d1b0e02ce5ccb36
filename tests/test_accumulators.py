"""Where a lane's check accumulators lie.  Every workgroup of a verification
adds to a few elements per layer, and how long that takes depends on their
addresses: in a block of their own, 12576 bytes apart, the batch SPDZ2K_CHECK
(two parties) takes 620 us in k_check_batch, up to 860 with other spacings or
behind the tables."""
import os
import re
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2311_04406_amd", "csrc")
# M x K x N, or M x K x N / C.H.W.k.s.p of an implicit convolution
SPDZ2K_CHECK = ("12x3577x52 2671x63x144/7.12.12.3.1.1 731x41x322 896x128x64 2834x133x1568 3098x644x764 64x192x1728 "
                "2624x128x64 11x10x2 200x13x12 512x128x1792 3006x188x169/188.13.13.1.1.0 94x755x1 192x64x320")


def test_spacing_and_block(tmp_path):
    src = tmp_path / "acc.cpp"
    src.write_text('#include <cstdio>\n#include "ct_internal.h"\nint main() { std::printf("%zu %zu", '
                   "sizeof(ct::u128) * ct::ACC_PER_LAYER, sizeof(ct::u128) * ct::ACC_RP); }\n")
    exe = str(tmp_path / "acc")
    subprocess.check_call(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-isystem",
                           os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include"),
                           "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-o", exe, str(src)])
    assert subprocess.check_output([exe]).split() == [b"12576", b"288"]
    api = open(os.path.join(CSRC, "ct_api.hip")).read()
    assert re.search(r"hipMalloc\(&ln\.acc_dev, sizeof\(u128\) \* ACC_PER_LAYER \* \(int64_t\)max_layers\)", api)
