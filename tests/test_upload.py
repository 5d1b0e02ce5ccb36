"""How a call's tables go to the device: copies of at most 16 KB, which the
device takes in 2.5 us each, up to 64 KB, and one copy (17 us) beyond."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_pieces(tmp_path):
    src = tmp_path / "up.cpp"
    src.write_text('#include <cstdio>\n#include "ct_host.h"\nint main() {\n'
                   "    for (long long b : {1, 16384, 16385, 26000, 65536, 65537, 1 << 20})\n"
                   '        std::printf("%lld ", (b + ct::upload_piece(b) - 1) / ct::upload_piece(b));\n}\n')
    exe = str(tmp_path / "up")
    subprocess.check_call(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-isystem",
                           os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include"),
                           "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2311_04406_amd", "csrc"),
                           "-o", exe, str(src)])
    assert subprocess.check_output([exe]).split() == [b"1", b"1", b"2", b"2", b"4", b"1", b"1"]
