"""The plan of the residue products (ct_rns_plan.h) on the host: on random
batches and scratch sizes the scratch ranges lie where they should and do not
meet, chunks cover K, and every workgroup of every launch finds its own piece
of work (tests/rns_plan_sim.cpp); and which path the rule gives an encoder."""
import os
import re
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_plans_and_rule(tmp_path):
    exe = str(tmp_path / "rns_plan_sim")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-Wall", "-Wextra", "-Werror", "-D__HIP_PLATFORM_AMD__",
                           "-isystem", os.path.join(rocm, "include"), "-I", os.path.join(ROOT, "include"),
                           "-I", os.path.join(ROOT, "paper_2311_04406_amd", "csrc"),
                           "-o", exe, os.path.join(ROOT, "tests", "rns_plan_sim.cpp")])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr + r.stdout
    got = {m.group(1): {k: int(v) for k, v in (kv.split("=") for kv in m.group(2).split())}
           for m in re.finditer(r"ok (\w+) (.*)", r.stdout)}
    # several groups a batch, on halves of the scratch too, and layers in K chunks
    assert got["plans"]["groups"] > got["plans"]["batches"] > 500
    assert got["plans"]["halves"] > 100 and got["plans"]["chunked"] > 100
    # layers by residues: an encoder's four with CompactTag, none in SPDZ2k or with three parties
    assert got["rule"] == {"compact": 4, "spdz2k": 0, "parties3": 0, "square": 1, "small": 0}
