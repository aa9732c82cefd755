"""CPU test of the link offsets that the FP16 odd step and the two-step passes
compute, with the kernels' own functions compiled for the host
(tests/host/link_offsets.cpp)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


def test_the_kernels_link_offsets_lead_to_the_tiled_slots(tmp_path):
    out = str(tmp_path / "link_offsets")
    src = os.path.join(ROOT, "tests", "host", "link_offsets.cpp")
    subprocess.run([os.path.join(ROCM, "bin", "hipcc"), "--offload-host-only", "-x", "hip", "-std=c++17", "-O1",
                    "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_1611_03329_amd", "csrc"),
                    src, "-o", out], check=True)
    r = subprocess.run([out], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
