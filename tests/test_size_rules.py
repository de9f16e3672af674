"""Rules on sizes that host and kernels share (csrc/pifcm_device.h), compiled
for the CPU and run over the whole range of volumes the library accepts."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2002_01981_amd", "csrc")
HIP = "/opt/rocm/include"


def run(tmp_path, body):
    """Output of a C++ program with `body` as its main, in namespace pifcm."""
    src, exe = tmp_path / "rules.cpp", tmp_path / "rules"
    src.write_text('#include <cstdio>\n#include "pifcm_device.h"\nnamespace pifcm { static void body() {\n' + body +
                   "\n} }\nint main() { pifcm::body(); }\n")
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-isystem", HIP, "-I", CSRC, str(src),
                    "-o", str(exe)], check=True, capture_output=True, text=True)
    return subprocess.run([str(exe)], check=True, capture_output=True, text=True, timeout=60).stdout.split()


pytestmark = pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir(HIP), reason="needs g++ and HIP's headers")


def test_only_a_single_voxel_has_no_neighbours(tmp_path):
    """Volumes of up to 4e9 voxels, whose count does not fit 32 bits."""
    sides = [(1, 1, 1), (2, 1, 1), (1, 2, 1), (1, 1, 2), (181, 217, 181), (2047, 1024, 1024), (2048, 1024, 1024),
             (2048, 1024, 1100), (2048, 1024, 1900), (1, 1, 2147483647), (65536, 1, 60000), (4096, 4096, 256)]
    out = run(tmp_path, "\n".join('std::printf("%%d\\n", (int)has_neighbours(%d, %d, %d));' % s for s in sides))
    assert [int(v) for v in out] == [int(s != (1, 1, 1)) for s in sides]


def test_a_thread_of_the_pointwise_pass_has_few_voxels(tmp_path):
    """At most eight runs of eight, whatever the volume; one up to 2^18 voxels."""
    sizes = [1, 255, 1 << 18, (1 << 18) + 1, 7109137, 1 << 24, (1 << 24) + 1, 1 << 30, 4000000000]
    out = run(tmp_path, "\n".join('std::printf("%%d\\n", fcm_vpt(%dull));' % n for n in sizes))
    assert [int(v) for v in out] == [min(64, max(1, -(-n // (1 << 18)))) for n in sizes]
