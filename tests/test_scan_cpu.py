"""The device-wide scan's header (scan.hpp) built for the CPU with a stand-in
for the device runtime (tests/native/hip_cpu): whichever workgroups of a scan
have started, their tiles are the first ones; the prefixes of the flat walk
and of the look-back; a bounded wait that runs out is reported."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_scan_on_the_cpu(tmp_path):
    exe = str(tmp_path / "scan_main")
    native = os.path.join(ROOT, "tests", "native")
    subprocess.check_call(["g++", "-O1", "-std=c++20", "-pthread", "-Wno-unknown-pragmas",
                           "-I" + os.path.join(native, "hip_cpu"),
                           "-I" + os.path.join(ROOT, "paper_2010_05337_amd", "csrc"),
                           os.path.join(native, "scan_main.cpp"), "-o", exe])
    r = subprocess.run([exe], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=240)
    assert r.returncode == 0 and r.stdout.endswith("ok\n"), r.stdout
