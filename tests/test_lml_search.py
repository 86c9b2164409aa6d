"""The search for an entry's bucket in llc_lml_bound's form by cells' sums stays within the buckets (CPU only): the kernel's own function,
compiled with AddressSanitizer, over arrays of the kernel's sizes; an entry that has target mass only lies at +inf."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_every_place_has_a_bucket(tmp_path):
    exe = tmp_path / "lml_search_driver"
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-Wno-unknown-pragmas", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                    os.path.join(ROOT, "tests", "lml_search_driver.cpp"), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, env=dict(os.environ, ASAN_OPTIONS="verify_asan_link_order=0"))
    assert out.returncode == 0, out.stdout[-2000:] + out.stderr[-4000:]
