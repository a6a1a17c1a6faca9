"""The pinned result slots of the diagnostics: when the page is allocated, and that it is never freed."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def test_the_page_is_allocated_once_when_it_pays(tmp_path):
    """Few reads per context, many contexts, no page to be had, and threads, on an allocator that counts."""
    exe = str(tmp_path / "probe")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-pthread", os.path.join(HERE, "host_slots_probe.cpp"), "-o", exe],
                   check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
