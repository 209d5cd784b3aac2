"""The scene upload's host side on the CPU under UndefinedBehaviorSanitizer
(tests/sanitize/scene_upload.cpp: a HIP runtime on the heap), built with the HIP
compiler's host pass."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
CSRC = os.path.join(ROOT, "paper_2305_04403_amd", "csrc")


@pytest.mark.skipif(not os.path.exists(HIPCC) and shutil.which("hipcc") is None, reason="no hipcc")
def test_scene_upload_under_sanitizer(tmp_path):
    flags = ["-std=c++17", "-O1", "-g", "-I", os.path.join(ROOT, "include")]
    host = ["-x", "hip", "--offload-host-only", "--offload-arch=gfx950",
            "-Xarch_host", "-fsanitize=undefined", "-Xarch_host", "-fno-sanitize-recover=undefined"]
    objs = []
    for src in (os.path.join(CSRC, "wob.hip"), os.path.join(ROOT, "tests", "sanitize", "scene_upload.cpp")):
        objs.append(str(tmp_path / (os.path.basename(src) + ".o")))
        subprocess.run([HIPCC, "-c", *host, *flags, src, "-o", objs[-1]], check=True)
    objs.append(str(tmp_path / "bvh_build.o"))
    subprocess.run(["g++", "-c", *flags, os.path.join(CSRC, "bvh_build.cpp"), "-o", objs[-1]], check=True)
    exe = str(tmp_path / "scene_upload")
    # the device code that a host pass leaves out is the one symbol that stays open
    clang = os.path.join(os.path.dirname(os.path.realpath(HIPCC)), "..", "lib", "llvm", "bin", "clang++")
    subprocess.run([clang if os.path.exists(clang) else "clang++", "-fsanitize=undefined", *objs,
                    "-Wl,--unresolved-symbols=ignore-all", "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), (r.stdout + r.stderr)[-3000:]
