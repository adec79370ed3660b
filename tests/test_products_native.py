"""Checks of the product launchers that need no GPU, through a small host program linked to the library."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="session")
def products(tmp_path_factory):
    from paper_2403_17031_amd import build
    if not os.path.exists(build.LIB):
        build.build()
    exe = str(tmp_path_factory.mktemp("native") / "products")
    cmd = [build._hipcc(), "-x", "hip", "--offload-host-only", "-std=c++17", "-O1", "-Wno-unused-result", "-I", build.CSRC,
           os.path.join(ROOT, "tests", "native", "products.cpp"), "-o", exe, "-L", build.HERE, "-l:librlhf_rollout.so",
           f"-Wl,-rpath,{build.HERE}"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return exe


def test_a_product_that_cannot_launch_reports_it(products):
    r = subprocess.run([products, "errors"], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stdout + r.stderr


def test_a_decode_product_with_scratch_is_split(products):
    r = subprocess.run([products, "split"], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stdout + r.stderr


def test_unaligned_operands_stay_off_the_few_rows_kernel(products):
    r = subprocess.run([products, "aligned"], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stdout + r.stderr
