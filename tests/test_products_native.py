"""Checks of the product launchers that need no GPU, through a small host program linked to the library."""
import os
import re
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


def test_a_second_bias_is_added_or_refused(products):
    r = subprocess.run([products, "bias2"], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stdout + r.stderr


def test_decode_passes_on_the_gpu_cover_every_form_of_the_kernel(products):
    """The shapes that the GPU tests grade against the oracle reach every form of the few-rows kernel in bf16, each but
    the short-K one (form 2) with a K loop that is long enough to be pipelined (2 * PF steps per wave), and a K split
    of eight."""
    from test_gpu_few_rows import DECODES, SHAPES, WIDE, WIDTHS
    runs = [(SHAPES[s][0], SHAPES[s][4], SHAPES[s][5], B) for s, B, *_ in DECODES if SHAPES[s][2] in (16, 64, 80, 128, 256)]
    runs += [(WIDTHS[w][0], WIDTHS[w][4], 515, B) for w, B in WIDE]
    seen, pipelined, splits = set(), set(), set()
    for d, F, V, B in runs:
        r = subprocess.run([products, "forms", *map(str, (d, F, V, min(B, 256)))], capture_output=True, text=True, timeout=100)
        assert r.returncode == 0, r.stdout + r.stderr
        for line in r.stdout.splitlines():
            name, _, split, _, steps = line.split()
            form = tuple(map(int, re.search(r"DF16_Li(\d)ELi(\d)ELi(\d)ELi(\d)ELi(\d)E", name).groups()))
            seen.add(form)
            splits.add(int(split))
            if int(steps) // int(split) // form[0] >= 2 * form[3]:
                pipelined.add(form)
    with open(os.path.join(ROOT, "paper_2403_17031_amd", "csrc", "few_rows.hip")) as f:
        forms = {tuple(map(int, m)) for m in re.findall(r"X\(\d, (\d), (\d), (\d), (\d), (\d)\)", f.read())}
    assert len(forms) == 9 and seen == forms
    assert {f for f in forms if f[:3] != (4, 1, 2)} <= pipelined
    assert max(splits) == 8
