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


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
def test_runs_on_the_gpu_cover_every_form_of_the_kernel(products, dtype):
    """The shapes that the GPU tests grade against the oracle reach every form of the few-rows kernel in either mode (3 x 5
    tiles are bf16's alone), each but the two that are taken for short K loops (1 x 2 tiles) with one that is long
    enough to be pipelined (2 * PF steps per wave) in bf16, those of 4 row tiles and up to 80 columns with several row tiles, and a K
    split of eight."""
    from test_gpu_few_rows import DECODES, MANY_FP32, SHAPES, WIDE, WIDE_FP32, WIDTHS
    fp32 = dtype == "fp32"
    runs = [("forms", SHAPES[s][0], SHAPES[s][4], SHAPES[s][5], min(B, 256)) for s, B, *_ in DECODES
            if SHAPES[s][2] in (16, 64, 80, 128, 256)]
    runs += [("forms", WIDTHS[w][0], WIDTHS[w][4], 515, B) for w, B in (WIDE_FP32 if fp32 else WIDE)]
    runs += [("many", WIDTHS[w][0], WIDTHS[w][4], 515, B * L) for w, B, L in MANY_FP32 if fp32]
    seen, pipelined, tiles, splits = set(), set(), set(), set()
    for what, *sizes in runs:
        args = [what, *(["0" if fp32 else "1"] if what == "forms" else []), *map(str, sizes)]
        r = subprocess.run([products, *args], capture_output=True, text=True, timeout=100)
        assert r.returncode == 0, r.stdout + r.stderr
        for line in r.stdout.splitlines():
            name, _, split, _, steps, _, rows = line.split()
            form = tuple(map(int, re.search(r"I(?:DF16_|f)Li(\d)ELi(\d)ELi(\d)ELi(\d)ELi(\d)E", name).groups()))
            seen.add(form)
            splits.add(int(split))
            if int(steps) // int(split) // form[0] >= 2 * form[3]:
                pipelined.add(form)
            if int(rows) > 64:
                tiles.add(form[:3])
    with open(os.path.join(ROOT, "paper_2403_17031_amd", "csrc", "few_rows.hip")) as f:
        forms = {tuple(map(int, m)) for m in re.findall(r"X\(\d+, (\d), (\d), (\d), (\d), (\d)\)", f.read())}
    assert len(forms) == 13
    assert seen == {f for f in forms if not fp32 or f[:3] != (4, 3, 5)}
    assert fp32 or {f for f in forms if f[1:3] != (1, 2)} <= pipelined
    assert {(4, 4, 2), (4, 4, 4), (4, 4, 5)} <= tiles and (not fp32 or (4, 4, 8) in tiles)
    assert max(splits) == 8


def _forms(products, dtype, d, rows, vocab=50304):
    """(waves, row tiles, column tiles) that a decode pass of a model of width d takes for QKV + FC1, for out-projection +
    FC2 and for the LM head."""
    args = ["forms", *(str(x) for x in (dtype, d, 4 * d, vocab, rows))]
    r = subprocess.run([products, *args], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stdout + r.stderr
    return [tuple(map(int, re.search(r"I(?:DF16_|f)Li(\d)ELi(\d)ELi(\d)E", line).groups())) for line in r.stdout.splitlines()]


@pytest.mark.parametrize("d", [512, 768, 1536, 2048, 4096])
@pytest.mark.parametrize("rows", [1, 16, 17, 32, 33, 48, 49, 64])
def test_no_idle_row_tiles_in_forms_of_two_and_four_column_tiles(products, d, rows):
    for _, row_tiles, column_tiles in _forms(products, 1, d, rows):
        assert column_tiles > 4 or row_tiles == (rows + 15) // 16


@pytest.mark.parametrize("rows", [1, 16, 17, 48])
def test_one_round_rather_than_a_second_that_is_not_full(products, rows):
    """Two column tiles would be 288 to 448 blocks where four are 144 to 224; at 512 blocks both rounds are full."""
    tiles = (rows + 15) // 16
    assert _forms(products, 1, 1152, rows)[1] == (4, tiles, 4)
    assert [f for f in _forms(products, 1, 1536, rows)[:2]] == [(4, tiles, 4)] * 2
    assert _forms(products, 1, 2048, rows)[0] == (4, tiles, 4)
    if rows <= 16:
        assert _forms(products, 1, 2048, rows)[1] == (4, 1, 2)


def test_eight_waves_for_the_lm_head_of_few_rows(products):
    head = {(d, rows): _forms(products, 1, d, rows)[2] for d in (1536, 2048, 2432, 2560, 3072, 4096) for rows in (1, 8, 16, 17)}
    eight = {k for k, form in head.items() if form == (8, 1, 2)}
    assert eight == {(2432, 1), (2432, 8), (2560, 1), (2560, 8), (3072, 1), (3072, 8), (2048, 16), (2432, 16)}


@pytest.mark.parametrize("d", [512, 768, 1024, 2048])
@pytest.mark.parametrize("rows", [1, 16, 17, 32, 33, 48, 49, 64, 100])
def test_no_idle_row_tiles_in_fp32(products, d, rows):
    for _, row_tiles, column_tiles in _forms(products, 0, d, rows):
        assert row_tiles == min((rows + 15) // 16, 4) and (row_tiles, column_tiles) != (3, 5)


@pytest.mark.parametrize("d,split", [(512, 4), (768, 8), (2560, 8), (3072, 8), (3136, 4), (3584, 4), (4032, 4), (4096, 8)])
def test_split_of_the_residual_product(products, d, split):
    """K in 8 but where that would be a second round of blocks that is not full, or fewer than seven steps to a block."""
    for rows in (1, 32, 64):
        r = subprocess.run([products, "forms", "1", str(d), str(4 * d), "515", str(rows)], capture_output=True, text=True, timeout=100)
        assert r.returncode == 0 and r.stdout.splitlines()[1].split()[1:3] == ["split", str(split)], r.stdout


def test_assembly_that_writes_m0_puts_it_back():
    """The register that holds a direct load's LDS address is the compiler's, and no clobber list may name it: assembly that
    sets it saves it first and restores it last."""
    from paper_2403_17031_amd import build
    seen = 0
    for name in sorted(os.listdir(build.CSRC)):
        with open(os.path.join(build.CSRC, name)) as f:
            for text in re.findall(r"\basm\b(?:\s+volatile)?\s*\(((?:\s*\"(?:[^\"\\]|\\.)*\")+)", f.read()):
                lines = "".join(re.findall(r"\"((?:[^\"\\]|\\.)*)\"", text)).replace("\\n\\t", "\\n").split("\\n")
                if not any(re.match(r"\s*s_\w+ m0\b", line) for line in lines):
                    continue
                seen += 1
                saved = re.fullmatch(r"s_mov_b32 (%\d+), m0", lines[0])
                assert saved and lines[-1] == f"s_mov_b32 m0, {saved[1]}", (name, lines)
    assert seen == 1
