"""Which launches store a trajectory by rows (csrc/cp_rows.h, built here with
the host compiler): every case of the rows tests on the GPU takes the kernel
that it is there for, and batches whose row blocks would leave CUs idle never
take them, however long the trajectory."""
import os
import subprocess

import pytest

from test_gpu_rows import CASES

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ELEM = {"f32": 4, "f64": 8, "f16": 2}


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("rows") / "rows_rule")
    subprocess.run(["g++", "-std=c++17", "-O1",
                    "-I" + os.path.join(ROOT, "paper_2301_13062_amd", "csrc"),
                    os.path.join(ROOT, "tests", "rows_rule.cpp"), "-o", exe], check=True)

    def ask(cases):
        text = "".join("%d %d %d %d %d\n" % c for c in cases)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout
        return [int(v) for v in out.split()]

    return ask


def test_cases_take_their_kernel(rule):
    base = 1 << 30  # allocations start on lines
    got = rule([(n, T, ELEM[prec], base + shift * ELEM[prec], base + shift * 4)
                for prec, n, T, _, shift, _ in CASES])
    assert got == [block for *_, block in CASES]
    # the other side of the comparison: launches too short for rows
    assert not any(rule([(n, 7, ELEM[prec], base, base) for prec, n, _, _, _, _ in CASES]))


@pytest.mark.parametrize("elem,least", [(4, 128000), (8, 97793), (2, 1000000)])
def test_small_batches_are_stored_by_waves(rule, elem, least):
    sizes = [1, 1000, 4097, 10001, 20001, 50001, 80001, 97791, least - 1]
    steps = [64, 800, 5000, 70000, 1 << 20]
    assert not any(rule([(n, T, elem, 4, 4) for n in sizes for T in steps]))


def test_rounds_of_blocks_full(rule):
    # 512 environments per block (1,024 from 400,000 on): rounds of 256 blocks
    assert rule([(n, 900, 4, 0, 0) for n in (127999, 128001, 131072 + 1, 150001, 196096 + 1)]) \
        == [0, 512, 0, 0, 512]
    # 0.98, 1.15, 1.53, 2.29 and 2.01 rounds
    assert rule([(n, 400, 8, 0, 0) for n in (128001, 150001, 200003, 300007, 526001)]) \
        == [512, 0, 512, 512, 0]
    # binary16, 2,048 per block: 1.91, 2.10, 3.00, 2.97, 6.10 and 3.32
    assert rule([(n, 1200, 2, 0, 0) for n in (1000003, 1100001, 1572001, 1559361, 3200001, 1740801)]) \
        == [1024, 0, 1024, 1024, 0, 0]


def test_bytes(rule):
    # 21 bytes per environment and step against 402,653,184; 13 against 838,860,800
    assert rule([(300007, T, 4, 0, 0) for T in (63, 64)]) == [0, 512]
    assert rule([(3000001, T, 2, 0, 0) for T in (21, 22)]) == [0, 1024]
    # 64-bit products
    assert rule([(2000000001, 1 << 30, 4, 0, 0)]) == [1024]


def test_rows_on_lines_are_stored_by_waves(rule):
    assert rule([(4194304, 64, e, 0, 0) for e in (2, 4, 8)]) == [0, 0, 0]
    assert rule([(4194304, 64, e, 0, 4) for e in (4, 8)]) == [1024, 1024]
