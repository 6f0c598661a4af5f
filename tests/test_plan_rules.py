"""The rules that choose a kernel's tile (csrc/nmfa_plan.h), compiled for the CPU: their choice at sizes on
both sides of a line where both were measured on a device of 256 CUs."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1806_08422_amd", "csrc")


def _run(tmp_path_factory, body):
    d = tmp_path_factory.mktemp("plan")
    src, exe = d / "plan.cpp", d / "plan"
    src.write_text(f'#include "nmfa_plan.h"\n#include <cstdio>\n#include <cstdlib>\nusing namespace nmfa;\n'
                   f'int main(int argc, char** argv) {{ auto arg = [&](int k) {{ return atoi(argv[k]); }}; {body} }}\n')
    subprocess.check_call(["g++", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)])
    return lambda *a: subprocess.check_output([str(exe), *map(str, a)], text=True).split()


@pytest.fixture(scope="module")
def step(tmp_path_factory):
    return _run(tmp_path_factory, 'printf("%d", (int)step_pick(arg(1), arg(2), arg(3), 256).tile); (void)argc;')


# 64x32 alone, 64x32, 128, 256x64, 256x128
@pytest.mark.parametrize("jfmt,n,R,tile", [
    (2, 1300, 3072, 4), (2, 2100, 2048, 4), (2, 2600, 4096, 4), (2, 3100, 1536, 4), (1, 600, 4096, 4),
    (1, 2600, 4096, 4), (0, 2000, 1536, 4), (0, 2000, 2048, 4), (0, 2600, 1536, 4), (0, 5500, 1536, 4), (0, 8192, 1280, 4),
    (2, 8192, 1024, 4), (2, 8192, 512, 3), (2, 2100, 64, 1), (2, 2100, 1024, 2), (1, 2000, 1536, 3), (0, 2100, 64, 0),
    (0, 8192, 64, 0), (0, 8192, 256, 2), (0, 2000, 1024, 2)])
def test_step_tile(step, jfmt, n, R, tile):
    assert step(jfmt, n, R) == [str(tile)]


@pytest.fixture(scope="module")
def small(tmp_path_factory):
    return _run(tmp_path_factory, 'SmallSplit s = small_split(arg(1), arg(2), arg(3), 256); '
                                  'printf("%d %d", s.split, s.ls); (void)argc;')


# waves of a workgroup (n / 16, rounded up), replicas -> waves per tile, columns per replica
@pytest.mark.parametrize("fp64,waves,R,want", [
    (1, 1, 64, (4, 2)), (1, 2, 256, (2, 2)), (1, 2, 5000, (1, 1)), (1, 3, 1024, (1, 4)), (1, 4, 1025, (1, 2)),
    (1, 5, 64, (1, 4)), (1, 7, 1000, (1, 4)), (1, 7, 1024, (1, 4)), (1, 7, 1025, (1, 2)), (1, 7, 2049, (1, 1)),
    (0, 1, 64, (1, 2)), (0, 7, 2048, (1, 2)), (0, 16, 2049, (1, 1))])
def test_small_split(small, fp64, waves, R, want):
    assert small(fp64, waves, R) == [str(x) for x in want]
