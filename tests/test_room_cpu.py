"""CPU: the room that a surrogate batch's network rows get
(paper_2410_05408_amd/csrc/gl_room.h), built for the host."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
MEM = 288 << 30


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("needs g++")
    exe = str(tmp_path_factory.mktemp("room") / "gl_room_check")
    subprocess.run([cxx, "-O2", "-std=c++17", "-I", os.path.join(ROOT, "paper_2410_05408_amd", "csrc"),
                    os.path.join(ROOT, "tests", "host", "gl_room_check.cpp"), "-o", exe], check=True)
    return lambda *a: subprocess.run([exe, *map(str, a)], capture_output=True, text=True, check=True).stdout


@pytest.mark.parametrize("n_out", [1, 300, 140000, (1 << 20) - 1, 1 << 20, 12288000, 1 << 26, 1 << 28])
def test_rows_of_a_first_batch(check, n_out):
    # 2^24 rows, the sub-samples that the lists of an earlier pipeline held, as
    # far as 16 per output need them
    rows = int(check("rows", n_out, 0, 0, MEM))
    assert rows >= min(16 * n_out, 1 << 24) and rows >= min(16 * n_out, n_out // 4)
    assert rows <= max(16 * n_out, 1)


def test_rows_follow_the_demand(check):
    assert int(check("rows", 300, 19200, 4800, MEM)) == 24000
    assert int(check("rows", 300, 4000, 4800, MEM)) == 4800
    assert int(check("rows", 1 << 26, 1 << 40, 1 << 24, MEM)) == MEM // 8 // 52
    assert int(check("rows", 1 << 26, 0, 0, 1 << 30)) == (1 << 30) // 8 // 52


@pytest.mark.parametrize("held", [0, 1])
@pytest.mark.parametrize("fail_at", [0, 1, 2, 9])
def test_rows_stay_where_no_more_can_be_had(check, held, fail_at):
    ok, good, kept, there, live = map(int, check("replace", held, fail_at).split())
    assert good
    if fail_at == 9:
        assert (ok, kept, there, live) == (1, 0, 3, 3)
    else:
        assert (ok, kept, there, live) == (0, 3, 3 * held, 3 * held)
