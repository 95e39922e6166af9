"""Host arithmetic of the two-launch wide block (csrc/cf_ffn_plan.h), walked
through on the CPU: the header is compiled into a small program."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2404_03617_amd", "csrc")


def run_cpp(tmp_path, body):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("g++ not found")
    src, exe = tmp_path / "plan.cpp", tmp_path / "plan"
    src.write_text('#include "cf_ffn_plan.h"\n#include <stdio.h>\nusing namespace cf::ffn;\n'
                   "int main() {\n%s\nreturn 0;\n}\n" % body)
    subprocess.run([cxx, "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout[-2000:]


def test_every_group_that_is_counted_holds_chunks(tmp_path):
    """For every chunk count, wish and room: the groups that the kernel's
    grid covers with group_chunks chunks each are all of those counted, none
    is empty, they fit the room, and the count is a fixed point (what
    launch_ffn_block asks for)."""
    run_cpp(tmp_path, """
    for (int chunks = 1; chunks <= 130; chunks++)
        for (int want = 1; want <= 70; want++)
            for (int room = 0; room <= 70; room++) {
                const int g = fitting_groups(chunks, want, 1000, (size_t)room * 1000 + 999);
                const int per = group_chunks(chunks, g);
                const bool ok = g >= 1 && g <= want && (g == 1 || g <= room) && (g - 1) * per < chunks &&
                                g * per >= chunks && filled_groups(chunks, g) == g;
                if (!ok) {
                    printf("chunks %d want %d room %d: %d groups of %d\\n", chunks, want, room, g, per);
                    return 1;
                }
            }
    """)
