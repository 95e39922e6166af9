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


def test_depthwise_launches_stay_below_the_thread_limit(tmp_path):
    """Every call that the two-launch block takes has a depth-wise grid of
    fewer than 2^32 threads, by the kernel's own count (strips of four or
    seven pixels, C / 8 threads each, 256 to a workgroup), up to the 2^31 pixels
    that the entry points take; what it takes of narrow images ends at 64 GiB
    for one column and 128 GiB for two."""
    run_cpp(tmp_path, """
    const int Cs[] = {128, 256, 512};
    for (int C : Cs)
        for (int W = 1; W <= 600; W++)
            for (int64_t P = 1; P < (int64_t)1 << 31; P += P / 3 + 1) {
                const int64_t rows = P / W;
                if (rows < 1 || !dw_launchable(rows, W, C))
                    continue;
                const bool seven = (W + 6) / 7 * 7 <= (W + 3) / 4 * 4;
                for (int tw = 4; tw <= (seven ? 7 : 4); tw += 3) {
                    const int64_t strips = rows * ((W + tw - 1) / tw), per = 256 / (C / 8);
                    const int64_t threads = (strips + per - 1) / per * 256;
                    if (threads >= (int64_t)1 << 32 || strips >= (int64_t)1 << 31) {
                        printf("C %d W %d rows %lld: %lld threads\\n", C, W, (long long)rows, (long long)threads);
                        return 1;
                    }
                }
            }
    for (int C : Cs) {
        const int64_t one = ((int64_t)1 << 36) / (2 * C), two = ((int64_t)1 << 37) / (4 * C);
        if (dw_launchable(one, 1, C) || !dw_launchable(one - 64, 1, C) || dw_launchable(two, 2, C) ||
            !dw_launchable(two - 64, 2, C) || !dw_launchable(((int64_t)1 << 37) / (16 * C), 8, C))
            return 2;
    }
    """)
