"""What the sample that the sort's intervals come from may overlook (csrc/sd_sample.h), for every size of an index on the CPU: tokens
of a block get equal parts of its interval only where none of them has more than some two hundred entries too many."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2411_04975_amd", "csrc")


def test_what_equal_parts_overlook(tmp_path):
    src = tmp_path / "sample.cpp"
    src.write_text("""
#include <stdio.h>
#include "%s/sd_sample.h"
int main() {
    long long n;
    while (scanf("%%lld", &n) == 1) printf("%%lld %%u %%u %%u\\n", (long long)sd_sample_runs(n), sd_even_slack(n), SIGHTING, UNSEEN);
}
""" % CSRC)
    exe = str(tmp_path / "sample")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-o", exe, str(src)], check=True)
    top = (1 << 31) - 4096
    sizes = [0, 1, 63, 64, 65, 4096, 262_143, 262_144, 262_145, 1 << 24, 1 << 27, (1 << 27) + 64, 134_217_728 * 3 // 2, 1 << 28, 537_000_000,
             10 ** 9, 1 << 30, top - 1, top]
    r = subprocess.run([exe], input="\n".join(map(str, sizes)), capture_output=True, text=True, check=True)
    for n, line in zip(sizes, r.stdout.splitlines(), strict=True):
        runs, slack, sighting, unseen = map(int, line.split())
        assert runs <= -(-n // 64) and runs <= 32768, n
        assert (sighting * 64 * runs + unseen * (1 << 24)) < 1 << 27, n  # no interval is empty
        if n == 0:
            continue
        tokens = slack / sighting * max(n / (64 * runs), 1)  # that `slack` stands for
        assert tokens <= 192 * (1 + 1e-6), (n, tokens)
        if n <= 1 << 27:
            assert slack == 3 * sighting, n
        else:  # and not much less: weights are whole numbers
            assert slack >= 1 and tokens > 192 * (slack / (slack + 1)) - 1, n
