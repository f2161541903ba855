"""How many waves and how much LDS a drafting launch gets (csrc/sd_plan.h), held to its promises for every tree size on
the CPU: the launch is one that the device takes, and the workgroups that the numbers count on fit a compute
unit's LDS together, the kernel's own static part included."""
import os
import re
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2411_04975_amd", "csrc")

LDS, PIECE, CUS = 160 * 1024, 1280, 256   # gfx950
LEAST = 16384                             # what the occurrence sort needs


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    """{(requests, static LDS, LDS of a wave): (waves, resident, dynamic LDS)}."""
    d = tmp_path_factory.mktemp("plan")
    src = d / "plan.cpp"
    src.write_text("""
#include <stdio.h>
#include "%s/sd_plan.h"
int main() {
    unsigned q, s, w;
    while (scanf("%%u %%u %%u", &q, &s, &w) == 3) {
        const sd_plan p = sd_plan_waves((int)q, %d, %d, %d - s - 256, s, w, %d);
        printf("%%d %%d %%zu\\n", p.waves, p.resident, p.lds);
    }
}
""" % (CSRC, CUS, LDS, LDS, LEAST))
    exe = str(d / "plan")
    subprocess.run(["g++", "-std=c++17", "-O1", "-o", exe, str(src)], check=True)

    def ask(keys):
        r = subprocess.run([exe], input="".join("%d %d %d\n" % k for k in keys), capture_output=True, text=True, check=True)
        return {k: tuple(map(int, line.split())) for k, line in zip(keys, r.stdout.splitlines(), strict=True)}
    return ask


def _wave_lds(nodes):  # frontier and two trees per node, and the staging, as launch_speculate lays them out
    return (60 * nodes + 4 * (3 * 64 + 256) + 7) // 8 * 8


@pytest.mark.parametrize("static", [3040, 8104, 12000])
def test_every_tree_size_has_a_launch_that_fits(plans, static):
    keys = [(q, static, _wave_lds(n)) for n in range(1, 257)
            for q in (1, 255, 256, 257, 512, 513, 768, 769, 1024, 1025, 1280, 1536, 2048, 2049, 8192, 100_000)]
    for (q, _, wave), (waves, resident, lds) in plans(keys).items():
        at = (q, wave, waves, resident, lds)
        assert 1 <= waves <= 16 and resident >= 1, at
        assert lds >= LEAST and lds >= waves * wave, at
        assert lds <= LDS - static - 256, at          # what the device is told to allow
        whole = -(-(lds + static) // PIECE) * PIECE
        assert resident * whole <= LDS, at
        assert resident <= -(-q // CUS), at


def test_the_usual_sizes(plans):
    """Trees of 32 and 64 nodes with the kernel's 8104 bytes: the waves that the launches of one to many requests
    per compute unit are measured with, and one more wave would not have fitted where there are fewer."""
    want = {32: {256: 16, 512: 12, 768: 8, 1024: 6, 2048: 5, 8192: 4},
            64: {256: 16, 512: 12, 768: 8, 1024: 5, 2048: 5, 8192: 4},
            128: {256: 16, 512: 7, 768: 4, 1024: 3, 2048: 3, 8192: 3}}
    for n, rows in want.items():
        got = plans([(q, 8104, _wave_lds(n)) for q in rows])
        assert {k[0]: v[0] for k, v in got.items()} == rows, n


def test_the_launch_plans_with_the_lds_of_the_kernel():
    """The static part that the plan is made with is the kernel's own, whatever it grows to."""
    src = open(os.path.join(CSRC, "sd_speculate.hip")).read()
    call = re.search(r"sd_plan_waves\(([^;]*)\);", src).group(1)
    assert "sizeof(WgShared)" in call
    kernel = src[src.index("void k_speculate("):]
    kernel = kernel[:kernel.index("\n}\n")]
    assert re.findall(r"__shared__ ([^;]*);", kernel) == ["double smem[]", "WgShared sh"]


def test_the_waves_that_are_resident():
    """The launch's own call, with a node of 48 bytes: six workgroups of four waves and the kernel's registers, LDS that would lie idle for the
    occurrence sort, and a launch that the device takes for every tree size."""
    src = """
#include <stdio.h>
#include <initializer_list>
#include "%s/sd_plan.h"
int main() {
    for (int nodes = 1; nodes <= 256; nodes++)
        for (int q : {1, 256, 257, 512, 768, 769, 1024, 1025, 1280, 1281, 1536, 2048, 2049, 4096, 8192, 100000}) {
            const size_t wave = (48 * (size_t)nodes + 4 * (2 * 64 + 256) + 7) / 8 * 8;
            const sd_plan p = sd_plan_waves(q, %d, %d, %d - 8104 - 256, 8104, wave, %d, 2 * %d, 24);
            printf("%%d %%d %%zu %%d %%d %%zu\\n", nodes, q, wave, p.waves, p.resident, p.lds);
        }
}
""" % (CSRC, CUS, LDS, LDS, LEAST, LEAST)
    import tempfile
    with tempfile.TemporaryDirectory() as d:
        path = os.path.join(d, "plan.cpp")
        open(path, "w").write(src)
        subprocess.run(["g++", "-std=c++17", "-O1", "-o", os.path.join(d, "plan"), path], check=True)
        out = subprocess.run([os.path.join(d, "plan")], capture_output=True, text=True, check=True).stdout
    waves_at = {}
    for nodes, q, wave, waves, resident, lds in (map(int, line.split()) for line in out.splitlines()):
        at = (nodes, q, waves, resident, lds)
        assert 1 <= waves <= 16 and resident >= 1 and lds >= LEAST and lds >= waves * wave, at
        assert lds <= LDS - 8104 - 256, at
        whole = -(-(lds + 8104) // PIECE) * PIECE
        assert resident * whole <= LDS and resident <= -(-q // CUS), at
        waves_at[nodes, q] = waves
        if (nodes, q) == (64, 8192):
            assert LDS // whole == 6
    assert [waves_at[64, q] for q in (1024, 1025, 1280, 1281, 2048, 8192)] == [6, 5, 5, 4, 4, 4]
    assert [waves_at[32, q] for q in (1024, 1025, 1280, 1281, 2048, 8192)] == [6, 4, 4, 4, 4, 4]
