"""The hand-over between a workgroup's waves (csrc/sd_handover.h) under ThreadSanitizer: the header's own code, a
thread for a wave, its atomics taken as the host's of the same order.  One wave appends to the row, the others
put down their hits; every one counts itself in, waits for all and reads what all have written, as the decode
step does with a frequent token's occurrences.  The same with relaxed orders in the header must be reported."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "paper_2411_04975_amd", "csrc", "sd_handover.h")

PROGRAM = r"""
#include <thread>
#include <vector>
#include <stdio.h>
#define __device__
#define __forceinline__ inline
#define __HIP_MEMORY_SCOPE_WORKGROUP 0
#define __hip_atomic_fetch_add(p, v, order, scope) __atomic_fetch_add(p, v, order)
#define __hip_atomic_load(p, order, scope) __atomic_load_n(p, order)
#define __builtin_amdgcn_s_sleep(n) std::this_thread::yield()
%s
enum { WAVES = 6, EACH = 50 };
int row[EACH], hits[WAVES][EACH], count;
int main() {
    long sum[WAVES] = {};
    for (int rep = 0; rep < 20; rep++) {
        count = 0;
        std::vector<std::thread> waves;
        for (int w = 0; w < WAVES; w++)
            waves.emplace_back([&, w] {
                for (int i = 0; i < EACH; i++) hits[w][i] = rep + w;
                if (w == WAVES - 1)
                    for (int i = 0; i < EACH; i++) row[i] = rep;
                count_in(&count);
                wait_for_count(&count, WAVES);
                for (int i = 0; i < EACH; i++) {
                    sum[w] += row[i];
                    for (int v = 0; v < WAVES; v++) sum[w] += hits[v][i];
                }
            });
        for (auto &t : waves) t.join();
    }
    for (int w = 0; w < WAVES; w++) printf("%%ld\n", sum[w]);
}
"""


def _run(tmp_path, header):
    (tmp_path / "t.cpp").write_text(PROGRAM % header)
    exe = str(tmp_path / "t")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-pthread", "-fsanitize=thread", "-o", exe, str(tmp_path / "t.cpp")],
                       capture_output=True, text=True)
    if r.returncode != 0 and "tsan" in r.stderr:
        pytest.skip("no thread sanitizer runtime for g++ here: " + r.stderr[-300:])
    assert r.returncode == 0, r.stderr
    return subprocess.run([exe], capture_output=True, text=True, timeout=120)


def _header():
    return "".join(line for line in open(HEADER) if not line.startswith(("#pragma", "#include")))


def test_what_counted_waves_stored_is_seen(tmp_path):
    r = _run(tmp_path, _header())
    assert r.returncode == 0 and "WARNING" not in r.stderr, r.stderr[:3000]
    want = 50 * sum(rep * 7 + 15 for rep in range(20))
    assert [int(v) for v in r.stdout.split()] == [want] * 6


@pytest.mark.parametrize("order", ["RELEASE", "ACQUIRE"])
def test_a_relaxed_order_is_reported(tmp_path, order):
    weak = _header().replace("__ATOMIC_" + order, "__ATOMIC_RELAXED")
    assert weak != _header()
    r = _run(tmp_path, weak)
    assert "data race" in r.stderr


def test_the_early_parts_use_it():
    src = open(os.path.join(os.path.dirname(HEADER), "sd_speculate.hip")).read()
    body = src[src.index("unsigned occ_take_chunks("):]
    body = body[:body.index("\n}\n")]
    assert "wait_for_count(&sh.scan_done, nw);" in body and "__restrict__ x" not in body
    scan = src[src.index("void request_occurrences("):]
    scan = scan[:scan.index("\n}\n")]
    assert scan.index("settle();") < scan.index("count_in(&sh.scan_done)") < scan.index("between();")
    assert "__restrict__ x" not in scan
    uses = re.findall(r"(\w+\(&)?sh\.scan_done( = 0)?", src)
    assert sorted(uses) == [("", " = 0"), ("count_in(&", ""), ("wait_for_count(&", "")]
