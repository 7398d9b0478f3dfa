"""The wait of the redo kernels (csrc/redo_wait.h), on the CPU: it ends when the count is there, when more than the count is there, and
when the count never comes."""
import os
import re
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1905_06900_amd", "csrc")

PROGRAM = r"""
#include "redo_wait.h"
#include <cstdio>
int main()
{
    // a counter that grows by one a look, from 0 up to `most`
    auto wait = [](uint32_t most, uint32_t n, uint32_t patience, uint32_t &looks, uint32_t &pauses) {
        uint32_t value = 0;
        looks = pauses = 0;
        return dcpq::wait_until([&] { ++looks; return value < most ? value++ : most; }, [&] { ++pauses; }, n, patience);
    };
    uint32_t looks, pauses;
    bool ok = true;
    ok = ok && wait(7, 5, 100, looks, pauses) && looks == 6 && pauses == 5;           // there after some looks
    ok = ok && wait(0, 0, 0, looks, pauses) && looks == 1 && pauses == 0;             // there at once
    ok = ok && !wait(4, 5, 100, looks, pauses) && looks == 101 && pauses == 100;      // never there
    uint32_t past = 9;                                                                // more than what is waited for, at once
    ok = ok && dcpq::wait_until([&] { return past; }, [] {}, 5u, 0u);
    ok = ok && (dcpq::kRedoGivenUp & ((1ull << 62) - 1)) == 0;                        // (no number of items reaches the bit)
    std::puts(ok ? "ok" : "wrong");
    return ok ? 0 : 1;
}
"""


def test_wait_always_ends(tmp_path):
    src = tmp_path / "wait.cpp"
    src.write_text(PROGRAM)
    exe = tmp_path / "wait"
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    assert subprocess.run([str(exe)], capture_output=True, text=True, timeout=20).stdout.strip() == "ok"


def test_no_other_wait_for_another_workgroup():
    # a loop over a load of what another workgroup writes stands in wait_until only
    for name in sorted(os.listdir(CSRC)):
        with open(os.path.join(CSRC, name)) as f:
            text = f.read()
        assert not re.search(r"while\s*\([^;{]*(agent_load|__hip_atomic_load)", text), name
        assert "s_sleep" not in text or "wait_until(" in text, name
