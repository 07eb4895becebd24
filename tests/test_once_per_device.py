"""What the launchers keep per device (csrc/tt_once.h), compiled for the host: every device gets its own turn, a failure is
tried again, threads agree.  And no launcher keeps a plain flag of its own beside it."""
import glob
import os
import re
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2101_11714_amd", "csrc")

PROGRAM = r"""
#include <cassert>
#include <thread>
#include <vector>
#include "tt_once.h"

int main()
{
    tt::OncePerDevice once;
    int calls = 0;
    auto ok = [&] { ++calls; return 0; };
    assert(once(0, [&] { ++calls; return 7; }) == 7 && calls == 1);      // failed: not done
    assert(once(0, ok) == 0 && once(0, ok) == 0 && calls == 2);
    assert(once(1, ok) == 0 && once(63, ok) == 0 && calls == 4);         // devices of their own
    assert(once(0, ok) == 0 && once(1, ok) == 0 && calls == 4);
    assert(once(64, ok) == 0 && once(64, ok) == 0 && calls == 6);        // beyond what is remembered: every time
    tt::OncePerDevice other;
    std::atomic<int> n{0};
    std::vector<std::thread> ts;
    for (int t = 0; t < 8; ++t) ts.emplace_back([&, t] { for (int i = 0; i < 1000; ++i) assert(other((t + i) % 8, [&] { ++n; return 0; }) == 0); });
    for (auto &t : ts) t.join();
    assert(n >= 8 && n <= 64);
    return 0;
}
"""


def test_every_device_has_its_turn(tmp_path):
    src = tmp_path / "once.cpp"
    src.write_text(PROGRAM)
    exe = str(tmp_path / "once")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-pthread", "-fsanitize=thread", "-I", CSRC, str(src), "-o", exe])
    subprocess.check_call([exe])


def test_kernel_attributes_are_set_through_it():
    for path in glob.glob(os.path.join(CSRC, "*")):
        text = open(path).read()
        assert not re.search(r"static bool \w+ = false", text), path
        if os.path.basename(path) not in ("tt_common.h", "tt_emb.hip"):      # the helper, and the one that sets it on every call
            assert "hipFuncSetAttribute" not in text, path
