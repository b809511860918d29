"""The encoder's threads (csrc/crew.h), compiled on their own: passes in step, and what one of them throws."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2604_02715_amd", "csrc")
PROGRAM = """
#include "crew.h"
#include <cstdio>
#include <cstdlib>
#include <string>
using namespace fluxmoe;
int main(int argc, char** argv) {
    const int n = std::atoi(argv[1]);
    const std::string who = argv[2];                         // none, caller, worker, once, last (pass): who throws
    try {
        Crew crew(n);
        const uint32_t thrower = who == "worker" ? crew.size() - 1 : 0;
        std::atomic<uint64_t> sum{0};
        uint64_t passes = 0;
        crew.run([&](uint32_t me) {
            for (int pass = 0; pass < 3; ++pass) {
                for (uint64_t u; (u = crew.take()) < 1000;) sum += u;
                if (pass == 1 && (who == "caller" || who == "worker") && me == thrower) throw std::bad_alloc();
                if (pass == 2 && who == "last" && me == thrower) throw std::bad_alloc();
                crew.wait([&]() { if (pass == 1 && who == "once") throw std::bad_alloc(); ++passes; });
            }
        });
        std::printf("%llu %llu", (unsigned long long)sum, (unsigned long long)passes);
    } catch (const std::bad_alloc&) {
        std::printf("thrown");
    }
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("crew")
    (d / "main.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-pthread", "-I", CSRC, str(d / "main.cpp"), "-o", str(d / "main")], check=True)
    return str(d / "main")


@pytest.mark.parametrize("threads", [1, 2, 7])
@pytest.mark.parametrize("who", ["none", "caller", "worker", "once", "last"])
def test_passes_and_exceptions(program, threads, who):
    for _ in range(20):
        out = subprocess.run([program, str(threads), who], capture_output=True, text=True, timeout=20)
        assert out.returncode == 0 and out.stdout == ("1498500 3" if who == "none" else "thrown")
