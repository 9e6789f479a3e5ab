"""The build's page-locked result words (csrc/pinned_info.h) when a build ends in an error, in a CPU program whose own
functions stand in for the HIP runtime."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2402_05396_amd", "csrc")

PROGRAM = r"""
#include "pinned_info.h"
#include <stdio.h>
#include <stdlib.h>
static int waits = 0;
static hipError_t wait_result = hipSuccess;
extern "C" hipError_t hipHostMalloc(void** p, size_t n, unsigned) { *p = calloc(n, 1); return hipSuccess; }
extern "C" hipError_t hipStreamSynchronize(hipStream_t) { ++waits; return wait_result; }
extern "C" hipError_t hipGetLastError() { return hipSuccess; }
#define EXPECT(x) do { if (!(x)) { printf("line %d: %s\n", __LINE__, #x); return 1; } } while (0)
int main() {
    const hipStream_t stream = reinterpret_cast<hipStream_t>(8);
    unsigned long long* first;
    { PinnedInfo a; first = a.words; EXPECT(first); PinnedInfo b; EXPECT(b.words && b.words != first); }
    { PinnedInfo a; EXPECT(a.words == first && waits == 0); a.launched(stream); a.settled(); }      // a build that went well
    EXPECT(waits == 0);
    { PinnedInfo a; EXPECT(a.words == first); a.launched(stream); }                                 // ended between launch and wait
    EXPECT(waits == 1);
    wait_result = hipErrorUnknown;
    { PinnedInfo a; EXPECT(a.words == first); a.launched(stream); }                                 // and the wait fails as well
    EXPECT(waits == 2);
    { PinnedInfo a; EXPECT(a.words && a.words != first); }                                          // that slot is left alone
    for (int i = 0; i < 63; ++i) { PinnedInfo a; EXPECT(a.words && a.words != first); a.launched(stream); }
    { PinnedInfo a; EXPECT(a.words == nullptr); a.launched(stream); }                               // none left: the build reads back
    EXPECT(waits == 65);
    return 0;
}
"""


def test_a_slot_is_not_handed_on_while_a_kernel_may_write_it(tmp_path):
    (tmp_path / "p.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__=1", "-I", CSRC, "-isystem", "/opt/rocm/include", "-o", str(tmp_path / "p"),
                    str(tmp_path / "p.cpp")], check=True)
    r = subprocess.run([str(tmp_path / "p")], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
