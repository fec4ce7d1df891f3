"""CPU: what a failed kernel launch leaves behind, with a stand-in for the HIP runtime's two functions."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = r"""
#include "flexiq_internal.h"

static hipError_t answer = hipSuccess, last = hipSuccess;   // (the runtime keeps the last error until it is asked for)
extern "C" hipError_t hipLaunchKernel(const void *, dim3, dim3, void **, size_t, hipStream_t)
{
    if (answer != hipSuccess) last = answer;
    return answer;
}
extern "C" hipError_t hipGetLastError(void)
{
    const hipError_t e = last;
    last = hipSuccess;
    return e;
}
struct Params {
    int a;
};
static void kernel(const Params) {}

int main()
{
    for (hipError_t e : {hipErrorInvalidConfiguration, hipErrorOutOfMemory, hipErrorStreamCaptureImplicit}) {
        answer = e;
        if (flexiq::launch_kernel<Params>(kernel, dim3(1), dim3(64), 0, nullptr, Params{1}) != e) return 1;
        if (last != hipSuccess) return 2;   // the caller has been told: nobody else is to hear of it
    }
    answer = hipSuccess;
    last = hipErrorNotReady;   // somebody else's, not for this call to report or to take away
    if (flexiq::launch_kernel<Params>(kernel, dim3(1), dim3(64), 0, nullptr, Params{1}) != hipSuccess) return 3;
    return last == hipErrorNotReady ? 0 : 4;
}
"""


def test_a_failed_launch_leaves_no_error_behind(tmp_path):
    source, program = tmp_path / "launch.cpp", tmp_path / "launch"
    source.write_text(PROGRAM)
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.check_call(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-isystem", os.path.join(rocm, "include"), "-I", os.path.join(ROOT, "include"),
                           "-I", os.path.join(ROOT, "paper_2510_02822_amd", "csrc"), str(source), "-o", str(program)])
    assert subprocess.call([str(program)]) == 0
