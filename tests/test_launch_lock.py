"""The lock that a call holds from taking its stream's scratch to its
launches: one per stream. Calls on one stream exclude each other, calls on
different streams do not wait (a small C++ program on the library's own
context object; no GPU)."""
import os
import subprocess

from paper_1807_09932_amd import build

PROGRAM = r"""
#include <chrono>
#include <cstdio>
#include <future>

#include "ebic_runtime_internal.h"

int main()
{
    ebic_ctx ctx;
    hipStream_t a = reinterpret_cast<hipStream_t>(16), b = reinterpret_cast<hipStream_t>(32);
    std::unique_lock<std::mutex> held = ebic::launch_lock(&ctx, a);
    auto other = std::async(std::launch::async, [&] { ebic::launch_lock(&ctx, b); });
    if (other.wait_for(std::chrono::seconds(20)) != std::future_status::ready) {
        std::printf("a call on another stream waits\n");
        std::fflush(stdout);
        std::_Exit(1);
    }
    auto same = std::async(std::launch::async, [&] { ebic::launch_lock(&ctx, a); });
    if (same.wait_for(std::chrono::milliseconds(300)) == std::future_status::ready) {
        std::printf("a call on the same stream does not wait\n");
        return 1;
    }
    held.unlock();
    same.wait();
    return 0;
}
"""


def test_streams_have_their_own_lock(tmp_path):
    source, program = tmp_path / "lock.cpp", tmp_path / "lock"
    source.write_text(PROGRAM)
    rocm = os.path.dirname(os.path.dirname(build.hipcc()))
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", build.CSRC, "-I", f"{rocm}/include",
                    str(source), build.LIB, f"-Wl,-rpath,{build.PKG}", f"-Wl,-rpath-link,{rocm}/lib", "-pthread",
                    "-o", str(program)], check=True)
    env = dict(os.environ, LD_LIBRARY_PATH=f"{rocm}/lib:" + os.environ.get("LD_LIBRARY_PATH", ""))
    r = subprocess.run([str(program)], capture_output=True, text=True, timeout=60, env=env)
    assert r.returncode == 0, r.stdout + r.stderr
