"""Which files of the tuning cache are read: those of this build's shapes. A
file without their number, or with another, holds shapes that were the fastest
of other kernels, and gives no entries (a small C++ program on the library's
own reader; no GPU)."""
import os
import subprocess

from paper_1807_09932_amd import build

PROGRAM = r"""
#include <cstdio>

#include "ebic_runtime_internal.h"

int main(int argc, char **argv)
{
    for (int i = 1; i < argc; ++i) {
        ebic_ctx ctx;
        ebic::load_tune_cache(&ctx, argv[i]);
        std::printf("%d ", (int)ctx.tuned.size());
    }
    return 0;
}
"""

ENTRIES = ('"entries": [\n'
           '  {"kind": 0, "rows_b": 18, "cols_b": 6, "n_b": 9, "k_b": 4, "L": 1, "W": 4, "P": 4, "staging": 6},\n'
           '  {"kind": 1, "rows_b": 18, "cols_b": 6, "n_b": 9, "k_b": 0, "L": 4, "W": 8, "P": 64, "staging": 3}\n]}\n')


def test_files_of_other_shapes_are_skipped(tmp_path):
    source, program = tmp_path / "cache.cpp", tmp_path / "cache"
    source.write_text(PROGRAM)
    rocm = os.path.dirname(os.path.dirname(build.hipcc()))
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", build.CSRC, "-I", f"{rocm}/include",
                    str(source), build.LIB, f"-Wl,-rpath,{build.PKG}", f"-Wl,-rpath-link,{rocm}/lib", "-pthread",
                    "-o", str(program)], check=True)
    heads = ['{"arch": "gfx950:sramecc+:xnack-", "shapes": 2, ', '{"arch": "gfx950", ', '{"shapes": 1, ',
             '{"shapes": 3, ']
    files = []
    for i, head in enumerate(heads):
        files.append(tmp_path / f"{i}.json")
        files[-1].write_text(head + ENTRIES)
    env = dict(os.environ, LD_LIBRARY_PATH=f"{rocm}/lib:" + os.environ.get("LD_LIBRARY_PATH", ""))
    r = subprocess.run([str(program), *map(str, files)], capture_output=True, text=True, timeout=60, env=env)
    assert r.returncode == 0, r.stderr
    assert r.stdout.split() == ["2", "0", "0", "0"]
