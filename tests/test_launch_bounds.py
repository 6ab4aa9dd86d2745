"""Host-side arithmetic of the kernels' loads and launches, compiled from their
own header with the host compiler: what a load may touch, against the memory
that the caller's buffer has, and a launch's size against its 32-bit count."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2602_05774_amd", "csrc")


def _run(tmp_path, body):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text("#include <cstdio>\n#include \"vsd_kernels.hpp\"\nint main() {\n" + body + "\nreturn 0; }\n")
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", CSRC, "-isystem", "/opt/rocm/include",
                    str(src), "-o", str(exe)], check=True, capture_output=True, text=True)
    return subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split()


@pytest.mark.parametrize("n", (1, 8, 40, 257, 1003, 32000))
def test_kmajor_load_stays_in_the_matrix(tmp_path, n):
    """Four rows of stride ld, 16 bytes per lane: within the n columns of the last row, and all of them."""
    strides = [(n + 7) // 8 * 8 + pad for pad in (0, 8, 64, 32000)]
    got = _run(tmp_path, "".join(f'std::printf("%u\\n", vsd::lm_kmajor_bytes({ld}, {n}));\n' for ld in strides))
    for ld, size in zip(strides, map(int, got)):
        # the last byte of the buffer whose columns are n of a wider one, in whole 16-byte chunks of its rows
        assert 2 * (3 * ld + n) <= size <= 2 * (3 * ld + (n + 7) // 8 * 8)


@pytest.mark.parametrize("Vd,Vt", ((1000, 1000), (32000, 32000), (32000, 128256), (70000, 70000), (6145, 65537)))
def test_score_launch_fits_its_grid(tmp_path, Vd, Vt):
    """64 W work-items a row (W = 1: four rows of 64 to a workgroup) stay below 2^32 up to the most rows a call takes."""
    rows = (1, 4, 256, 896, 897, 1024, 1792, 1793, 2 ** 20, 2 ** 22 - 1, 2 ** 22, 2 ** 24 - 1)
    calls = [(r, es, kl, rag) for r in rows for es in (2, 4) for kl in (0, 1) for rag in (0, 1)]
    got = _run(tmp_path, "".join(f'std::printf("%d\\n", vsd::score_waves({r}ll, {Vd}, {Vt}, {es}, {kl}, {rag}));\n'
                                 for r, es, kl, rag in calls))
    for (r, *_), w in zip(calls, map(int, got)):
        assert w in (1, 4, 16) and (r if w > 1 else (r + 3) // 4) * (64 * w if w > 1 else 256) < 2 ** 32
