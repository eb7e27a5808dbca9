"""The rules on sizes that pick a kernel for a block's layers, on the host.  The expected kernels are those that measured faster on 256 CUs
at sizes on both sides of each line."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _run(tmp_path, body):
    """Compiles `body` (the inside of main) against the rules and returns the lines it prints."""
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    src, exe = tmp_path / "choice.cpp", tmp_path / "choice"
    src.write_text('#include <stdio.h>\n#include "gemm_choice.hpp"\nusing namespace rs;\nint main() {\n' + body + "\nreturn 0;\n}\n")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I" + os.path.join(ROOT, "paper_2508_00367_amd", "csrc"),
                    str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
    return r.stdout.splitlines()


TILES = ["slim 64x64", "slim 128x64", "slim 128x128", "slim 256x128", "ring", "direct", "persistent"]


def _frag(tmp_path, cases):
    """Kernels and rows of each problem (M, N, K, residual): [[(kernel, rows), ...], ...]."""
    body = ""
    for M, N, K, res in cases:
        body += """{ int64_t left = %d; while (left > 0) { const GemmChoice c = gemm_choose_frag(left, %d, %d, 256, %d);
            if (c.rows < 1 || c.rows > left) return 1;
            printf("%%d %%lld ", (int)c.tile, (long long)c.rows); left -= c.rows; } printf("\\n"); }\n""" % (M, N, K, res)
    out = []
    for line in _run(tmp_path, body):
        v = list(map(int, line.split()))
        out.append([(TILES[t], rows) for t, rows in zip(v[::2], v[1::2])])
    assert len(out) == len(cases)
    return out


def _whole(tmp_path, cases):
    """One kernel for all rows, case by case (M, N, K, residual, kernel)."""
    got = _frag(tmp_path, [c[:4] for c in cases])
    assert got == [[(c[4], c[0])] for c in cases]


def test_fragments_small_tiles(tmp_path):
    _whole(tmp_path, [(1, 64, 64, 0, "slim 64x64"), (256 * 64, 64, 64, 1, "slim 64x64"), (256 * 64 + 1, 64, 64, 1, "slim 128x64"),
                      (256 * 128, 64, 512, 0, "slim 128x64"), (256 * 128 + 1, 64, 512, 0, "slim 256x128"),
                      (128 * 64, 256, 512, 1, "slim 128x64"), (128 * 64 + 1, 256, 512, 1, "slim 128x128"),
                      (128 * 128, 256, 512, 1, "slim 128x128"), (128 * 128 + 1, 256, 512, 1, "slim 256x128")])


def test_fragments_up_to_one_slim_tile_per_cu(tmp_path):
    """Ragged widths, where the direct kernel has more than one tile per CU, and residual layers stay with the slim tiles."""
    _whole(tmp_path, [(8612, 832, 832, 1, "slim 256x128"), (9152, 832, 832, 1, "slim 256x128"), (9100, 832, 1088, 0, "slim 256x128"),
                      (19656, 320, 768, 0, "slim 256x128"), (17000, 320, 1280, 1, "slim 256x128"), (9324, 576, 832, 1, "slim 256x128"),
                      (9244, 768, 768, 1, "slim 256x128"), (8036, 1024, 1024, 1, "slim 256x128"), (24600, 256, 1344, 1, "slim 256x128"),
                      (3368, 2304, 768, 0, "direct"), (2064, 3072, 1024, 0, "direct"), (1968, 3840, 1280, 0, "direct"),
                      (3368, 2304, 704, 0, "slim 256x128"), (3368, 2304, 1536, 0, "slim 256x128")])


def test_fragments_two_slim_tiles_per_cu(tmp_path):
    """More than two direct tiles per CU, but at most two slim ones."""
    _whole(tmp_path, [(13664, 1088, 1088, 1, "slim 256x128"), (23564, 576, 832, 1, "slim 256x128"), (33000, 320, 1280, 1, "slim 256x128"),
                      (10944, 1344, 256, 0, "slim 256x128"), (36000, 384, 1536, 1, "slim 256x128"),
                      (25216, 768, 768, 1, "direct"), (43800, 384, 1536, 1, "direct"), (20280, 768, 640, 0, "direct")])
