"""The choice of the bf16 GEMM kernel by shape, on the host: it ends, every row goes to exactly one kernel, and no
launch is empty, for every problem the linear layer accepts: M around the 256-row panels, N around the
widths at which one panel alone is a round of the chip (256 columns per CU) or several."""
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

DRIVER = r"""
#include <stdio.h>
#include <initializer_list>
#include "gemm_choice.hpp"
int main() {
    const int64_t cus_of[] = {8, 64, 256, 304};
    long problems = 0;
    for (int64_t cus : cus_of) {
        int64_t ms[400], ns[400];
        int nm = 0, nn = 0;
        for (int64_t p : {0, 1, 2, 3, 4, 7, 64, 197, 4096})
            for (int64_t d : {-1, 0, 1, 64, 65}) if (p * 256 + d > 0) ms[nm++] = p * 256 + d;
        for (int64_t n = 64; n <= 1024; n += 192) ns[nn++] = n;
        for (int r = 1; r <= 4; ++r)
            for (int64_t d : {-256, -64, 0, 64, 128, 192, 256, 8192, 32768})
                if (r * 256 * cus + d > 0 && r * 256 * cus + d <= (1 << 20)) ns[nn++] = r * 256 * cus + d;
        ns[nn++] = 1 << 20;
        for (int i = 0; i < nm; ++i)
            for (int j = 0; j < nn; ++j)
                for (int K : {64, 384, 448, 1984, 2048, 4096}) {
                    int64_t left = ms[i];
                    int parts = 0;
                    while (left > 0) {
                        const rs::GemmChoice c = rs::gemm_choose(left, ns[j], K, cus);
                        if (c.rows < 1 || c.rows > left || (c.rows < left && c.rows % 256) || ++parts > 64) {
                            printf("M %lld N %lld K %d cus %lld: part %d takes %lld of %lld rows\n", (long long)ms[i],
                                   (long long)ns[j], K, (long long)cus, parts, (long long)c.rows, (long long)left);
                            return 1;
                        }
                        left -= c.rows;
                    }
                    ++problems;
                }
    }
    for (int64_t n = 64; n <= (1 << 20); n += 64)
        for (int bm : {32, 64}) {
            const int64_t rows = rs::gemm_f32_launch_rows((int)n, bm), tiles = rows / bm * (n / 64);
            const bool full = tiles + n / 64 > (1 << 24) - 8;   // one more row of tiles would be too many
            if (rows < bm || rows % bm || (tiles + 7) / 8 * 8 * 256 >= (int64_t)1 << 32 || !full) {
                printf("fp32 N %lld tiles of %d rows: %lld rows per launch\n", (long long)n, bm, (long long)rows);
                return 1;
            }
        }
    printf("ok %ld\n", problems);
    return 0;
}
"""


def test_every_row_goes_to_one_kernel(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    src, exe = tmp_path / "choice.cpp", tmp_path / "choice"
    src.write_text(DRIVER)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I" + os.path.join(ROOT, "paper_2508_00367_amd", "csrc"),
                    str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.startswith("ok"), r.stdout


CALL = """
import ctypes, sys
import paper_2508_00367_amd as rs
M, N, K = map(int, sys.argv[1:])
p = [ctypes.c_void_p(0x1000 * i) for i in (1, 2, 3)]
print(rs.lib().rs_linear_fwd(p[0], p[1], None, None, p[2], ctypes.c_int64(M), N, K, rs.RS_EPI_BIAS, rs.RS_BF16, None))
"""


@pytest.mark.parametrize("M,N,K", [(64, 65536, 2048), (64, 65600, 2048), (1, 81920, 4096), (257, 65600, 2048), (256, 98304, 2048),
                                   (200, 1 << 20, 2048)])
def test_wide_linear_layer_returns_a_status(M, N, K):
    """In a process that sees no GPU every launch fails (the pointers are never read), and the call says so."""
    env = dict(os.environ, HIP_VISIBLE_DEVICES="-1", ROCR_VISIBLE_DEVICES="-1", PYTHONPATH=ROOT)
    r = subprocess.run([sys.executable, "-c", CALL, str(M), str(N), str(K)], capture_output=True, text=True, env=env, cwd=ROOT,
                       timeout=120)
    assert r.returncode == 0, (r.returncode, r.stderr[-500:])
    assert r.stdout.split()[-1] == "4"      # RS_ERR_DEVICE
