"""The rules on sizes that pick a kernel for a block's layers and for attention, on the host.  The expected kernels are those that measured faster on 256 CUs
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
    src.write_text('#include <stdio.h>\n#include <initializer_list>\n#include "gemm_choice.hpp"\n#include "attention_choice.hpp"\nusing namespace rs;\nint main() {\n' + body + "\nreturn 0;\n}\n")
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


def test_fragments_narrow(tmp_path):
    """At most 128 features: tiles no wider than that."""
    _whole(tmp_path, [(65536, 64, 64, 1, "slim 256x128"), (65537, 64, 64, 1, "ring"), (372288, 64, 64, 1, "ring"), (91520, 64, 256, 1, "ring"),
                      (75680, 128, 128, 1, "ring"), (300320, 128, 512, 1, "ring"), (300320, 128, 576, 1, "slim 256x128"),
                      (165252, 128, 1024, 1, "slim 256x128"), (121512, 64, 2048, 1, "slim 256x128"), (75732, 192, 64, 0, "direct")])


def test_fragments_few_tiles_beyond_whole_rounds(tmp_path):
    """Long K and a last round of 256 x 256 tiles at most a sixth full: whole rounds to the persistent kernel, the rest to a tile of its own."""
    got = _frag(tmp_path, [(16388, 1024, 4096, 1), (23000, 768, 3072, 1), (45568, 768, 3072, 1), (33200, 1024, 4096, 1)])
    assert got == [[("persistent", 16384), ("slim 64x64", 4)], [("persistent", 21760), ("slim 64x64", 1240)],
                   [("persistent", 43520), ("slim 128x64", 2048)], [("persistent", 32768), ("slim 64x64", 432)]]
    _whole(tmp_path, [(20000, 1024, 4096, 1, "direct"), (27392, 768, 3072, 1, "direct"), (50432, 768, 3072, 1, "direct"),
                      (36000, 448, 1792, 1, "direct"), (16384, 1024, 4096, 1, "persistent"), (21760, 768, 3072, 1, "persistent"),
                      (33536, 768, 3072, 1, "persistent"), (41216, 768, 3072, 1, "persistent"), (50432, 384, 1536, 1, "direct"),
                      (50000, 512, 2048, 1, "direct"), (25216, 384, 1536, 1, "persistent")])


def test_fragments_every_row_goes_to_one_kernel(tmp_path):
    """The choice ends, and leaves no row out and no launch empty, at all widths and chips."""
    out = _run(tmp_path, r"""
    long n = 0;
    for (int64_t cus : {8, 64, 256, 304})
        for (int64_t p : {0, 1, 2, 3, 7, 64, 85, 86, 197, 4096})
            for (int64_t d : {-1, 0, 1, 64, 65, 255})
                for (int64_t N : {64, 128, 192, 320, 768, 1024, 3072, 65536, 65600, 196608, 1048576})
                    for (int K : {64, 384, 512, 576, 768, 1472, 1536, 2048, 4096})
                        for (int res : {0, 1}) {
                            int64_t left = p * 256 + d;
                            for (int parts = 0; left > 0; ++n) {
                                const GemmChoice c = gemm_choose_frag(left, N, K, cus, res);
                                if (c.rows < 1 || c.rows > left || (c.rows < left && c.rows % 256) || ++parts > 64) return 1;
                                left -= c.rows;
                            }
                        }
    printf("ok\n");""")
    assert out == ["ok"]


def _f32(tmp_path, cases):
    """Workgroups per CU on shared tiles, 0 = split tiles, of each problem (M, N, K)."""
    return [int(l) for l in _run(tmp_path, "".join('printf("%%d\\n", gemm_f32_choose(%d, %d, %d, 256).per_cu);\n' % c for c in cases))]


def test_fp32_tiles(tmp_path):
    """A tile alone behind four rounds is what three workgroups per CU avoid; split tiles where the shared ones leave the chip empty."""
    cases = [((2176, 2304, 2048), 3), ((6544, 768, 3072), 3), ((25600, 192, 768), 3), ((4800, 1024, 1024), 3), ((7168, 1024, 4096), 3),
             ((30000, 192, 192), 4), ((65536, 64, 192), 4), ((65537, 64, 192), 3), ((81919, 64, 192), 4), ((81857, 64, 192), 4), ((81856, 64, 192), 3),
             ((12608, 768, 192), 4), ((12608, 768, 768), 4), ((3152, 576, 192), 4), ((10088, 192, 768), 4), ((20000, 192, 768), 4),
             ((12608, 192, 768), 0), ((8192, 192, 768), 0), ((788, 192, 768), 0), ((2000, 768, 3072), 0), ((4000, 768, 3072), 4),
             ((76800, 64, 2048), 0), ((48640, 64, 2048), 4), ((65536, 64, 2048), 4), ((65537, 64, 2048), 0), ((90048, 64, 2048), 0), ((90112, 64, 2048), 3), ((76800, 64, 1024), 3), ((1, 64, 64), 0)]
    assert _f32(tmp_path, [c for c, _ in cases]) == [n for _, n in cases]


def _attention(tmp_path, cases):
    """(query rows per workgroup, workgroups per head, tail) of each (heads in all, N)."""
    body = "".join('{ const AttentionPlan p = attention_plan(%d, %d, 256); printf("%%d %%d %%d\\n", p.rows, p.q_tiles, (int)p.tail); }\n' % c for c in cases)
    return [tuple(map(int, l.split())) for l in _run(tmp_path, body)]


def test_attention_plans_reach_what_the_gpu_tests_say(tmp_path):
    from test_gpu_attention_row_tiles import ROW_TILES
    from test_gpu_parity import ATT_PLANS
    got = _attention(tmp_path, [(B * H, N) for B, N, H, _ in ATT_PLANS])
    assert [-r if tail else r for r, _, tail in got] == [p[3] for p in ATT_PLANS]
    assert {p[3] for p in ATT_PLANS} == {128, 256, -256}
    assert [p[0:3:2] for p in _attention(tmp_path, [(h, N) for N, h in ROW_TILES])] == [(256, 0)] * len(ROW_TILES)
    assert [p[0:3:2] for p in _attention(tmp_path, [(1, N) for N, _ in ROW_TILES])] == [(128, 0)] * len(ROW_TILES)


def test_attention_plan_covers_every_row(tmp_path):
    cases = [(bh, n) for bh in (1, 7, 8, 49, 96, 128, 1000) for n in list(range(257, 2700, 7)) + [2304, 2305, 2368, 2369, 4096, 4097, 4160]]
    for (bh, n), (rows, tiles, tail) in zip(cases, _attention(tmp_path, cases)):
        assert rows in (128, 256)
        if tail:
            assert rows == 256 and 0 < n - rows * tiles <= 64, (bh, n)
        else:
            assert (tiles - 1) * rows < n <= tiles * rows, (bh, n)


def test_fragment_kernels_of_the_gpu_tests(tmp_path):
    from test_gpu_fragment_weights import BY_SHAPE
    got = _frag(tmp_path, [p for (B, N, D, Dm), _ in BY_SHAPE for p in ((B * N, 3 * D, D, 0), (B * N, D, D, 1), (B * N, Dm, D, 0), (B * N, D, Dm, 1))])
    names = [" + ".join(k for k, _ in g) for g in got]
    assert [names[i:i + 4] for i in range(0, len(names), 4)] == [want for _, want in BY_SHAPE]


def test_fp32_sizes_of_the_gpu_tests(tmp_path):
    """The whole call on shared tiles, the calls it is compared with on split ones."""
    from test_gpu_fp32_kernels import SHARED_TILES
    assert _f32(tmp_path, [(M, N, K) for M, K, N, _ in SHARED_TILES]) == [c[3] for c in SHARED_TILES]
    parts = [(m, N, K) for M, K, N, _ in SHARED_TILES for step in [1024 if N > 64 else 2048] for m in (step, M % step or step)]
    assert set(_f32(tmp_path, parts)) == {0}
