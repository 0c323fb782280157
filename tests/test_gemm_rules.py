"""The rules that send a GEMM call to a kernel (csrc/gemm_rules.h), compiled with the host compiler."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2510_04147_amd", "csrc")
PROGRAM = """
#include <cstdio>
#include "gemm_rules.h"
int main() {
    int M, N, K, split, wn;
    while (std::scanf("%d %d %d %d %d", &M, &N, &K, &split, &wn) == 5) {
        const GemmPass p = gemm_few_row_pass(M, N, split, wn);
        std::printf("%d %d %d %d", gemm_rows_tile((const void*)4096, M, N, split, wn), p.mt, p.passes, (int)p.cached);
        for (uintptr_t x = 4098; x <= 4112; x += 2) std::printf(" %d", gemm_rows_tile((const void*)x, M, N, split, wn));
        std::printf("\\n");
    }
}
"""
# N, K, split, 32-row weight tiles per few-row work-group
SHAPES = [(12288, 4096, 2, 3), (4096, 4096, 4, 2), (24576, 4096, 1, 3), (4096, 12288, 8, 4), (126464, 4096, 1, 4),
          (4608, 3584, 4, 2), (37888, 3584, 1, 4), (3584, 18944, 8, 4), (768, 512, 4, 2), (512, 512, 4, 2), (3072, 512, 1, 3),
          (512, 1536, 4, 2), (2080, 512, 1, 4), (4800, 1600, 1, 2), (1600, 1600, 1, 2), (12800, 1600, 1, 4),
          (1600, 6400, 5, 4), (5632, 1024, 1, 4), (1024, 2816, 4, 2), (11264, 2048, 1, 4), (32, 64, 1, 2)]


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    (d / "rules.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(d / "rules.cpp"), "-o", str(d / "rules")], check=True)

    def ask(calls):
        text = "".join("%d %d %d %d %d\n" % c for c in calls)
        out = subprocess.run([str(d / "rules")], input=text, capture_output=True, text=True, check=True).stdout
        return [tuple(int(v) for v in line.split()) for line in out.splitlines()]
    return ask


def test_passes_cover_the_rows(rules):
    calls = [(M, *s) for s in SHAPES for M in (1, 31, 32, 33, 64, 65, 96, 97, 160, 161, 192, 193, 320, 321, 384, 385, 1000, 2304, 16384)]
    for (M, N, K, split, wn), (rows_tile, mt, passes, cached) in zip(calls, (r[:4] for r in rules(calls))):
        assert rows_tile in (0, 3, 4, 5) and 1 <= mt <= 6, (M, N)
        assert (passes - 1) * mt * 32 < M <= passes * mt * 32, (M, N, mt, passes)
        assert rows_tile == 0 or (M > 192 and -(-N // 256) * split * -(-M // (32 * rows_tile)) >= 128), (M, N)


def test_weights_that_several_passes_read_are_cached(rules):
    calls = [(M, *s) for s in SHAPES for M in (1, 32, 33, 64, 160, 192, 193, 384, 1000, 2304)]
    for call, (_, mt, passes, cached) in zip(calls, (r[:4] for r in rules(calls))):
        assert cached == (passes > 1), call


def test_two_full_passes_are_kept_where_they_are_faster(rules):
    """8B shape: two 192-row passes of QKV and gate/up beat the many-row kernel at 321 to 384 rows; down, attention
    output and LM head, and every matrix at the rows around them, do not."""
    qkv, o, gu, down, lm = SHAPES[:5]
    for M in (321, 352, 384):
        assert [r[0] == 0 for r in rules([(M, *s) for s in (qkv, o, gu, down, lm)])] == [True, False, True, False, False], M
    for M in (193, 256, 257, 320, 385, 448, 576, 640, 705, 768, 1000, 2304):
        assert all(r[0] > 0 for r in rules([(M, *s) for s in (qkv, o, gu, down, lm)])), M


def test_unaligned_rows_stay_with_the_few_row_kernel(rules):
    """The many-row kernel copies 16 bytes at a time: x at byte offsets 2, 4 ... 14 never goes there, at 16 as at 0."""
    for r in rules([(M, *s) for s in SHAPES for M in (160, 193, 256, 640, 1000, 2304)]):
        assert r[4:] == (0,) * 7 + (r[0],)


def test_gpu_test_reaches_every_tile(rules):
    """Row counts and shapes of test_gpu_many_rows.py: every tile height with every epilogue, the fp32 one with K whole and
    in 2, 4 and 8 slices, and every tile height among the row counts compared with fp64."""
    from paper_2510_04147_amd import synth
    from test_gpu_many_rows import ROWS, ROWS64, SHAPES as MODELS
    seen, seen64 = set(), set()
    for m in MODELS:
        cfg = synth.model_config("8b", **m)
        d, F, nq = cfg["d_model"], cfg["d_ffn"], cfg["n_q_heads"] * cfg["head_dim"]
        for epi, N, K in (("f32", nq + 2 * cfg["n_kv_heads"] * cfg["head_dim"], d), ("f32", d, nq), ("f32", d, F),
                          ("swiglu", 2 * F, d), ("lm", cfg["vocab"], d)):
            if K % 64 or N % 32:
                continue                                     # the plain kernel's
            wn, split = (3 if N // 32 % 3 == 0 else 4) if epi == "swiglu" else 4, 1
            if epi == "f32":                                 # as launch_gemm_mfma_f32 chooses
                wn, split = (3 if N // 32 % 3 == 0 else 4, 2) if N > 8192 else (2, 4) if K <= 4096 else (4, 8)
                while K % (split * 64):
                    split -= 1
            for M, r in zip(ROWS, rules([(M, N, K, split, wn) for M in ROWS])):
                if r[0]:
                    seen.add((epi, split, r[0]))
                    if M in ROWS64 and epi != "swiglu":
                        seen64.add((epi, r[0]))
    assert {(e, t) for e, _, t in seen} == {(e, t) for e in ("f32", "swiglu", "lm") for t in (3, 4, 5)}
    assert {(s, t) for e, s, t in seen if e == "f32"} >= {(s, t) for s in (1, 2, 4, 8) for t in (3, 4, 5)}, sorted(seen)
    assert seen64 == {(e, t) for e in ("f32", "lm") for t in (3, 4, 5)}, sorted(seen64)


def test_plain_gemm_gpu_test_crosses_the_switch(tmp_path):
    """Shapes and row counts of test_gpu_small_tiles.py: every epilogue with at most 256 tiles of 64x64 and with more, close to
    the limit on either side; unaligned operands never take the small tiles."""
    from paper_2510_04147_amd import synth
    from test_gpu_small_tiles import SHAPES as MODELS, rows_of
    (tmp_path / "p.cpp").write_text(
        '#include <cstdio>\n#include "gemm_rules.h"\nint main() { int M, N; while (std::scanf("%d %d", &M, &N) == 2) { '
        'auto f = [&](uintptr_t x, uintptr_t w) { return (int)gemm_plain_small_tiles((const void*)x, (const void*)w, M, N); }; '
        'std::printf("%d %d %d\\n", f(4096, 8192), f(4100, 8192), f(4096, 8194)); } }')
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(tmp_path / "p.cpp"), "-o", str(tmp_path / "p")], check=True)
    calls = []
    for m in MODELS:
        cfg = synth.model_config("tiny", **m)
        for epi, N in (("f32", (cfg["n_q_heads"] + 2 * cfg["n_kv_heads"]) * cfg["head_dim"]), ("f32", cfg["d_model"]),
                       ("swiglu", cfg["d_ffn"]), ("lm", cfg["vocab"])):
            calls += [(epi, M, N, -(-N // 64) * -(-M // 64)) for M in rows_of(m)]
    out = subprocess.run([str(tmp_path / "p")], input="".join("%d %d\n" % c[1:3] for c in calls), capture_output=True, text=True, check=True)
    small = [tuple(int(v) for v in line.split()) for line in out.stdout.splitlines()]
    assert small == [(int(c[3] <= 256), 0, 0) for c in calls]
    for epi in ("f32", "swiglu", "lm"):
        tiles = [c[3] for c in calls if c[0] == epi]
        assert any(246 < t <= 256 for t in tiles) and any(256 < t < 280 for t in tiles), (epi, sorted(tiles)[-6:])
