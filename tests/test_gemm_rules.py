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
        std::printf("%d %d %d", p.mt, p.passes, (int)p.cached);
        const GemmOut outs[3] = {GEMM_SUMS, GEMM_CHANNELS, GEMM_LM};
        for (GemmOut out : outs) std::printf(" %d", gemm_tile(M, N, K / split / 64, split, wn, out));
        std::printf("\\n");
    }
}
"""
SUMS, CHANNELS, LM = 3, 4, 5                                 # columns of the answer
FEW, SMALL, WIDE, HALVES = 0, (256096, 256128, 256160), (192256, 192320, 256256), (2192128, 2256128)
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
    for (M, N, K, split, wn), (mt, passes, _, *tiles) in zip(calls, rules(calls)):
        assert 1 <= mt <= 6 and (passes - 1) * mt * 32 < M <= passes * mt * 32, (M, N, mt, passes)
        for t in tiles:
            assert t in (FEW, *SMALL, *WIDE, *HALVES), (M, N)
            if t:
                parts = 2 if t in HALVES else split
                assert M > 192 and -(-N // (t // 1000 % 1000)) * parts * -(-M // (t % 1000)) >= 112, (M, N, t)
        assert tiles[1] not in HALVES and tiles[2] not in HALVES and (split > 2 or tiles[0] not in HALVES), (M, N)


def test_weights_that_several_passes_read_are_cached(rules):
    calls = [(M, *s) for s in SHAPES for M in (1, 32, 33, 64, 160, 192, 193, 384, 1000, 2304)]
    for call, (_, passes, cached, *_) in zip(calls, rules(calls)):
        assert cached == (passes > 1), call


def test_choices_that_measure_at_least_5_percent_faster_than_another_kind(rules):
    """Attention output of the 8B shape: one partial sum per slice at 448 to 512 rows, two halves at 896 and 1000; its down projection
    in halves from 576 to 1000 rows, not at 512.  Gate/up of a 3072 and a 1600 wide model: the few-row kernel at 193 to 288 rows."""
    qkv, o, gu, down, lm = SHAPES[:5]
    ask = lambda shape, rows, col: [r[col] for r in rules([(M, *shape) for M in rows])]
    assert all(t in SMALL for t in ask(o, (448, 480, 512), SUMS))
    assert all(t in HALVES for t in ask(o, (896, 1000), SUMS))
    assert all(t in HALVES for t in ask(down, (576, 704, 768, 896, 1000), SUMS)) and ask(down, (512,), SUMS) == [256256]
    for shape in ((16384, 3072, 1, 4), (12800, 1600, 1, 4)):
        assert ask(shape, (193, 224, 256, 288), CHANNELS) == [FEW] * 4


def test_gate_up_blocks(tmp_path):
    """Blocks of three tiles where they divide the matrix, for one row tile, and up to 192 rows with at least 160 of them; the row
    counts and shapes of test_gpu_few_row_passes.py meet blocks of three that do not divide the matrix, and of four."""
    (tmp_path / "p.cpp").write_text('#include <cstdio>\n#include "gemm_rules.h"\nint main() { int M, N; while (std::scanf("%d %d", &M, &N) == 2) '
                                    'std::printf("%d\\n", gemm_channels_block(M, N)); }')
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(tmp_path / "p.cpp"), "-o", str(tmp_path / "p")], check=True)
    ask = lambda calls: [int(v) for v in subprocess.run([str(tmp_path / "p")], input="".join("%d %d\n" % c for c in calls), capture_output=True,
                                                        text=True, check=True).stdout.split()]
    assert ask([(M, 24576) for M in (1, 32, 33, 192, 193, 2304)]) == [3] * 6
    assert ask([(M, 37888) for M in (1, 32, 33, 192, 193)]) == [3, 3, 3, 3, 4]
    assert ask([(M, 400 * 32) for M in (1, 32, 33, 192, 193)]) == [3, 3, 4, 4, 4]
    from test_gpu_few_row_passes import SHAPES as MODELS
    assert any(2 * m["d_ffn"] // 32 % 3 for m in MODELS)


def test_gpu_test_reaches_every_tile(rules):
    """Row counts and shapes of test_gpu_many_rows.py, through the whole rule: every height of the 256-row blocks with every epilogue,
    the fp32 one with K whole and in 2, 4 and 8 slices, and every height among the row counts compared with fp64."""
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
                t = r[{"f32": SUMS, "swiglu": CHANNELS, "lm": LM}[epi]]
                if t in SMALL:
                    seen.add((epi, split, t))
                    if M in ROWS64 and epi != "swiglu":
                        seen64.add((epi, t))
    assert {(e, t) for e, _, t in seen} == {(e, t) for e in ("f32", "swiglu", "lm") for t in SMALL}
    assert {(s, t) for e, s, t in seen if e == "f32"} >= {(s, t) for s in (1, 2, 4, 8) for t in SMALL}, sorted(seen)
    assert seen64 == {(e, t) for e in ("f32", "lm") for t in SMALL}, sorted(seen64)


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
