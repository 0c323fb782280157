"""The many-row GEMM that walks half of the k-slices in one work-group (two partial sums instead of one per slice), alone through
ssd_k_linear: slice counts of eight, seven, four and three (halves of unequal length), slices of one, two and ten chunks, weight
rows that leave the last block part empty, ragged row counts.

Each slice is a chain of its own and the halves are added as the consumers add partial sums, so every call must equal the
same rows sent in 160-row calls (one partial sum per slice) bit for bit; against fp64 on the identical operands the sums
differ by fp32 rounding only (operands of order 0.5 * 0.02, sums below 4; K <= 4480 makes at most 290 additions: 290 * 2^-24 * 4
< 7e-5 < 2e-4)."""
import os
import subprocess

import pytest
import torch

from paper_2510_04147_amd import synth

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2510_04147_amd", "csrc")
# (d_model, query heads of 128 channels, d_ffn, slices of the attention output projection and of down)
SHAPES = [(4128, 2, 4608, 4, 8), (4192, 4, 4480, 4, 7), (3616, 3, 512, 3, 4), (8160, 2, 256, 4, 4)]
ROWS = (500, 640, 897, 1000, 1281)
TILES = (2256128, 2192128)


def test_rows_and_shapes_reach_both_tiles(tmp_path):
    (tmp_path / "p.cpp").write_text(
        '#include <cstdio>\n#include "gemm_rules.h"\nint main() { int M, N, n, s, w; while (std::scanf("%d %d %d %d %d", &M, &N, &n, &s, &w) == 5) '
        'std::printf("%d\\n", gemm_tile(M, N, n, s, w, GEMM_SUMS)); }')
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(tmp_path / "p.cpp"), "-o", str(tmp_path / "p")], check=True)

    def ask(calls):
        out = subprocess.run([str(tmp_path / "p")], input="".join("%d %d %d %d %d\n" % c for c in calls), capture_output=True, text=True, check=True)
        return [int(v) for v in out.stdout.split()]

    seen = set()
    for d, heads, F, so, sd in SHAPES:
        for K, split, wn in ((heads * 128, so, 2), (F, sd, 2 if F <= 4096 else 4)):
            for M, t in zip(ROWS, ask([(M, d, K // split // 64, split, wn) for M in ROWS])):
                if t in TILES:
                    seen.add((t, split, K // split // 64))
    assert {s[0] for s in seen} == set(TILES), seen
    assert {s[1] for s in seen} == {3, 4, 7, 8}, seen
    assert {s[2] for s in seen} >= {1, 2, 10}, seen
    # a matrix in one or two slices, and rows that one pass of the few-row kernel takes, never
    assert not set(TILES) & set(ask([(1000, 4096, 32, s, 4) for s in (1, 2)] + [(M, 4096, 24, 8, 4) for M in (1, 160, 192)]))


@pytest.mark.gpu
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: f"d{s[0]}")
def test_halves_equal_one_partial_sum_per_slice(shape):
    from paper_2510_04147_amd import binding
    d, heads, F, _, _ = shape
    cfg = synth.model_config("8b", n_layers=1, d_model=d, n_q_heads=heads, n_kv_heads=heads, d_ffn=F, vocab=64)
    w = synth.gen_weights(cfg, 5, device="cuda")
    eng = binding.SSD(cfg, w, max_seqs=1, max_seq_len=64, block=32, max_draft=4, max_rows=max(ROWS))
    g = torch.Generator(device="cuda").manual_seed(7)
    try:
        for M in ROWS:
            for which, K, wt in ((1, heads * 128, w["layers"][0]["wo"]), (3, F, w["layers"][0]["wdown"])):
                x = (torch.randn(M, K, device="cuda", generator=g) * 0.5).bfloat16()

                def call(rows):
                    out = torch.full((rows.shape[0], d), float("nan"), device="cuda")
                    eng.k_linear(which, 0, rows, out)
                    return out

                got = call(x)
                ref = torch.cat([call(x[m:m + 160].contiguous()) for m in range(0, M, 160)])
                assert torch.equal(got, ref), (shape, M, which)
                assert (got.double() - x.double() @ wt.double().T).abs().max() < 2e-4, (shape, M, which)
    finally:
        eng.close()
