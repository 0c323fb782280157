"""The large tiles of the many-row GEMM (256 x 256, 192 x 320 and 192 x 256 weight rows x rows), alone through ssd_k_linear:
row counts around multiples of their 256 and 320 rows; weight rows that leave the last 192- or 256-row block part empty; K
slices of one to six chunks, which is fewer and more than the rings have stages (two or three of activations, three or four of weights).

Every sum is one chain in the order of the few-row kernel, so every call must equal the same rows sent in 160-row calls bit
for bit; against fp64 on the identical operands the fp32 sums differ by fp32 rounding only (operands of order 0.5 * 0.02, sums
below 1; K <= 384 makes at most 24 additions of 16 products each and two slices: 26 * 2^-24 < 2e-6 < 1e-5)."""
import os
import subprocess

import pytest
import torch

from paper_2510_04147_amd import synth

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2510_04147_amd", "csrc")
SHAPES = [dict(d_model=64, d_ffn=8240, vocab=18016, n_q_heads=35, n_kv_heads=35),
          dict(d_model=128, d_ffn=9232, vocab=21152, n_q_heads=35, n_kv_heads=35),
          dict(d_model=192, d_ffn=9008, vocab=17952, n_q_heads=34, n_kv_heads=17),
          dict(d_model=256, d_ffn=8256, vocab=21152, n_q_heads=35, n_kv_heads=35),
          dict(d_model=320, d_ffn=9232, vocab=18016, n_q_heads=34, n_kv_heads=17),
          dict(d_model=384, d_ffn=8240, vocab=17952, n_q_heads=33, n_kv_heads=33)]
ROWS = (447, 512, 513, 577, 640, 641, 768, 769, 960, 1000, 1280, 1281)
WIDE = (256256, 192320, 192256)


def linears(cfg):
    """(which, epilogue, K, output columns, N, split, few-row n-tiles) of the steps whose shapes the matrix-core kernels take."""
    d, F, nq = cfg["d_model"], cfg["d_ffn"], cfg["n_q_heads"] * cfg["head_dim"]
    nqkv = nq + 2 * cfg["n_kv_heads"] * cfg["head_dim"]
    split = 2 if nqkv > 8192 and d % 128 == 0 else 1
    wn = lambda N: 3 if N // 32 % 3 == 0 else 4
    return [(0, "f32", d, nqkv, nqkv, split, wn(nqkv)), (2, "swiglu", d, F, 2 * F, 1, wn(2 * F)), (4, "lm", d, 3, cfg["vocab"], 1, 4)]


def test_rows_and_shapes_reach_every_large_tile(tmp_path):
    (tmp_path / "p.cpp").write_text(
        '#include <cstdio>\n#include "gemm_rules.h"\nint main() { int M, N, n, s, w, o; while (std::scanf("%d %d %d %d %d %d", &M, &N, &n, &s, &w, &o) == 6) '
        'std::printf("%d\\n", gemm_tile(M, N, n, s, w, (GemmOut)o)); }')
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(tmp_path / "p.cpp"), "-o", str(tmp_path / "p")], check=True)

    def ask(calls):
        out = subprocess.run([str(tmp_path / "p")], input="".join("%d %d %d %d %d %d\n" % c for c in calls), capture_output=True, text=True, check=True)
        return [int(v) for v in out.stdout.split()]

    seen = set()
    for m in SHAPES:
        for _, epi, K, _, N, split, wn in linears(synth.model_config("8b", **m)):
            nch = K // split // 64
            for M, t in zip(ROWS, ask([(M, N, nch, split, wn, ("f32", "swiglu", "lm").index(epi)) for M in ROWS])):
                if t in WIDE:
                    block = t // 1000
                    assert -(-N // block) * split * -(-M // (t % 1000)) >= 112, (M, N, t)
                    seen.add((epi, t, nch, N % block != 0, M % (t % 1000) != 0))
    for epi in ("f32", "swiglu", "lm"):
        for t in WIDE:
            mine = [s for s in seen if s[:2] == (epi, t)]
            assert {s[2] for s in mine} >= {1, 2, 3}, (epi, t, sorted(mine))
            assert {s[4] for s in seen if s[1] == t} == {False, True}, t
            assert any(s[3] for s in mine), (epi, t)
    assert {s[2] for s in seen} == {1, 2, 3, 4, 5, 6}
    # no tile of the many-row kernel for rows that one pass of the few-row kernel takes, nor for grids that leave half of the chip idle
    assert not any(ask([(M, 24576, 64, 1, 3, 1) for M in (1, 32, 160, 192)] + [(M, 1024, 64, 1, 2, 1) for M in (193, 640, 1000)]))


@pytest.mark.gpu
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: f"k{s['d_model']}")
def test_large_tiles_equal_few_row_passes(shape):
    from paper_2510_04147_amd import binding
    cfg = synth.model_config("8b", n_layers=1, **shape)
    w = synth.gen_weights(cfg, 5, device="cuda")
    eng = binding.SSD(cfg, w, max_seqs=1, max_seq_len=64, block=32, max_draft=4, max_rows=1300)
    g = torch.Generator(device="cuda").manual_seed(7)
    try:
        for M in ROWS:
            x = (torch.randn(M, cfg["d_model"], device="cuda", generator=g) * 0.5).bfloat16()

            def call(which, rows, cols):
                out = torch.full((rows.shape[0] * cols,), float("nan"), device="cuda",
                                 dtype=torch.bfloat16 if which == 2 else torch.float32)
                eng.k_linear(which, 0, rows, out)
                return out.view(-1, cols) if which != 4 else out.view(3, -1).T

            for which, _, _, cols, *_ in linears(cfg):
                got = call(which, x, cols)
                ref = torch.cat([call(which, x[m:m + 160].contiguous(), cols) for m in range(0, M, 160)])
                assert torch.equal(got, ref), (shape, M, which)
                if which == 2 or M not in (447, 641, 1281):
                    continue
                want = x.double() @ (w["layers"][0]["wqkv"] if which == 0 else w["lm_head"]).double().T
                if which == 4:
                    want[:, cfg["mask_id"]] = -float("inf")
                    got, want = got[:, 0], want.amax(-1)
                assert (got.double() - want).abs().max() < 1e-5, (shape, M, which)
    finally:
        eng.close()
