"""The many-row GEMM (k_gemm_rows) at the edges of its tiles, alone through ssd_k_linear: row counts around the
switch from the few-row kernel and around multiples of its 96-, 128- and 160-row tiles; weight-row counts that do
not fill the last 256-row block; K of one to three chunks past a multiple of its unroll of four, and fewer than four;
K whole and cut into two, four (attention output) and eight slices (down).  tests/test_gemm_rules.py checks on the CPU that
these row counts reach every tile height with every epilogue, and the fp32 one with K whole and cut.

Its sums are those of the few-row kernel bit for bit, so every call must equal the same rows sent in 160-row calls;
against fp64 on the identical operands the fp32 sums differ by fp32 rounding only (operands of order 0.5 * 0.02, partial
sums below 4; K <= 6144 makes at most 400 additions of 16 products each and eight slices: 408 * 2^-24 * 4 < 1e-4 < 2e-4)."""
import pytest
import torch

from paper_2510_04147_amd import synth

pytestmark = pytest.mark.gpu

# d_model (chunks of 64: 13, 14, 15, 3), with row counts of the outputs that leave the last block of 256 part empty
SHAPES = [dict(d_model=832, d_ffn=8240, vocab=18016), dict(d_model=896, d_ffn=9232, vocab=21152),
          dict(d_model=960, d_ffn=9008, vocab=17952), dict(d_model=192, d_ffn=8208, vocab=16416),
          # attention output in four slices of eight chunks, down in eight of twelve
          dict(d_model=2048, n_q_heads=16, n_kv_heads=4, d_ffn=6144, vocab=1056),
          # QKV in two slices of 19 chunks, attention output in four of twelve, down in eight of nine
          dict(d_model=2432, n_q_heads=24, n_kv_heads=8, d_ffn=4608, vocab=1056)]
ROWS = (192, 193, 224, 256, 257, 289, 385, 480, 513, 640, 641, 801, 1281)
ROWS64 = (193, 257, 289, 480, 641, 1281)                # also compared with fp64


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: f"k{s['d_model']}")
def test_many_rows_equal_few_row_passes(shape):
    from paper_2510_04147_amd import binding
    cfg = synth.model_config("8b", n_layers=1, **shape)
    w = synth.gen_weights(cfg, 5, device="cuda")
    eng = binding.SSD(cfg, w, max_seqs=1, max_seq_len=64, block=32, max_draft=4, max_rows=1300)
    lw, d, F, nq = w["layers"][0], cfg["d_model"], cfg["d_ffn"], cfg["n_q_heads"] * cfg["head_dim"]
    nqkv = nq + 2 * cfg["n_kv_heads"] * cfg["head_dim"]
    g = torch.Generator(device="cuda").manual_seed(7)
    try:
        for M in ROWS:
            xs = {k: (torch.randn(M, k, device="cuda", generator=g) * 0.5).bfloat16() for k in (d, nq, F)}

            def call(which, rows, cols):
                out = torch.full((rows.shape[0] * cols,), float("nan"), device="cuda",
                                 dtype=torch.bfloat16 if which == 2 else torch.float32)
                eng.k_linear(which, 0, rows, out)
                return out.view(-1, cols) if which != 4 else out.view(3, -1).T

            for which, k, cols in ((0, d, nqkv), (1, nq, d), (2, d, F), (3, F, d), (4, d, 3)):
                x = xs[k]
                got = call(which, x, cols)
                ref = torch.cat([call(which, x[m:m + 160].contiguous(), cols) for m in range(0, M, 160)])
                assert torch.equal(got, ref), (shape, M, which)
                if M not in ROWS64 or which == 2:
                    continue
                want = x.double() @ {0: lw["wqkv"], 1: lw["wo"], 3: lw["wdown"], 4: w["lm_head"]}[which].double().T
                if which == 4:
                    want[:, cfg["mask_id"]] = -float("inf")
                    got, want = got[:, 0], want.amax(-1)
                assert (got.double() - want).abs().max() < 2e-4, (shape, M, which)
    finally:
        eng.close()
