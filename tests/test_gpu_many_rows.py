"""The many-row GEMM (k_gemm_rows) at the edges of its tiles, alone through ssd_k_linear: row counts around the
switch from the few-row kernel and around multiples of its 96-, 128- and 160-row tiles; weight-row counts that do
not fill the last 256-row block; K of one to three chunks past a multiple of its unroll of four, and fewer than four.

Its sums are those of the few-row kernel bit for bit, so every call must equal the same rows sent in 160-row calls;
against fp64 on the identical operands the fp32 sums differ by fp32 rounding only (K <= 2560 products of operands of
order 0.5 * 0.02, partial sums below 2: < 2e-4)."""
import pytest
import torch

from paper_2510_04147_amd import synth

pytestmark = pytest.mark.gpu

# d_model (chunks of 64: 13, 14, 15, 3), with row counts of the outputs that leave the last block of 256 part empty
SHAPES = [dict(d_model=832, d_ffn=8240, vocab=18016), dict(d_model=896, d_ffn=9232, vocab=21152),
          dict(d_model=960, d_ffn=9008, vocab=17952), dict(d_model=192, d_ffn=8208, vocab=16416)]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: f"k{s['d_model']}")
def test_many_rows_equal_few_row_passes(shape):
    from paper_2510_04147_amd import binding
    cfg = synth.model_config("8b", n_layers=1, **shape)
    w = synth.gen_weights(cfg, 5, device="cuda")
    eng = binding.SSD(cfg, w, max_seqs=1, max_seq_len=64, block=32, max_draft=4, max_rows=1300)
    lw, d, F, V = w["layers"][0], cfg["d_model"], cfg["d_ffn"], cfg["vocab"]
    nqkv = (cfg["n_q_heads"] + 2 * cfg["n_kv_heads"]) * cfg["head_dim"]
    g = torch.Generator(device="cuda").manual_seed(7)
    for M in (192, 193, 224, 256, 257, 289, 385, 480, 513, 640, 801, 1281):
        x = (torch.randn(M, d, device="cuda", generator=g) * 0.5).bfloat16()

        def call(which, rows, cols, dtype):
            out = torch.full((rows.shape[0] * cols,), float("nan"), device="cuda", dtype=dtype)
            eng.k_linear(which, 0, rows, out)
            return out.view(-1, cols) if which != 4 else out.view(3, -1).T

        for which, cols, dtype in ((0, nqkv, torch.float32), (2, F, torch.bfloat16), (4, 3, torch.float32)):
            got = call(which, x, cols, dtype)
            ref = torch.cat([call(which, x[m:m + 160].contiguous(), cols, dtype) for m in range(0, M, 160)])
            assert torch.equal(got, ref), (shape, M, which)
        if M in (193, 641, 1281):
            want = x.double() @ lw["wqkv"].double().T
            assert (call(0, x, nqkv, torch.float32).double() - want).abs().max() < 2e-4
            logits = x.double() @ w["lm_head"].double().T
            logits[:, cfg["mask_id"]] = -float("inf")
            assert (call(4, x, 3, torch.float32)[:, 0].double() - logits.amax(-1)).abs().max() < 2e-4
    eng.close()
