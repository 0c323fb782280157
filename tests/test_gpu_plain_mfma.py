"""The fp32 matrix-core GEMM of the plain path (k_gemm_plain, k_gemm_plain_small), alone through ssd_k_linear, where its tiles and
chains end: row counts around 16 and 64 and on both sides of 160 tiles of 64x64, output widths that fill no tile, K of less
than one step of 16 columns, of fewer steps than the eight chains, and of chains that are cut short or empty.

Every output is the same eight chains in both kernels, so a call must equal the same rows sent one by one; against fp64 the
sums differ by fp32 rounding only (K <= 680 products of order 0.5 * 0.02: K * 2^-24 * 0.04 < 2e-6, below 1e-5 through SwiGLU).
A row of infinities or NaN leaves every other row as it is."""
import pytest
import torch

from paper_2510_04147_amd import synth

pytestmark = pytest.mark.gpu

# steps of 16: 1 (half), 2 (one half), 7, 8, 9, 43 (chains of six, the last of one)
SHAPES = [dict(d_model=8, d_ffn=24, vocab=70), dict(d_model=24, d_ffn=104, vocab=131), dict(d_model=128, d_ffn=144, vocab=129),
          dict(d_model=680, d_ffn=680, vocab=1025)]
ROWS = (15, 16, 17, 63, 64, 65, 640, 705)


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: f"k{s['d_model']}")
@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
def test_edges(shape, dtype):
    from paper_2510_04147_amd import binding
    cfg = synth.model_config("tiny", n_layers=1, dtype=dtype, **shape)
    w = synth.gen_weights(cfg, 5, device="cuda")
    eng = binding.SSD(cfg, w, max_seqs=1, max_seq_len=64, block=32, max_draft=4, max_rows=max(ROWS))
    eng.set_kernel_path(0)
    lw, d, F = w["layers"][0], cfg["d_model"], cfg["d_ffn"]
    dt = torch.float32 if dtype == "fp32" else torch.bfloat16
    nqkv = (cfg["n_q_heads"] + 2 * cfg["n_kv_heads"]) * cfg["head_dim"]
    g = torch.Generator(device="cuda").manual_seed(7)
    try:
        for M in ROWS:
            xs = {k: (torch.randn(M, k, device="cuda", generator=g) * 0.5).to(dt) for k in (d, F)}

            def call(which, rows, cols):
                out = torch.full((rows.shape[0] * cols,), float("nan"), device="cuda", dtype=dt if which == 2 else torch.float32)
                eng.k_linear(which, 0, rows, out)
                return out.view(-1, cols) if which != 4 else out.view(3, -1).T

            for which, k, cols in ((0, d, nqkv), (2, d, F), (3, F, d), (4, d, 3)):
                x = xs[k]
                got = call(which, x, cols)
                some = sorted({0, M // 2, M - 1})
                for m in some:
                    assert torch.equal(got[m:m + 1], call(which, x[m:m + 1].contiguous(), cols)), (shape, M, which, m)
                y = x.clone()
                y[M // 2] = float("inf")
                y[M // 2, 0] = float("nan")
                keep = torch.arange(M, device="cuda") != M // 2
                assert torch.equal(got[keep], call(which, y, cols)[keep]), (shape, M, which)
                lin = lambda m: x.double() @ m.double().T
                if which in (0, 3):
                    assert (got.double() - lin(lw["wqkv"] if which == 0 else lw["wdown"])).abs().max() < 1e-5, (shape, M, which)
                elif which == 4:
                    lg = lin(w["lm_head"])
                    lg[:, cfg["mask_id"]] = -float("inf")
                    assert (got[:, 0].double() - lg.amax(-1)).abs().max() < 1e-5, (shape, M, which)
                elif dtype == "fp32":
                    gu = lin(lw["wgu"])
                    assert (got.double() - torch.nn.functional.silu(gu[:, :F]) * gu[:, F:]).abs().max() < 1e-5, (shape, M, which)
    finally:
        eng.close()
