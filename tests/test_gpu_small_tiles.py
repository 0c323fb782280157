"""The small-tile plain GEMM (k_gemm_plain_small) at the edges of its tiles, alone through ssd_k_linear: row counts around
multiples of 8 and 16 and on both sides of the limit of 256 tiles of 64x64 (tests/test_gemm_rules.py checks on the CPU that
every epilogue meets both), output widths that fill no tile, and K that is no multiple of a step of 16 columns or shorter
than one.

Both kernels add every output in the same eight chains, so a call must equal the same rows sent in other calls bit for bit,
whichever kernel they take, aligned operands or not.  Against fp64 on the identical operands the sums differ by fp32 rounding
only (K <= 1032 products of operands of order 0.5 * 0.02: K * 2^-24 * 0.04 < 3e-6, and up to 1e-5 through SwiGLU)."""
import pytest
import torch

from paper_2510_04147_amd import synth

pytestmark = pytest.mark.gpu

SHAPES = [dict(d_model=256, d_ffn=768, vocab=1024), dict(d_model=264, d_ffn=776, vocab=1001),
          dict(d_model=8, d_ffn=24, vocab=33), dict(d_model=72, d_ffn=8, vocab=65), dict(d_model=1032, d_ffn=1032, vocab=1100)]
ROWS = (1, 7, 8, 9, 32, 65, 160, 333, 700)
# the widest shape: 255 and 256 ... 264 of the 64x64 tiles, and more
ROWS_WIDE = (9, 896, 960, 961, 1344, 1345)


def rows_of(shape):
    return ROWS_WIDE if shape["d_model"] == 1032 else ROWS


@pytest.mark.parametrize("path", [0, 1])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: f"k{s['d_model']}")
@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
def test_small_tiles_equal_any_split_of_the_rows(shape, dtype, path):
    from paper_2510_04147_amd import binding
    if dtype == "fp32" and path == 1:
        pytest.skip("fp32 models have the plain path only")
    cfg = synth.model_config("tiny", n_layers=1, dtype=dtype, **shape)
    w = synth.gen_weights(cfg, 5, device="cuda")
    eng = binding.SSD(cfg, w, max_seqs=1, max_seq_len=64, block=32, max_draft=4, max_rows=max(rows_of(shape)))
    eng.set_kernel_path(path)
    lw, d, F = w["layers"][0], cfg["d_model"], cfg["d_ffn"]
    dt = torch.float32 if dtype == "fp32" else torch.bfloat16
    nqkv = (cfg["n_q_heads"] + 2 * cfg["n_kv_heads"]) * cfg["head_dim"]
    g = torch.Generator(device="cuda").manual_seed(7)
    try:
        for M in rows_of(shape):
            xs = {k: (torch.randn(M, k, device="cuda", generator=g) * 0.5).to(dt) for k in (d, F)}

            def call(which, rows, cols):
                out = torch.full((rows.shape[0] * cols,), float("nan"), device="cuda",
                                 dtype=dt if which == 2 else torch.float32)
                eng.k_linear(which, 0, rows, out)
                return out.view(-1, cols) if which != 4 else out.view(3, -1).T

            for which, k, cols in ((0, d, nqkv), (2, d, F), (3, F, d), (4, d, 3)):
                x = xs[k]
                got = call(which, x, cols)
                ref = torch.cat([call(which, x[m:m + 23].contiguous(), cols) for m in range(0, M, 23)])
                assert torch.equal(got, ref), (shape, M, which)
                if path == 1:
                    continue
                odd = torch.empty(x.numel() + 1, device="cuda", dtype=dt)[1:].view_as(x).copy_(x)
                assert torch.equal(got, call(which, odd, cols)), (shape, M, which)
                if dtype == "fp32":
                    lin = lambda m: x.double() @ m.double().T
                    if which == 2:
                        gu = lin(lw["wgu"])
                        want = torch.nn.functional.silu(gu[:, :F]) * gu[:, F:]
                    elif which == 4:
                        lg = lin(w["lm_head"])
                        lg[:, cfg["mask_id"]] = -float("inf")
                        top = lg.max(-1)
                        assert torch.equal(got[:, 1].long(), top.indices)
                        got, want = got[:, ::2], torch.stack([top.values, torch.softmax(lg, -1).amax(-1)], 1)
                    else:
                        want = lin(lw["wqkv"] if which == 0 else lw["wdown"])
                    assert (got.double() - want).abs().max() < 1e-5, (shape, M, which)
    finally:
        eng.close()
