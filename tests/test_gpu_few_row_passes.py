"""The few-row GEMM in several passes over the weights (small matrices), alone through ssd_k_linear: every number of row tiles
a pass can have, with the chunk counts that run as straight-line code and with others, for every epilogue.

The rows of a pass share nothing but the weights, so a call must equal the same rows sent 32 at a time (one pass of one
tile, weights loaded non-temporally) bit for bit."""
import pytest
import torch

from paper_2510_04147_amd import synth

pytestmark = pytest.mark.gpu

# K = 4096 (gate/up, LM head) and K = 1536; attention output with K = 4096, down with K = 12288; all few work-groups wide
SHAPES = [dict(d_model=4096, d_ffn=1536, vocab=2080), dict(d_model=1024, d_ffn=12288, vocab=4128),
          dict(d_model=320, d_ffn=848, vocab=1056, n_q_heads=5, n_kv_heads=5)]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: f"d{s['d_model']}")
def test_passes_equal_single_tiles(shape):
    from paper_2510_04147_amd import binding
    cfg = synth.model_config("8b", n_layers=1, **shape)
    w = synth.gen_weights(cfg, 5, device="cuda")
    eng = binding.SSD(cfg, w, max_seqs=1, max_seq_len=64, block=32, max_draft=4, max_rows=700)
    d, F, nq = cfg["d_model"], cfg["d_ffn"], cfg["n_q_heads"] * cfg["head_dim"]
    nqkv = nq + 2 * cfg["n_kv_heads"] * cfg["head_dim"]
    g = torch.Generator(device="cuda").manual_seed(7)
    try:
        for M in (33, 64, 65, 97, 128, 160, 192, 193, 225, 321, 385, 700):
            for which, k, cols in ((0, d, nqkv), (1, nq, d), (2, d, F), (3, F, d), (4, d, 3)):
                x = (torch.randn(M, k, device="cuda", generator=g) * 0.5).bfloat16()

                def call(rows):
                    out = torch.full((rows.shape[0] * cols,), float("nan"), device="cuda",
                                     dtype=torch.bfloat16 if which == 2 else torch.float32)
                    eng.k_linear(which, 0, rows, out)
                    return out.view(-1, cols) if which != 4 else out.view(3, -1).T

                ref = torch.cat([call(x[m:m + 32].contiguous()) for m in range(0, M, 32)])
                assert torch.equal(call(x), ref), (shape, M, which)
    finally:
        eng.close()


def test_unaligned_rows_equal_aligned_ones():
    """x off a 16-byte boundary: the call copies it to one first, same rows."""
    from paper_2510_04147_amd import binding
    cfg = synth.model_config("8b", n_layers=1, d_model=896, d_ffn=9232, vocab=21152)
    w = synth.gen_weights(cfg, 5, device="cuda")
    eng = binding.SSD(cfg, w, max_seqs=1, max_seq_len=64, block=32, max_draft=4, max_rows=700)
    d, F, nqkv = cfg["d_model"], cfg["d_ffn"], (cfg["n_q_heads"] + 2 * cfg["n_kv_heads"]) * cfg["head_dim"]
    try:
        for M in (193, 641):
            x = (torch.randn(M, d, device="cuda") * 0.5).bfloat16()
            for which, cols in ((0, nqkv), (2, F), (4, 3)):
                outs = []
                for off in (0, 2, 4):                    # elements: byte offsets 0, 4, 8
                    y = torch.empty(x.numel() + 8, device="cuda", dtype=x.dtype)[off:off + x.numel()].view_as(x).copy_(x)
                    assert y.data_ptr() % 16 == 2 * off
                    out = torch.full((M * cols,), float("nan"), device="cuda", dtype=torch.bfloat16 if which == 2 else torch.float32)
                    eng.k_linear(which, 0, y, out)
                    outs.append(out)
                assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2]), (M, which)
    finally:
        eng.close()
