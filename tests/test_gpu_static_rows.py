"""ssd_k_lm_head_static with rows that start off a 16-byte boundary: the results of the aligned call, with more rows than its copy
area holds at a time too, and the context's workspace left as it was, byte for byte."""
import pytest
import torch

from paper_2510_04147_amd import synth

pytestmark = pytest.mark.gpu


# 16 KB a row: 256 rows at a time; 128 bytes a row: one part; K that the matrix-core kernels do not take
@pytest.mark.parametrize("d_model,rows", [(8192, (3, 256, 257, 600)), (64, (33, 600)), (72, (33,))])
def test_rows_off_16_bytes(d_model, rows):
    from paper_2510_04147_amd import binding
    cfg = synth.model_config("8b", n_layers=1, d_model=d_model, n_q_heads=1, n_kv_heads=1, d_ffn=64, vocab=1056)
    eng = binding.SSD(cfg, synth.gen_weights(cfg, 3, device="cuda"), max_seqs=1, max_seq_len=64, block=8, max_draft=1, max_rows=max(rows))
    g = torch.Generator(device="cuda").manual_seed(17)
    try:
        for M in rows:
            x = torch.randn(M, d_model, generator=g, device="cuda").bfloat16()
            want = torch.empty(3, M, device="cuda")
            eng.k_lm_head_static(x, want)
            for off in (1, 2, 4):                        # elements
                y = torch.empty(x.numel() + 8, device="cuda", dtype=x.dtype)[off:off + x.numel()].view_as(x).copy_(x)
                assert y.data_ptr() % 16 == 2 * off
                before, got = eng.workspace.clone(), torch.full((3, M), -7.0, device="cuda")
                eng.k_lm_head_static(y, got)
                assert torch.equal(got, want), (M, off)
                assert torch.equal(eng.workspace, before), (M, off)
    finally:
        eng.close()
