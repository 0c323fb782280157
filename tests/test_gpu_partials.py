"""The consumers of split-K partial sums at every number of them: the first half in order, the second half in order, then both.  A
call with p partial sums must equal the call with their sum, added in that order in fp32, bit for bit: the rotary stage apart and
inside the attention kernel, the residual + norm step."""
import pytest
import torch

from paper_2510_04147_amd import synth

pytestmark = pytest.mark.gpu


def by_halves(parts):
    def run(ps):
        t = ps[0].clone()
        for p in ps[1:]:
            t += p
        return t
    half = (len(parts) + 1) // 2
    return run(parts[:half]) + run(parts[half:]) if len(parts) > 1 else parts[0]


@pytest.mark.parametrize("dh,dtype", [(128, "bf16"), (64, "bf16"), (64, "fp32"), (128, "fp32")])
def test_consumers_add_by_halves(dh, dtype):
    from paper_2510_04147_amd import binding
    cfg = synth.model_config("tiny", n_layers=1, dtype=dtype, d_model=512, n_q_heads=4, n_kv_heads=2, head_dim=dh, d_ffn=512, vocab=64)
    t = torch.bfloat16 if dtype == "bf16" else torch.float32
    eng = binding.SSD(cfg, synth.gen_weights(cfg, 5, device="cuda"), max_seqs=1, max_seq_len=128, block=32, max_draft=4, max_rows=160)
    g = torch.Generator(device="cuda").manual_seed(3)
    nodes, M, Hq, Hkv = [(0, 40, 24, 0)] * 3, 72, 4, 2
    try:
        k, v = (torch.randn(40, Hkv, dh, device="cuda", generator=g).to(t) for _ in range(2))
        eng.k_write_cache(0, 0, 0, k, v)
        for p in range(1, 9):
            qkv = torch.randn(p, M, (Hq + 2 * Hkv) * dh, device="cuda", generator=g)
            one = by_halves(list(qkv))[None].contiguous()
            for fused in (0, 1) if dtype == "bf16" and dh == 128 else (0,):
                outs = []
                for x in (qkv, one):
                    out = torch.empty(M, Hq * dh, device="cuda", dtype=t)
                    own = [] if fused else [torch.empty(M, h, dh, device="cuda", dtype=t) for h in (Hq, Hkv, Hkv)]
                    eng.k_attention(0, nodes, x, fused, out, *own)
                    outs.append([out, *own])
                assert all(torch.equal(a, b) for a, b in zip(*outs)), (dh, dtype, p, fused)
            parts, gain = torch.randn(p, M, 512, device="cuda", generator=g), torch.rand(512, device="cuda", generator=g) + 0.5
            h0 = torch.randn(M, 512, device="cuda", generator=g)
            # the norm adds the first half's sum to the row, then the second's
            want = h0.clone()
            for ps in (parts[:(p + 1) // 2], parts[(p + 1) // 2:]):
                if len(ps):
                    s = ps[0].clone()
                    for q in ps[1:]:
                        s += q
                    want += s
            h, out = h0.clone(), torch.empty(M, 512, device="cuda", dtype=t)
            eng.k_norm(h, parts, gain, out)
            h2, out2 = want.clone(), torch.empty(M, 512, device="cuda", dtype=t)
            eng.k_norm(h2, torch.zeros(1, M, 512, device="cuda"), gain, out2)
            assert torch.equal(h, want) and torch.equal(out, out2), (dtype, p)
    finally:
        eng.close()
