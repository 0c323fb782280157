"""Plain attention in both of its variants (few waves: many loads in flight; many waves: few), alone through ssd_k_attention: a
node's rows in a call of many nodes, which takes the second variant, must equal the node's own call, which takes the first, bit for
bit: both add in channel and key order.  (16-bit operands with head size 128 have one variant.)  Prefixes that are whole tiles, end
in one at an odd position or leave 32 keys behind them, blocks shorter and longer than a tile, a cached suffix."""
import os
import subprocess

import pytest
import torch

from paper_2510_04147_amd import synth

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2510_04147_amd", "csrc")
HEADS, NODES = 8, 13
# prefix, block, end of the cached suffix
NODE_SHAPES = [(0, 16, 0), (1, 9, 0), (64, 16, 0), (45, 24, 0), (381, 11, 0), (96, 32, 0), (100, 16, 407), (36, 64, 0)]


def test_the_two_calls_take_different_variants(tmp_path):
    (tmp_path / "p.cpp").write_text(
        '#include <cstdio>\n#include "gemm_rules.h"\nint main() { long long w; int d, b; while (std::scanf("%lld %d %d", &w, &d, &b) == 3) '
        'std::printf("%d\\n", (int)attn_plain_deep(w, d, b)); }')
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(tmp_path / "p.cpp"), "-o", str(tmp_path / "p")], check=True)

    def deep(calls):
        out = subprocess.run([str(tmp_path / "p")], input="".join("%d %d %d\n" % c for c in calls), capture_output=True, text=True, check=True)
        return [v == "1" for v in out.stdout.split()]

    blens = [b for _, b, _ in NODE_SHAPES]
    for dh, size in ((64, 4), (64, 2), (128, 4)):
        assert all(deep([(b * HEADS, dh, size) for b in blens]))
        assert deep([(NODES * b * HEADS, dh, size) for b in blens]).count(False) >= 6
    assert not any(deep([(1, 128, 2), (4096, 128, 2)]))


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("dh", [64, 128])
def test_rows_of_many_nodes_equal_the_node_alone(dh, dtype):
    from paper_2510_04147_amd import binding
    cfg = synth.model_config("tiny", n_layers=1, d_model=128, n_q_heads=HEADS, n_kv_heads=2, head_dim=dh, d_ffn=64, vocab=64, dtype=dtype)
    w = synth.gen_weights(cfg, 5, device="cuda")
    t = torch.float32 if dtype == "fp32" else torch.bfloat16
    g = torch.Generator(device="cuda").manual_seed(dh)
    eng = binding.SSD(cfg, w, max_seqs=1, max_seq_len=512, block=64, max_draft=NODES - 1, max_rows=NODES * 64)
    eng.set_kernel_path(0)
    try:
        k, v = (torch.randn(410, 2, dh, device="cuda", generator=g).to(t) for _ in range(2))
        eng.k_write_cache(0, 0, 0, k, v)
        for S, blen, T in NODE_SHAPES:
            qkv = torch.randn(1, NODES * blen, (HEADS + 4) * dh, device="cuda", generator=g)
            out = torch.empty(NODES * blen, HEADS * dh, device="cuda", dtype=t)
            eng.k_attention(0, [(0, S, blen, T)] * NODES, qkv, 0, out)
            assert out.isfinite().all()
            for i in (0, 5, NODES - 1):
                rows = slice(i * blen, (i + 1) * blen)
                one = torch.empty(blen, HEADS * dh, device="cuda", dtype=t)
                eng.k_attention(0, [(0, S, blen, T)], qkv[:, rows].contiguous(), 0, one)
                assert torch.equal(out[rows], one), (S, blen, T, i)
    finally:
        eng.close()
