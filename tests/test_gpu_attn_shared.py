"""The matrix-core attention kernel with two work-groups on a CU (four waves of two strands) against the one with eight waves:
more than 256 work-groups take the first, a node alone the second, and a node's output may not depend on which.  Key tiles of
fewer than eight, exactly eight and nine strands, a strand of several tiles, ragged prefixes and blocks, cached suffixes, both head
sizes, the rotary stage inside and apart.  (tests/test_gpu_kernels_tight.py holds the kernels against fp64.)"""
import os
import subprocess

import pytest
import torch

from paper_2510_04147_amd import synth

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2510_04147_amd", "csrc")
M128 = dict(dtype="bf16", n_layers=1, d_model=512, n_q_heads=32, n_kv_heads=8, head_dim=128, d_ffn=512, vocab=512)
M64 = dict(dtype="bf16", n_layers=1, d_model=512, n_q_heads=32, n_kv_heads=4, head_dim=64, d_ffn=512, vocab=512)
# (S, block length, T) per node, one sequence each
PREFIXES = [(0, 32, 0), (5, 8, 0), (64, 32, 0), (96, 31, 0), (223, 32, 0), (224, 20, 0), (225, 32, 0), (256, 1, 0), (515, 32, 0), (600, 24, 0)]
SUFFIXES = [(0, 32, 300), (37, 24, 290), (64, 32, 97), (250, 30, 600), (33, 7, 600), (300, 32, 0), (96, 32, 128), (1, 31, 33), (129, 32, 545)]
LONG = [(0, 200, 0), (70, 64, 0), (224, 100, 0), (515, 33, 0)]
CASES = [("m128", M128, PREFIXES, (0, 1)), ("m128_suffix", M128, SUFFIXES, (0, 1)), ("m128_long", M128, LONG, (0,)),
         ("m64", M64, PREFIXES, (0,)), ("m64_suffix", M64, SUFFIXES, (0,)), ("m64_long", M64, LONG, (0,))]


def test_cases_take_the_kernel_they_mean(tmp_path):
    (tmp_path / "p.cpp").write_text('#include <cstdio>\n#include "gemm_rules.h"\nint main() { long long n; while (std::scanf("%lld", &n) == 1) '
                                    'std::printf("%d\\n", (int)attn_two_per_cu(n)); }')
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(tmp_path / "p.cpp"), "-o", str(tmp_path / "p")], check=True)
    ask = lambda n: bool(int(subprocess.run([str(tmp_path / "p")], input=str(n), capture_output=True, text=True, check=True).stdout))
    for name, m, nodes, _ in CASES:
        tiles = -(-max(n[1] for n in nodes) // 32)                   # the grid has this many query tiles for every node
        assert ask(len(nodes) * m["n_q_heads"] * tiles), name
        for n in nodes:
            assert not ask(m["n_q_heads"] * -(-n[1] // 32)), (name, n)


@pytest.mark.gpu
@pytest.mark.parametrize("name,model,nodes,fused", CASES, ids=[c[0] for c in CASES])
def test_a_node_is_the_same_alone_and_among_many(name, model, nodes, fused):
    from paper_2510_04147_amd import binding
    cfg = synth.model_config("tiny", **model)
    w = synth.gen_weights(cfg, 5, device="cuda")
    torch.cuda.synchronize()
    Hq, Hkv, dh, rows = cfg["n_q_heads"], cfg["n_kv_heads"], cfg["head_dim"], sum(n[1] for n in nodes)
    eng = binding.SSD(cfg, w, max_seqs=len(nodes), max_seq_len=704, block=32, max_draft=1, max_rows=max(rows, 64 * len(nodes)))
    g = torch.Generator(device="cuda").manual_seed(7)
    try:
        for i, (S, bl, T) in enumerate(nodes):
            if max(S, T):
                k = (torch.randn(max(S, T), Hkv, dh, generator=g, device="cuda") * 0.7).bfloat16()
                eng.k_write_cache(i, 0, 0, k, torch.randn(max(S, T), Hkv, dh, generator=g, device="cuda").bfloat16())
        qkv = torch.randn(2, rows, (Hq + 2 * Hkv) * dh, generator=g, device="cuda") * 0.8
        for f in fused:
            out = torch.full((rows, Hq * dh), float("nan"), device="cuda").bfloat16()
            eng.k_attention(0, [(i, *n) for i, n in enumerate(nodes)], qkv, f, out)
            assert not out.isnan().any()
            row = 0
            for i, n in enumerate(nodes):
                one = torch.full((n[1], Hq * dh), float("nan"), device="cuda").bfloat16()
                eng.k_attention(0, [(i, *n)], qkv[:, row:row + n[1]].contiguous(), f, one)
                assert torch.equal(out[row:row + n[1]], one), (name, f, n)
                row += n[1]
    finally:
        eng.close()
