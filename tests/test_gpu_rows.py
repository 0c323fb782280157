"""Staging and the row kernel (tree build, embedding, first norm) of forwards with many nodes: sixteen sequences of up to six
nodes each, more than one wave of node descriptors, odd block lengths, draft counts and prefixes that differ between sequences.
The sequences share nothing, so every sequence's outputs must equal those of a call with that sequence alone, bit for bit; a
wrong node, token or position of a row changes them."""
import random

import pytest
import torch

from paper_2510_04147_amd import synth

pytestmark = pytest.mark.gpu

SMALL = dict(dtype="bf16", n_layers=2, d_model=512, n_q_heads=8, n_kv_heads=2, head_dim=64, d_ffn=1536, vocab=2080)


@pytest.mark.parametrize("block", [7, 24])
@pytest.mark.parametrize("name", ["fp32", "bf16"])
def test_sequences_of_one_forward_equal_their_own_forwards(name, block):
    from paper_2510_04147_amd import binding
    cfg = synth.model_config("tiny", **(SMALL if name == "bf16" else {}))
    w = synth.gen_weights(cfg, 5, device="cuda")
    torch.cuda.synchronize()
    n, N, mask = 16, 5, cfg["mask_id"]
    rng = random.Random(block)
    eng = binding.SSD(cfg, w, max_seqs=n, max_seq_len=80, block=block, max_draft=N, max_rows=n * (N + 1) * block)
    try:
        pos0 = [rng.randrange(1, 50) for _ in range(n)]
        for i in range(n):
            eng.prefill_kv(i, synth.gen_prompt(cfg, 100 + i, pos0[i]), 0)
        toks, masks, drafts = [], [], []
        for i in range(n):
            open_ = sorted(rng.sample(range(block), rng.randrange(1, block + 1)))
            row = [mask if p in open_ else rng.randrange(cfg["vocab"] - 1) for p in range(block)]
            toks.append(row)
            masks.append(sum(1 << p for p in open_))
            order = rng.sample(open_, len(open_))
            drafts.append([(p, rng.randrange(cfg["vocab"] - 1)) for p in order[:min(N, len(open_) - 1)]])
        assert sum(len(d) + 1 for d in drafts) > 64
        whole = eng.new_out(n)
        eng.verify_tree(list(range(n)), toks, masks, pos0, drafts, N, whole)
        whole = whole.host()
        for i in range(n):
            one = eng.new_out(1)
            eng.verify_tree([i], [toks[i]], [masks[i]], [pos0[i]], [drafts[i]], N, one)
            one = one.host()
            nodes, acc, nxt = len(drafts[i]) + 1, int(one["n_accept"][0]), int(one["n_next"][0])
            for k, cnt in (("n_accept", None), ("n_next", None), ("acc_pos", acc), ("acc_tok", acc), ("next_pos", nxt), ("next_tok", nxt),
                           ("row_maxlogit", nodes), ("row_argmax", nodes), ("row_conf", nodes)):
                a, b = (whole[k][i], one[k][0]) if cnt is None else (whole[k][i][:cnt], one[k][0][:cnt])
                assert (a == b).all(), (name, block, i, k)
    finally:
        eng.close()
