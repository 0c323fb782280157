"""ssd_generate has waited for its last forward when it returns, also where that forward only appends keys and values, and its
statistics count every forward: on a stream that the null stream does not wait for, with graphs on, earlier work on the stream and
other work on the device, another prompt in every call (the output buffer holds the tokens of the call before)."""
import numpy as np
import pytest
import torch

from paper_2510_04147_amd import synth

pytestmark = pytest.mark.gpu

P, BLOCK, GEN, N = 8, 8, 48, 3


@pytest.fixture(scope="module")
def tiny():
    cfg = synth.model_config("tiny")
    wg = synth.weights_to(synth.gen_weights(cfg, 0), "cuda")
    torch.cuda.synchronize()
    return cfg, wg


def engine(cfg, wg):
    from paper_2510_04147_amd import binding
    return binding.SSD(cfg, wg, max_seqs=1, max_seq_len=128, block=BLOCK, max_draft=N, max_rows=(N + 3) * BLOCK)


@pytest.mark.parametrize("fuse", [0, 1])
def test_tokens_and_stream_when_the_call_returns(tiny, fuse):
    cfg, wg = tiny
    prompts = [synth.gen_prompt(cfg, 200 + i, P) for i in range(6)]
    ref = engine(cfg, wg)                                # on the default stream, stepwise
    try:
        want = [ref.generate([p], GEN, BLOCK, 0)[0] for p in prompts]
    finally:
        ref.close()
    assert len({tuple(t[0, -BLOCK:]) for t in want}) > 1     # a stale last block would show
    a = torch.randn(1024, 1024, device="cuda")
    torch.cuda.synchronize()
    stream, other = torch.cuda.Stream(), torch.cuda.Stream()
    with torch.cuda.stream(stream):
        eng = engine(cfg, wg)
        try:
            eng.set_graphs(1)
            eng.set_boundary_fusion(fuse)
            for rep in range(3):                         # the second call captures, later ones replay
                for p, t in zip(prompts, want):
                    with torch.cuda.stream(other):
                        for _ in range(8):
                            b = a @ a
                    for _ in range(8):
                        c = a @ a
                    got, st = eng.generate([p], GEN, BLOCK, N)
                    assert stream.query(), (rep, "work left on the stream")
                    assert np.array_equal(got, t), rep
                    assert st["kv_passes"] == (2 if fuse else 1 + GEN // BLOCK)
                    assert st["decode_ms"] + st["kv_ms"] <= st["total_ms"]
        finally:
            torch.cuda.synchronize()
            eng.close()


@pytest.mark.parametrize("fuse", [0, 1])
def test_kv_ms_counts_every_kv_pass(tiny, fuse):
    """The prompt is as long as a block, so every KV pass is a forward of the same size: the passes behind the prompt's take at
    least a quarter of its time each."""
    cfg, wg = tiny
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        eng = engine(cfg, wg)
        try:
            eng.set_boundary_fusion(fuse)
            prompt = synth.gen_prompt(cfg, 300, P)
            prefill, kv = [], []
            for rep in range(8):
                _, st = eng.generate([prompt], GEN, BLOCK, N)
                kv.append(st["kv_ms"])
                t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                eng.reset(0)
                t0.record(stream)
                eng.prefill_kv(0, prompt, 0)
                t1.record(stream)
                t1.synchronize()
                prefill.append(t0.elapsed_time(t1))
            first = min(prefill[1:])
            assert min(kv[1:]) >= first * (1 + 0.25 * (st["kv_passes"] - 1)), (kv, prefill, st["kv_passes"])
        finally:
            eng.close()
