"""Decode steps of many sequences (the decoder layers' matrices through the
tiled GEMM) against the same sequences stepped in small batches (through the
decode GEMVs), and against the oracle.

Both carry X as bf16 pairs and sum in fp32; a different order of the sums moves
some new keys and values to the other bf16 neighbour, which the tolerances of
the small-batch parity tests against the oracle cover (3e-3 of the 2-norm; a
confidence within 1e-3 of the oracle's on each side, so 2e-3 between them).
The draft and the confidence follow the backbone token, so they are compared
where both sides chose the same one: nearly everywhere, as the choices differ
only where two logits lie within that rounding of each other.
"""
import os
import sys

import numpy as np
import pytest

from synth import rspec
from synth.configs import DENSE_4B, ModelConfig
from oracle import pipo_oracle as O

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
from parity import run_parity, run_regular_parity  # noqa: E402

pytestmark = pytest.mark.gpu

REL, CONF = 3e-3, 2e-3


def log(msg):
    print(msg, flush=True)


def _rel(a, b):
    return float((a - b).double().norm() / b.double().norm())


@pytest.mark.parametrize("hidden,nq,nkv,d,ffn", [(2560, 32, 8, 128, 9728), (416, 6, 2, 64, 992), (96, 3, 1, 128, 160)])
@pytest.mark.parametrize("B", [40, 41, 47, 64])
@pytest.mark.parametrize("heads", [0, 7])
def test_batched_step_matches_small_batches(hidden, nq, nkv, d, ffn, B, heads):
    import torch
    from paper_2605_27255_amd import PipoModel
    cfg = ModelConfig(**{**DENSE_4B.with_layers(3).__dict__, "hidden": hidden, "n_q_heads": nq, "n_kv_heads": nkv,
                         "head_dim": d, "ffn": ffn, "vocab": 1008, "heads": heads})
    gen = torch.Generator(device="cuda").manual_seed(B)
    n = 90
    tokens = torch.randint(0, 1007, (B, n), generator=gen, device="cuda", dtype=torch.int32)
    lens = [max(1, n - (7919 * b) % (n - 1)) for b in range(B)]
    pairs = [torch.randint(0, 1007, (B, 2), generator=gen, device="cuda", dtype=torch.int32) for _ in range(3)]
    print(f"hidden {hidden} B {B} heads {heads}", flush=True)

    def steps(lo, hi):
        m = PipoModel(cfg, seed=0, max_batch=hi - lo, max_latent=64, prefill_chunk=64)
        outs = [m.prefill(tokens[lo:hi].contiguous(), tau=0.95, lens=lens[lo:hi], logits=True)]
        for p in pairs:
            outs.append(m.decode_step(in_pairs=p[lo:hi].contiguous(), logits=True))
        torch.cuda.synchronize()
        m.close()
        return outs

    got = steps(0, B)
    parts = [steps(lo, min(lo + 8, B)) for lo in range(0, B, 8)]
    for i, (out, lb, ld) in enumerate(got):
        w_out, w_lb, w_ld = (torch.cat([p[i][j] for p in parts]) for j in range(3))
        assert _rel(lb, w_lb) <= REL
        same = out[:, 0] == w_out[:, 0]
        assert int(same.sum()) >= B - max(2, B // 16), (i, int(same.sum()))
        assert _rel(ld[same], w_ld[same]) <= REL
        conf = (out[same, 2].view(torch.float32) - w_out[same, 2].view(torch.float32)).abs().max()
        assert float(conf) <= CONF, (i, float(conf))


@pytest.mark.parametrize("heads", [0, 7])
def test_batched_steps_against_the_oracle(heads):
    """4B widths, two layers, 41 ragged prompts."""
    from paper_2605_27255_amd import PipoModel
    cfg = ModelConfig(**{**DENSE_4B.with_layers(2).__dict__, "vocab": 4096, "heads": heads, "gain_mode": 1})
    B, steps = 41, 3
    lens = [1 + (13 * b) % 80 for b in range(B)]
    prompts = rspec.prompt_tokens(B, max(lens), cfg.vocab, seed=30)
    m = PipoModel(cfg, seed=6, max_batch=B, max_latent=48, prefill_chunk=16)
    W = O.OracleWeights.generate(cfg, seed=6, precision="bf16")
    rep, _ = run_parity(m, W, prompts, steps, O.Sampling(tau=0.6), log, lens=lens, seqs=[0, 7, 31, 32, 40])
    rep.check()
    m.close()


def test_batched_regular_steps_against_the_oracle():
    from paper_2605_27255_amd import PipoModel
    cfg = ModelConfig(n_layers=2, hidden=256, n_q_heads=4, n_kv_heads=2, head_dim=64, ffn=1024, vocab=1008,
                      rope_base=1e4, gain_mode=1)
    B, steps = 45, 4
    lens = [1 + (7 * b) % 40 for b in range(B)]
    prompts = rspec.prompt_tokens(B, max(lens), cfg.vocab, seed=31)
    m = PipoModel(cfg, seed=7, max_batch=B, max_latent=48, prefill_chunk=16)
    W = O.OracleWeights.generate(cfg, seed=7, precision="bf16")
    rep, _ = run_regular_parity(m, W, prompts, steps, O.Sampling(tau=0.0), log, lens=lens)
    rep.check()
    m.close()


# one and two KV groups: 6 to 16 splits, merged on their XCD or by the merge launch
@pytest.mark.parametrize("nq,nkv,d,B", [(16, 1, 64, 41), (4, 2, 128, 48), (12, 2, 64, 64), (3, 1, 128, 64)])
@pytest.mark.parametrize("xcd", [True, False])
def test_batched_attention_splits(monkeypatch, nq, nkv, d, B, xcd):
    from paper_2605_27255_amd import PipoModel
    monkeypatch.setenv("PIPO_NO_XCD_MERGE", "0" if xcd else "1")
    cfg = ModelConfig(n_layers=2, hidden=256, n_q_heads=nq, n_kv_heads=nkv, head_dim=d, ffn=512, vocab=1008,
                      rope_base=1e4)
    n, steps = 1201, 2
    lens = [n - (7919 * b) % n for b in range(B)]
    prompts = rspec.prompt_tokens(B, n, cfg.vocab, seed=32)
    m = PipoModel(cfg, seed=8, max_batch=B, max_latent=1024, prefill_chunk=512)
    W = O.OracleWeights.generate(cfg, seed=8, precision="bf16")
    rep, _ = run_parity(m, W, prompts, steps, O.Sampling(tau=0.5), log, lens=lens, seqs=[0, 1, B // 2, B - 1])
    rep.check()
    m.close()


@pytest.mark.parametrize("B", [3, 41, 64])
@pytest.mark.parametrize("captured", [False, True])
def test_noalloc_steps_match_the_graph_steps(B, captured):
    """pipo_decode_step_noalloc, launched and recorded into a caller's graph, against
    pipo_decode_step on a second context in the same state; the replays have eager
    work and a synchronisation between them."""
    import torch
    from paper_2605_27255_amd import PipoModel
    cfg = ModelConfig(n_layers=2, hidden=416, n_q_heads=6, n_kv_heads=2, head_dim=64, ffn=992, vocab=1008,
                      rope_base=1e4, heads=7)
    lens = [1 + (11 * b) % 60 for b in range(B)]
    prompts = torch.from_numpy(rspec.prompt_tokens(B, max(lens), cfg.vocab, seed=33)).cuda()
    ref, new = (PipoModel(cfg, seed=9, max_batch=B, max_latent=64, prefill_chunk=32) for _ in range(2))
    for m in (ref, new):
        m.prefill(prompts, 0.5, lens=lens)
    out = torch.empty((B, 4), dtype=torch.int32, device="cuda")
    lb, ld = (torch.empty((B, cfg.vocab), device="cuda") for _ in range(2))
    step = lambda: new.decode_step_noalloc(out, logits_b=lb, logits_d=ld)  # noqa: E731
    torch.cuda.synchronize()
    if captured:
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            step()
        step = graph.replay
    for k in range(5):
        w_out, w_lb, w_ld = ref.decode_step(logits=True)
        for t in (out, lb, ld):
            t.fill_(-1)
        step()
        torch.cuda.synchronize()
        got, want = out.cpu().numpy(), w_out.cpu().numpy()
        np.testing.assert_array_equal(got[:, [0, 1, 3]], want[:, [0, 1, 3]], err_msg=f"step {k}")
        assert np.abs(got[:, 2].view(np.float32) - want[:, 2].view(np.float32)).max() <= CONF
        assert _rel(lb, w_lb) <= REL and _rel(ld, w_ld) <= REL
    if captured:
        del graph
    ref.close()
    new.close()
