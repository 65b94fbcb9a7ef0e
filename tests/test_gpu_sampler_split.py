"""Evaluation sampler over split rows against the same logits selected in float64.

The selection rule is the oracle's (repetition penalty, temperature, top-k with
ties kept, top-p, draw): the device and the rule see the same fp32 logits, so
the tokens are equal except where a threshold falls within the rounding of the
fp32 exponentials (about 1e-6 of the mass): those draws may give either side.
"""
import numpy as np
import pytest

from synth import rspec
from synth.configs import TINY, ModelConfig
from oracle import pipo_oracle as O

pytestmark = pytest.mark.gpu


# vocabularies on both sides of the sizes from which rows are split (12304 ids up to
# 16 sequences, 16400 with more; ends of segments, sub-tiles and rows), top-k of one,
# within and past a segment's list
@pytest.mark.parametrize("V", [16, 1008, 4096, 12288, 12304, 16384, 16400, 33024, 151936])
@pytest.mark.parametrize("B,top_k", [(1, 1), (3, 20), (3, 64), (3, 65), (20, 20), (64, 200), (64, 512)])
def test_eval_sampler_split_rows(V, B, top_k):
    import torch
    from paper_2605_27255_amd import PipoModel
    if top_k >= V:
        pytest.skip("top-k of the whole vocabulary takes the one-workgroup kernel")
    cfg = ModelConfig(**{**TINY.__dict__, "vocab": V})
    gen = torch.Generator(device="cuda").manual_seed(V + B)
    tokens = torch.randint(0, V - 1, (B, 24), generator=gen, device="cuda", dtype=torch.int32)
    seeds = [1000 + b for b in range(B)]
    m = PipoModel(cfg, seed=0, max_batch=B, max_latent=32, prefill_chunk=16)
    print(f"V {V} B {B} top_k {top_k}", flush=True)
    out, lb, ld = m.prefill(tokens, tau=0.5, temperature=1.0, top_p=0.95, top_k=top_k, rep_penalty=1.5, seeds=seeds,
                            logits=True)
    torch.cuda.synchronize()
    got = out.cpu().numpy()[:, :2].astype(np.int64)
    lb, ld, prompt = lb.cpu().numpy(), ld.cpu().numpy(), tokens.cpu().numpy()
    for b in range(B):
        seen = set(prompt[b].tolist())
        for slot, logits in ((0, lb), (1, ld)):
            penal = seen | ({int(got[b, 0])} if slot else set())
            u = rspec.uniform_draw(seeds[b], 0, slot)
            want = {int(O.select_eval(logits[b].astype(np.float64), penal, 1.0, top_k, tp, 1.5, min(max(u + du, 0.0), 1.0 - 1e-9)))
                    for tp in (0.95 - 1e-6, 0.95, 0.95 + 1e-6) for du in (-2e-6, 0.0, 2e-6)}
            assert int(got[b, slot]) in want, (b, slot, got[b, slot], want)
    m.close()


def test_ties_that_do_not_fit_a_list():
    """An infinite repetition penalty makes every penalised logit 0 or -inf: where a
    prompt holds all but a few tokens of a segment, hundreds tie at the segment's
    k-th largest, more than its list holds, and the row is selected from its logits;
    the other rows of the call still come from their lists."""
    import torch
    from paper_2605_27255_amd import PipoModel
    V, B, top_k = 16400, 3, 20
    cfg = ModelConfig(**{**TINY.__dict__, "vocab": V})
    rng = np.random.default_rng(5)
    free = rng.choice(V - 1, 60, replace=False)              # tokens the full row's prompt leaves out
    full = rng.permutation(np.setdiff1d(np.arange(V - 1), free))
    prompt = rng.integers(0, V - 1, (B, full.size)).astype(np.int32)
    prompt[1] = full
    lens = [24, full.size, 301]
    seeds = [77, 78, 79]
    m = PipoModel(cfg, seed=0, max_batch=B, max_latent=V // 2 + 8, prefill_chunk=4096)
    out, lb, ld = m.prefill(torch.from_numpy(prompt).cuda(), tau=0.5, temperature=1.0, top_p=0.95, top_k=top_k,
                            rep_penalty=float("inf"), seeds=seeds, logits=True, lens=lens)
    torch.cuda.synchronize()
    got = out.cpu().numpy()[:, :2].astype(np.int64)
    lb, ld = lb.cpu().numpy(), ld.cpu().numpy()
    # (the full row: segments of 1024 ids whose ties at 0 outnumber their 64-entry lists)
    seen1 = np.zeros(V, bool)
    seen1[full] = True
    ties = np.add.reduceat(seen1 & (lb[1] > 0), np.arange(0, V, 1024))
    assert (ties[:-1] > 64).all() and (np.add.reduceat(~seen1 & (lb[1] > 0), np.arange(0, V, 1024))[:-1] < top_k).all()
    for b in range(B):
        seen = set(prompt[b, :lens[b]].tolist())
        for slot, logits in ((0, lb), (1, ld)):
            penal = seen | ({int(got[b, 0])} if slot else set())
            u = rspec.uniform_draw(seeds[b], 0, slot)
            want = {int(O.select_eval(logits[b].astype(np.float64), penal, 1.0, top_k, tp, float("inf"),
                                      min(max(u + du, 0.0), 1.0 - 1e-9)))
                    for tp in (0.95 - 1e-6, 0.95, 0.95 + 1e-6) for du in (-2e-6, 0.0, 2e-6)}
            assert int(got[b, slot]) in want, (b, slot, got[b, slot], want)
    m.close()
