"""Decode steps of many sequences (the decoder layers' matrices through the
tiled GEMM) against the same sequences stepped in small batches (through the
decode GEMVs).

Both carry X as bf16 pairs and sum in fp32; a different order of the sums moves
some new keys and values to the other bf16 neighbour, which the tolerances of
the small-batch parity tests against the oracle cover (3e-3 of the 2-norm).
"""
import pytest

from synth.configs import DENSE_4B, ModelConfig

pytestmark = pytest.mark.gpu

REL = 3e-3


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
        outs = [m.prefill(tokens[lo:hi].contiguous(), tau=0.95, lens=lens[lo:hi], logits=True)[1].clone()]
        for p in pairs:
            outs.append(m.decode_step(in_pairs=p[lo:hi].contiguous(), logits=True)[1].clone())
        torch.cuda.synchronize()
        m.close()
        return outs

    got = steps(0, B)
    parts = [steps(lo, min(lo + 8, B)) for lo in range(0, B, 8)]
    for i, g in enumerate(got):
        w = torch.cat([p[i] for p in parts])
        assert float((g - w).double().norm() / w.double().norm()) <= REL
