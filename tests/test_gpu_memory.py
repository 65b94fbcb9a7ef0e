"""Device memory a context takes, from what the runtime reports as free before and after."""
import pytest

from synth.configs import TINY, ModelConfig

pytestmark = pytest.mark.gpu


def _taken(cfg, **kw):
    import torch
    from paper_2605_27255_amd import PipoModel
    PipoModel(cfg, seed=0, **kw).close()     # (anything the runtime allocates on first use)
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    m = PipoModel(cfg, seed=0, **kw)
    torch.cuda.synchronize()
    taken = before - torch.cuda.mem_get_info()[0]
    m.close()
    return taken / 2**20


def test_chunk_workspaces_follow_the_capacity():
    """Positions for 49 latents need no room for a chunk of 4096: 16 MiB of k-range
    partial sums and about 10 of weights, cache and the rest, not 64 and 40 more."""
    assert _taken(TINY, max_batch=1, max_latent=49, prefill_chunk=4096) <= 40


def test_one_layer_holds_no_fp16_cache():
    """One layer runs no prefill attention, so its cache is all the key and value
    memory it takes: 79 MiB for eight sequences of 20000 latents, not twice that."""
    cfg = ModelConfig(**{**TINY.__dict__, "n_layers": 1})
    cache = 2 * 8 * TINY.kv_dim * (20000 + 128) * 2 / 2**20
    small = _taken(cfg, max_batch=8, max_latent=64, prefill_chunk=64)
    assert _taken(cfg, max_batch=8, max_latent=20000, prefill_chunk=64) - small <= 1.15 * cache
