"""The prefill over one chunk (every GEMM tile shape and k split the sizes
choose) against the same prompt in 32-position chunks.

Both sides round their own keys and values to the cache's bf16; against 64-bit
sums each is within 7e-4 to 1.1e-3 (2-norm) at these widths, so they may differ
by up to about twice that; 3e-3 leaves a margin of 1.5.
"""
import pytest

from synth.configs import DENSE_4B, ModelConfig

pytestmark = pytest.mark.gpu

REL = 3e-3


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available(), "GPU tests need a GPU"
    return t


def _rel(a, b):
    return float((a - b).double().norm() / b.double().norm())


def _logits(torch, cfg, tokens, lens, positions, chunk, regular=False):
    from paper_2605_27255_amd import PipoModel
    m = PipoModel(cfg, seed=0, max_batch=tokens.shape[0], max_latent=positions + 8, prefill_chunk=chunk)
    if regular:
        tok, first = m.regular_prefill(tokens, lens=lens, logits=True)
        outs = [first.clone()]
    else:
        _, lb, ld = m.prefill(tokens, tau=0.95, lens=lens, logits=True)
        outs = [lb.clone(), ld.clone()]
        # a teacher-forced step reads the keys and values of every position
        _, lb, ld = m.decode_step(in_pairs=tokens[:, :2].contiguous(), logits=True)
        outs += [lb.clone(), ld.clone()]
    torch.cuda.synchronize()
    m.close()
    return outs


# positions per sequence (lens: ragged prompts, in tokens)
CASES = [(1, 1, None), (1, 31, None), (1, 33, None), (1, 65, None), (1, 129, None), (1, 257, None), (1, 600, None),
         (1, 1100, None), (1, 4100, None), (3, 200, [400, 7, 129]), (5, 333, [1, 665, 666, 64, 301])]


@pytest.mark.parametrize("B,positions,lens", CASES)
@pytest.mark.parametrize("heads", [0, 7])
def test_prefill_in_one_chunk_matches_small_chunks(torch, B, positions, lens, heads):
    if heads and positions > 1100:
        pytest.skip("the App. B heads take the same GEMMs")
    cfg = ModelConfig(**{**DENSE_4B.with_layers(2).__dict__, "vocab": 4096, "heads": heads})
    gen = torch.Generator(device="cuda").manual_seed(positions)
    n = max(lens) if lens else 2 * positions
    tokens = torch.randint(0, 4095, (B, n), generator=gen, device="cuda", dtype=torch.int32)
    print(f"B {B} positions {positions} heads {heads}", flush=True)
    want = _logits(torch, cfg, tokens, lens, positions, 32)
    got = _logits(torch, cfg, tokens, lens, positions, 4096)
    for w, g in zip(want, got):
        assert _rel(g, w) <= REL


# widths that are not whole GEMM tiles: 16-row strips left over, odd k tiles
@pytest.mark.parametrize("hidden,nq,nkv,d,ffn", [(96, 6, 2, 64, 160), (416, 3, 1, 128, 992), (1120, 10, 5, 64, 2080)])
@pytest.mark.parametrize("positions", [1, 63, 300])
@pytest.mark.parametrize("regular", [False, True])
def test_prefill_odd_widths(torch, hidden, nq, nkv, d, ffn, positions, regular):
    cfg = ModelConfig(**{**DENSE_4B.with_layers(2).__dict__, "hidden": hidden, "n_q_heads": nq, "n_kv_heads": nkv,
                         "head_dim": d, "ffn": ffn, "vocab": 1008})
    gen = torch.Generator(device="cuda").manual_seed(hidden + positions)
    tokens = torch.randint(0, 1007, (2, positions * (1 if regular else 2)), generator=gen, device="cuda",
                           dtype=torch.int32)
    print(f"hidden {hidden} positions {positions} regular {regular}", flush=True)
    want = _logits(torch, cfg, tokens, None, positions, 32, regular)
    got = _logits(torch, cfg, tokens, None, positions, 4096, regular)
    for w, g in zip(want, got):
        assert _rel(g, w) <= REL
