"""Where a step's results go: one launch into the context's own device memory,
copies into anything else, and an error for a buffer that ends too early."""
import ctypes

import pytest

from synth import rspec
from synth.configs import TINY

pytestmark = pytest.mark.gpu


@pytest.fixture()
def models():
    """Two contexts in the same state, so that one step of each gives the same results."""
    import torch
    from paper_2605_27255_amd import PipoModel
    ms = [PipoModel(TINY, seed=0, max_batch=2, max_latent=24, prefill_chunk=16) for _ in range(2)]
    prompts = torch.from_numpy(rspec.prompt_tokens(2, 20, TINY.vocab, seed=3)).cuda()
    for m in ms:
        m.prefill(prompts, 0.5)
    yield ms
    torch.cuda.synchronize()
    for m in ms:
        m.close()


def _check(want, got):
    import torch
    torch.cuda.synchronize()
    for w, g in zip(want, got):
        assert torch.equal(w.cpu().view(torch.int32), g.cpu().view(torch.int32))


@pytest.mark.parametrize("off", [0, 1, 2, 3, 4])
@pytest.mark.parametrize("noalloc", [False, True])
def test_outputs_at_any_alignment(models, off, noalloc):
    """Logits buffers 4 * off bytes past a 16-byte boundary; the words around them stay."""
    import torch
    ref, m = models
    n = 2 * TINY.vocab
    want = ref.decode_step(logits=True)
    buf = [torch.full((n + 8,), 7.0, device="cuda") for _ in range(2)]
    out = torch.empty((2, 4), dtype=torch.int32, device="cuda")
    lb, ld = (b[off:off + n].view(2, TINY.vocab) for b in buf)
    (m.decode_step_noalloc if noalloc else m.decode_into)(out, logits_b=lb, logits_d=ld)
    _check(want, (out, lb, ld))
    for b in buf:
        assert (b[:off] == 7).all() and (b[off + n:] == 7).all()


@pytest.mark.parametrize("shift", [0, 4, 16, 4096])
def test_overlapping_outputs_are_written_in_order(models, shift):
    """The draft logits over the backbone's, from `shift` values on: the pairs, then
    the backbone logits, then the draft logits, as separate copies leave them."""
    import torch
    ref, m = models
    n = 2 * TINY.vocab
    w_out, w_lb, w_ld = ref.decode_step(logits=True)
    buf = torch.full((n + shift,), 7.0, device="cuda")
    out = torch.empty((2, 4), dtype=torch.int32, device="cuda")
    m.decode_into(out, logits_b=buf[:n], logits_d=buf[shift:])
    want = torch.cat([w_lb.flatten()[:shift], w_ld.flatten()])
    _check((w_out, want), (out, buf))


def test_outputs_in_pinned_host_memory(models):
    import torch
    ref, m = models
    want = ref.decode_step(logits=True)
    out = torch.empty((2, 4), dtype=torch.int32, pin_memory=True)
    lb, ld = (torch.empty((2, TINY.vocab), pin_memory=True) for _ in range(2))
    m.decode_into(out, logits_b=lb, logits_d=ld)
    _check(want, (out, lb, ld))


def test_buffer_that_ends_too_early_is_refused(models):
    """An allocation 64 bytes shorter than the logits (its last page still holds
    them): the call reports an error, and the memory is left as it was."""
    import torch
    from paper_2605_27255_amd import PipoError, PIPO_EHIP
    ref, m = models
    hip = m.lib     # (the HIP runtime's own symbols, through the library that links it)
    size = 4 * 2 * TINY.vocab - 64
    ptr = ctypes.c_void_p()
    assert hip.hipMalloc(ctypes.byref(ptr), ctypes.c_size_t(size)) == 0
    try:
        host = torch.full((size // 4,), 7.0)
        assert hip.hipMemcpy(ptr, ctypes.c_void_p(host.data_ptr()), ctypes.c_size_t(size), 1) == 0
        out = torch.empty((2, 4), dtype=torch.int32, device="cuda")
        full = torch.empty((2, TINY.vocab), device="cuda")
        for lb, ld in ((ptr, None), (ctypes.c_void_p(full.data_ptr()), ptr)):
            with pytest.raises(PipoError) as e:
                m._check(m.lib.pipo_decode_step(m.ctx, None, ctypes.c_void_p(out.data_ptr()), lb, ld, m._stream()))
            assert e.value.code == PIPO_EHIP
        torch.cuda.synchronize()
        back = torch.zeros(size // 4)
        assert hip.hipMemcpy(ctypes.c_void_p(back.data_ptr()), ptr, ctypes.c_size_t(size), 2) == 0
        assert (back == 7).all()
    finally:
        hip.hipFree(ptr)
