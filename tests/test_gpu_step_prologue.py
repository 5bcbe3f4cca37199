"""The step prologue takes the hidden state eight elements at a time, and from any address."""
import pytest

import synth
from harness import GpuModel, fixed_step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hidden", [256, 8192 + 256])
def test_hidden_state_at_any_address(hidden):
    """Fewer pieces than threads, and more than two rounds of the loop take at a time: the bits that an aligned hidden state gives."""
    import torch
    import paper_2604_13327_amd as etc
    s = synth.ModelShape("address", 1, hidden, 4, 2, 64, 512)
    model = GpuModel(s, seed=29, n_pool_pages=16)
    dec = etc.Decoder(s, kv_chunk_tokens=32, sampled_batches=[3], max_kv_len=32, debug_flags=etc.DEBUG_LAYER_HIDDEN, spin_budget=400000)
    model.bind(dec)
    dec.bind_step(fixed_step(s, 3, [5, 17, 30], 16, seed=5))
    x, got = model.hidden(0, 3), []
    assert x.data_ptr() % 16 == 0
    room = torch.full((x.numel() + 16,), float("nan"), dtype=x.dtype, device="cuda")
    for start in (0, 1, 3, 4, 7):
        room.fill_(float("nan"))
        here = room[start:start + x.numel()].view(x.shape)
        here.copy_(x)
        out = torch.empty_like(x)
        dec.launch(here, out)
        torch.cuda.synchronize()
        assert (dec.error_word() == 0).all() and torch.isfinite(out.float()).all()
        got.append((out, dec.layer_hidden(0)))
    dec.close()
    for out, layer in got[1:]:
        assert torch.equal(out, got[0][0]) and (layer == got[0][1]).all()
