"""Router tiles per task of the stand-alone MoE layer: with 256 experts (16 tiles a block of 64 tokens) 16 blocks fill the 256 queues
with one tile per task, 17 take two and 33 four; the last block with one token, with all, and absent (fewer tokens than the plan)."""
import dataclasses

import numpy as np
import pytest

import synth
from test_gpu_moe_layer import SPIN, _check_against_oracle, _etc, _routing, _run, _weights

pytestmark = pytest.mark.gpu

FN_ROUTER_LOGITS = 10


@pytest.mark.parametrize("sampled,tokens,tiles", [(1024, 1024, 1), (1025, 1025, 2), (1088, 1000, 2), (1088, 9, 2), (2112, 2112, 4), (2112, 90, 4)])
def test_router_tiles_per_task(sampled, tokens, tiles):
    from synth import gpu as sgpu
    etc = _etc()
    s, seed, tile_m = dataclasses.replace(synth.TINY_MOE, n_experts=256), 61, 32
    w, x = _weights(s, seed), sgpu.hidden_gpu(s, seed, tokens, tokens)
    plan = etc.moe_layer_plan_build(s, sampled, 256, kind=0, moe_tile_m=tile_m)
    t = plan["tasks"][plan["tasks"]["fn"] == FN_ROUTER_LOGITS]
    assert (t["c2"] & 255 == tiles).all() and len(t) == 16 // tiles * -(-sampled // 64)
    outs = []
    for kind in (0, 1):
        layer = etc.MoeLayer(s, [sampled], kind=kind, moe_tile_m=tile_m, debug_flags=etc.DEBUG_ROUTING, spin_budget=SPIN)
        layer.bind_weights(w)
        layer.bind_tokens(tokens)
        for _ in range(2):
            y = _run(layer, x)
            assert (layer.error_word() == 0).all() and (layer.event_counters() == 0).all()
        r = _routing(layer, s, tokens)
        outs.append(y)
        if kind == 0:
            _check_against_oracle(s, seed, x, y, r, tile_m)
        layer.close()
    np.testing.assert_array_equal(outs[1], outs[0])


@pytest.mark.parametrize("sampled,tokens,cols", [(16, 16, 64), (17, 17, 16), (64, 64, 16), (64, 33, 16), (64, 3, 16), (512, 512, 16), (512, 90, 16), (513, 513, 64)])
def test_router_columns_per_task(sampled, tokens, cols):
    """Hidden 1024, 128 experts (8 tiles): 16 columns a task while one round of 256 covers all, else 64; column blocks that the bound
    tokens leave part or all of empty."""
    from synth import gpu as sgpu
    etc = _etc()
    s, seed, tile_m = dataclasses.replace(synth.TINY_MOE, H=1024, n_experts=128), 67, 32
    w, x = _weights(s, seed), sgpu.hidden_gpu(s, seed, tokens, tokens)
    t = etc.moe_layer_plan_build(s, sampled, 256, kind=0, moe_tile_m=tile_m)["tasks"]
    t = t[t["fn"] == FN_ROUTER_LOGITS]
    assert (t["c2"] >> 8 == cols).all() and len(t) == 8 * -(-sampled // cols)
    outs = []
    for kind in (0, 1):
        layer = etc.MoeLayer(s, [sampled], kind=kind, moe_tile_m=tile_m, debug_flags=etc.DEBUG_ROUTING, spin_budget=SPIN)
        layer.bind_weights(w)
        layer.bind_tokens(tokens)
        for _ in range(2):
            y = _run(layer, x)
            assert (layer.error_word() == 0).all() and (layer.event_counters() == 0).all()
        outs.append(y)
        if kind == 0:
            _check_against_oracle(s, seed, x, y, _routing(layer, s, tokens), tile_m)
        layer.close()
    np.testing.assert_array_equal(outs[1], outs[0])
