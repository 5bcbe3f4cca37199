"""Row blocks of the stand-alone MoE layer under skewed routings: experts with no, one, a few, just under, exactly and just over a
block's rows, so that every length class of blocks occurs next to the others, in the slots the static grid gives them (longest
first, neighbours on one XCD where enough slots are left over, in order where not) and in those the dynamic scheduler releases."""
import numpy as np
import pytest

import synth
from test_gpu_moe_layer import SPIN, _check_against_oracle, _etc, _routing, _run, _weights

pytestmark = pytest.mark.gpu


def _forced(counts, seed):
    """Top-2 routing whose experts get `counts` pairs: pairs dealt to tokens, never the same expert twice in a token."""
    tokens = sum(counts) // 2
    order = np.argsort([-c for c in counts])
    flat = np.concatenate([np.full(counts[e], e, np.int32) for e in order])
    ids = np.stack([flat[:tokens], flat[tokens:]], 1)            # an expert of at most `tokens` pairs never meets itself
    assert (ids[:, 0] != ids[:, 1]).all()
    return np.ascontiguousarray(ids[np.random.default_rng(seed).permutation(tokens)])


@pytest.mark.parametrize("tile_m", [64, 48, 40, 16])
@pytest.mark.parametrize("counts", [
    [300, 129, 128, 127, 65, 64, 63, 33, 32, 31, 17, 16, 15, 1, 0, 1],
    [257, 256, 255, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0],
    [200, 200] + [0] * 14,
    [64] * 16,
    [1, 1] + [0] * 14,
])
def test_blocks_of_every_length(counts, tile_m):
    from synth import gpu as sgpu
    etc = _etc()
    s, seed = synth.TINY_MOE, 53
    forced = _forced(counts, 3)
    tokens = len(forced)
    w, x = _weights(s, seed), sgpu.hidden_gpu(s, seed, tokens, tokens)
    outs = []
    for kind in (0, 1, 2):
        layer = etc.MoeLayer(s, [tokens], kind=kind, moe_tile_m=tile_m, debug_flags=etc.DEBUG_ROUTING, spin_budget=SPIN)
        layer.bind_weights(w)
        layer.bind_tokens(tokens)
        layer.force_routing(0, forced)
        for _ in range(2):
            y = _run(layer, x)
            assert (layer.error_word() == 0).all() and (layer.event_counters() == 0).all()
        r = _routing(layer, s, tokens)
        assert (np.diff(r["tok_indptr"]) == counts).all()
        outs.append(y)
        _check_against_oracle(s, seed, x, y, r, tile_m, forced=forced)
        layer.close()
    for y in outs[1:]:
        np.testing.assert_array_equal(y, outs[0])
