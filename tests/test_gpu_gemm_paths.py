"""The projection and GroupGEMM loop forms at the sizes where each can go wrong: column counts on and around their limits
(8 and 16 columns per product group, 16 / 32 / 64 / 128 per block), K of fewer 64-element units than wavefronts and of a
number of units they cannot share evenly, task shapes of one and of several passes (few queues make the tasks large).
Against the CPU oracle, within the bar of the other parity tests (max|err| <= 2e-2 of the RMS: the outputs are bf16, half a
unit is up to 4e-3 of a value); every scheduler gives the same bits."""
import numpy as np
import pytest

import synth
from harness import GpuModel, bf16_to_f32_np, fixed_step, oracle_step, rel_err
from test_gpu_moe_layer import SPIN, TOL, _check_against_oracle, _routing, _run, _weights

pytestmark = pytest.mark.gpu

# K = 768 = 12 units over 8 wavefronts, 1280 = 20, 256 = 4
ODD_K = synth.ModelShape("odd-k", 2, 768, 4, 2, 64, 1280)
MOE_EDGES = synth.ModelShape("moe-edges", 1, 512, 4, 2, 64, 0, n_experts=16, top_k=2, moe_F=768)


@pytest.mark.parametrize("batch", [1, 8, 9, 16, 17, 33, 64])
@pytest.mark.parametrize("shape,n_queues", [(synth.TINY, 0), (ODD_K, 0), (ODD_K, 8)])
def test_projection_paths(shape, n_queues, batch):
    import torch

    import paper_2604_13327_amd as etc
    pages = batch * 3 + 4
    model = GpuModel(shape, seed=71, n_pool_pages=pages)
    step = fixed_step(shape, batch, [(7 * b + 3) % 40 for b in range(batch)], pages, seed=72)
    x = model.hidden(0, batch)
    ref = oracle_step(shape, model.seed, pages, step, 0)["final"]
    outs = []
    for kind in (etc.SCHED_STATIC, etc.SCHED_DYNAMIC):
        model.reset_pools()
        dec = etc.Decoder(shape, kv_chunk_tokens=32, sampled_batches=[batch], max_kv_len=41, kind=kind, spin_budget=SPIN,
                          n_queues=n_queues)
        model.bind(dec)
        dec.bind_step(step)
        out = torch.full_like(x, float("nan"))
        dec.launch(x, out)
        torch.cuda.synchronize()
        assert (dec.error_word() == 0).all() and (dec.event_counters() == 0).all()
        outs.append(bf16_to_f32_np(out))
        dec.close()
    assert rel_err(outs[0], ref) <= TOL
    np.testing.assert_array_equal(outs[0], outs[1])


@pytest.mark.parametrize("tile_m,n_queues", [(64, 0), (64, 4), (48, 4), (16, 4), (64, 1)])
def test_group_gemm_row_blocks(tile_m, n_queues):
    """Experts with 0, 1, 7, 8, 9, ... 128, 130 and 175 rows in one block of tokens (forced routing)."""
    import paper_2604_13327_amd as etc
    from synth import gpu as sgpu
    s, seed = MOE_EDGES, 73
    first, second = [1, 8, 9, 16, 17, 33, 130, 175], [32, 64, 65, 0, 128, 15, 7, 78]
    tokens = sum(first)
    assert tokens == sum(second) == 389
    ids = np.stack([np.repeat(np.arange(8), first), np.repeat(np.arange(8, 16), second)[::-1]], 1).astype(np.int32)
    w = _weights(s, seed)
    x = sgpu.hidden_gpu(s, seed, tokens, tokens)
    outs = []
    for kind, kbk in ((0, False), (0, True), (1, False), (2, False)):
        layer = etc.MoeLayer(s, [tokens], kind=kind, moe_tile_m=tile_m, debug_flags=etc.DEBUG_ROUTING, spin_budget=SPIN,
                             n_queues=n_queues)
        layer.bind_weights(w)
        layer.bind_tokens(tokens)
        layer.force_routing(0, ids)
        for rep in range(2):
            y = _run(layer, x, kbk)
            assert (layer.error_word() == 0).all(), layer.error_word()
        outs.append((y, _routing(layer, s, tokens)))
        layer.close()
    _check_against_oracle(s, seed, x, outs[0][0], outs[0][1], tile_m, forced=ids)
    for y, r in outs[1:]:
        np.testing.assert_array_equal(y, outs[0][0])


@pytest.mark.parametrize("shift", [0, 64])
def test_moe_layer_output_over_its_input(shift):
    """y may lie over x, whole or shifted by some rows."""
    import torch

    import paper_2604_13327_amd as etc
    from synth import gpu as sgpu
    s, seed, tokens = MOE_EDGES, 74, 300
    w = _weights(s, seed)
    x = sgpu.hidden_gpu(s, seed, tokens, tokens)
    layer = etc.MoeLayer(s, [tokens], moe_tile_m=64, spin_budget=SPIN)
    layer.bind_weights(w)
    layer.bind_tokens(tokens)
    want = _run(layer, x)
    both = torch.zeros(tokens + shift, s.H, dtype=x.dtype, device="cuda")
    both[shift:] = x
    layer.launch(both[shift:], both[:tokens])
    torch.cuda.synchronize()
    np.testing.assert_array_equal(bf16_to_f32_np(both[:tokens]), want)
    layer.close()


@pytest.mark.parametrize("batch", [1, 3, 5, 8])
def test_attention_slots_of_a_batch_below_the_sampled_one(batch):
    """The slots of the sampled batch (8) are shared out to the bound one: chunk counts from 1 to all slots, lengths on and
    around the chunk and page boundaries those give."""
    import torch

    import paper_2604_13327_amd as etc
    s, lens = synth.TINY, [300, 0, 31, 32, 255, 127, 128, 511][:batch]
    pages = sum(n // 16 + 1 for n in lens) + 4
    model = GpuModel(s, seed=75, n_pool_pages=pages)
    step = fixed_step(s, batch, lens, pages, seed=76)
    x = model.hidden(0, batch)
    ref = oracle_step(s, model.seed, pages, step, 0)["final"]
    outs = []
    for kind in (etc.SCHED_STATIC, etc.SCHED_DYNAMIC, etc.SCHED_UNFUSED):
        model.reset_pools()
        dec = etc.Decoder(s, kv_chunk_tokens=32, sampled_batches=[8], max_kv_len=512, kind=kind, spin_budget=SPIN)
        model.bind(dec)
        dec.bind_step(step)
        out = torch.full_like(x, float("nan"))
        for _ in range(2):
            dec.launch(x, out)
        torch.cuda.synchronize()
        assert (dec.error_word() == 0).all() and (dec.event_counters() == 0).all()
        outs.append(bf16_to_f32_np(out))
        dec.close()
    assert rel_err(outs[0], ref) <= TOL
    for o in outs[1:]:
        np.testing.assert_array_equal(o, outs[0])


@pytest.mark.parametrize("n_experts,top_k,batch,tile_m", [(256, 16, 64, 3), (256, 1, 9, 16), (240, 16, 8, 7), (16, 16, 1, 1)])
def test_router_sums_over_experts(n_experts, top_k, batch, tile_m):
    """Ids, permutation and both index arrays bit for bit where the sums over experts end: a full last lane, one in the middle of
    the wavefront, one and four tokens in flight, row tiles that divide nothing, the most pairs a step can have."""
    import paper_2604_13327_amd as etc
    from test_gpu_moe import check_moe_step
    s = synth.ModelShape("moe-sums", 1, 256, 4, 2, 64, 0, n_experts=n_experts, top_k=top_k, moe_F=256)
    pages = batch * 2 + 4
    model = GpuModel(s, seed=77, n_pool_pages=pages)
    step = fixed_step(s, batch, [(5 * b + 1) % 30 for b in range(batch)], pages, seed=78)
    for kind in (etc.SCHED_STATIC, etc.SCHED_DYNAMIC):
        model.reset_pools()
        dec = etc.Decoder(s, kv_chunk_tokens=32, sampled_batches=[batch], max_kv_len=129, moe_tile_m=tile_m, kind=kind,
                          spin_budget=SPIN, debug_flags=etc.DEBUG_ROUTING | etc.DEBUG_LAYER_HIDDEN | etc.DEBUG_EXEC_COUNT)
        model.bind(dec)
        dec.bind_step(step)
        check_moe_step(dec, model, s, step, tile_m)
        dec.close()


@pytest.mark.parametrize("bound", [5, 8, 9, 12, 16])
@pytest.mark.parametrize("shape,sliced", [(synth.TINY, False), (synth.ModelShape("small-sliced", 2, 1024, 8, 2, 64, 3072), True)])
def test_staged_only_plan_of_up_to_16_sequences(shape, sliced, bound):
    """A plan of 16 whose projections all fit the staged path, with and without slices of K: bound batches on both sides of
    the 8 columns of one product group, on the instances for one and for two groups, against the oracle."""
    import torch

    import paper_2604_13327_amd as etc
    fns = etc.plan_build(shape, 32, 16, 256, 41)["tasks"]["fn"]
    assert (fns == 16).any() == sliced                    # the sums of a down projection cut along K
    pages = bound * 3 + 4
    model = GpuModel(shape, seed=79, n_pool_pages=pages)
    step = fixed_step(shape, bound, [(7 * b + 3) % 40 for b in range(bound)], pages, seed=80)
    x = model.hidden(0, bound)
    ref = oracle_step(shape, model.seed, pages, step, 0)["final"]
    outs = []
    for kind in (etc.SCHED_STATIC, etc.SCHED_DYNAMIC, etc.SCHED_UNFUSED):
        model.reset_pools()
        dec = etc.Decoder(shape, kv_chunk_tokens=32, sampled_batches=[16], max_kv_len=41, kind=kind, spin_budget=SPIN)
        model.bind(dec)
        dec.bind_step(step)
        out = torch.full_like(x, float("nan"))
        for _ in range(2):
            dec.launch(x, out)
        torch.cuda.synchronize()
        assert (dec.error_word() == 0).all() and (dec.event_counters() == 0).all()
        outs.append(bf16_to_f32_np(out))
        dec.close()
    assert rel_err(outs[0], ref) <= TOL
    for o in outs[1:]:
        np.testing.assert_array_equal(o, outs[0])


@pytest.mark.parametrize("tile_m,n_queues,gate_up,down", [(64, 32, 48, 24), (40, 64, 24, 12), (40, 32, 48, 24), (64, 48, 32, 16)])
def test_group_gemm_three_tiles_per_wavefront(tile_m, n_queues, gate_up, down):
    """Task shapes of 24 and 48 row tiles (three per wavefront, one pass and two), at 33 .. 64 columns, at more on an expert's
    only block and on one of several; three row tiles of 40 to a block of 120 columns."""
    import paper_2604_13327_amd as etc
    from synth import gpu as sgpu
    s, seed = synth.ModelShape("moe-edges-3", 1, 768, 4, 2, 64, 0, n_experts=16, top_k=2, moe_F=768), 81
    first, second = [1, 8, 9, 16, 17, 33, 130, 175], [32, 64, 65, 0, 128, 15, 7, 78]
    tokens = sum(first)
    t = etc.moe_layer_plan_build(s, tokens, n_queues, moe_tile_m=tile_m)["tasks"]
    assert set(t["c2"][t["fn"] == 12]) == {gate_up} and set(t["c2"][t["fn"] == 13]) == {down}
    ids = np.stack([np.repeat(np.arange(8), first), np.repeat(np.arange(8, 16), second)[::-1]], 1).astype(np.int32)
    w = _weights(s, seed)
    x = sgpu.hidden_gpu(s, seed, tokens, tokens)
    outs = []
    for kind in (etc.SCHED_STATIC, etc.SCHED_DYNAMIC, etc.SCHED_UNFUSED):
        layer = etc.MoeLayer(s, [tokens], kind=kind, moe_tile_m=tile_m, debug_flags=etc.DEBUG_ROUTING, spin_budget=SPIN,
                             n_queues=n_queues)
        layer.bind_weights(w)
        layer.bind_tokens(tokens)
        layer.force_routing(0, ids)
        for rep in range(2):
            y = _run(layer, x)
            assert (layer.error_word() == 0).all(), layer.error_word()
        outs.append((y, _routing(layer, s, tokens)))
        layer.close()
    _check_against_oracle(s, seed, x, outs[0][0], outs[0][1], tile_m, forced=ids)
    for y, r in outs[1:]:
        np.testing.assert_array_equal(y, outs[0][0])
