"""Attention chunks at the edges of their steps: 16 keys a wavefront step (128 a chunk at most: one step; longer chunks of staged-only
plans: several) and 32 (the other plans), chunks of the step's own token alone, more pages than the window of page ids in LDS holds,
every (head dim, heads per KV head) there is a body for.  The place of the step's own token in the cache holds NaN beforehand: its
row must come from the projection, not from the cache."""
import numpy as np
import pytest

import synth
from harness import GpuModel, bf16_to_f32_np, fixed_step, oracle_step, rel_err

pytestmark = pytest.mark.gpu
SPIN = 400000
# Hidden states of a layer are fp32: what is rounded on the way are the projections' operands to 16 mantissa bits, 2^-17 = 7.6e-6 of a
# value under sums of up to 512 terms of either sign.  4.8e-6 of RMS is the largest difference of an element measured here, in two
# layers; 2e-5 is four times that, and attention with queries or probabilities of one bf16 part is 1.9e-4 off and more.
TOL_LAYER, TOL_BF16 = 2e-5, 2e-2


def _check(shape, lens, kv_chunk, max_len, kind=0):
    import torch
    import paper_2604_13327_amd as etc
    n_pool = int(sum(synth.pages_needed(int(n), shape.page) for n in lens)) + 8
    model = GpuModel(shape, seed=31, n_pool_pages=n_pool)
    step = fixed_step(shape, len(lens), lens, n_pool, seed=5)
    for b, n in enumerate(lens):
        page = int(step.page_ids[step.page_indptr[b] + n // shape.page])
        model.kpool[:, page, n % shape.page] = float("nan")
        model.vpool[:, page, n % shape.page] = float("nan")
    dec = etc.Decoder(shape, kv_chunk_tokens=kv_chunk, sampled_batches=[len(lens)], max_kv_len=max_len, kind=kind,
                      debug_flags=etc.DEBUG_EXEC_COUNT | etc.DEBUG_LAYER_HIDDEN, spin_budget=SPIN)
    model.bind(dec)
    x = model.hidden(0, len(lens))
    out = torch.empty_like(x)
    dec.bind_step(step)
    dec.launch(x, out)
    torch.cuda.synchronize()
    assert (dec.error_word() == 0).all() and (dec.event_counters() == 0).all() and (dec.exec_counts() == 1).all()
    ref = oracle_step(shape, model.seed, n_pool, step, 0)
    for l in range(shape.n_layers):
        got, want = dec.layer_hidden(l), ref["layers"][l]
        for b, n in enumerate(lens):
            assert rel_err(got[b], want[b]) <= TOL_LAYER, f"layer {l}, sequence {b} (kv_len {n})"
    assert rel_err(bf16_to_f32_np(out), ref["final"]) <= TOL_BF16
    for b, n in enumerate(lens):                       # the appended rows replaced the NaN
        page = int(step.page_ids[step.page_indptr[b] + n // shape.page])
        assert torch.isfinite(model.kpool[:, page, n % shape.page].float()).all()
        assert torch.isfinite(model.vpool[:, page, n % shape.page].float()).all()
    dec.close()


SHAPES = [(128, 1, False), (128, 1, True), (128, 4, False), (128, 8, True), (64, 2, True), (64, 4, False)]


def _shape(d, grp, norm, page=16):
    return synth.ModelShape(f"d{d}-g{grp}", 2, 256, 2 * grp, 2, d, 512, qk_norm=norm, page=page)


@pytest.mark.parametrize("d,grp,norm", SHAPES)
@pytest.mark.parametrize("lens,kv_chunk", [
    ([0, 15, 16, 17, 127], 128),                                  # one step of 16 keys each
    ([128, 129, 255, 300, 127], 128),                             # chunks of 128 keys, one of the new token alone
    ([256, 257, 271, 512, 700], 512),                             # several steps of 16 keys
    ([600, 767, 768, 831, 40], 768),                              # the same, six rounds
    ([0, 1, 31, 32, 33, 128, 129, 255, 256, 257, 287, 288, 289, 511, 512, 513, 700], 512),      # steps of 32 keys
])
def test_steps_and_chunks(d, grp, norm, lens, kv_chunk):
    _check(_shape(d, grp, norm), lens, kv_chunk, max(lens) + 1)


@pytest.mark.parametrize("batch", [2, 17])
@pytest.mark.parametrize("d,grp", [(128, 1), (128, 8), (64, 4)])
def test_more_pages_than_the_window_holds(d, grp, batch):
    """Pages of one token, chunks of 8192 keys: two windows of page ids, the second one key, 200 keys and 904 keys long."""
    lens = ([4097, 5000] if batch == 2 else [4097, 4296, 5000, 4096, 4095] + [7] * (batch - 5))
    _check(_shape(d, grp, False, page=1), lens, 8192, 8192)


@pytest.mark.parametrize("page", [1 << 18, 1 << 19, 1 << 20])
def test_pages_of_many_tokens(page):
    """A contiguous cache as one page a sequence: the same bits as with the same keys in pages of 16 (one chunk either way), where
    4096 pages are 2^30 tokens and where they are more than 32 bits count."""
    import torch
    import paper_2604_13327_amd as etc
    lens, outs = [1000, 0, 4095], []
    small = synth.ModelShape("pages", 1, 256, 4, 1, 64, 512)
    n_pool = sum(synth.pages_needed(n, 16) for n in lens)
    model = GpuModel(small, seed=37, n_pool_pages=n_pool)
    x = model.hidden(0, len(lens))
    rows = [torch.arange(n, device="cuda") for n in lens]                    # pages in order: position i of sequence b
    first = np.cumsum([0] + [synth.pages_needed(n, 16) for n in lens])
    for size in (16, page):
        s = synth.ModelShape("pages", 1, 256, 4, 1, 64, 512, page=size)
        if size == 16:
            indptr, ids, k, v = first, np.arange(n_pool), model.kpool.clone(), model.vpool.clone()
        else:
            indptr, ids = np.arange(len(lens) + 1), np.arange(len(lens))
            k, v = (torch.zeros((1,) + synth.kv_pool_shape(s, len(lens)), dtype=torch.bfloat16, device="cuda") for _ in range(2))
            for b, r in enumerate(rows):
                for pool, to in ((model.kpool, k), (model.vpool, v)):
                    to[0, b, :len(r)] = pool[0, first[b]:].flatten(0, 1)[:len(r)]
        dec = etc.Decoder(s, kv_chunk_tokens=page, sampled_batches=[len(lens)], max_kv_len=max(lens) + 1, spin_budget=SPIN)
        dec.bind_layer_weights(0, model.weights[0])
        dec.bind_kv_pool(k, v)
        dec.bind_step(synth.Step(len(lens), np.asarray(lens, np.int32), indptr.astype(np.int32), ids.astype(np.int32)))
        out = torch.empty_like(x)
        dec.launch(x, out)
        torch.cuda.synchronize()
        assert (dec.error_word() == 0).all() and torch.isfinite(out.float()).all()
        outs.append(out)
        dec.close()
    assert torch.equal(outs[0], outs[1])


@pytest.mark.parametrize("d,grp,norm", SHAPES)
@pytest.mark.parametrize("lens,kv_chunk", [([20, 127, 100], 128), ([300, 511, 500], 512), ([16, 300, 511] * 6, 512)])
def test_infinite_keys(d, grp, norm, lens, kv_chunk):
    """Keys with an infinite element whose score is -inf for every head of the group have weight 0, whichever lane, step or wavefront
    meets them, be it a whole step; a NaN in a key stays a NaN, in its own sequence."""
    import torch
    import oracle
    import paper_2604_13327_amd as etc
    s = synth.ModelShape(f"inf-d{d}-g{grp}", 1, 256, 2 * grp, 2, d, 512, qk_norm=norm)
    n_pool, seed = int(sum(synth.pages_needed(n, s.page) for n in lens)) + 2, 41
    step = fixed_step(s, len(lens), lens, n_pool, seed=5)
    w, x0 = synth.layer_weights_f32(s, seed, 0), synth.hidden_f32(s, seed, 0, len(lens))
    model = GpuModel(s, seed, n_pool)
    k, v = synth.kv_pool_f32(s, seed, 0, n_pool)
    _, dbg = oracle.layer(oracle.shape_of(s), x0.copy(), w, k.copy(), v.copy(), step.kv_len, step.page_indptr, step.page_ids, debug=True)
    q, hit = dbg["q_rot"].reshape(len(lens), 2, grp, d), 0
    for b, n in enumerate(lens):
        for h in range(2):
            same = np.flatnonzero(np.abs(np.sign(q[b, h]).sum(0)) == grp)
            if len(same) == 0:
                continue
            for j in {0, 5, n // 2, n - 1} | set(range(16, min(n - 1, 64))):
                e = same[j % len(same)]
                page = step.page_ids[step.page_indptr[b] + j // s.page]
                k[page, j % s.page, h, e] = -np.sign(q[b, h, 0, e]) * np.inf
                hit += 1
    assert hit > 0
    bad = len(lens) - 1
    k[step.page_ids[step.page_indptr[bad]], 3, 0, 1] = np.nan
    model.kpool.copy_(torch.from_numpy(k[None]))
    dec = etc.Decoder(s, kv_chunk_tokens=kv_chunk, sampled_batches=[len(lens)], max_kv_len=max(lens) + 1,
                      debug_flags=etc.DEBUG_LAYER_HIDDEN, spin_budget=SPIN)
    model.bind(dec)
    x = model.hidden(0, len(lens))
    dec.bind_step(step)
    dec.launch(x, torch.empty_like(x))
    torch.cuda.synchronize()
    got = dec.layer_hidden(0)
    dec.close()
    ref = oracle.decode_step(s, 1, x0, lambda l: w, lambda l: (k, v), step)["layers"][0]
    for b in range(bad):
        assert np.isfinite(ref[b]).all()
        assert rel_err(got[b], ref[b]) <= TOL_LAYER, f"sequence {b}"
    assert np.isnan(ref[bad]).all() and np.isnan(got[bad]).all()
