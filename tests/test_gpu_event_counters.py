"""Where events count on the device: an event of 16 or more producers has 16 counters among which they are divided, and counters have
lines of their own, unless a plan has many of them and few of such events.  Row sums of small whole numbers are exact, whatever the
layout."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
SPIN = 400000


def _coarse_graph(etc, kind, consumers_first=False, in_front=3, **kw):
    """partial_sum (n, 4) -> one event -> final_sum (n) -> another event; events nobody notifies lie in front of them."""
    from paper_2604_13327_amd import binding as b
    g = etc.EventGraph(kind=kind, **kw)
    n, one = g.dim(sym=0, mul=1, add=0), g.dim(add=1)
    g.add_event([g.dim(add=in_front)])
    e1, e2 = g.add_event([one]), g.add_event([one])
    whole = lambda e: g.edge(e, [(b.MAP_CONST, 0, 0)])
    calls = [lambda: g.add_call(b.FN_ROWSUM_PARTIAL, [n, g.dim(add=4)], out_edges=[whole(e1)]),
             lambda: g.add_call(b.FN_ROWSUM_FINAL, [n], in_edges=[whole(e1)], out_edges=[whole(e2)])]
    for add in reversed(calls) if consumers_first else calls:
        add()
    return g


def _buffers(g, n, seed):
    import torch
    gen = torch.Generator(device="cuda").manual_seed(seed)
    A = torch.randint(-8, 9, (n * 32, 128), device="cuda", generator=gen).float()
    B = torch.full((n * 32, 4), float("nan"), device="cuda")
    C = torch.full((n * 32,), float("nan"), device="cuda")
    for slot, t in enumerate((A, B, C)):
        g.bind_buffer(slot, t)
    g.bind_shape([n])
    return A, C


@pytest.mark.parametrize("kind", [0, 1])
def test_plans_around_the_number_of_counters_that_have_lines(kind):
    """n row blocks with an event of four producers each and, with `common`, one event of all final sums: its 16 counters are too few
    for lines above 2048 counters, and 2032 + 16 of them the last plan that has them anyway."""
    import torch
    import paper_2604_13327_amd as etc
    from paper_2604_13327_amd import binding as b
    for common in (False, True):
        g = etc.EventGraph(kind=kind, debug_flags=etc.DEBUG_EXEC_COUNT, spin_budget=SPIN)
        n = g.dim(sym=0, mul=1, add=0)
        ev, last = g.add_event([n]), g.add_event([g.dim(add=1)])
        g.add_call(b.FN_ROWSUM_PARTIAL, [n, g.dim(add=4)], out_edges=[g.edge(ev, [(b.MAP_DIM, 0, 1)])])
        g.add_call(b.FN_ROWSUM_FINAL, [n], in_edges=[g.edge(ev, [(b.MAP_DIM, 0, 1)])], out_edges=[g.edge(last, [(b.MAP_CONST, 0, 0)])] if common else [])
        for blocks in (2031, 2032, 2033, 2047, 2048, 100):
            A, C = _buffers(g, blocks, blocks)
            for rep in range(2):
                C.fill_(float("nan"))
                g.launch()
                torch.cuda.synchronize()
                assert torch.equal(C, A.sum(1)), (blocks, rep)
                assert (g.event_counters() == 0).all() and (g.exec_counts() == rep + 1).all(), (blocks, rep)
        g.close()


@pytest.mark.parametrize("kind", [0, 1, 2])
def test_events_around_the_number_of_producers_that_spreads_them(kind):
    import torch
    import paper_2604_13327_amd as etc
    g = _coarse_graph(etc, kind, debug_flags=etc.DEBUG_EXEC_COUNT, spin_budget=SPIN)
    for n in (3, 4, 5, 15, 16, 17, 67):          # 4 n producers of the first event, n of the second
        A, C = _buffers(g, n, n)
        for rep in range(3):                     # the later launches run on re-armed counters
            C.fill_(float("nan"))
            g.launch()
            torch.cuda.synchronize()
            assert torch.equal(C, A.sum(1)), (n, rep)
            assert (g.event_counters() == 0).all() and (g.exec_counts() == rep + 1).all(), (n, rep)
        assert g.step_info().n_events == (2 if kind == 2 else 5)
    g.close()


def test_more_counters_than_lines():
    """65600 row blocks with an event each: counters side by side; then a plan with lines."""
    import torch
    import paper_2604_13327_amd as etc
    from paper_2604_13327_amd import binding as b
    g = etc.EventGraph(kind=0, spin_budget=SPIN)
    n = g.dim(sym=0, mul=1, add=0)
    ev = g.add_event([n])
    g.add_call(b.FN_ROWSUM_PARTIAL, [n, g.dim(add=4)], out_edges=[g.edge(ev, [(b.MAP_DIM, 0, 1)])])
    g.add_call(b.FN_ROWSUM_FINAL, [n], in_edges=[g.edge(ev, [(b.MAP_DIM, 0, 1)])])
    for blocks in (65600, 7):
        A, C = _buffers(g, blocks, 1)
        for _ in range(2):
            C.fill_(float("nan"))
            g.launch()
            torch.cuda.synchronize()
            assert torch.equal(C, A.sum(1))
            assert (g.event_counters() == 0).all()
    g.close()


def test_more_events_than_24_bits_count():
    import torch
    import paper_2604_13327_amd as etc
    g = _coarse_graph(etc, 0, in_front=(1 << 24) + 5, spin_budget=SPIN)
    A, C = _buffers(g, 20, 3)
    for _ in range(2):
        C.fill_(float("nan"))
        g.launch()
        torch.cuda.synchronize()
        assert torch.equal(C, A.sum(1)) and (g.event_counters() == 0).all()
    assert g.step_info().n_events == (1 << 24) + 7
    g.close()


def test_a_wait_that_gives_up_names_the_event():
    """One queue, consumers listed ahead of their 20 producers, a tiny budget: the kernel drains, and the error word names the
    event (3: behind the three nobody notifies), not one of its counters."""
    import torch
    import paper_2604_13327_amd as etc
    g = _coarse_graph(etc, 0, consumers_first=True, spin_budget=2000, n_queues=1)
    _buffers(g, 5, 1)
    g.launch()
    torch.cuda.synchronize()
    word = g.error_word()
    assert word[0] == 1 and word[2] == 3, np.asarray(word)
    with pytest.raises(etc.EtcError):
        g.event_counters()
    g.close()


def test_a_wait_that_gives_up_names_the_event_of_the_plan_it_ran():
    """A launch of one plan gives up (nearly every task heads a queue of its own, with a budget of one look), and another plan is
    bound before anybody looks: the error word names an event that tasks of its function wait for in the plan that was launched."""
    import torch
    import synth
    from harness import GpuModel, fixed_step
    import paper_2604_13327_amd as etc
    from paper_2604_13327_amd import binding as b
    s = synth.ModelShape("give-up", 2, 256, 4, 2, 64, 512)
    model = GpuModel(s, seed=3, n_pool_pages=128)
    for launched, bound in [(1, 64), (64, 1)] * 3:
        dec = etc.Decoder(s, kv_chunk_tokens=32, sampled_batches=[1, 64], max_kv_len=32, spin_budget=1)
        model.bind(dec)
        first, then = (fixed_step(s, n, [9] * n, 128, seed=5) for n in (launched, bound))
        dec.bind_step(first)
        tasks = b.plan_build(s, 32, launched, dec.step_info().n_queues, 32)["tasks"]
        x = model.hidden(0, launched)
        out = torch.empty_like(x)
        work = torch.zeros(8192, 8192, device="cuda")
        side = torch.cuda.Stream()               # (the first launch copies weight tables and waits for the default stream)
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            for _ in range(8):                   # in front of the launch on its stream: it has not run when the other step is bound
                work = work @ work
        dec.launch(x, out, stream=side)
        dec.bind_step(then)
        torch.cuda.synchronize()
        word = dec.error_word()
        mine = tasks[tasks["fn"] == word[1]]
        waits = set(mine["wait1"]) | {w + i for w, f in zip(mine["wait0"], mine["flags"]) for i in range(8 if f & 1 else 1)}
        assert word[0] == 1 and word[2] in waits - {-1}, (launched, np.asarray(word), sorted(waits))
        dec.close()


def test_only_the_dynamic_scheduler_holds_dispatch_counters():
    """4000 events of 17 producers: two buffers of 64000 lines, 16 MB, and as much again for the counts of producers not dispatched."""
    import torch
    import paper_2604_13327_amd as etc
    from paper_2604_13327_amd import binding as b
    held = []
    for kind in (0, 1):
        g = etc.EventGraph(kind=kind)
        n = g.dim(sym=0, mul=1, add=0)
        ev = g.add_event([n])
        g.add_call(b.FN_ROWSUM_PARTIAL, [n, g.dim(add=17)], out_edges=[g.edge(ev, [(b.MAP_DIM, 0, 1)])])
        before = torch.cuda.mem_get_info()[0]
        g.bind_shape([4000])
        held.append(before - torch.cuda.mem_get_info()[0])
        g.close()
    assert 16 << 20 <= held[0] <= 24 << 20 and held[1] >= 32 << 20, held
