// Where the events of a plan count (place_counters): the producers of every event bring all its counters to zero and no other, and
// lines and spread events are where the rule wants them.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <initializer_list>
#include <vector>

#include "graph.h"

using namespace etc;

static void check(bool ok, const char *what, int at = 0)
{
    if (ok) return;
    printf("%s (%d)\n", what, at);
    exit(1);
}

// n tasks with an event each, and n final tasks that notify one more event; events nobody notifies in front of them
static Plan rows(int n, int producers, bool common, int in_front = 0)
{
    GraphDecl g;
    if (in_front) g.add_event({dim_const(in_front)});
    const int ev = g.add_event({dim_const(n)}), last = g.add_event({dim_const(1)});
    CallDecl a, b;
    a.fn = FN_ROWSUM_PARTIAL; a.rank = 2; a.shape[0] = dim_const(n); a.shape[1] = dim_const(producers);
    b.fn = FN_ROWSUM_FINAL; b.rank = 1; b.shape[0] = dim_const(n); b.stage = 1;
    EdgeMap m, k;
    m.event = ev; m.rank = 1; m.kind[0] = MAP_DIM; m.src[0] = 0; m.div[0] = 1;
    k.event = last; k.rank = 1; k.kind[0] = MAP_CONST; k.src[0] = 0; k.div[0] = 0;
    a.out = {m};
    b.in = {m};
    if (common) b.out = {k};
    g.calls = {a, b};
    Plan p;
    const int sym[4] = {0, 0, 0, 0};
    check(instantiate(g, sym, 256, false, &p).empty(), "instantiate");
    return p;
}

static Counters placed(const Plan &p, bool dynamic)
{
    Plan q = p;
    Counters c = place_counters(q, dynamic);
    std::vector<int32_t> left = c.init;
    check(q.tasks.size() == p.tasks.size() && q.queue_tasks.size() == p.queue_tasks.size(), "tasks");
    for (const Task &t : q.tasks) {
        const int32_t e = p.tasks[t.id].notify0;
        for (auto w : {&Task::wait0, &Task::wait1}) check(t.*w == (p.tasks[t.id].*w < 0 ? -1 : c.wait[p.tasks[t.id].*w]), "a wait", t.id);
        check((e < 0) == (t.notify0 < 0), "a notify lost", t.id);
        if (e < 0) continue;
        const int32_t at = notify_counter(t.notify0);
        check(at >= 0 && at < (int32_t)left.size() && c.event[at] == e, "a notify that misses its event", t.id);
        check(notify_event(t.notify0) == (c.wait[e] & kEvIndex), "an event's first counter", t.id);
        --left[at];
    }
    for (size_t i = 0; i < left.size(); ++i) check(left[i] == 0, "a counter that does not end at zero", (int)i);
    for (size_t i = 0; i < q.queue_tasks.size(); ++i) {
        const Task &t = q.queue_tasks[i];
        check(t.id == p.queue_tasks[i].id && !memcmp(&t, &q.tasks[t.id], sizeof(Task)), "queue record", t.id);
    }
    return c;
}

static int spread(const Counters &c)
{
    int n = 0;
    for (int32_t w : c.wait) n += (w & kEvSpread) != 0;
    return n;
}

int main()
{
    for (bool dynamic : {false, true}) {
        for (int n : {1, 15, 16, 17, 300}) {         // events of four producers, and one of n
            const Counters c = placed(rows(n, 4, true), dynamic);
            check(c.shift == 5 && spread(c) == (n >= kSpreadMinProducers), "small plans", n);
        }
        for (int n : {2031, 2032, 2033, 5000, 60000}) {      // ... of which the one has 16 counters: too few for lines above 2048
            const Counters c = placed(rows(n, 4, true), dynamic);
            const bool lines = n + kEvSpreadN <= kLinesAnyway;
            check(c.shift == (lines ? 5 : 0) && spread(c) == lines && (int)c.init.size() == n + (lines ? kEvSpreadN : 1), "many plain events", n);
        }
        for (int n : {200, 4000, 4095, 4096}) {      // all of 16 producers and more: lines up to 65536 counters
            const Counters c = placed(rows(n, 17, false), dynamic);
            const bool lines = n < 4096;             // (and the counter of the event nobody notifies)
            check(c.shift == (lines ? 5 : 0) && spread(c) == (lines ? n : 0), "spread events", n);
        }
    }
    for (int in_front : {(1 << 24) - 2, (1 << 24) + 5}) {      // counters that take more than 24 bits
        const Counters c = placed(rows(20, 17, true, in_front), false);
        check(c.shift == 0 && spread(c) == 0 && (int)c.init.size() == in_front + 21, "many events", in_front);
    }
    // the decoders' plans have lines, at every batch
    struct { ModelDims d; int batch, kv; } models[] = {
        {{32, 4096, 32, 8, 128, 14336, 0, 0, 0, 16, 128, 16}, 1, 1025}, {{80, 8192, 64, 8, 128, 28672, 0, 0, 0, 16, 128, 16}, 64, 8193},
        {{48, 2048, 32, 4, 128, 0, 128, 8, 768, 16, 128, 16}, 1, 1025}, {{48, 2048, 32, 4, 128, 0, 128, 8, 768, 16, 128, 1}, 64, 1025}};
    for (auto &m : models)
        for (bool dynamic : {false, true}) {
            GraphDecl g;
            Plan p;
            check(build_decoder_graph(m.d, m.batch, 256, !dynamic, &g).empty(), "graph");
            const int chunk = effective_kv_chunk(m.d.kv_chunk, m.d.page, m.kv, m.batch, m.d.nkv, 256);
            const int sym[4] = {m.batch, (m.kv + chunk - 1) / chunk, 0, 0};
            check(instantiate(g, sym, 256, false, &p).empty(), "instantiate");
            const Counters c = placed(p, dynamic);
            check(c.shift == 5 && spread(c) > 0, "decoder", m.batch);
        }
    puts("ok");
    return 0;
}
