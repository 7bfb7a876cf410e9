// Host unit test of the server's queues for launches of their own (gr_sched.h):
// injected sizes, no GPU.  Exits non-zero on failure.
#include <cstdio>
#include <cstdlib>

#include "gr_sched.h"

#define CHECK(c)                                             \
    do {                                                     \
        if (!(c)) {                                          \
            std::printf("FAIL line %d: %s\n", __LINE__, #c); \
            std::exit(1);                                    \
        }                                                    \
    } while (0)

using namespace gr;

static SchedQuery q(uint64_t t, int32_t g) { return SchedQuery{t, g, (int32_t)t, nullptr, (int64_t)t}; }

int main() {
    const auto bytes = [](int32_t g) -> size_t { return g == 0 ? 100 : 300; };
    LaunchQueue own(400, bytes);
    SlotPolicy fifo(400, [&](int32_t g) { return QuerySize{bytes(g), 1, 1}; });
    const SessionRoom room{8, 1000, 1000};
    size_t in_flight = 0;

    // as many as fit the budget, in arrival order, up to the maximum
    CHECK(own.take(64, &in_flight).empty() && in_flight == 0);
    for (uint64_t t = 1; t <= 6; ++t) own.push(q(t, 0));
    std::vector<SchedQuery> a = own.take(64, &in_flight);
    CHECK(a.size() == 4 && a[0].ticket == 1 && a[3].ticket == 4 && in_flight == 400 && own.pending() == 2);
    CHECK(own.take(64, &in_flight).empty());
    in_flight -= 400;
    a = own.take(1, &in_flight);
    CHECK(a.size() == 1 && a[0].ticket == 5 && in_flight == 100);
    a = own.take(64, &in_flight);
    CHECK(a.size() == 1 && a[0].ticket == 6 && in_flight == 200);

    // the budget is shared with the sessions: what they hold counts here, and the reverse
    fifo.push(q(7, 0));
    fifo.push(q(8, 0));
    CHECK(fifo.admit(room, &in_flight).size() == 2 && in_flight == 400);
    own.push(q(9, 0));
    CHECK(own.take(64, &in_flight).empty());
    in_flight -= 200;

    // an older head that does not fit yet keeps later ones of the other queue out ...
    fifo.push(q(10, 1));  // 300
    own.push(q(11, 0));
    OlderHeads h;
    fifo.head_into(&h);
    CHECK(h.n == 1 && h.before(10) == 0 && h.before(11) == 300);
    a = own.take(64, &in_flight, h);  // 9 arrived before it, 11 did not
    CHECK(a.size() == 1 && a[0].ticket == 9 && in_flight == 300);
    CHECK(own.take(64, &in_flight, h).empty());
    in_flight = 100;
    CHECK(own.take(64, &in_flight, h).empty());  // 100 + 100 + 300 kept
    OlderHeads o;
    own.head_into(&o);
    a = fifo.admit(room, &in_flight, o);  // ... and is let in once it fits (nothing is kept for 11, which is later)
    CHECK(a.size() == 1 && a[0].ticket == 10 && in_flight == 400);
    in_flight = 0;
    CHECK(own.take(64, &in_flight).size() == 1 && in_flight == 100);
    // the same the other way round
    own.push(q(12, 1));
    fifo.push(q(13, 0));
    OlderHeads w;
    own.head_into(&w);
    in_flight = 200;
    CHECK(fifo.admit(room, &in_flight, w).empty() && own.take(64, &in_flight).empty());
    in_flight = 100;
    CHECK(own.take(64, &in_flight).size() == 1 && in_flight == 400 && own.pending() == 0);

    std::printf("ok\n");
    return 0;
}
