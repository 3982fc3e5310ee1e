// Every interleaving of blocks that reserve places in the pool of tasks, by
// the library's own reserve_places.  Test infrastructure.
//
// usage: task_pool [--take-back] room start count...
//
// Block b asks for the b-th count while `start` of `room` places are given.
// A block's next access to the counter depends only on what its earlier ones
// returned, so it is found by running the block again on the log of those;
// the explorer lets each unfinished block make its next access in turn.  At
// the end the places given must be [start, places_given), each once, and no
// block may have been refused while the pool never ran out.  With --take-back
// a block takes an add that did not fit back, which must be found out.
// stdout: the number of orders, and of those that broke a rule.  Exit 1 if any did.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "task_pool.hpp"

namespace {

struct Access {
    enum { kAdd, kClose } what;
    uint64_t v;
};

// One block's view of the pool: answers from the log, then throws the access.
struct Word {
    const std::vector<uint64_t> *log;
    size_t *at;
    uint64_t next(Access x)
    {
        if (*at < log->size()) return (*log)[(*at)++];
        throw x;
    }
    uint64_t add(uint64_t v) { return next({Access::kAdd, v}); }
    void close(uint32_t v) { next({Access::kClose, v}); }
};

bool take_back(Word word, uint32_t cnt, uint32_t room, uint32_t *first)
{
    const uint64_t at = word.add(cnt);
    *first = (uint32_t)at;
    const bool fits = at <= room && room - at >= cnt;
    if (!fits) word.add(0 - (uint64_t)cnt);
    return fits;
}

struct State {
    uint64_t counter;
    uint32_t end;
    std::vector<std::vector<uint64_t>> log;
};

bool run(const State &s, size_t b, bool back, uint32_t room, uint32_t cnt, uint32_t *first)
{
    size_t at = 0;
    const Word w{&s.log[b], &at};
    return back ? take_back(w, cnt, room, first) : lbvh::reserve_places(w, cnt, room, first);
}

bool broken_rule(const State &s, bool back, uint32_t room, uint32_t start, const std::vector<uint32_t> &count)
{
    std::vector<int> given(room, 0);
    for (size_t b = 0; b < count.size(); ++b) {
        uint32_t first = 0;
        if (run(s, b, back, room, count[b], &first)) {
            for (uint32_t k = 0; k < count[b]; ++k)
                if (first + k >= room || given[first + k]++) return true;
        } else if (!back && s.counter <= room) {
            return true;
        }
    }
    const uint32_t end = lbvh::places_given(s.counter, s.end, room);
    if (end > room) return true;
    for (uint32_t k = 0; k < room; ++k)
        if (given[k] != (k >= start && k < end)) return true;
    return false;
}

void explore(const State &s, bool back, uint32_t room, uint32_t start, const std::vector<uint32_t> &count,
             long &orders, long &broken)
{
    bool ended = true;
    for (size_t b = 0; b < count.size(); ++b) {
        uint32_t first = 0;
        try {
            run(s, b, back, room, count[b], &first);
        } catch (const Access &x) {
            ended = false;
            State t = s;
            t.log[b].push_back(t.counter);
            if (x.what == Access::kAdd) t.counter += x.v;
            else t.end = (uint32_t)x.v;
            explore(t, back, room, start, count, orders, broken);
        }
    }
    if (ended) {
        ++orders;
        broken += broken_rule(s, back, room, start, count);
    }
}

}  // namespace

int main(int argc, char **argv)
{
    const bool back = argc > 1 && std::strcmp(argv[1], "--take-back") == 0;
    const int a0 = back ? 2 : 1;
    if (argc < a0 + 3) return 2;
    const uint32_t room = (uint32_t)std::atol(argv[a0]), start = (uint32_t)std::atol(argv[a0 + 1]);
    std::vector<uint32_t> count;
    for (int k = a0 + 2; k < argc; ++k) count.push_back((uint32_t)std::atol(argv[k]));
    long orders = 0, broken = 0;
    explore(State{start, 0xffffffffu, std::vector<std::vector<uint64_t>>(count.size())}, back, room, start, count,
            orders, broken);
    std::printf("%ld %ld\n", orders, broken);
    return broken ? 1 : 0;
}
