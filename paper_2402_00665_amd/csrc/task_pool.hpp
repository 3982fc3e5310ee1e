// The reservation of consecutive places in a pool by blocks that do not wait
// for each other.  Nothing here needs the GPU: `Word` is the access to the
// counter, add(count), which returns the value before, and to the pool's end,
// close(end).
#pragma once

#include <cstdint>

namespace lbvh {

// Reserves cnt of the pool's `room` places from *first on, or refuses.  An add
// is never taken back: the starts only rise, the first add that does not fit
// carries the counter past `room`, and no later one fits.  So the places given
// are those below that add's start, which it alone, starting at or below
// `room`, records as the pool's end.  (Taken back, an add could make others
// fail meanwhile, whose taking back then uncovers places already given.  A
// compare-and-swap loop gives the places out as well but makes every block
// wait for all others: 500 heavy packets of 2^20 box queries 756 -> 1273 us.)
// The counter has 64 bits, which 2^32 packets' adds of 2^10 do not wrap.
template <class Word>
constexpr bool reserve_places(Word word, uint32_t cnt, uint32_t room, uint32_t *first)
{
    const uint64_t at = word.add(cnt);
    if (at > room) return false;
    if (cnt > room - at) {
        word.close((uint32_t)at);
        return false;
    }
    *first = (uint32_t)at;
    return true;
}

// The places given: [0, places_given).
constexpr uint32_t places_given(uint64_t counter, uint32_t end, uint32_t room)
{
    return counter <= room ? (uint32_t)counter : end;
}

}  // namespace lbvh
