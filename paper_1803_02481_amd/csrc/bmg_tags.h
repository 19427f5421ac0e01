// bmg_tags.h -- the tags by which a host that polls a slot knows a result.
#pragma once
#include <cstdint>

namespace hbmg {

// A handle's tags count up from 1 and never repeat: a double holds every
// integer up to 2^53, enough for 1.8e13 solves of up to 500 cycles.  So no tag is
// 0 (what a slot holds that no launch has written, and k3_sum_out's "one more
// than the last") and none is one that an earlier solve left in a slot.
struct Tags {
    std::uint64_t last = 0;
    double next() { return (double)++last; }
    // n tags in a row: the first
    double take(std::uint64_t n)
    {
        const double first = (double)(last + 1);
        last += n;
        return first;
    }
};

}  // namespace hbmg
