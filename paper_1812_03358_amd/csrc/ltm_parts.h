// The parts in which a list of rays is taken.
#pragma once

// A list of `groups` groups, whole or, where a part fails, in its two halves: a walk
// over the tree of halves that visits each part at most once.  A part that failed is
// never met again, and past its halves the walk is back at the larger parts beside it,
// so one bad group costs a part per level of the tree, not the rest of the list.
struct Parts {
    int groups;
    int depth = 0, at = 0;   // the at-th of 2^depth parts

    constexpr int begin() const { return (groups * at) >> depth; }
    constexpr int end() const { return (groups * (at + 1)) >> depth; }
    constexpr bool done() const { return at >> depth != 0; }
    // the first half of this part, which has two groups or more
    constexpr void halve()
    {
        ++depth;
        at *= 2;
    }
    // what follows this part
    constexpr void next()
    {
        for (++at; depth > 0 && (at & 1) == 0; at >>= 1) --depth;
    }
};
