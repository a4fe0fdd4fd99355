// Slots of the combining tables (linear.hpp): which slots a key may take, in
// what order. Plain constexpr code, so that a host program can look at it.
#pragma once

namespace coffee {
namespace dev {

// Probes of one key before it is given up (added to global memory directly):
// one turn through the groups of a table of 128 slots, half of one with 256.
// Where a wave has more keys than slots (cell-major values, scattered cells)
// the probes that fail are what counts: Helmholtz gradients of P1 and P2 cells
// in random order took 0.80 of the time with 32 single slots, of which the
// last 16 were the first again, and take 0.63 so (geometric means, 1,293 to
// 2,045 cells, against keys hashed one by one); 12 and 8 gain little more.
constexpr int kCombineProbes = 16;

// First slot of a key in a table of ts slots (a power of two, at least 128).
// Keys are hashed in groups of eight consecutive ones that share eight
// neighbouring slots, so that the flush finds neighbouring dofs together. The
// hash also turns the group inside its slots: with key & 7 alone, keys that
// share a residue modulo 8 (dofs stored with a stride) had only ts / 8 slots
// between them.
constexpr unsigned combine_first(unsigned long long key, unsigned ts) {
    const unsigned long long h = (key >> 3) * 0x9E3779B97F4A7C15ull;
    return ((unsigned)(h >> 40) * 8u + (((unsigned)key + (unsigned)(h >> 61)) & 7u)) & (ts - 1);
}

// The slot of the next probe: the same place of the next group, so that a
// displaced group stays together.
constexpr unsigned combine_next(unsigned slot, unsigned ts) { return (slot + 8u) & (ts - 1); }

}  // namespace dev
}  // namespace coffee
