// DNA windows read three letters at a time (libprojmotif, gfx950).
#pragma once

#include "pm_common.h"

namespace pm {

// 32 symbols from symbol P (MSB-first): P .. P+15 in hi, P+16 .. P+31 in lo
struct Win {
    uint32_t hi, lo;
};

__device__ __forceinline__ Win load_win(const uint32_t *W, int64_t P)
{
    Win w;
    dna_window(W, P, w.hi, w.lo);
    return w;
}

// letters 3Q .. 3Q+2 of a window as a number below 64, first letter on top
// (letters past the 32nd are zero)
template <int Q>
__device__ __forceinline__ uint32_t three_letters(const Win &w)
{
    if (Q < 5) return (w.hi >> (26 - 6 * (Q < 5 ? Q : 0))) & 63u;
    if (Q == 5) return ((w.hi << 4) | (w.lo >> 28)) & 63u;
    if (Q < 10) return (w.lo >> (58 - 6 * (Q > 5 && Q < 10 ? Q : 9))) & 63u;
    return (w.lo << 2) & 63u;
}

}  // namespace pm
