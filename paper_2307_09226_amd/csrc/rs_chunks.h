// How a plan cuts P pixels into chunks (split-K): plain C++, so that the host
// tests can sweep it.  A chunk's sum is one partial cube, added to the others
// in a fixed order, so the chunks decide a cube's last bits: a request cuts its
// pixels the same way alone, in a batch and in a session.
#pragma once
#include <stdint.h>

struct rs_chunk_rule {
    int64_t tiles = 1;          // chunks aimed at: items_target / tiles
    int64_t items_target = 1;
    int64_t items = 1;          // work items of one chunk
    int64_t min_chunk = 1;
    int64_t step = 16;          // chunks are whole multiples of it
    int64_t ncu = 1;            // compute units
    int64_t fine = 0;           // smallest chunk where compute units would idle, 0: min_chunk
    int64_t cube_bytes = 1;     // one chunk's partial sums
};

inline int64_t rs_round_up(int64_t v, int64_t m) { return (v + m - 1) / m * m; }

// Pixels per chunk for P > 0 pixels.
inline int64_t rs_chunk_pixels(const rs_chunk_rule &r, int64_t P)
{
    int64_t s = r.items_target / r.tiles;
    if (s < 1) s = 1;
    int64_t ch = rs_round_up((P + s - 1) / s, r.step);
    if (ch < r.min_chunk) ch = r.min_chunk;
    // Few pixels: where the smallest chunk leaves compute units without a work
    // item, finer chunks as long as the partial sums stay within 16 MiB (plain
    // form, 2 x 4, 64 x 32, 4,096 pixels: 31.6 us with chunks of 256, 28.7 us with
    // 128).  Not for the matrix-core form, whose requests share a session's
    // launches and arena with others, where more partial sums only cost: 1 x 4,
    // 128 x 64, requests of about 3,000 pixels, 32 of them in a session 320 us
    // with chunks of 1,024 and 414 us with 640 (542 and 845 us where 8 MiB hold
    // them), in a batch 114 and 127 us; one of them alone 42 and 32 us.
    if (r.fine > 0 && (P + ch - 1) / ch * r.items < r.ncu) {
        int64_t s2 = r.ncu / r.items;
        if (s2 > ((int64_t)16 << 20) / r.cube_bytes) s2 = ((int64_t)16 << 20) / r.cube_bytes;
        if (s2 >= 1) {
            int64_t c2 = rs_round_up((P + s2 - 1) / s2, r.step);
            if (c2 < r.fine) c2 = r.fine;
            if (c2 < ch) ch = c2;
        }
    }
    return ch;
}

inline int64_t rs_chunk_count(const rs_chunk_rule &r, int64_t P)
{
    const int64_t ch = rs_chunk_pixels(r, P);
    return (P + ch - 1) / ch;
}

// The most chunks that any pixel count up to P > 0 is cut into.  The count
// itself falls here and there as P grows: from 1,024 s pixels on, s chunks become
// fewer by the rounding of their size, and where finer chunks end.
inline int64_t rs_chunk_count_upto(const rs_chunk_rule &r, int64_t P)
{
    int64_t s = r.items_target / r.tiles;
    if (s < 1) s = 1;
    int64_t most = (P + r.min_chunk - 1) / r.min_chunk;   // reached up to P = s min_chunk
    if (most > s) most = s;
    if (r.fine > 0 && r.items < r.ncu) {
        int64_t s2 = r.ncu / r.items;
        if (s2 > ((int64_t)16 << 20) / r.cube_bytes) s2 = ((int64_t)16 << 20) / r.cube_bytes;
        const int64_t f = (P + r.fine - 1) / r.fine;       // reached up to P = s2 fine
        if (f < s2) s2 = f;
        if (s2 > most) most = s2;
    }
    return most;
}
