// Host test of the chunk rule (paper_2307_09226_amd/csrc/rs_chunks.h), built
// with g++ under the sanitizers.  Prints "ALL OK" and exits 0 on success.
#include "rs_chunks.h"

#include <cstdio>
#include <cstdlib>
#include <initializer_list>

#define CHECK(cond)                                                                       \
    do {                                                                                  \
        if (!(cond)) {                                                                    \
            std::fprintf(stderr, "%s:%d: CHECK failed: %s\n", __FILE__, __LINE__, #cond); \
            std::exit(1);                                                                 \
        }                                                                                 \
    } while (0)

// The rules of a matrix-core plan (step 64 for mirrored pairs, 16 sample by
// sample) and of a plain plan with `items` work items a chunk.
static rs_chunk_rule matrix_core(int64_t items, int64_t step)
{
    rs_chunk_rule r;
    r.tiles = r.items = items;
    r.items_target = r.ncu = 256;
    r.min_chunk = 1024;
    r.step = step;
    r.cube_bytes = items * 128 * 64 * 8;
    return r;
}

static rs_chunk_rule plain(int64_t items, int64_t tiles)
{
    rs_chunk_rule r;
    r.items = items;
    r.tiles = tiles;
    r.items_target = 1024;
    r.ncu = 256;
    r.min_chunk = 256;
    r.fine = 128;
    r.cube_bytes = items * 64 * 32 * 16;
    return r;
}

// The bound for every pixel count up to P is the largest count seen so far.
static void sweep_bound(const rs_chunk_rule &r)
{
    int64_t most = 0;
    for (int64_t P = 1; P < 600000; ++P) {
        const int64_t S = rs_chunk_count(r, P);
        if (S > most) most = S;
        if (P < 5000 || P % 64 < 2) CHECK(rs_chunk_count_upto(r, P) == most);
    }
}

int main()
{
    for (int64_t items : {1, 3, 4, 12, 64, 300}) {
        for (int64_t step : {16, 64}) sweep_bound(matrix_core(items, step));
        sweep_bound(plain(items, items));
        sweep_bound(plain(items, 2 * items));
        sweep_bound(plain(2 * items, items));
        rs_chunk_rule r = plain(items, items);
        r.cube_bytes = (int64_t)3 << 20;   // finer chunks stop at 16 MiB
        sweep_bound(r);
        r.cube_bytes = (int64_t)17 << 20;
        sweep_bound(r);
    }
    for (int64_t items : {1, 2, 4, 12, 21, 64, 100, 300})
        for (int64_t step : {16, 64}) {
            const rs_chunk_rule r = matrix_core(items, step);
            for (int64_t P = 1; P < 400000; P += P < 3000 ? 1 : 997) {
                const int64_t ch = rs_chunk_pixels(r, P), S = rs_chunk_count(r, P);
                CHECK(ch % step == 0 && ch * S >= P && ch * (S - 1) < P);
                // a request holds no more partial sums than 1,024-pixel chunks
                // make, so a session of small requests admits as many of them
                CHECK(ch >= 1024 && S <= (P + 1023) / 1024);
                CHECK(S <= (256 / items < 1 ? 1 : 256 / items));
            }
        }
    for (int64_t items : {1, 3, 8, 32, 200})
        for (int64_t tiles : {items, 4 * items}) {
            const rs_chunk_rule r = plain(items, tiles);
            for (int64_t P = 1; P < 300000; P += P < 3000 ? 1 : 997) {
                const int64_t ch = rs_chunk_pixels(r, P), S = rs_chunk_count(r, P);
                CHECK(ch % 16 == 0 && ch >= 128 && ch * S >= P && ch * (S - 1) < P);
                CHECK(ch >= 256 || S * r.cube_bytes <= (int64_t)16 << 20);
            }
        }
    std::puts("ALL OK");
    return 0;
}
