// Host check of the decode attention's launch rule (attn_route) against what was measured on 256 compute
// units: each line is a shape, and the routes that were as fast as the fastest, within the spread.
#include <cstdio>
#include "kernels.h"
using namespace dvi;
int main() {
    constexpr int L4 = 1 << ATTN_LOCAL4, L8 = 1 << ATTN_LOCAL8, K1 = 1 << ATTN_IN_KERNEL, K2 = 1 << ATTN_TWO_LAUNCHES;
    const DType F = DType::F32, H = DType::BF16;
    struct Line { DType t; int hd, rows, chunks; long heads; int fast; };
    const Line lines[] = {
        // up to 4 chunks
        {F, 64, 1, 4, 4, L4}, {F, 64, 4, 4, 32, L4}, {F, 64, 1, 4, 2048, L4}, {F, 128, 1, 4, 4, L4}, {F, 128, 1, 4, 1024, L4},
        {H, 64, 16, 4, 8, L4}, {H, 64, 1, 4, 32, L4}, {H, 128, 1, 4, 32, L4}, {H, 128, 4, 4, 320, L4}, {H, 128, 1, 4, 2560, L4},
        // 5 to 8 chunks, fp32
        {F, 64, 1, 8, 4, K1}, {F, 64, 4, 8, 4, K1}, {F, 64, 1, 8, 16, K1}, {F, 64, 1, 8, 32, K1}, {F, 64, 1, 8, 64, K1},
        {F, 64, 1, 8, 128, L8}, {F, 64, 4, 8, 128, L8}, {F, 64, 1, 8, 256, L8}, {F, 64, 1, 8, 2048, L8},
        {F, 128, 1, 8, 4, K1}, {F, 128, 4, 8, 16, K1}, {F, 128, 1, 8, 32, K1}, {F, 128, 1, 8, 64, K1},
        {F, 128, 1, 8, 256, L8}, {F, 128, 1, 8, 512, L8}, {F, 128, 1, 8, 1024, L8 | K2},
        // 5 to 8 chunks, bf16
        {H, 64, 4, 8, 8, L8 | K1}, {H, 64, 16, 8, 8, L8 | K2}, {H, 64, 1, 8, 32, L8}, {H, 64, 4, 8, 64, L8}, {H, 64, 1, 8, 128, L8},
        {H, 64, 1, 8, 256, L8}, {H, 64, 4, 8, 512, L8}, {H, 64, 1, 8, 2048, L8},
        {H, 128, 1, 8, 32, K1 | L8}, {H, 128, 1, 8, 40, K1 | L8}, {H, 128, 1, 8, 64, L8}, {H, 128, 8, 8, 96, L8},
        {H, 128, 4, 8, 120, L8}, {H, 128, 1, 8, 128, L8}, {H, 128, 4, 8, 160, L8}, {H, 128, 1, 8, 256, L8},
        {H, 128, 1, 8, 320, K2}, {H, 128, 1, 8, 512, L8}, {H, 128, 1, 8, 640, K2}, {H, 128, 1, 8, 1024, L8}, {H, 128, 1, 8, 1280, L8},
        {H, 128, 1, 8, 2560, L8},
        // more than 4 query rows with more than 8 chunks, more than 16 rows
        {H, 128, 6, 12, 32, K2}, {F, 64, 8, 12, 4, K2}, {H, 128, 24, 4, 32, K2}, {H, 64, 32, 8, 8, K2},
        // one workgroup a compute unit, and just above
        {H, 128, 1, 32, 32, K1}, {H, 128, 4, 32, 32, K1 | K2}, {H, 64, 1, 32, 32, K1 | K2}, {F, 64, 1, 32, 32, K1}, {F, 128, 1, 32, 32, K1},
        {H, 64, 4, 16, 64, K2}, {F, 128, 4, 16, 64, K2}, {F, 128, 4, 8, 128, K2}, {H, 128, 1, 32, 40, K2}, {H, 128, 4, 32, 40, K2},
        // more than 8 chunks: clear on both sides of the line
        {H, 128, 1, 12, 32, K1}, {H, 128, 1, 16, 40, K1}, {H, 64, 1, 24, 32, K1}, {H, 64, 4, 32, 8, K1}, {F, 64, 1, 32, 4, K1},
        {F, 64, 1, 24, 32, K1}, {F, 128, 1, 32, 16, K1}, {H, 128, 1, 12, 128, K2}, {H, 128, 1, 32, 64, K2}, {F, 64, 1, 12, 128, K2},
        {F, 128, 1, 24, 64, K2}, {H, 64, 4, 24, 64, K2}, {H, 128, 4, 24, 256, K2},
    };
    for (const Line &l : lines) {
        const AttnRoute r = attn_route(l.t, l.hd, l.rows, l.chunks, l.heads, 256);
        if (!(l.fast >> r & 1)) {
            printf("%s hd %d rows %d chunks %d heads %ld: route %d\n", l.t == F ? "fp32" : "bf16", l.hd, l.rows, l.chunks, l.heads, (int)r);
            return 1;
        }
    }
    // the local kernels hold at most 16 rows and as many chunks as they have waves
    for (int hd : {64, 128})
        for (DType t : {F, H})
            for (int rows = 1; rows <= 64; ++rows)
                for (int n = 1; n <= 40; ++n)
                    for (long heads = 1; heads <= 4096; heads *= 2) {
                        const AttnRoute r = attn_route(t, hd, rows, n, heads, 256);
                        if ((r == ATTN_LOCAL4 && (rows > 16 || n > 4)) || (r == ATTN_LOCAL8 && (rows > 16 || n > 8)) ||
                            (r == ATTN_IN_KERNEL && rows > 16)) { printf("route %d holds no %d rows, %d chunks\n", (int)r, rows, n); return 1; }
                    }
    printf("ok\n");
    return 0;
}
