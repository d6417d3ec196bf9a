// launch_in_parts: every sequence in one part, in order, and no part of more work items than a grid dimension holds.
// Built by tests/test_launch_parts.py (host pass only).
#include <cstdio>

#include "../../paper_2505_14969_amd/csrc/launch.hpp"

int main() {
    int fails = 0, parts = 0;
    const int heads[] = {1, 3, 80, 127, 128, 4096, 16384, 32768, 65535};
    const int batches[] = {0, 1, 31, 32, 33, 64, 65, 512, 1000, 65535};
    for (int h : heads)
        for (int b : batches) {
            stree_dims d = {};
            d.batch = b, d.nheads = h, d.headdim = 128, d.nnodes = 200;
            int next = 0;
            const hipError_t e = stree::launch_in_parts(d, [&](const stree_dims &s, int first) {
                // two workgroups of 512 lanes per head, in eights: below 2^32
                const unsigned long long items = (2ull * s.batch * s.nheads + 7) / 8 * 8 * 512;
                if (first != next || s.batch < 1 || s.nheads != h || s.nnodes != 200 || items >= (1ull << 32)) {
                    printf("%d heads, batch %d: part of %d from %d (%llu work items)\n", h, b, s.batch, first, items);
                    ++fails;
                }
                next = first + s.batch;
                ++parts;
                return hipSuccess;
            });
            if (e != hipSuccess || next != b) {
                printf("%d heads, batch %d: ended at %d\n", h, b, next);
                ++fails;
            }
        }
    stree_dims d = {};
    d.batch = 100, d.nheads = 65535;
    int calls = 0;
    if (stree::launch_in_parts(d, [&](const stree_dims &, int) { ++calls; return hipErrorInvalidValue; }) != hipErrorInvalidValue || calls != 1) {
        printf("a failed part was followed by another\n");
        ++fails;
    }
    printf("%d mismatches, %d parts\n", fails, parts);
    return fails != 0;
}
