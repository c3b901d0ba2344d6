// Whole or split routed tiles of a decode layer's up projection: which side of the line the number of named experts lies on,
// and that what is launched holds every tile for every number of experts.
#include <cstdio>
#include <cstdlib>
#include <initializer_list>
#include "../../paper_2502_12224_amd/csrc/up_tiles.h"

static void expect(bool ok, const char* what, int n) {
    if (ok) return;
    std::printf("up tiles: %s (%d experts)\n", what, n);
    std::exit(1);
}

int main() {
    using fate::up_tiles_whole;
    const int slots = 512;
    // 60 experts, 4 selected, tiles 11 and 88 shared, 7 and 8 tokens: about 23 and 25 experts of a uniform gate, 9 to 15 of
    // a Zipf gate, and as few as 4 if all tokens are equal
    for (int n : {4, 9, 12, 13, 15, 19}) expect(!up_tiles_whole(n, 11, 88, slots, 2048), "one round of split tiles is taken whole", n);
    for (int n : {20, 22, 25}) expect(up_tiles_whole(n, 11, 88, slots, 2048), "more than a round of split tiles stays split", n);
    // 64 experts, 6 selected, 8 tokens
    expect(up_tiles_whole(35, 11, 44, slots, 2048), "more than a round of split tiles stays split", 35);
    expect(!up_tiles_whole(6, 11, 44, slots, 2048), "one round of split tiles is taken whole", 6);
    // H = 4096, few large experts: 2 tokens name 3 or 4
    expect(!up_tiles_whole(3, 112, 0, slots, 4096), "an uneven share of large whole tiles", 3);
    expect(up_tiles_whole(4, 112, 0, slots, 4096), "two whole rounds stay split", 4);
    expect(!up_tiles_whole(5, 112, 0, slots, 4096), "whole tiles beyond a round", 5);
    // what is launched
    for (int H : {1024, 3072, 3073, 4096})
        for (int tiles : {1, 3, 11, 22, 112, 1 << 24})
            for (unsigned shared : {0u, 12u, 88u, 600u, 1u << 29})
                for (int experts = 1; experts <= 64; ++experts) {
                    bool any = false, seen = false, reached = false;
                    const long long most = fate::up_tiles_most(experts, tiles, shared, slots, H, &any);
                    for (int n = 1; n <= experts; ++n) {
                        const bool whole = up_tiles_whole(n, tiles, shared, slots, H);
                        const long long need = (whole ? 1LL : 2LL) * n * tiles;
                        expect(need <= most, "a tile is not launched", n);
                        reached = reached || need == most;
                        seen = seen || whole;
                    }
                    expect(reached && seen == any, "more is launched than any number needs", experts);
                }
    std::puts("up tiles driver: ok");
    return 0;
}
