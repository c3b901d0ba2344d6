// The division of P pairs among the waves of the permutation, against 64-bit arithmetic: every pair belongs to one wave,
// and the waves that hold pairs are counted right, up to the largest P that the C entry accepts.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include "../../paper_2502_12224_amd/csrc/perm_split.h"

static void check(int64_t P, int nw) {
    const int64_t want = ((P + nw - 1) / nw + 63) / 64 * 64;
    const int chunk = fate::perm_chunk((int)P, nw);
    bool ok = chunk == want;
    int64_t next = 0;
    int holding = 0;
    for (int w = 0; ok && w < nw; ++w) {
        const int beg = w * chunk, end = fate::perm_end((int)P, beg, chunk);
        if (beg >= P) ok = end <= beg;
        else {
            ok = beg == next && end == (beg + want < P ? beg + want : P);
            next = end;
            ++holding;
        }
    }
    ok = ok && next == P && fate::perm_holding((int)P, chunk) == holding;
    if (!ok) {
        std::printf("perm split: wrong for P = %lld, %d waves\n", (long long)P, nw);
        std::exit(1);
    }
}

int main() {
    const int64_t top = INT32_MAX;
    auto at = [&](int64_t P) {
        if (P < 0 || P > top) return;
        const int waves = fate::perm_waves((int)P, 64);
        const int64_t groups = (P + 63) / 64;
        const int64_t want = P <= 64 ? 1 : groups < 4 ? 4 : groups > fate::kPermMaxWaves ? fate::kPermMaxWaves : groups;
        if (waves != want || fate::perm_waves((int)P, 65) != (P <= 64 ? 1 : fate::kPermMaxWaves)) {
            std::printf("perm split: %d waves for P = %lld\n", waves, (long long)P);
            std::exit(1);
        }
        check(P, waves);
        if (P > 0) check(P, fate::kPermMaxWaves);       // (the routing call's workgroup always has 16)
    };
    for (int64_t P = 0; P <= 5000; ++P) at(P);
    for (int64_t c = 1; c <= top; c *= 2)               // both sides of every power of two, and of the 16 waves' share of it
        for (int64_t d = -1100; d <= 1100; ++d) at(c + d);
    for (int64_t P = top - 3000; P <= top; ++P) at(P);
    for (int64_t P = 2013265920 - 2000; P <= 2013265920 + 20000; ++P) at(P);
    for (int64_t P = 6151; P <= top; P += 6151 * 97) at(P);
    std::puts("perm split driver: ok");
    return 0;
}
