// Decode layer (2 to 8 tokens), up projection: whether the routed experts are taken in whole tiles (128 neurons, a wave
// takes all columns) or in split ones (64 neurons, the columns over pairs of waves).  Same bits.  It hangs on how many
// experts the tokens name, which a skewed gate, or equal tokens, make far fewer than a uniform one, and which no host knows: every
// workgroup counts them for itself.  No device code: the CPU tests compile this header by itself.
#pragma once

namespace fate {

#ifdef __HIPCC__
#define FATE_TILE_FN __host__ __device__ inline
#else
#define FATE_TILE_FN inline
#endif

// experts: named by the tokens; tiles_whole: whole tiles of one; tiles_shared: tiles of the shared experts, split in both
// cases; slots: workgroups that the device holds at once.
// With room for all, split tiles spread the weights further (H = 2048, split / whole tiles of a layer: 440 / 264 41.0 us
// split, 43.2 whole; 484 / 286 42.8 / 44.8).  Beyond that the second round's tiles start, and select, when the first
// one's end, and whole ones are faster (513 / 279 50.0 us split, 47.8 whole; 568 / 328 48.4 / 45.6; 829 / 436 61.9 /
// 57.9), also where they are more than a round themselves (852 96.4 / 90.8; H = 3072: 546 / 317 68.9 / 61.4, 1113 / 601
// 97.9 / 96.0).  With longer rows the second round's start counts less than an uneven share of the tiles: H = 4096, 683 /
// 341 78.2 / 80.4, 747 / 373 78.8 / 80.7, 849 / 447 92.0 / 88.4, 875 / 437 88.2 / 86.0, 1152 / 576 121.1 / 125.3.
// (4-bit experts.  8-bit ones always take split tiles: whole ones at H = 2048 622 / 333 68.7 / 69.6, 852 / 448 83.9 /
// 81.1, but H = 4096 682 / 363 112.2 / 123.1, 1568 / 784 239.8 / 264.3.)
// (I of less than 2^31, 64 pairs and 16 shared experts: no sum passes 2^32.)
FATE_TILE_FN bool up_tiles_whole(unsigned experts, unsigned tiles_whole, unsigned tiles_shared, unsigned slots, int H) {
    const unsigned routed = experts * tiles_whole, whole = routed + tiles_shared, split = routed + whole;
    return H <= 3072 ? split > slots : whole <= slots && 2 * split > 3 * slots;
}

// Most routed tiles that up to `experts` named experts make, which is what has to be launched: a workgroup without a tile
// ends when it has selected.  *any: whether some number of them is taken whole.
inline long long up_tiles_most(int experts, unsigned tiles_whole, unsigned tiles_shared, unsigned slots, int H, bool* any) {
    long long most = 0;
    *any = false;
    for (int n = 1; n <= experts; ++n) {
        const bool whole = up_tiles_whole(n, tiles_whole, tiles_shared, slots, H);
        const long long tiles = (whole ? 1LL : 2LL) * n * tiles_whole;
        most = tiles > most ? tiles : most;
        *any = *any || whole;
    }
    return most;
}

}  // namespace fate
