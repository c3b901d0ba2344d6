// How block_permute divides P pairs among the waves of its workgroup.  P may be anything up to 2^31 - 1, so a sum that
// passes it is taken in unsigned arithmetic.  No device code: the CPU tests compile this header by itself.
#pragma once

namespace fate {

#ifdef __HIPCC__
#define FATE_PERM_FN __host__ __device__ inline
#else
#define FATE_PERM_FN inline
#endif

constexpr int kPermMaxWaves = 16;

// Waves of a permutation's workgroup: one per 64 pairs, at least four (64 pairs are one wave's work altogether).  More than
// 64 experts: all of them, for the popularity order, which they divide among themselves.
FATE_PERM_FN int perm_waves(int P, int E) {
    if (P <= 64) return 1;
    if (E > 64) return kPermMaxWaves;
    const unsigned n = ((unsigned)P + 63u) / 64u;
    return n < 4u ? 4 : (n > (unsigned)kPermMaxWaves ? kPermMaxWaves : (int)n);
}

// Pairs of one wave of nw, a multiple of 64.
FATE_PERM_FN int perm_chunk(int P, int nw) { return (int)((((unsigned)P + (unsigned)nw - 1u) / (unsigned)nw + 63u) & ~63u); }

// End of the pairs that start at beg (a multiple of chunk; past P: there are none).
FATE_PERM_FN int perm_end(int P, int beg, int chunk) { return P - beg < chunk ? P : beg + chunk; }

// Waves that hold pairs.
FATE_PERM_FN int perm_holding(int P, int chunk) { return chunk > 0 ? (int)(((unsigned)P + (unsigned)chunk - 1u) / (unsigned)chunk) : 0; }

}  // namespace fate
