// Prefill-side expert FFN: MFMA grouped GEMM over quantised experts.
//
// Four launches per layer:
//   prep     x (bf16) -> fp16 copy, shared-expert gate values, and the tile
//            tables (prefix sums of tiles per expert segment) of both GEMMs;
//   up       grouped GEMM  h = silu(X W1^T) * (X W3^T)   -> fp16 [rows, I]
//   down     grouped GEMM  Yp = h W2^T                     -> fp16 [rows, H]; fp32 [K parts][rows, H]
//            where the reduction dimension is cut into parts
//   combine  y[t] = sum_j w[t,j] Yp[inv_perm[t*k+j]] + sum_s g_s(t) Yp_s[t]
// Rows are (token, expert) pairs in the sorted order of the permutation, so
// an expert's rows are contiguous; shared experts are extra segments of N rows.
//
// GEMM tile: a workgroup of four waves owns up to 128 rows (64 of other widths than 4 bits) and, per wave, two
// 32-row blocks of weights (the same block of W1 and W3, or two neighbouring
// blocks of W2): 8 accumulators of 32x32, so that a dequantised operand serves
// four matrix products.  Two workgroups share a compute unit.
// Everything the loop reads - activations, raw codes, scales - travels from
// memory to LDS without passing through registers (global_load_lds), in a
// ring of stages of 64 columns (128 for int2); the waits count the loads that
// may still be in flight, so the stages ahead are never drained.  A wave
// dequantises its own codes from LDS into the A operand of
// v_mfma_f32_32x32x16_f16 (exact code, one rounding in code*scale) and
// multiplies them with the workgroup's activation rows; accumulation is fp32.
// What bounds it, by counters.  Full tiles (2048 tokens of the Mixtral shape, E = 8, H = 4096, I = 14336): the chip
// holds 1.5 GHz under the up GEMM and the matrix pipe is busy 73 % of the cycles (down 60 %), with 5.6 (4.9) vector
// instructions per matrix instruction.  Tiles of at most 32 rows have a form of their own (below).
// Measured (before: 64-row tiles, codes in registers): up 1125 -> 867 us and down 645 -> 515 us at 2048 tokens
// of the Mixtral shape, 271 -> 200 and 148 -> 124 us at 2048 tokens of the Qwen shape.
#include <hip/hip_fp16.h>
#include <algorithm>
#include <type_traits>
#include "common.h"
#include "qformat.h"
#include "ffn_internal.h"
#include "async_lds.h"
#include "tile_table.h"
#include "up_tiles.h"
#include "route_device.h"

namespace fate {

typedef _Float16 f16x2v_t __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

constexpr int kBM = 1 << kTileRowsLog2;   // most rows of a workgroup tile
constexpr int kBNUp = 128;          // weight rows per workgroup tile of the up GEMM (of each matrix)
constexpr int kBNDown = 256;        // weight rows per workgroup tile of the down GEMM
constexpr int kCombineRows = 64;    // rows whose addresses and weights a combination block keeps in LDS
constexpr int kKQ = 128;            // H and I must be multiples of this
constexpr int kGemmLds = 80 * 1024 - 128;   // two workgroups per compute unit
constexpr int kGemmSlots = 2 * 256; // workgroups the device holds at once

struct GemmArgs {
    const __half* A_r; int lda_r;      // activations fp16 of routed segments
    const __half* A_s; int lda_s;      // activations fp16 of shared segments
    int H;                             // hidden size
    const fate_qexpert* experts; const fate_qexpert* shared;
    int E, n_shared, N, k;
    const int32_t* perm;
    const int4* segs;                  // [E + n_shared + 1]: first tile, expert, first row and rows of a segment
    void* out_r; int ldo_r;            // routed rows, by sorted position
    void* out_s; int ldo_s;            // shared rows, s*N + t
    int nb_r, nb_s;                    // column blocks per routed / shared segment
    int rows_r, rows_s;                // most rows of a tile, log2
    int kp_r, kp_s;                    // parts of the reduction dimension (down GEMM), each with an output of its own
    size_t part_r, part_s;             // elements between those outputs
    int f32_r, f32_s;                  // down GEMM: output elements are fp32 (else fp16)
    int bits_r, group_r, bits_s, group_s;              // decode layer: entries of another format, or with zero-points, count as absent
    LayerOut lo;                       // decode layer only
    int32_t* status;
};

// Rows of one prefill tile: a segment's rows are cut into as few tiles as hold them, of equal size up to
// a whole number of 32-row products.
__device__ __forceinline__ int tile_rows(int T, int most_log2) {
    const int nt = (T + (1 << most_log2) - 1) >> most_log2;
    return ((T + nt - 1) / nt + 31) & ~31;
}

// x to fp16 and the shared experts' gate, one workgroup per token, and before them one for the tile
// tables: a serial chain of its own, which starts first and runs beside the conversion (built by token 0's
// workgroup behind its row, whole passes of 13 to 2048 tokens took the same within 1 %).  A later piece of a
// layer processed in pieces finds x and the gate values in place: it launches the tables' workgroup only.
__global__ __launch_bounds__(256) void prefill_prep_kernel(const uint16_t* __restrict__ x, int N, int H, int E,
                                                           int n_shared, const int32_t* __restrict__ offsets,
                                                           const int32_t* __restrict__ order,
                                                           const uint16_t* __restrict__ shared_gate,
                                                           __half* __restrict__ xh, float* __restrict__ sgate,
                                                           int4* __restrict__ tab_up, int4* __restrict__ tab_down,
                                                           TileBlocks nb, PartSel sel) {
    __shared__ float red[4];
    const int t = (int)blockIdx.x - 1, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int nvec = H >> 3;
    if (t < 0) {
        if (wave == 0) wave_tile_tables(offsets, order, E, n_shared, N, nb, sel, tab_up, tab_down);
        return;
    }
    const uint4* xr = reinterpret_cast<const uint4*>(x) + (size_t)t * nvec;
    uint4* xo = reinterpret_cast<uint4*>(xh) + (size_t)t * nvec;
    const uint4* gv = reinterpret_cast<const uint4*>(shared_gate);
    float acc = 0.f;
    for (int c = tid; c < nvec; c += 256) {
        const uint4 v = xr[c];
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
        uint32_t o[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            __half2 h = __floats2half2_rn(bf16_lo(w[i]), bf16_hi(w[i]));
            o[i] = *reinterpret_cast<uint32_t*>(&h);
        }
        store_pairs(xo, c, make_uint4(o[0], o[1], o[2], o[3]));
        if (gv) {
            const uint4 g = gv[c];
            const uint32_t gw[4] = {g.x, g.y, g.z, g.w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                acc = fmaf(bf16_lo(w[i]), bf16_lo(gw[i]), acc);
                acc = fmaf(bf16_hi(w[i]), bf16_hi(gw[i]), acc);
            }
        }
    }
    if (gv) {
        acc = wave_sum(acc);
        if (lane == 0) red[wave] = acc;
        __syncthreads();
        if (tid == 0) sgate[t] = 1.0f / (1.0f + expf(-((red[0] + red[1]) + (red[2] + red[3]))));
    }
}

// Pair p (0..3) of the 8 columns that a lane holds of matrix-core step d of the stage whose raw tile pieces are `raw`
// (the activations' pair order: int4 step d takes columns 2d, 2d + 1 of every dword), dequantised to a pair of fp16.  The
// code becomes an exact fp16 integer (its bits OR-ed into the mantissa of a power of two, which is subtracted again) and
// is rounded once in code * scale; with a zero-point (u - z) * s is rounded twice.
template <int BITS, bool ZP, int TPS>
__device__ __forceinline__ uint32_t dequant_pair(const uint4 (&raw)[TPS], int d, int p, f16x2v_t s2, f16x2v_t z2) {
    auto dword = [&](int tl, int i) { return i == 0 ? raw[tl].x : i == 1 ? raw[tl].y : i == 2 ? raw[tl].z : raw[tl].w; };
    auto both = [](float v) { return f16x2v_t{(_Float16)v, (_Float16)v}; };
    f16x2v_t w;
    if constexpr (BITS == 2) {
        // sixteen fields per dword, two dwords per 32 columns; signed code 2u - 3 without a zero-point
        const uint32_t r = dword(0, 2 * (d >> 2) + (p >> 1)), x = p & 1 ? r >> 8 : r;
        const int f = d & 3;
        const uint32_t v = f == 0 ? and_or_b32(x, 0x00030003u, 0x64006400u) : f == 1 ? and_or_b32(x, 0x000c000cu, 0x5c005c00u)
                         : f == 2 ? and_or_b32(x, 0x00300030u, 0x54005400u) : and_or_b32(x, 0x00c000c0u, 0x4c004c00u);
        w = __builtin_bit_cast(f16x2v_t, v) - both(f == 0 ? 1024.f : f == 1 ? 256.f : f == 2 ? 64.f : 16.f);
        w = ZP ? w - z2 : w * both(2.f) - both(3.f);
    } else if constexpr (BITS == 4) {
        const uint32_t r = dword(0, p), x = d < 2 ? r : r >> 8;
        const uint32_t v = d & 1 ? and_or_b32(x, 0x00f000f0u, 0x54005400u) : and_or_b32(x, 0x000f000fu, 0x64006400u);
        w = __builtin_bit_cast(f16x2v_t, v) - both((d & 1 ? 64.f : 1024.f) + (ZP ? 0.f : 8.f));
        if constexpr (ZP) w = w - z2;
    } else {
        const uint32_t v = __builtin_amdgcn_perm(0x64646464u, dword(d >> 1, 2 * (p & 1) + (d & 1)), p & 2 ? 0x04030402u : 0x04010400u);
        w = __builtin_bit_cast(f16x2v_t, v) - both(1152.f);       // 1024 + 128
    }
    return __builtin_bit_cast(uint32_t, w * s2);
}

// Eight activations of a lane: one piece of 16 bytes, or 8 bytes of two pieces.
template <int N>
__device__ __forceinline__ f16x8_t load_piece(const char* base, const uint32_t (&off)[N]) {
    if constexpr (N == 1) {
        return *reinterpret_cast<const f16x8_t*>(base + off[0]);
    } else {
        const uint2 a = *reinterpret_cast<const uint2*>(base + off[0]), b = *reinterpret_cast<const uint2*>(base + off[1]);
        return __builtin_bit_cast(f16x8_t, u32x4_t{a.x, a.y, b.x, b.y});
    }
}

// A value that is the same in all lanes, told to the compiler (it keeps what it loaded from memory
// in vector registers otherwise).
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
template <class T>
__device__ __forceinline__ T* uniform(T* p) {
    const uint64_t v = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((int)(uint32_t)v), hi = __builtin_amdgcn_readfirstlane((int)(v >> 32));
    return reinterpret_cast<T*>((uint64_t)hi << 32 | lo);
}

// What one tile needs; everything is the same in all lanes of a wave unless said otherwise.
struct TileCtx {
    const fate_qexpert* ex;
    const __half* A; int lda;
    const int32_t* rows; int div;      // activation row of tile row r: rows[r] / div, or r itself when rows is NULL
    int nrows;                         // live rows of the tile (the rest read the first one and are not stored)
    int wrow[2];                       // first weight row of the wave's two blocks
    bool wlive[2];                     // whether they exist (a wave without weights still stages activations)
    int Nout, K, col0, ncol;           // weight rows of the matrix, its columns, this part's columns
    int group;
    void* out; int ldo;                // output row 0 of the tile
    bool f32;                          // its elements: fp32 or fp16
    const int32_t* orows;              // decode-sized form: output row of tile row r, or NULL: r itself
};

template <int BITS>
struct GemmFmt {
    static constexpr int KT = QFmt<BITS>::KT;
    static constexpr int BK = KT < 64 ? 64 : KT;          // columns per stage
    static constexpr int TPS = BK / KT;                   // weight tiles per stage and block
    static constexpr int XROW = BK * 2;                   // bytes per activation row of a stage
    static constexpr int xbytes(int nmt) { return nmt * 32 * XROW; }
    static constexpr int stage(int nmt) { return xbytes(nmt) + 4 * 2 * TPS * 1024 + 4 * 256; }
    static constexpr int depth(int nmt) { return kGemmLds / stage(nmt) < 6 ? kGemmLds / stage(nmt) : 6; }
};

// One tile with NMT 32-row products.  UP: two matrices and SwiGLU; else one matrix, two row blocks.  only: rows that are
// stored (of a single product).
// Stage layout: activation rows (16-byte pieces of row r permuted by r & 7: conflict-free
// ds_read_b128), then per wave the raw weight tiles of both blocks, then per wave 256 bytes of
// scales and zero-points (lanes 0-15 / 16-31: scales of block 0 / 1, 32-47 / 48-63: zero-points).
template <int BITS, bool ZP, bool UP, int NMT>
__device__ __forceinline__ void gemm_pipe(const TileCtx& c, char* smem, uint32_t only = ~0u) {
    typedef GemmFmt<BITS> F;
    constexpr int KT = F::KT, BK = F::BK, TPS = F::TPS, XROW = F::XROW;
    constexpr int SPT = KT / 16;                          // matrix-core steps per weight tile
    constexpr int NX = NMT * 32 * XROW / 4096;            // activation loads per wave and stage
    constexpr int RPL = 1024 / XROW;                      // activation rows per load
    constexpr int S = F::depth(NMT), SB = F::stage(NMT);
    constexpr int LPS = NX + 2 * TPS + 1;
    static_assert(S >= 2, "at least one stage ahead");
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 31, half = lane >> 5;
    const int nstage = c.ncol / BK, tiles_k = c.K / KT;
    const uint32_t lds0 = lds_offset(smem);
    const char* abase = uniform(reinterpret_cast<const char*>(c.A));

    // activation loads: load i of this wave fills rows (i*4 + wave)*RPL + lane / (64 / RPL)
    uint32_t xoff[NX];
    {
        constexpr int LPR = XROW / 16;                    // lanes (16-byte pieces) per row
        const int rl = lane / LPR, q = lane % LPR;
#pragma unroll
        for (int i = 0; i < NX; ++i) {
            const int r = (i * 4 + wave) * RPL + rl;
            const int rr = r < c.nrows ? r : 0;
            const int ar = c.rows ? c.rows[rr] / c.div : rr;
            xoff[i] = ((uint32_t)ar * (uint32_t)c.lda + (uint32_t)c.col0) * 2u + (uint32_t)((q ^ (r & 7)) * 16);
        }
    }
    // weights: tile (row block, column tile) is 1 KiB; scales: group-major [groups][Nout]
    const char* wbase[2];
    const char* sbase;                                    // this lane's scale (or zero-point) address at group 0
    {
        const void* wp[2] = {UP ? c.ex->w1 : c.ex->w2, UP ? c.ex->w3 : c.ex->w2};
        const void* sp[2] = {UP ? c.ex->s1 : c.ex->s2, UP ? c.ex->s3 : c.ex->s2};
        const void* zp[2] = {UP ? c.ex->z1 : c.ex->z2, UP ? c.ex->z3 : c.ex->z2};
#pragma unroll
        for (int i = 0; i < 2; ++i)
            wbase[i] = static_cast<const char*>(uniform(wp[i])) + ((size_t)(c.wrow[i] >> 5) * tiles_k + c.col0 / KT) * 1024;
        const int b = (lane >> 4) & 1;
        const void* p0 = ZP && half ? zp[0] : sp[0];          // (these differ between lanes)
        const void* p1 = ZP && half ? zp[1] : sp[1];
        sbase = static_cast<const char*>(b ? p1 : p0) + (size_t)(b ? c.wrow[1] : c.wrow[0]) * 2 + (lane & 15) * 4;
    }
    const uint32_t lane16 = lane * 16;
    // the next stage to be requested: stages are requested in order (group = 64 columns at least)
    int gcol = c.col0 % c.group;
    sbase += (size_t)(c.col0 / c.group) * c.Nout * 2;
    // load l (0 .. LPS - 1) of stage st into ring slot `slot`
    auto issue_one = [&](int st, int slot, int l) {
        const uint32_t base = lds0 + slot * SB;
        if (l < NX) {
            lds_load16(base + (l * 4 + wave) * 1024, abase + (size_t)st * XROW, xoff[l]);
        } else if (l < NX + 2 * TPS) {
            const int i = (l - NX) / TPS, tl = (l - NX) % TPS;
            lds_load16(base + F::xbytes(NMT) + (wave * 2 * TPS + i * TPS + tl) * 1024, wbase[i] + (size_t)(st * TPS + tl) * 1024,
                       lane16);
        } else {
            lds_load4(base + F::xbytes(NMT) + 4 * 2 * TPS * 1024 + wave * 256, sbase);
            gcol += BK;
            if (gcol >= c.group) {
                gcol -= c.group;
                sbase += (size_t)c.Nout * 2;
            }
        }
    };
    auto issue = [&](int st, int slot) {
#pragma unroll
        for (int l = 0; l < LPS; ++l) issue_one(st, slot, l);
    };

    f32x16_t acc[2][NMT];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int mt = 0; mt < NMT; ++mt)
#pragma unroll
            for (int j = 0; j < 16; ++j) acc[i][mt][j] = 0.f;
    // this lane's activation pieces of a stage, in the order of the weight operands
    // (8-bit tiles: a step's 8 columns are half of two pieces)
    constexpr int APS = BITS == 8 ? 2 : 1;
    uint32_t aoff[TPS * SPT][APS];
#pragma unroll
    for (int tl = 0; tl < TPS; ++tl)
#pragma unroll
        for (int d = 0; d < SPT; ++d)
#pragma unroll
            for (int i = 0; i < APS; ++i) {
                const int piece = BITS == 8 ? tl * 4 + 2 * d + i : (tl * KT + half * (KT / 2)) / 8 + d;
                aoff[tl * SPT + d][i] = n * XROW + (piece ^ (n & 7)) * 16 + (BITS == 8 ? half * 8 : 0);
            }

    constexpr int KS = TPS * SPT;                         // matrix-core steps per stage
    int slot = 0, slot_in = S - 1;                        // stage being multiplied, stage being filled
    auto next = [](int i) { return i + 1 == S ? 0 : i + 1; };
#pragma unroll
    for (int s = 0; s < S - 1; ++s)
        if (s < nstage) issue(s, s);
    auto step = [&](int st, auto more) {                  // more: whether stage st + S - 1 exists
        if constexpr (more) wait_loads<(S - 2) * LPS>();
        else wait_stages<LPS, S - 2>(nstage - 1 - st);
        lds_only_barrier();                               // stage st is in LDS, everyone is done with stage st - 1
        const char* base = smem + slot * SB;
        const char* wl = base + F::xbytes(NMT) + wave * (2 * TPS * 1024) + lane16;
        const char* sl = base + F::xbytes(NMT) + 4 * 2 * TPS * 1024 + wave * 256 + n * 2;
        uint4 raw[2][TPS];
        f16x2v_t s2[2], z2[2];
        f16x8_t av[2][NMT];                               // activations of the current and the next step
        u32x4_t b[2][2];                                  // dequantised codes: [step parity][block]
        auto read_av = [&](int d, int mt) {
            av[d & 1][mt] = load_piece<APS>(base + mt * 32 * XROW, aoff[d]);
        };
        // the e-th of the 8 pairs of a step: 4 of each block
        auto dequant = [&](int d, int e) { b[d & 1][e >> 2][e & 3] = dequant_pair<BITS, ZP>(raw[e >> 2], d, e & 3, s2[e >> 2], z2[e >> 2]); };
#pragma unroll
        for (int i = 0; i < 2; ++i) {
#pragma unroll
            for (int tl = 0; tl < TPS; ++tl) raw[i][tl] = *reinterpret_cast<const uint4*>(wl + (i * TPS + tl) * 1024);
            const _Float16 sv = *reinterpret_cast<const _Float16*>(sl + i * 64);
            const _Float16 zv = ZP ? *reinterpret_cast<const _Float16*>(sl + 128 + i * 64) : (_Float16)0.f;
            s2[i] = f16x2v_t{sv, sv};
            z2[i] = f16x2v_t{zv, zv};
        }
#pragma unroll
        for (int mt = 0; mt < NMT; ++mt) read_av(0, mt);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int e = 0; e < 8; ++e) dequant(0, e);
        // Matrix products of a step with the next step's dequantisation and LDS reads between them: a product
        // occupies the matrix pipe for 32 cycles, so the dequantisation of a step runs beside the products
        // of four row blocks.  (The
        // fences keep the compiler from collecting the vector instructions in front of the products.)
#pragma unroll
        for (int d = 0; d < KS; ++d) {
#pragma unroll
            for (int mt = 0; mt < NMT; ++mt) {
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = 0; i < 2; ++i)
                    acc[i][mt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8_t, b[d & 1][i]), av[d & 1][mt],
                                                                        acc[i][mt], 0, 0, 0);
                // (the next stage's loads go out one at a time: the memory path of a compute unit takes 64 bytes
                // per cycle, and a wave that asks for a whole stage at once waits for it)
                if constexpr (more) {
                    constexpr int G = KS * NMT;
#pragma unroll
                    for (int l = LPS * (d * NMT + mt) / G; l < LPS * (d * NMT + mt + 1) / G; ++l) issue_one(st + S - 1, slot_in, l);
                }
                if (d + 1 < KS) {
                    read_av(d + 1, mt);
#pragma unroll
                    for (int e = 8 * mt / NMT; e < 8 * (mt + 1) / NMT; ++e) dequant(d + 1, e);
                }
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        slot = next(slot);
        slot_in = next(slot_in);
    };
    int st = 0;
    for (; st + S - 1 < nstage; ++st) step(st, std::true_type{});
    for (; st < nstage; ++st) step(st, std::false_type{});
    // epilogue: lane holds tile row mt*32 + n, weight rows 8*(j/4) + 4*half + j%4 of each block
#pragma unroll
    for (int mt = 0; mt < NMT; ++mt) {
        const int r = mt * 32 + n;
        if (r < c.nrows && (NMT > 1 || (only >> n) & 1)) {
            if constexpr (UP) {
                // in pair order a lane's 16 neurons are two pieces of 16 bytes
                uint4* o = reinterpret_cast<uint4*>(static_cast<__half*>(c.out) + (size_t)r * c.ldo + c.wrow[0]) + 2 * half;
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    __half h[8];
#pragma unroll
                    for (int q = 0; q < 4; ++q)
#pragma unroll
                        for (int j = 0; j < 2; ++j) {
                            const float g = acc[0][mt][4 * q + 2 * u + j];
                            h[2 * q + j] = __float2half(g / (1.0f + __expf(-g)) * acc[1][mt][4 * q + 2 * u + j]);
                        }
                    if (c.wlive[0]) o[u] = *reinterpret_cast<uint4*>(h);
                }
            } else {
                __half* o = static_cast<__half*>(c.out) + (size_t)r * c.ldo + 4 * half;
                float* of = static_cast<float*>(c.out) + (size_t)r * c.ldo + 4 * half;
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        if (!c.wlive[i]) continue;
                        if (c.f32) {
                            *reinterpret_cast<float4*>(of + c.wrow[i] + 8 * q) =
                                make_float4(acc[i][mt][4 * q], acc[i][mt][4 * q + 1], acc[i][mt][4 * q + 2], acc[i][mt][4 * q + 3]);
                        } else {
                            __half h[4];
#pragma unroll
                            for (int j = 0; j < 4; ++j) h[j] = __float2half(acc[i][mt][4 * q + j]);
                            *reinterpret_cast<uint2*>(o + c.wrow[i] + 8 * q) = *reinterpret_cast<uint2*>(h);
                        }
                    }
            }
        }
    }
}

// ---- few rows ------------------------------------------------------------------------------------
// Tiles of at most 32 rows (decode-sized calls and decode layers: 16 and 8): the codes stream once and everything else is
// small, so a tile is bounded by the memory path and by the vector instructions that widen the codes.  A code enters the
// matrix cores as an exact integer counted from the middle of its range (an AND-OR and a subtraction per pair of codes, for
// int4 half a shift), and the fp16 scale multiplies the fp32 sum of a stage's columns (which lie in one group): weights
// enter without rounding.  With a zero-point in memory its distance to the middle times the sum of the activations (a
// product with ones) is added.  (int4 as u + 16, a shift and an AND-OR, with the constant's share taken off the sum,
// is 0.6 to 1.6 % faster per layer of 1 to 48 tokens - 8 tokens of the DeepSeek shape 470.9 us for 8 layers, now 477.5; 13
// of the Qwen shape 353.7 for 6, now 359.5 - but makes an infinite activation NaN and sums through terms four times as
// large as the products.)  16x16x32 products: 16 rows of activations
// against 16 rows of weights, whose 16-byte pieces lane (cl = lane / 16, n = lane % 16) reads from the raw tiles in LDS.
// D: lane (cl, n) holds weight row n, activation rows 4cl .. 4cl + 3.
// NM: 16-row blocks of activations, R: rows staged (8, or 16 * NM).  KW: waves over which the reduction dimension is split
// (up projection of a decode layer: tiles of 64 neurons instead of 128).  QT: the columns add up in quarters, whether one
// wave takes them all or two take two each: h is rounded to fp16 and must not depend on that.
// Stages: 128 columns for int4 with groups of a multiple of 128 and for int2, 64 for int8 and for int4 otherwise.  HS = 2:
// int4 stages of 128 columns with two groups of 64 each, for decode-sized calls and decode layers, where the barrier of a
// stage counts: lanes 32..63 bring the second group's scales, zero-points are a load of their own.  Groups of 64 against
// stages of 64: 13 tokens of the Qwen shape 399 -> 379 us (6 layers), 8 of the DeepSeek shape 394 -> 376 (6).
// Against 32x32x16 products of codes made exact by a subtraction (16 rows) or of code * scale (32 rows): 48 tokens of the
// DeepSeek shape (5 rows a tile) up 51.1 -> 41.0, down 34.1 -> 29.2 us; 13 tokens of the Qwen shape 28.7 -> 24.6 (106 MB
// of codes and scales: 4.3 TB/s) and 17.2 -> 15.7; one token of the Mixtral shape 30.2 -> 26.8 and 17.5 -> 14.8.  By counters
// (these three, 1.8 to 2.1 GHz): 13 vector instructions per matrix instruction, the matrix pipe busy 9 to 15 %, waves
// waiting for memory or a barrier 28 to 40 % and for an issue slot 13 to 34 % of their time.
template <int BITS, bool ZP, int R, int KW, int BK, int HS>
struct RowsFmt {
    static constexpr int KT = QFmt<BITS>::KT;
    static constexpr int TPS = BK / KT;                   // weight tiles per stage and block
    static constexpr int GC = BK / HS;                    // columns of a sum that takes one scale
    static constexpr int KS = GC / 32;                    // matrix-core steps of it
    static constexpr bool split = BITS == 8 || (BITS == 4 && GC == 64); // a step's 8 columns are half of two pieces
    static constexpr int XROW = BK * 2;
    static constexpr int xwave = R * XROW;                // of the waves that share a range of columns
    static constexpr int xbytes = KW * xwave;
    static constexpr int SL = HS == 2 && ZP ? 2 : 1;      // loads of scales and zero-points
    static constexpr int sc0 = xbytes + 4 * 2 * TPS * 1024;
    static constexpr int stage = sc0 + 4 * SL * 256;
    static constexpr int depth = kGemmLds / stage < 8 ? kGemmLds / stage : 8;
};

// What a code is counted from: u - 8, u - 1.5 (2u - 3 of the symmetric format, halved) and u - 128, exact in fp16.
constexpr float code_mid(int bits) { return bits == 4 ? 8.f : bits == 2 ? 1.5f : 128.f; }

// the codes of step k of a lane's piece (16 or 8 bytes; GC: columns of the sum), less code_mid
template <int BITS, int GC>
__device__ __forceinline__ f16x8_t code_step(const uint4& r, int k) {
    u32x4_t v;
    // a pair whose bits are the code's, in the mantissa of a power of two: that and the middle are taken off again
    auto less = [](uint32_t w, float one) {
        const _Float16 h = (_Float16)(one + code_mid(BITS));
        return __builtin_bit_cast(uint32_t, __builtin_bit_cast(f16x2v_t, w) - f16x2v_t{h, h});
    };
    if constexpr (BITS == 4) {
        // pair i of a dword (bits 4i of both halves)
        auto pair = [&](uint32_t r, int i) {
            const uint32_t x = i < 2 ? r : r >> 8;
            return i & 1 ? less(and_or_b32(x, 0x00f000f0u, 0x54005400u), 64.f) : less(and_or_b32(x, 0x000f000fu, 0x64006400u), 1024.f);
        };
        if constexpr (GC == 128) v = u32x4_t{pair(r.x, k), pair(r.y, k), pair(r.z, k), pair(r.w, k)};
        else v = u32x4_t{pair(r.x, k), pair(r.y, k), pair(r.x, k + 2), pair(r.y, k + 2)};
    } else if constexpr (BITS == 2) {
        // field k of both bytes of both halves; field 0 is moved up (1024 + 1.5 is no fp16 number)
        const int f = k ? k : 1;
        const uint32_t m = 0x00030003u << (2 * f), o = 0x64006400u - 0x08000800u * f;           // 256, 64, 16
        const float one = f == 1 ? 256.f : f == 2 ? 64.f : 16.f;
        auto pair = [&](uint32_t r, int hi) {
            return less(and_or_b32(hi ? (k ? r >> 8 : r >> 6) : (k ? r : r << 2), m, o), one);
        };
        v = u32x4_t{pair(r.x, 0), pair(r.x, 1), pair(r.y, 0), pair(r.y, 1)};
    } else {
        const uint32_t a = k ? r.y : r.x, b = k ? r.w : r.z;
        auto pair = [&](uint32_t w, uint32_t sel) { return less(__builtin_amdgcn_perm(0x64646464u, w, sel), 1024.f); };
        v = u32x4_t{pair(a, 0x04010400u), pair(b, 0x04010400u), pair(a, 0x04030402u), pair(b, 0x04030402u)};
    }
    return __builtin_bit_cast(f16x8_t, v);
}

// a * b rounded to fp16 once.  Spelled out: from the plain expression the compiler makes this instruction in most copies
// of the code below and, where it joins the ends of two copies, a product and a conversion, which round twice (about one
// value in 2^15 differs) - the bits of h would hang on which kernels a copy is compiled into.
__device__ __forceinline__ uint16_t half_of_product(float a, float b) {
    uint32_t r;
    asm("v_fma_mixlo_f16 %0, %1, %2, 0" : "=v"(r) : "v"(a), "v"(b));
    return (uint16_t)r;
}

// Returns, the same in all waves, the rows that are not stored since one of their activations is infinite (or none): with
// zero-points only, where an infinite activation times a code and times the zero-point's distance can have both signs.
template <int BITS, bool ZP, bool UP, int NM, int R, int KW, bool QT, int BK, int HS = 1>
__device__ __forceinline__ uint32_t gemm_rows(const TileCtx& c, char* smem) {
    typedef RowsFmt<BITS, ZP, R, KW, BK, HS> F;
    constexpr int KT = F::KT, TPS = F::TPS, KS = F::KS, GC = F::GC, SL = F::SL, XROW = F::XROW;
    constexpr int S = F::depth, SB = F::stage;
    constexpr int NX = (F::xwave / 1024 + 4 / KW - 1) / (4 / KW);          // activation loads per wave and stage
    constexpr int LPS = NX + 2 * TPS + SL;
    static_assert(S >= 2, "at least one stage ahead");
    static_assert(HS == 1 || (BITS == 4 && BK == 128), "two groups of 64 columns");
    static_assert(KW == 1 || (KW == 2 && UP && QT && NM == 1), "the split of the reduction dimension belongs to the up projection");
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 15, cl = lane >> 4;
    const int kw = wave & (KW - 1);                       // this wave's range of columns
    const int ncol = c.ncol / KW, col0 = c.col0 + kw * ncol;
    const int nstage = uniform(ncol / BK), tiles_k = c.K / KT;
    const char* abase = uniform(reinterpret_cast<const char*>(c.A));
    const uint32_t lds0 = lds_offset(smem);
    constexpr int LPR = XROW / 16, RPL = 64 / LPR;        // lanes per row, rows per load
    constexpr int XL = F::xwave / 1024;                   // activation loads of a range; waves beyond them repeat one
    uint32_t xoff[NX];
    auto xpiece = [&](int i) { return (i * (4 / KW) + wave / KW) % XL; };
#pragma unroll
    for (int i = 0; i < NX; ++i) {
        const int r = xpiece(i) * RPL + lane / LPR, q = lane % LPR;
        const int rr = r < c.nrows ? r : 0;
        const int ar = c.rows ? c.rows[rr] / c.div : rr;
        xoff[i] = ((uint32_t)ar * (uint32_t)c.lda + (uint32_t)col0) * 2u + (uint32_t)((q ^ (r & 7)) * 16);
    }
    const char* wbase[2];
    // this lane's scale (HS = 1: lanes 0..31) or zero-point address, HS = 2 with zero-points: theirs
    const char *sbase, *zbase;
    {
        const void* wp[2] = {UP ? c.ex->w1 : c.ex->w2, UP ? c.ex->w3 : c.ex->w2};
        const void* sp[2] = {UP ? c.ex->s1 : c.ex->s2, UP ? c.ex->s3 : c.ex->s2};
        const void* zp[2] = {UP ? c.ex->z1 : c.ex->z2, UP ? c.ex->z3 : c.ex->z2};
#pragma unroll
        for (int i = 0; i < 2; ++i)
            wbase[i] = uniform(static_cast<const char*>(wp[i]) + ((size_t)(c.wrow[i] >> 5) * tiles_k + col0 / KT) * 1024);
        const int b = (lane >> 4) & 1;
        const bool zs = ZP && HS == 1 && lane >= 32;
        const size_t off = (size_t)(b ? c.wrow[1] : c.wrow[0]) * 2 + (lane & 15) * 4 +
                           (size_t)(col0 / c.group + (HS == 2 && lane >= 32 ? 1 : 0)) * c.Nout * 2;
        const void* p0 = zs ? zp[0] : sp[0];
        const void* p1 = zs ? zp[1] : sp[1];
        sbase = static_cast<const char*>(b ? p1 : p0) + off;
        zbase = SL == 2 ? static_cast<const char*>(b ? zp[1] : zp[0]) + off : nullptr;
    }
    const uint32_t lane16 = lane * 16;
    int gcol = col0 % c.group;                            // of the next stage to be requested
    auto issue_one = [&](int st, int slot, int l) {
        const uint32_t base = lds0 + slot * SB;
        if (l < NX) {
            lds_load16(base + kw * F::xwave + xpiece(l) * 1024, abase + (size_t)st * XROW, xoff[l]);
        } else if (l < NX + 2 * TPS) {
            const int i = (l - NX) / TPS, tl = (l - NX) % TPS;
            lds_load16(base + F::xbytes + (wave * 2 * TPS + i * TPS + tl) * 1024, wbase[i] + (size_t)(st * TPS + tl) * 1024, lane16);
        } else if (l == NX + 2 * TPS) {
            lds_load4(base + F::sc0 + wave * SL * 256, sbase);
            if constexpr (HS == 2) {
                sbase += (size_t)c.Nout * 4;
            } else {
                gcol += BK;
                if (gcol >= c.group) {
                    gcol -= c.group;
                    sbase += (size_t)c.Nout * 2;
                }
            }
        } else {
            lds_load4(base + F::sc0 + (wave * SL + 1) * 256, zbase);
            zbase += (size_t)c.Nout * 4;
        }
    };
    // by block of weight rows (half of the wave's block i) and block of activation rows
    f32x4_t out[2][2][NM], tot[2][2][NM];
    const f32x4_t zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int mb = 0; mb < NM; ++mb) out[i >> 1][i & 1][mb] = tot[i >> 1][i & 1][mb] = zero;
    f32x4_t xall[NM];                                     // sums of the activations: the same in all waves
#pragma unroll
    for (int mb = 0; mb < NM; ++mb) xall[mb] = zero;
    // stages done and the end of the current quarter (two waves: of the first one of this wave's two)
    const int nq = c.K / BK;
    int sidx = kw * (nq / 2), quarter = nq * (2 * kw + 1) / 4;
    auto close_quarter = [&]() {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int mb = 0; mb < NM; ++mb) {
                tot[i >> 1][i & 1][mb] += out[i >> 1][i & 1][mb];
                out[i >> 1][i & 1][mb] = zero;
            }
    };
    // this lane's piece of a block's raw tiles (rows 0..15 of it; rows 16..31 lie 256 bytes on) and of the activations
    constexpr bool wide = BITS == 8 || (BITS == 4 && GC == 128);          // the piece: 16 or 8 bytes
    const uint32_t woff = ((cl & 1) * 32 + n) * 16 + (cl >> 1) * (wide ? 1024 : 8);
    uint32_t aoff[KS][F::split ? 2 : 1];
#pragma unroll
    for (int k = 0; k < KS; ++k)
#pragma unroll
        for (int i = 0; i < (F::split ? 2 : 1); ++i) {
            const int piece = BITS == 8 ? (cl >> 1) * 4 + 2 * k + i
                            : BITS == 2 ? ((cl & 1) * 2 + (cl >> 1)) * 4 + k
                            : GC == 64 ? (cl & 1) * 4 + k + 2 * i : cl * 4 + k;
            aoff[k][i] = kw * F::xwave + (n & (R - 1)) * XROW + (piece ^ (n & 7)) * 16 +
                         (BITS == 8 ? (cl & 1) * 8 : F::split ? (cl >> 1) * 8 : 0);
        }
    const f16x8_t ones = {(_Float16)1.f, (_Float16)1.f, (_Float16)1.f, (_Float16)1.f, (_Float16)1.f, (_Float16)1.f, (_Float16)1.f, (_Float16)1.f};
    int slot = 0, slot_in = S - 1;
    auto next = [](int i) { return i + 1 == S ? 0 : i + 1; };
#pragma unroll
    for (int s = 0; s < S - 1; ++s)
        if (s < nstage) {
#pragma unroll
            for (int l = 0; l < LPS; ++l) issue_one(s, s, l);
        }
    auto step = [&](int st, auto more) {                  // more: whether stage st + S - 1 exists
        if constexpr (more) wait_loads<(S - 2) * LPS>();
        else wait_stages<LPS, S - 2>(nstage - 1 - st);
        lds_only_barrier();                               // stage st is in LDS, everyone is done with stage st - 1
        const char* base = smem + slot * SB;
        // the columns of one scale (HS = 2: the stage's halves, a weight tile each)
        auto columns = [&](auto half) {
            constexpr int h = half;
            const char* wl = base + F::xbytes + wave * (2 * TPS * 1024) + h * 1024 + woff;
            const char* sl = base + F::sc0 + wave * SL * 256 + h * 128 + n * 2;
            f16x8_t av[NM][KS];
            uint4 raw[4];
            float sv[4], zv[4];
#pragma unroll
            for (int k = 0; k < KS; ++k)
#pragma unroll
                for (int mb = 0; mb < NM; ++mb) av[mb][k] = load_piece<F::split ? 2 : 1>(base + mb * 16 * XROW + h * 128, aoff[k]);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const char* p = wl + (q >> 1) * TPS * 1024 + (q & 1) * 256;
                if constexpr (wide) raw[q] = *reinterpret_cast<const uint4*>(p);
                else {
                    const uint2 v = *reinterpret_cast<const uint2*>(p);
                    raw[q] = make_uint4(v.x, v.y, 0, 0);
                }
                sv[q] = (float)*reinterpret_cast<const _Float16*>(sl + q * 32);
                zv[q] = ZP ? code_mid(BITS) - (float)*reinterpret_cast<const _Float16*>(sl + (SL == 2 ? 256 : 128) + q * 32) : 0.f;
            }
            f32x4_t xsum[NM], acc[4][NM];
            // a block's products, then (behind the next block's) its sums
            auto products = [&](int q) {
#pragma unroll
                for (int k = 0; k < KS; ++k) {
                    const f16x8_t b = code_step<BITS, GC>(raw[q], k);
#pragma unroll
                    for (int mb = 0; mb < NM; ++mb)
                        acc[q][mb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(av[mb][k], b, k ? acc[q][mb] : zero, 0, 0, 0);
                }
            };
            if constexpr (ZP) {
#pragma unroll
                for (int mb = 0; mb < NM; ++mb)
#pragma unroll
                    for (int k = 0; k < KS; ++k)
                        xsum[mb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(av[mb][k], ones, k ? xsum[mb] : zero, 0, 0, 0);
#pragma unroll
                for (int mb = 0; mb < NM; ++mb) xall[mb] += xsum[mb];
            }
            auto sums = [&](int q) {
                const float s = BITS == 2 && !ZP ? 2.0f * sv[q] : sv[q];
#pragma unroll
                for (int mb = 0; mb < NM; ++mb)
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const float t = ZP ? fmaf(zv[q], xsum[mb][j], acc[q][mb][j]) : acc[q][mb][j];
                        out[q >> 1][q & 1][mb][j] = fmaf(s, t, out[q >> 1][q & 1][mb][j]);
                    }
            };
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                products(q);
                if constexpr (more) {
#pragma unroll
                    for (int l = LPS * (4 * h + q) / (4 * HS); l < LPS * (4 * h + q + 1) / (4 * HS); ++l) issue_one(st + S - 1, slot_in, l);
                }
                if (q) sums(q - 1);
            }
            sums(3);
        };
        columns(std::integral_constant<int, 0>{});
        if constexpr (HS == 2) columns(std::integral_constant<int, 1>{});
        if constexpr (QT && UP) {
            ++sidx;
            if constexpr (KW == 1) {
                if (sidx >= quarter) {
                    close_quarter();
                    // the next quarter that holds a stage ends at nq * q / 4
                    int qn = 4 * sidx / nq + 1;
                    while (qn < 4 && nq * qn / 4 <= sidx) ++qn;
                    quarter = nq * qn / 4;
                }
            } else if (sidx == quarter) {
                close_quarter();
            }
        }
        slot = next(slot);
        slot_in = next(slot_in);
    };
    int st = 0;
    for (; st + S - 1 < nstage; ++st) step(st, std::true_type{});
    for (; st < nstage; ++st) step(st, std::false_type{});
    if constexpr (QT && UP && KW == 1) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int mb = 0; mb < NM; ++mb) out[i >> 1][i & 1][mb] = tot[i >> 1][i & 1][mb];
    }
    if constexpr (KW > 1) {
        // the quarters' sums meet in LDS: the first range's wave of every block adds the others in order
        f32x4_t* red = reinterpret_cast<f32x4_t*>(smem);  // [quarter of the second range][block of the tile][4][64 lanes]
        lds_only_barrier();                               // the rings are done with
        const int blk = wave / KW;
        auto at = [&](int q, int i) { return red + ((q * (4 / KW) + blk) * 4 + i) * 64 + lane; };
        if (kw > 0) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                *at(0, i) = tot[i >> 1][i & 1][0];
                *at(1, i) = out[i >> 1][i & 1][0];
            }
        }
        lds_only_barrier();
        if (kw > 0) return 0;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            out[i >> 1][i & 1][0] = ((tot[i >> 1][i & 1][0] + out[i >> 1][i & 1][0]) + *at(0, i)) + *at(1, i);
    }
    uint32_t left = 0;
    if constexpr (ZP) {
#pragma unroll
        for (int mb = 0; mb < NM; ++mb)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const unsigned long long m = __ballot(!__builtin_isfinite(xall[mb][j]));
#pragma unroll
                for (int q = 0; q < 4; ++q) left |= (m >> (16 * q)) & 1 ? 1u << (mb * 16 + 4 * q + j) : 0u;
            }
    }
#pragma unroll
    for (int mb = 0; mb < NM; ++mb)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int r = mb * 16 + 4 * cl + j;
            if (r < c.nrows && !(ZP && (left >> r) & 1)) {
                const int ro = c.orows ? c.orows[r] : r;
                const size_t row = (size_t)ro * c.ldo;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    if constexpr (UP) {
                        const float g = out[0][h][mb][j];
                        if (c.wlive[0])
                            static_cast<uint16_t*>(c.out)[row + c.wrow[0] + pair_place(h * 16 + n)] =
                                half_of_product(g / (1.0f + expf(-g)), out[1][h][mb][j]);
                    } else {
#pragma unroll
                        for (int i = 0; i < 2; ++i)
                            if (c.wlive[i]) {
                                const float v = out[i][h][mb][j];
                                if (QT || c.f32) static_cast<float*>(c.out)[row + c.wrow[i] + h * 16 + n] = v;
                                else static_cast<__half*>(c.out)[row + c.wrow[i] + h * 16 + n] = __float2half(v);
                            }
                    }
                }
            }
        }
    return left;
}

template <int BITS, bool ZP, bool UP, int NM, int R, int KW, bool QT>
__device__ __forceinline__ void rows_tile(const TileCtx& c, char* smem) {
    uint32_t left;
    if constexpr (BITS == 4) {
        if (c.group % 128 == 0) left = gemm_rows<4, ZP, UP, NM, R, KW, QT, 128>(c, smem);
        else if (QT && c.K % 128 == 0) left = gemm_rows<4, ZP, UP, NM, R, KW, QT, 128, QT ? 2 : 1>(c, smem);
        else left = gemm_rows<4, ZP, UP, NM, R, KW, QT, 64>(c, smem);
    } else {
        left = gemm_rows<BITS, ZP, UP, NM, R, KW, QT, BITS == 2 ? 128 : 64>(c, smem);
    }
    if constexpr (ZP) {
        // rows with an infinite activation (an h past the range of fp16): from the weights' own values
        if (left) {
            wait_loads<0>();
            lds_only_barrier();
            gemm_pipe<BITS, true, UP, 1>(c, smem, left);
        }
    }
}

// A tile of any number of rows (at most kBM): the few-row form up to 32 rows, else as many 32-row products as it has
// rows, in one pass if the stages of that many rows fit into LDS twice (int4), else in passes of 64 rows.
template <int BITS, bool ZP, bool UP>
__device__ __forceinline__ void gemm_tile(const TileCtx& c, char* smem) {
    if constexpr (BITS == 4) {
        if (c.nrows <= 16) rows_tile<4, ZP, UP, 1, 16, 1, false>(c, smem);
        else if (c.nrows <= 32) rows_tile<4, ZP, UP, 2, 32, 1, false>(c, smem);
        else if (c.nrows <= 64) gemm_pipe<BITS, ZP, UP, 2>(c, smem);
        else if (c.nrows <= 96) gemm_pipe<BITS, ZP, UP, 3>(c, smem);
        else gemm_pipe<BITS, ZP, UP, 4>(c, smem);
    } else {
        TileCtx p = c;
        for (int r0 = 0; r0 < c.nrows; r0 += 64) {
            if (r0) {
                lds_only_barrier();
                if (c.rows) p.rows = c.rows + r0;
                else p.A = c.A + (size_t)r0 * c.lda;
                p.out = static_cast<char*>(c.out) + (size_t)r0 * c.ldo * (c.f32 ? sizeof(float) : sizeof(__half));
            }
            p.nrows = min(64, c.nrows - r0);
            if (p.nrows <= 16) rows_tile<BITS, ZP, UP, 1, 16, 1, false>(p, smem);
            else if (p.nrows <= 32) rows_tile<BITS, ZP, UP, 2, 32, 1, false>(p, smem);
            else gemm_pipe<BITS, ZP, UP, 2>(p, smem);
        }
    }
}

// The routing outputs of a decode layer, by one workgroup beside the layer's up GEMM: selection, prediction,
// permutation and popularity (at most 64 pairs).  One entry at a time: nothing waits for this workgroup, and sixteen in
// straight-line code cost the kernel around it 8 spilled scalar registers.
__device__ __forceinline__ void layer_outputs(const LayerOut& o, char* smem) {
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), P = o.N * o.k;
    float* z = reinterpret_cast<float*>(smem);            // [gates][N][E]
    int32_t* ids = reinterpret_cast<int32_t*>(z + 2 * o.N * o.E);
    int32_t* pop = ids + 64;
    const int njobs = (o.pids ? 2 : 1) * o.N;
    for (int i = tid; i < njobs * o.E; i += 256) z[i] = o.z[i];
    for (int i = tid; i < o.E; i += 256) pop[i] = 0;
    __syncthreads();
    for (int j = wave; j < njobs; j += 4) {
        const int t = j < o.N ? j : j - o.N;
        if (j < o.N) wave_softmax_topm<1>(z + (size_t)j * o.E, o.E, o.k, o.renorm, ids + t * o.k, o.w + (size_t)t * o.k, nullptr, nullptr);
        else wave_softmax_topm<1>(z + (size_t)j * o.E, o.E, o.m, 0, o.pids + (size_t)t * o.m, o.pw + (size_t)t * o.m, nullptr, pop);
    }
    __syncthreads();
    if (tid < P) o.ids[tid] = ids[tid];
    if (o.pids)
        for (int i = tid; i < o.E; i += 256) o.pop[i] = pop[i];
    if (wave == 0) wave_permute_small<1>(ids, P, o.E, o.counts, o.offsets, o.perm, o.inv_perm, o.order);
    if (tid == 0) *o.calls += 1;
}

// MODE 0: prefill.  MODE 1: decode-sized (tiles of at most 16 rows, all in the few-row form), fp32 outputs of the down GEMM.
// MODE 2: the same inside a decode layer (at most 8 tokens, 64 pairs): no tile table; a workgroup finds its
// expert and rows by itself, the up GEMM's from the logits and the down GEMM's from the selection; rows of h
// and of the outputs are pairs.  The up GEMM's first workgroup writes the layer's routing outputs.  KW: waves over which its
// columns are split; CHOOSE: routed tiles are whole where the number of named experts asks for it.
template <bool UP, int MODE, int KW, bool CHOOSE>
__device__ __forceinline__ void grouped_gemm_body(const GemmArgs& a) {
    extern __shared__ uint4 gemm_smem[];
    char* smem = reinterpret_cast<char*>(gemm_smem);
    __shared__ int32_t rowlist[MODE == 2 ? 8 : 1];
    constexpr bool EXACT = MODE != 0;
    const int lane = threadIdx.x & 63;
    bool is_shared, whole = false;
    int local, e = 0, sbeg = 0, T = 0;
    if constexpr (MODE == 2) {
        int b = (int)blockIdx.x;
        if (UP && b-- == 0) {
            layer_outputs(a.lo, smem);
            return;
        }
        const int ks = a.nb_s * (UP ? 1 : a.kp_s);
        is_shared = b < a.n_shared * ks;
        if (is_shared) {
            e = b / ks;
            local = b - e * ks;
            T = a.N;
        } else {
            b -= a.n_shared * ks;
            // slot s is the s-th pair, in pair order, whose expert no earlier pair has
            const int P = a.N * a.k;
            int key;
            if constexpr (UP) {
                float* z = reinterpret_cast<float*>(smem);
                int32_t* ids = reinterpret_cast<int32_t*>(z + a.N * a.E);
                for (int i = threadIdx.x; i < a.N * a.E; i += 256) z[i] = a.lo.z[i];
                __syncthreads();
                for (int t = threadIdx.x >> 6; t < a.N; t += 4) wave_topk_ids(z + t * a.E, a.E, a.k, ids + t * a.k);
                __syncthreads();
                key = lane < P ? ids[lane] : -1;
            } else {
                key = lane < P ? a.lo.ids[lane] : -1;
            }
            unsigned long long same = __ballot(key >= 0);
#pragma unroll
            for (int i = 0; i < 8; ++i) {                 // E <= 256
                const unsigned long long m = __ballot((key >> i) & 1);
                same &= (key >> i) & 1 ? m : ~m;
            }
            const unsigned long long lt = lane == 0 ? 0ull : (~0ull >> (64 - lane));
            const bool lead = key >= 0 && (same & lt) == 0;
            const unsigned long long leads = __ballot(lead);
            if constexpr (CHOOSE) whole = up_tiles_whole(__popcll(leads), a.nb_r >> 1, a.n_shared * ks, kGemmSlots, a.H);
            const int kr = CHOOSE && whole ? a.nb_r >> 1 : a.nb_r * (UP ? 1 : a.kp_r);
            const int slot = __popcll(__ballot(lane * kr <= b)) - 1;      // b / kr (at most 64 slots)
            local = b - slot * kr;
            const unsigned long long mine = __ballot(lead && __popcll(leads & lt) == slot);
            if (mine == 0) return;                        // fewer activated experts than slots
            const int l = __ffsll((long long)mine) - 1;
            e = __builtin_amdgcn_readlane(key, l);
            const unsigned long long rows = ((unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(same >> 32), l) << 32) |
                                            (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)same, l);
            T = __popcll(rows);
            if (threadIdx.x < 64 && ((rows >> lane) & 1)) rowlist[__popcll(rows & lt)] = lane;
            __syncthreads();                              // (and the selection's LDS is free for the ring)
        }
    } else {
        const int nseg = a.E + a.n_shared;
        // Which tile: the segments' first tiles, one per lane, all requested at once.  The shared experts'
        // segments come last in the table and hold the fullest tiles: they go first.
        constexpr int kSegRegs = (kMaxE + 16 + 1 + 63) / 64;
        int4 seg[kSegRegs];
#pragma unroll
        for (int i = 0; i < kSegRegs; ++i)
            if (64 * i <= nseg) seg[i] = a.segs[min(64 * i + lane, nseg)];
        int ntile = 0;
#pragma unroll
        for (int i = 0; i < kSegRegs; ++i)
            if ((nseg >> 6) == i) ntile = __builtin_amdgcn_readlane(seg[i].x, nseg & 63);
        if ((int)blockIdx.x >= ntile) return;
        const int b = ntile - 1 - (int)blockIdx.x;
        int sidx = 0, first = 0;                           // last segment that starts at or before tile b
#pragma unroll
        for (int i = 0; i < kSegRegs; ++i)
            if (64 * i < nseg) {
                const unsigned long long m = __ballot(64 * i + lane < nseg && seg[i].x <= b);
                if (m) {
                    const int l = 63 - __clzll((long long)m);
                    sidx = 64 * i + l;
                    first = __builtin_amdgcn_readlane(seg[i].x, l);
                    e = __builtin_amdgcn_readlane(seg[i].y, l);
                    sbeg = __builtin_amdgcn_readlane(seg[i].z, l);
                    T = __builtin_amdgcn_readlane(seg[i].w, l);
                }
            }
        is_shared = sidx >= a.E;
        local = b - first;
    }
    const int nb = is_shared ? a.nb_s : a.nb_r, kp = UP ? 1 : (is_shared ? a.kp_s : a.kp_r);
    const int mb = MODE == 2 ? 0 : local / (nb * kp);       // (a decode layer's experts have at most 8 rows)
    local -= mb * (nb * kp);
    const int part = MODE == 2 && UP ? 0 : local / nb, nblk = local - part * nb;
    const fate_qexpert* ex = (is_shared ? a.shared : a.experts) + e;
    const int trows = EXACT ? 1 << kExactTileRowsLog2 : tile_rows(T, is_shared ? a.rows_s : a.rows_r);
    const int row0 = mb * trows;
    TileCtx c;
    c.ex = ex;
    c.nrows = min(trows, T - row0);
    // waves over which the columns are split, weight rows of the tile
    const int kw = whole ? 1 : KW, bn = UP ? kBNUp / kw : kBNDown;
    c.Nout = UP ? uniform(ex->I) : a.H;
    c.K = UP ? a.H : uniform(ex->I);
    if (c.nrows <= 0) return;
    const int out_row0 = (is_shared ? e * a.N : sbeg) + row0;      // (MODE 2, routed: 0, rows are pairs)
    c.ldo = is_shared ? a.ldo_s : a.ldo_r;
    c.f32 = !UP && (EXACT || (is_shared ? a.f32_s : a.f32_r));
    {
        const size_t osz = c.f32 ? sizeof(float) : sizeof(__half);
        c.out = static_cast<char*>(is_shared ? a.out_s : a.out_r) +
                ((size_t)part * (is_shared ? a.part_s : a.part_r) + (size_t)out_row0 * c.ldo) * osz;
    }
    // width and group of THIS expert's copy: a layer may hold copies of several widths (the
    // popularity-aware hybrid of section 4.5 moves the least popular experts at 2 bits)
    const int bits = uniform(ex->bits);
    c.group = uniform(ex->group);
    const int kt = bits == 4 ? 64 : (bits == 8 ? 32 : 128);
    const bool has_z = ex->z1 != nullptr;
    const bool absent = ex->w1 == nullptr || ex->w3 == nullptr || ex->w2 == nullptr ||
                        (MODE == 2 && (has_z || bits != (is_shared ? a.bits_s : a.bits_r) ||
                                               c.group != (is_shared ? a.group_s : a.group_r)));
    const bool bad = (bits != 2 && bits != 4 && bits != 8) || c.group < kt || c.group % kt || c.group % 64 || (EXACT && c.group != 64 && c.group % 128) || a.H % c.group ||
                     uniform(ex->I) % c.group || (has_z && (bits == 8 || ex->z2 == nullptr || ex->z3 == nullptr));   // zero-points: 4 and 2 bits
    if (absent || bad) {
        // nothing to multiply: the pairs of this expert contribute zeros
        if (UP) {
            if (threadIdx.x == 0) atomicOr(a.status, absent ? 1 : 4);
        } else {
            for (int i = threadIdx.x; i < c.nrows * (kBNDown / 4); i += 256) {
                int r = i / (kBNDown / 4);
                const int col = nblk * kBNDown + (i % (kBNDown / 4)) * 4;
                if (MODE == 2 && !is_shared) r = rowlist[r];
                if (col < a.H) {
                    if (c.f32) reinterpret_cast<float4*>(static_cast<float*>(c.out) + (size_t)r * c.ldo + col)[0] = make_float4(0.f, 0.f, 0.f, 0.f);
                    else reinterpret_cast<uint2*>(static_cast<__half*>(c.out) + (size_t)r * c.ldo + col)[0] = make_uint2(0, 0);
                }
            }
        }
        return;
    }
    if (UP && nblk * bn >= c.Nout) return;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int wr = UP ? nblk * bn + wave / kw * 32 : nblk * kBNDown + wave * 64 + i * 32;
        c.wlive[i] = wr < c.Nout;
        c.wrow[i] = c.wlive[i] ? wr : 0;
    }
    // columns of this part: a whole number of 128-column pieces (none is possible: an expert smaller than I_max), with
    // the last part the 64 columns that an expert's own I may have beyond them
    const int pieces = c.K / kKQ;
    const int p0 = pieces * part / kp, p1 = pieces * (part + 1) / kp;
    c.col0 = p0 * kKQ;
    c.ncol = (p1 - p0) * kKQ;
    if (!UP && part + 1 == kp) c.ncol += c.K % kKQ;
    c.lda = is_shared ? a.lda_s : a.lda_r;
    c.A = is_shared ? a.A_s : a.A_r;
    c.rows = c.orows = nullptr;
    c.div = 1;
    if (MODE == 2 && !is_shared) {
        c.rows = c.orows = rowlist;
        if (UP) c.div = a.k;
    } else if (UP) {
        if (is_shared) c.A += (size_t)row0 * c.lda;
        else { c.rows = a.perm + sbeg + row0; c.div = a.k; }
    } else {
        c.A += (size_t)out_row0 * c.lda;
    }
    if constexpr (MODE == 2) {
        if (CHOOSE && whole) rows_tile<4, false, UP, 1, 8, 1, true>(c, smem);       // (routed, of the layer's width: 4 bits)
        else if (bits == 4) rows_tile<4, false, UP, 1, 8, KW, true>(c, smem);
        else rows_tile<8, false, UP, 1, 8, KW, true>(c, smem);
    } else if constexpr (MODE == 1) {
        if (has_z && bits == 4) rows_tile<4, true, UP, 1, 16, 1, true>(c, smem);
        else if (has_z) rows_tile<2, true, UP, 1, 16, 1, true>(c, smem);
        else if (bits == 4) rows_tile<4, false, UP, 1, 16, 1, true>(c, smem);
        else if (bits == 2) rows_tile<2, false, UP, 1, 16, 1, true>(c, smem);
        else rows_tile<8, false, UP, 1, 16, 1, true>(c, smem);
    } else {
        if (has_z && bits == 4) gemm_tile<4, true, UP>(c, smem);
        else if (has_z) gemm_tile<2, true, UP>(c, smem);
        else if (bits == 4) gemm_tile<4, false, UP>(c, smem);
        else if (bits == 2) gemm_tile<2, false, UP>(c, smem);
        else gemm_tile<8, false, UP>(c, smem);
    }
}

template <bool UP, int MODE, int KW, bool CHOOSE = false>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void grouped_gemm_kernel(GemmArgs a) {
    grouped_gemm_body<UP, MODE, KW, CHOOSE>(a);
}

// acc += wgt[i] * row i of src, columns c*V .. c*V + V - 1.  With few tokens the rows' latency is all there
// is, so a thread asks for 128 bytes of rows at once.
template <class T, int V>
__device__ __forceinline__ void add_rows(const void* const* src, const float* wgt, int n, int c, float (&acc)[V]) {
    constexpr int L = V * (int)sizeof(T) / 16, B = 8 / L;  // loads per row, rows per batch
    for (int i0 = 0; i0 < n; i0 += B) {
        uint4 v[B][L];
#pragma unroll
        for (int u = 0; u < B; ++u) {
            const uint4* q = static_cast<const uint4*>(src[min(i0 + u, n - 1)]);
#pragma unroll
            for (int l = 0; l < L; ++l) v[u][l] = q ? q[c * L + l] : make_uint4(0, 0, 0, 0);
        }
#pragma unroll
        for (int u = 0; u < B; ++u) {
            if (i0 + u >= n) break;
            const float w = wgt[i0 + u];
            const T* e = reinterpret_cast<const T*>(v[u]);
#pragma unroll
            for (int i = 0; i < V; ++i) acc[i] = fmaf(w, (float)e[i], acc[i]);
        }
    }
}

// y[t,:] = sum_j w[t,j] * Yp_r[pos(t,j), :] + sum_s g_s(t) * Yp_s[s*N+t, :], each Yp the sum of its K parts;
// pos = inv_perm, or the pair itself when that is NULL.  TR / TS: elements of the routed / shared outputs.
// A block of 64 to 256 threads per token and slice of H.
template <class TR, class TS>
__global__ void combine_kernel(const TR* __restrict__ yp_r, const TS* __restrict__ yp_s, const int32_t* __restrict__ inv_perm,
                               const float* __restrict__ topk_w, const float* __restrict__ sgate, int H, int k, int n_shared,
                               int N, int kp_r, int kp_s, size_t part_r, size_t part_s, float* __restrict__ y32,
                               uint16_t* __restrict__ y16) {
    constexpr bool same = sizeof(TR) == sizeof(TS);
    constexpr int V = same ? 16 / sizeof(TR) : 8;         // outputs per thread: 16 bytes of the narrower rows
    __shared__ const void* src[kCombineRows];
    __shared__ float wgt[kCombineRows];
    const int t = blockIdx.x;
    const int c = blockIdx.y * blockDim.x + threadIdx.x;
    const int nr = k * kp_r, nrows = nr + n_shared * kp_s;
    float acc[V];
#pragma unroll
    for (int i = 0; i < V; ++i) acc[i] = 0.f;
    for (int r0 = 0; r0 < nrows; r0 += kCombineRows) {
        const int lim = min(kCombineRows, nrows - r0);
        if (r0) __syncthreads();
        for (int i = threadIdx.x; i < lim; i += blockDim.x) {
            const int r = r0 + i;
            if (r < nr) {
                const int j = r / kp_r, p = r - j * kp_r;
                const int pos = inv_perm ? inv_perm[t * k + j] : t * k + j;
                src[i] = yp_r + p * part_r + (size_t)max(pos, 0) * H;
                wgt[i] = pos < 0 ? 0.f : topk_w[t * k + j];        // (a pair whose expert id was out of range: no row of its own)
                if (pos < 0) src[i] = nullptr;
            } else {
                const int s = (r - nr) / kp_s, p = r - nr - s * kp_s;
                src[i] = yp_s + p * part_s + ((size_t)s * N + t) * H;
                wgt[i] = sgate ? sgate[t] : 1.0f;
            }
        }
        __syncthreads();
        if (c * V < H) {
            const int lim_r = same ? lim : max(0, min(lim, nr - r0));
            add_rows<TR, V>(src, wgt, lim_r, c, acc);
            if constexpr (!same) add_rows<TS, V>(src + lim_r, wgt + lim_r, lim - lim_r, c, acc);
        }
    }
    if (c * V >= H) return;
    if (y32) {
        float4* o = reinterpret_cast<float4*>(y32 + (size_t)t * H + c * V);
#pragma unroll
        for (int i = 0; i < V / 4; ++i) o[i] = make_float4(acc[4 * i], acc[4 * i + 1], acc[4 * i + 2], acc[4 * i + 3]);
    } else {
        uint2* o = reinterpret_cast<uint2*>(y16 + (size_t)t * H + c * V);
#pragma unroll
        for (int i = 0; i < V / 4; ++i)
            o[i] = make_uint2(f32_to_bf16_bits(acc[4 * i]) | (f32_to_bf16_bits(acc[4 * i + 1]) << 16),
                              f32_to_bf16_bits(acc[4 * i + 2]) | (f32_to_bf16_bits(acc[4 * i + 3]) << 16));
    }
}

// Parts of the reduction dimension of the down GEMM.  A tile's time is its K; with `tiles` of
// length K over 2 workgroups per compute unit, a tile longer than the average load of a
// workgroup would run on after everything else has ended, so it is cut into parts.  Every part
// has an output of its own in fp32, which combine adds up (512 columns at least, 8 parts at most).
void mfma_k_parts(const fate_ffn_desc& d, int* kp_r, int* kp_s) {
    const long long P = (long long)d.N * d.k, nb = (d.H + kBNDown - 1) / kBNDown;
    const long long tr = (P / kBM + std::min<long long>(d.E, P)) * nb;
    const long long ts = (long long)d.n_shared * ((d.N + kBM - 1) / kBM) * nb;
    const long long load = std::max<long long>((tr * d.I_max + ts * (d.n_shared ? d.I_shared_max : 0)) / kGemmSlots, 512);
    auto parts = [&](long long K) { return (int)std::min<long long>(std::max<long long>((K + load - 1) / load, 1), 8); };
    *kp_r = parts(d.I_max);
    *kp_s = d.n_shared ? parts(d.I_shared_max) : 1;
}

TileBlocks mfma_tile_blocks(const fate_ffn_desc& d, bool exact) {
    int kp_r = 1, kp_s = 1;
    mfma_k_parts(d, &kp_r, &kp_s);
    const int nb_down = (d.H + kBNDown - 1) / kBNDown;
    auto rows = [&](int bits) { return exact ? kExactTileRowsLog2 : (bits == 4 ? kTileRowsLog2 : kTileRowsLog2Wide); };
    return TileBlocks{(d.I_max + kBNUp - 1) / kBNUp, d.n_shared ? (d.I_shared_max + kBNUp - 1) / kBNUp : 0, nb_down * kp_r,
                      nb_down * kp_s, rows(d.bits), rows(d.shared_bits)};
}

fate_status launch_ffn_mfma(hipStream_t st, const fate_ffn_desc& d, DecodeArgs da, const MfmaScratch& ms,
                            void* y_out, const PartSel& sel, const MfmaMode& mode) {
    const int phase = mode.phase;
    const bool exact = mode.exact;
    if (d.H % kKQ || d.I_max % kKQ || (d.n_shared && d.I_shared_max % kKQ))
        FATE_FAIL(FATE_ESHAPE, "the MFMA path needs H and I to be multiples of %d", kKQ);
    const int P = d.N * d.k;
    // the GEMM addresses activation rows with 32-bit element offsets
    const long long amax = std::max({(long long)d.N * d.H, (long long)P * da.ldh_r,
                                     (long long)d.n_shared * d.N * da.ldh_s});
    if (amax >= (1LL << 31))
        FATE_FAIL(FATE_ESHAPE, "the MFMA path needs activation matrices of fewer than 2^31 elements (%lld)", amax);
    const TileBlocks nb = mfma_tile_blocks(d, exact);
    int kp_r = 1, kp_s = 1;
    mfma_k_parts(d, &kp_r, &kp_s);
    const int nb_down = nb.r_down / kp_r;
    // upper bounds of the routed row blocks, and the shared experts' row blocks
    // (a decode layer has no tile table: its experts have at most 8 rows)
    const long long mb_r = (mode.layer ? 0 : P >> nb.rows_r) + (d.E < P ? d.E : P);
    const long long mb_s = (d.N + (1 << nb.rows_s) - 1) >> nb.rows_s;
    const bool do_up = phase != 2, do_down = phase != 1;
    static bool attr_done = false;
    if (!attr_done) {
#define FATE_GEMM_ATTR(...)                                                                 \
    FATE_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(grouped_gemm_kernel<__VA_ARGS__>),  \
                                 hipFuncAttributeMaxDynamicSharedMemorySize, kGemmLds));
        FATE_GEMM_ATTR(true, 0, 1) FATE_GEMM_ATTR(false, 0, 1)
        FATE_GEMM_ATTR(true, 1, 1) FATE_GEMM_ATTR(false, 1, 1)
        FATE_GEMM_ATTR(true, 2, 1) FATE_GEMM_ATTR(false, 2, 1)
        FATE_GEMM_ATTR(true, 2, 2) FATE_GEMM_ATTR(true, 2, 2, true)
#undef FATE_GEMM_ATTR
        attr_done = true;
    }
    // Decode layer: the columns of the up projection are split over pairs of waves if they can be (whole stages of 128,
    // whole groups), tiles of 64 neurons instead of 128; 4-bit routed experts go back to whole tiles where the workgroups
    // count more experts than split ones have places for (up_tiles.h).  Where no count can ask for that: the kernel that
    // does not choose.  Per layer, always split / chosen from an expected count of uniform routing / now: 8 tokens of the
    // DeepSeek shape 60.8 / 57.0 / 56.9 us, of the Qwen shape 47.6 / 45.4 / 44.4, of that with a Zipf gate (13 experts
    // instead of 22) 38.4 / 39.8 / 38.2; 2 of the Mixtral shape 76.7 / 80.0 / 76.7.
    const int kw = mode.layer && d.H % 256 == 0 && (d.H / d.group) % 2 == 0 && (!d.n_shared || (d.H / d.shared_group) % 2 == 0) ? 2 : 1;
    const unsigned shared_tiles = (unsigned)(kw * d.n_shared * nb.s_up);
    bool choose = false;
    long long tiles_r = mb_r * nb.r_up * kw;
    if (kw == 2 && d.bits == 4) tiles_r = up_tiles_most((int)mb_r, nb.r_up, shared_tiles, kGemmSlots, d.H, &choose);
    if (do_up && !mode.layer) {
        prefill_prep_kernel<<<sel.first ? d.N + 1 : 1, 256, 0, st>>>(da.x, d.N, d.H, d.E, d.n_shared, da.offsets,
                                                                 da.order, da.shared_gate, ms.xh, ms.sgate, ms.tab_up, ms.tab_down,
                                                                 nb, sel);
        FATE_HIP(hipGetLastError());
    }
    GemmArgs g{};
    g.experts = da.experts; g.shared = da.shared; g.E = d.E; g.n_shared = d.n_shared; g.N = d.N; g.k = d.k;
    g.perm = da.perm;
    g.rows_r = nb.rows_r; g.rows_s = nb.rows_s;
    g.status = da.status;
    if (mode.layer) g.lo = *mode.layer;
    g.bits_r = da.bits_r; g.group_r = da.group_r; g.bits_s = da.bits_s; g.group_s = da.group_s;
    g.H = d.H;
    if (do_up) {
        g.A_r = ms.xh; g.lda_r = d.H; g.A_s = ms.xh; g.lda_s = d.H; g.segs = ms.tab_up;
        g.out_r = da.h_r; g.ldo_r = da.ldh_r; g.out_s = da.h_s; g.ldo_s = da.ldh_s;
        g.nb_r = nb.r_up * kw; g.nb_s = nb.s_up * kw;
        g.kp_r = g.kp_s = 1;
        const long long grid = tiles_r + d.n_shared * mb_s * g.nb_s + (mode.layer ? 1 : 0);
        if (grid > 0x7fffffffLL) FATE_FAIL(FATE_ESHAPE, "too many tiles");
        const unsigned ng = (unsigned)grid;
        if (choose) grouped_gemm_kernel<true, 2, 2, true><<<ng, 256, kGemmLds, st>>>(g);
        else if (mode.layer && kw == 2) grouped_gemm_kernel<true, 2, 2><<<ng, 256, kGemmLds, st>>>(g);
        else if (mode.layer) grouped_gemm_kernel<true, 2, 1><<<ng, 256, kGemmLds, st>>>(g);
        else if (exact) grouped_gemm_kernel<true, 1, 1><<<ng, 256, kGemmLds, st>>>(g);
        else grouped_gemm_kernel<true, 0, 1><<<ng, 256, kGemmLds, st>>>(g);
        FATE_HIP(hipGetLastError());
    }
    if (do_down) {
        g.A_r = da.h_r; g.lda_r = da.ldh_r; g.A_s = da.h_s; g.lda_s = da.ldh_s;
        g.segs = ms.tab_down; g.nb_r = nb_down; g.nb_s = nb_down;
        g.out_r = ms.yp_r; g.ldo_r = d.H; g.out_s = ms.yp_s; g.ldo_s = d.H;
        g.kp_r = kp_r; g.kp_s = kp_s;
        g.f32_r = mfma_out_bytes(exact, kp_r) == 4; g.f32_s = d.n_shared && mfma_out_bytes(exact, kp_s) == 4;
        g.part_r = (size_t)P * d.H; g.part_s = (size_t)d.n_shared * d.N * d.H;
        const long long grid = (mb_r * kp_r + d.n_shared * mb_s * kp_s) * nb_down;
        if (grid > 0x7fffffffLL) FATE_FAIL(FATE_ESHAPE, "too many tiles");
        const unsigned ng = (unsigned)grid;
        if (mode.layer) grouped_gemm_kernel<false, 2, 1><<<ng, 256, kGemmLds, st>>>(g);
        else if (exact) grouped_gemm_kernel<false, 1, 1><<<ng, 256, kGemmLds, st>>>(g);
        else grouped_gemm_kernel<false, 0, 1><<<ng, 256, kGemmLds, st>>>(g);
        FATE_HIP(hipGetLastError());
        if (sel.last) {
            float* y32 = d.y_is_fp32 ? static_cast<float*>(y_out) : nullptr;
            uint16_t* y16 = d.y_is_fp32 ? nullptr : static_cast<uint16_t*>(y_out);
            const float* gate = da.shared_gate ? ms.sgate : nullptr;
            const int32_t* inv = mode.layer ? nullptr : da.inv_perm;
            const int threads = d.N >= 64 ? 256 : 64;
#define FATE_COMBINE(TR, TS)                                                                                          \
    combine_kernel<TR, TS><<<dim3(d.N, (d.H / (sizeof(TR) == sizeof(TS) ? 16 / (int)sizeof(TR) : 8) + threads - 1) / threads), \
                             threads, 0, st>>>(static_cast<const TR*>(ms.yp_r), static_cast<const TS*>(ms.yp_s), inv,   \
                                               da.topk_w, gate, d.H, d.k, d.n_shared, d.N, kp_r, kp_s, g.part_r,        \
                                               g.part_s, y32, y16)
            if (g.f32_r && (g.f32_s || !d.n_shared)) FATE_COMBINE(float, float);
            else if (g.f32_r) FATE_COMBINE(float, __half);
            else if (g.f32_s) FATE_COMBINE(__half, float);
            else FATE_COMBINE(__half, __half);
#undef FATE_COMBINE
        }
        FATE_HIP(hipGetLastError());
    }
    return FATE_OK;
}

}  // namespace fate
