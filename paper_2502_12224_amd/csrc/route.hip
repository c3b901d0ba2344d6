// Gate routing, cross-layer prediction, permutation: kernels and C entry points.
//
// fate_gate_route / fate_cross_layer_predict: a workgroup per token (decode-sized calls and
// hidden sizes that are no multiple of 1024) or the gate as a GEMM on the matrix cores.
//
// fate_route_fused, up to 16 tokens: a workgroup per (token, gate), the last one to leave does
// popularity and permutation; prefill sizes: both gates in one GEMM launch, then the permutation.
#include "common.h"
#include "route_device.h"
#include "async_lds.h"
#include "decode_device.h"
#include "layer_decode.h"

namespace fate {

__global__ void fill_i32_kernel(int32_t* p, int n, int32_t v) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

// Logits of TPW tokens (rows of x) for every expert into z [TPW][E], by a whole workgroup of NW
// waves; wave w takes experts w, w + NW, .., four at a time, so that up to 16 rows
// of 1 KiB are requested before the first is used.  Rows past the last expert read row 0.
// A lane sums columns lane*8 + 512*j in order, then the lanes add up: the same bits for a
// (token, expert) whichever workgroup, batch size or call evaluates it.
constexpr int kTokWaves = 16;
template <int TPW, int NW = kTokWaves>
__device__ __forceinline__ void token_logits(const uint4* __restrict__ x, const uint4* __restrict__ Wg,
                                             const float* __restrict__ bias, int ntok, int nvec, int E, float* z) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    constexpr int NE = 4, NJ = TPW == 1 ? 4 : 2;       // operands of one batch: within the 128 registers of 16 waves
    for (int e0 = wave; e0 < E; e0 += NW * NE) {
        float acc[NE][TPW];
        const uint4* wr[NE];
#pragma unroll
        for (int i = 0; i < NE; ++i) {
            const int e = e0 + NW * i;
            wr[i] = Wg + (size_t)(e < E ? e : 0) * nvec;
#pragma unroll
            for (int t = 0; t < TPW; ++t) acc[i][t] = 0.f;
        }
        for (int c0 = lane; c0 < nvec; c0 += 64 * NJ) {
            uint4 wv[NJ][NE], xv[NJ][TPW];
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                const int c = c0 + 64 * j;
                const bool in = c < nvec;
                const int cc = in ? c : 0;
#pragma unroll
                for (int i = 0; i < NE; ++i) wv[j][i] = wr[i][cc];
#pragma unroll
                for (int t = 0; t < TPW; ++t) {
                    // columns past the row read column 0; both operands are zero there, which leaves the sums as they are
                    const uint4 v = x[(size_t)(t < ntok ? t : 0) * nvec + cc];
                    xv[j][t] = in ? v : make_uint4(0, 0, 0, 0);
                }
            }
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                if (c0 - lane + 64 * (j + 1) > nvec && c0 + 64 * j >= nvec) {
#pragma unroll
                    for (int i = 0; i < NE; ++i) wv[j][i] = make_uint4(0, 0, 0, 0);
                }
#pragma unroll
                for (int i = 0; i < NE; ++i)
#pragma unroll
                    for (int t = 0; t < TPW; ++t) acc[i][t] = dot8_bf16(xv[j][t], wv[j][i], acc[i][t]);
            }
        }
#pragma unroll
        for (int i = 0; i < NE; ++i) {
            const int e = e0 + NW * i;
            if (e < E) {
                const float b = bias ? bias[e] : 0.f;
#pragma unroll
                for (int t = 0; t < TPW; ++t) {
                    const float s = wave_sum(acc[i][t]);
                    if (lane == 0) z[t * E + e] = s + b;
                }
            }
        }
    }
}

// A workgroup of 16 waves per TPW tokens.  A decode-sized call is a handful of dependent memory
// round trips, so a token gets a whole compute unit: the gate matrix (a few hundred KB, from L2
// after the first workgroup) is requested at once by 16 waves.  48 tokens, E = 64, H = 2048:
// 7.8 us, of which the selection is 1.5 (one wave per token, rows one after the other: 109 us).  NW: waves, 16, or 4 where there are more tokens than the
// device holds workgroups of 16.
template <int TPW, int NW>
__global__ __launch_bounds__(64 * NW) void route_rows_kernel(const uint16_t* __restrict__ x, const uint16_t* __restrict__ Wg,
                                                           const float* __restrict__ bias, int N, int H, int E, int m,
                                                           int renorm, int32_t* __restrict__ ids, float* __restrict__ w,
                                                           float* __restrict__ probs, int32_t* __restrict__ pop) {
    __shared__ float z[TPW * kMaxE];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nvec = H >> 3, tok0 = blockIdx.x * TPW, ntok = min(TPW, N - tok0);
    token_logits<TPW, NW>(reinterpret_cast<const uint4*>(x) + (size_t)tok0 * nvec, reinterpret_cast<const uint4*>(Wg), bias,
                      ntok, nvec, E, z);
    __syncthreads();
    if (wave < ntok) {
        const int tok = tok0 + wave;
        wave_softmax_topm(z + wave * E, E, m, renorm, ids + (size_t)tok * m, w + (size_t)tok * m,
                          probs ? probs + (size_t)tok * E : nullptr, pop);
    }
}

// Many tokens (prefill): the gate is a small GEMM, z[N,E] = x[N,H] . Wg[E,H]^T, done on the matrix
// cores.  A workgroup (8 waves) owns TOK tokens; wave w takes expert tile (w & 1) of a pair of
// 32-expert tiles and quarter (w >> 1) of the reduction dimension; the quarters add up in LDS.
// bf16 products are exact in fp32; accumulation is fp32.  The logits meet in LDS, then one wave
// per token does softmax and selection as in the other kernels.
// What bounds it is the way of the gate matrix (a few hundred KB per workgroup) into the compute
// unit.  Every wave brings its own rows and columns to LDS by itself, 64 columns at a time in a ring
// of stages, whole 128-byte lines per row (read straight into the operand registers, a load
// touches 32 rows for 32 bytes each); no barrier before the logits meet.  Both gates, E = 60, H = 2048: 131
// tokens 18.3 -> 10.8 us, 2048 tokens 25.4 -> 16.6 us; with the selection by straight-line counting 9.6 and 15.3.
struct RouteSecond {             // arguments of the second gate (grid.y = 2); unused when grid.y = 1
    const uint16_t* Wg; const float* bias; int m; int32_t* ids; float* w; int32_t* pop;
    int32_t* pop_part;           // [workgroups][E] each: when set, a workgroup leaves its counts of predicted /
    int32_t* cnt_part;           // selected experts there (plain stores) for permute_parts_kernel to add up
};
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(16))) float rf32x16_t;
constexpr int kGateWaves = 8;
constexpr int gate_stage(int tok) { return 32 * 128 + tok * 128; }       // bytes per wave: 32 gate rows, the tokens
constexpr int gate_depth(int tok) { return tok == 32 ? 2 : 3; }
constexpr int gate_lds(int tok, int ne) {
    const int ring = kGateWaves * gate_depth(tok) * gate_stage(tok), logits = 4 * tok * ne * 64 * 4;
    return ring > logits ? ring : logits;
}

// NE = pairs of expert tiles (E <= 64 * NE)
template <int TOK, int NE>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void route_mfma_kernel(
    const uint16_t* __restrict__ x, const uint16_t* __restrict__ Wg, const float* __restrict__ bias, int N, int H, int E,
    int m, int renorm, int32_t* __restrict__ ids, float* __restrict__ w, float* __restrict__ probs,
    int32_t* __restrict__ pop, RouteSecond g2) {
    extern __shared__ uint4 smem[];
    // counts of this workgroup's tokens: added up here first, so that a device-wide histogram
    // takes one atomic per workgroup and expert instead of one per token and expert
    __shared__ int32_t pop_s[kMaxE];
    int32_t* part = g2.cnt_part;
    if (blockIdx.y == 1) {                        // the second gate of the same launch (next layer's)
        Wg = g2.Wg; bias = g2.bias; m = g2.m; renorm = 0; ids = g2.ids; w = g2.w; probs = nullptr; pop = g2.pop;
        part = g2.pop_part;
    }
    constexpr int S = gate_depth(TOK), SB = gate_stage(TOK), NX = TOK / 8, LPS = 4 + NX;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 31, half = lane >> 5;
    const int etile = wave & 1, kq = wave >> 1;
    const int t0 = blockIdx.x * TOK;
    const int nchunk = H >> 8, nst = NE * nchunk;  // stages: the quarter's chunks of 64 columns for every pair of tiles
    const bool counted = pop != nullptr || part != nullptr;
    if (counted)
        for (int i = threadIdx.x; i < E; i += 512) pop_s[i] = 0;

    // a load brings 8 rows of 128 bytes; piece p of row r goes to place p ^ (r & 7)
    char* ring = reinterpret_cast<char*>(smem) + wave * (S * SB);
    const uint32_t lds0 = lds_offset(ring);
    const int rl = lane >> 3, q = (lane & 7) ^ rl;
    uint32_t xoff[NX], woff[4];
#pragma unroll
    for (int i = 0; i < NX; ++i) {
        const int t = t0 + i * 8 + rl;
        xoff[i] = (uint32_t)((i * 8 + rl) * (t < N ? 1 : 0)) * (uint32_t)H * 2u + q * 16;      // no token: the first one's row
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) woff[i] = (uint32_t)(i * 8 + rl) * (uint32_t)H * 2u + q * 16;
    const char* xb = reinterpret_cast<const char*>(x + (size_t)t0 * H + kq * (H >> 2));
    const char* wb = reinterpret_cast<const char*>(Wg + kq * (H >> 2));
    auto issue = [&](int st, int slot) {
        const int e0 = st / nchunk, c = st - e0 * nchunk;
        const uint32_t base = lds0 + slot * SB;
        const int r0 = e0 * 64 + etile * 32;          // rows past the last expert read row 0 (their logits are not looked at)
#pragma unroll
        for (int i = 0; i < 4; ++i)
            lds_load16(base + i * 1024, wb + c * 128, r0 + i * 8 + rl < E ? (uint32_t)r0 * (uint32_t)H * 2u + woff[i] : (uint32_t)q * 16);
#pragma unroll
        for (int i = 0; i < NX; ++i) lds_load16(base + 4096 + i * 1024, xb + c * 128, xoff[i]);
    };
    rf32x16_t acc[NE];
#pragma unroll
    for (int e = 0; e < NE; ++e)
#pragma unroll
        for (int j = 0; j < 16; ++j) acc[e][j] = 0.f;
    const int xr = n & (TOK - 1);
#pragma unroll
    for (int s = 0; s < S - 1; ++s) issue(s, s);      // (H >= 1024: four stages at least)
    int slot = 0, slot_in = S - 1, st = 0;
#pragma unroll
    for (int e = 0; e < NE; ++e)
        for (int c = 0; c < nchunk; ++c, ++st) {
            wait_stages<LPS, S - 2>(nst - 1 - st);
            // the wave's reads of the stage that is about to be overwritten have returned
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            if (st + S - 1 < nst) issue(st + S - 1, slot_in);
            const char* base = ring + slot * SB;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int p = 2 * u + half;
                const uint4 av = *reinterpret_cast<const uint4*>(base + 4096 + xr * 128 + ((p ^ (xr & 7)) * 16));
                const uint4 bv = *reinterpret_cast<const uint4*>(base + n * 128 + ((p ^ (n & 7)) * 16));
                acc[e] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, av),
                                                                 __builtin_bit_cast(bf16x8_t, bv), acc[e], 0, 0, 0);
            }
            slot = slot + 1 == S ? 0 : slot + 1;
            slot_in = slot_in + 1 == S ? 0 : slot_in + 1;
        }
    __syncthreads();                                  // the rings are done with: the logits take their place
    float* zs = reinterpret_cast<float*>(smem);       // [4 quarters][TOK][64 * NE]
    constexpr int Epad = 64 * NE;
    // lane (half, n) holds expert column n, token rows 8*(j/4) + 4*half + j%4
#pragma unroll
    for (int e = 0; e < NE; ++e)
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const int t = 8 * (j >> 2) + 4 * half + (j & 3);
            if (t < TOK) zs[((size_t)kq * TOK + t) * Epad + e * 64 + etile * 32 + n] = acc[e][j];
        }
    __syncthreads();
    for (int t = wave; t < TOK; t += kGateWaves) {
        const int tk = t0 + t;
        if (tk < N) {
            float* z = zs + (size_t)t * Epad;
            constexpr size_t Q = (size_t)TOK * Epad;
#pragma unroll
            for (int e = lane; e < Epad; e += 64)
                if (e < E) z[e] = ((z[e] + z[e + Q]) + (z[e + 2 * Q] + z[e + 3 * Q])) + (bias ? bias[e] : 0.f);
            __builtin_amdgcn_wave_barrier();
            wave_softmax_topm(z, E, m, renorm, ids + (size_t)tk * m, w + (size_t)tk * m,
                              probs ? probs + (size_t)tk * E : nullptr, counted ? pop_s : nullptr);
        }
    }
    if (counted) {
        __syncthreads();
        for (int i = threadIdx.x; i < E; i += 512) {
            if (part) part[(size_t)blockIdx.x * E + i] = pop_s[i];
            else if (pop_s[i]) atomicAdd(&pop[i], pop_s[i]);
        }
    }
}

__global__ __launch_bounds__(1024) void permute_kernel(const int32_t* __restrict__ ids, int P, int E,
                                                       int32_t* counts, int32_t* offsets, int32_t* perm,
                                                       int32_t* inv_perm, int32_t* order) {
    __shared__ int32_t sm[kPermSmemInts];
    if (P <= 64) {
        if (threadIdx.x < 64) wave_permute_small(ids, P, E, counts, offsets, perm, inv_perm, order);
        return;
    }
    block_permute(ids, P, E, counts, offsets, perm, inv_perm, order, sm);
}

// The permutation after route_mfma_kernel, a workgroup per routing workgroup: the rows of counts
// that those left (cnt_part [nparts][E]) give the place of every expert and, summed up to this
// workgroup's row, of its pairs among the expert's; the pairs of its own tokens (pairs_wg of them)
// are ranked by one wave in order.  Same outputs as permute_kernel, which one workgroup works
// through on its own (131 tokens, k = 4: 8.9 -> 5.0 us, 2048 tokens 21.9 -> 9.7 us; the first workgroup, which also adds
// up the predictions, asks for eight of their rows at once: 13.9 -> 9.7).
// The first workgroup writes what is not per pair.
__global__ __launch_bounds__(256) void permute_parts_kernel(const int32_t* __restrict__ ids, int P, int pairs_wg, int E,
                                                            int nparts, const int32_t* __restrict__ cnt_part,
                                                            const int32_t* __restrict__ pop_part, int32_t* counts,
                                                            int32_t* offsets, int32_t* perm, int32_t* inv_perm,
                                                            int32_t* order, int32_t* pop_out) {
    __shared__ int32_t tot[kMaxE], before[kMaxE], pops[kMaxE], wsum[4];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int b = blockIdx.x;
    const int beg = b * pairs_wg, end = min(P, beg + pairs_wg);
    const int id0 = wave == 0 && beg + lane < end ? ids[beg + lane] : -1;      // under way with the counts
    for (int i = tid; i < E; i += 256) tot[i] = before[i] = pops[i] = 0;
    __syncthreads();
    // column sums: a thread takes one expert (of Ew = 64, 128 or 256 columns) and every (256 / Ew)-th row
    const int Ew = E <= 64 ? 64 : (E <= 128 ? 128 : 256);
    const int e0 = tid & (Ew - 1), rstep = 256 / Ew;
    if (e0 < E) {
        int t = 0, bf = 0, pp = 0;
        const bool want_pop = b == 0 && pop_part != nullptr;
        for (int p = tid / Ew; p < nparts; p += 8 * rstep) {
            int v[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = p + i * rstep < nparts ? cnt_part[(size_t)(p + i * rstep) * E + e0] : 0;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                t += v[i];
                bf += p + i * rstep < b ? v[i] : 0;
            }
        }
        if (want_pop)
            for (int p = tid / Ew; p < nparts; p += 8 * rstep) {
                int v[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) v[i] = p + i * rstep < nparts ? pop_part[(size_t)(p + i * rstep) * E + e0] : 0;
#pragma unroll
                for (int i = 0; i < 8; ++i) pp += v[i];
            }
        if (rstep == 1) {
            tot[e0] = t; before[e0] = bf; pops[e0] = pp;
        } else {
            atomicAdd(&tot[e0], t);
            atomicAdd(&before[e0], bf);
            if (want_pop) atomicAdd(&pops[e0], pp);
        }
    }
    __syncthreads();
    // exclusive scan of the totals over experts (one per thread)
    const int c = tid < E ? tot[tid] : 0;
    int inc = c;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int up = __shfl_up(inc, o, 64);
        if (lane >= o) inc += up;
    }
    if (lane == 63) wsum[wave] = inc;
    __syncthreads();
    int carry = 0;
    for (int i = 0; i < wave; ++i) carry += wsum[i];
    const int off = carry + inc - c;
    if (tid < E) before[tid] += off;                   // where this workgroup's pairs of the expert start
    if (b == 0) {
        if (tid < E) {
            counts[tid] = c;
            offsets[tid] = off;
            if (pop_part) pop_out[tid] = pops[tid];
        }
        if (tid == 0) offsets[E] = wsum[0] + wsum[1] + wsum[2] + wsum[3];
    }
    __syncthreads();
    if (wave == 0) {
        int nbits = 0;
        while ((1 << nbits) < E) ++nbits;
        const unsigned long long lt = lane == 0 ? 0ull : (~0ull >> (64 - lane));
        volatile int32_t* at = before;
        for (int i0 = beg; i0 < end; i0 += 64) {
            const int i = i0 + lane;
            const int e = i0 == beg ? id0 : (i < end ? ids[i] : -1);
            const bool valid = i < end && e >= 0 && e < E;
            const unsigned long long mk = wave_match(e, valid, nbits);
            const int start = valid ? at[e] : 0;
            if (valid) {
                const int pos = start + __popcll(mk & lt);
                perm[pos] = i;
                inv_perm[i] = pos;
                if ((mk & lt) == 0) at[e] = start + __popcll(mk);
            }
        }
    } else if (b == 0) {
        // experts by (count descending, id ascending): rank = experts that come before
        for (int e = tid - 64; e < E; e += 192) {
            const int ce = tot[e];
            int r = 0;
            for (int j = 0; j < E; ++j) {
                const int cj = tot[j];
                r += cj > ce || (cj == ce && j < e);
            }
            order[r] = e;
        }
    }
}

// ---- fused decode-side routing --------------------------------------------
// grid (N, gates): a workgroup evaluates one gate for one token as route_rows_kernel does (same
// bits) and selects; what the permutation and the popularity need goes out with device-scope
// stores, and the workgroup that leaves last (ticket counter at the start of the workspace, zero
// between calls) adds them up.  13 tokens, E = 60, H = 2048: 11.7 us (selection and
// permutation entry by entry in loops: 16; a wave per gate row for all tokens, then every selection in the last workgroup: 52).
__global__ __launch_bounds__(64 * kTokWaves) void route_fused_kernel(FusedRouteArgs a, int32_t* ticket) {
    __shared__ float z[kMaxE];
    __shared__ int32_t sel[kMaxM];
    __shared__ float selw[kMaxM];
    __shared__ int32_t all[kFusedMaxN * kMaxM];
    __shared__ int32_t pop[kMaxE];
    __shared__ int32_t sm_perm[kPermSmemInts];
    __shared__ int sm_last;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int t = blockIdx.x, g = blockIdx.y, nvec = a.H >> 3, E = a.E;
    token_logits<1>(reinterpret_cast<const uint4*>(a.x) + (size_t)t * nvec, reinterpret_cast<const uint4*>(g ? a.Wg2 : a.Wg),
                    g ? a.bias2 : a.bias, 1, nvec, E, z);
    for (int i = tid; i < E; i += 64 * kTokWaves) pop[i] = 0;
    __syncthreads();
    const int m = g ? a.m : a.k;
    if (wave == 0) {
        wave_softmax_topm(z, E, m, g ? 0 : a.renorm, sel, selw, nullptr, nullptr);
        __builtin_amdgcn_wave_barrier();
        if (tid < m) {
            st_dev((g ? a.pids : a.ids) + (size_t)t * m + tid, sel[tid]);
            (g ? a.pw : a.w)[(size_t)t * m + tid] = selw[tid];
        }
        wait_own_stores();      // the ids have been acknowledged before the ticket counts this workgroup
        if (tid == 0) sm_last = (atomicAdd(ticket, 1) == (int)(gridDim.x * gridDim.y) - 1);
    }
    __syncthreads();
    if (!sm_last) return;
    const int P = a.N * a.k, Q = a.Wg2 ? a.N * a.m : 0;
    // (at most 1024 of each: one per thread, requested together)
    const int id = tid < P ? ld_dev(a.ids + tid) : -1;
    const int pid = tid < Q ? ld_dev(a.pids + tid) : -1;
    if (tid < P) all[tid] = id;
    if (pid >= 0) atomicAdd(&pop[pid], 1);
    __syncthreads();
    if (Q)
        for (int i = tid; i < E; i += 64 * kTokWaves) a.pop[i] = pop[i];
    if (P <= 64) {
        if (wave == 0) wave_permute_small(all, P, E, a.counts, a.offsets, a.perm, a.inv_perm, a.order);
    } else {
        block_permute(all, P, E, a.counts, a.offsets, a.perm, a.inv_perm, a.order, sm_perm);
    }
    if (tid == 0) *ticket = 0;
}

// Logits of a decode layer: a workgroup of four waves per 16 experts, token and gate (a compute unit takes the
// gate matrix at 64 bytes per cycle; one workgroup for all of 60 experts took 9 us, of which 4 were that); the
// first gate's first workgroup of a token also writes the token's row as fp16 and its shared gate.
__global__ __launch_bounds__(256) void layer_logits_kernel(FusedRouteArgs a, RoutePrep prep) {
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int t = blockIdx.x, g = blockIdx.y, e0 = blockIdx.z * 16, nvec = a.H >> 3, E = a.E;
    const uint4* xrow = reinterpret_cast<const uint4*>(a.x) + (size_t)t * nvec;
    if (e0 >= E) {                                        // the preparation has workgroups of its own
        if (g) return;
        uint4* xo = reinterpret_cast<uint4*>(prep.xh) + (size_t)t * nvec;
        for (int c = tid; c < nvec; c += 256) store_pairs(xo, c, bf16x8_to_f16x8(xrow[c]));
        if (wave == 3 && prep.shared_gate != nullptr) {
            const float v = wave_sigmoid_dot_bf16(xrow, reinterpret_cast<const uint4*>(prep.shared_gate), nvec);
            if ((tid & 63) == 0) prep.sgate[t] = v;
        }
        return;
    }
    const float* bias = g ? a.bias2 : a.bias;
    token_logits<1, 4>(xrow, reinterpret_cast<const uint4*>(g ? a.Wg2 : a.Wg) + (size_t)e0 * nvec, bias ? bias + e0 : nullptr, 1,
                       nvec, min(16, E - e0), prep.z + ((size_t)g * a.N + t) * E + e0);
}

fate_status launch_layer_logits(hipStream_t st, const FusedRouteArgs& r, const RoutePrep& prep) {
    layer_logits_kernel<<<dim3(r.N, r.Wg2 ? 2 : 1, (r.E + 15) / 16 + 1), 256, 0, st>>>(r, prep);
    FATE_HIP(hipGetLastError());
    return FATE_OK;
}

static fate_status check_route_args(const void* x, const void* Wg, const float* bias, int N, int H, int E, int k,
                                    int m, const void* ids, const void* w) {
    if (N < 0) FATE_FAIL(FATE_EINVAL, "N = %d < 0", N);
    if (E < 1 || E > kMaxE) FATE_FAIL(FATE_ESHAPE, "E = %d outside [1, %d]", E, kMaxE);
    if (H < 64 || (H % 64) != 0) FATE_FAIL(FATE_ESHAPE, "H = %d must be a positive multiple of 64", H);
    if (k < 1 || k > m) FATE_FAIL(FATE_EINVAL, "need 1 <= k <= m (k = %d, m = %d)", k, m);
    if (m > E || m > kMaxM) FATE_FAIL(FATE_EINVAL, "m = %d exceeds min(E, %d)", m, kMaxM);
    if (N == 0) return FATE_OK;
    FATE_CHECK_PTR(x);
    FATE_CHECK_PTR(Wg);
    FATE_CHECK_PTR_OPT(bias);
    FATE_CHECK_PTR(ids);
    FATE_CHECK_PTR(w);
    return FATE_OK;
}

// tokens per workgroup of the gate GEMM: enough workgroups for the device before the tile is
// filled with tokens
static int route_mfma_ntok(int N) { return N > 4096 ? 32 : (N > 1024 ? 16 : 8); }

template <int TOK, int NE>
static fate_status launch_route_mfma_v(hipStream_t st, dim3 grid, const uint16_t* x, const uint16_t* Wg, const float* bias,
                                       int N, int H, int E, int m, bool renorm, int32_t* ids, float* w, float* probs,
                                       int32_t* pop, const RouteSecond& second) {
    constexpr int lds = gate_lds(TOK, NE);
    static bool attr_done = false;
    if (!attr_done) {
        FATE_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(route_mfma_kernel<TOK, NE>),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, lds));
        attr_done = true;
    }
    route_mfma_kernel<TOK, NE><<<grid, 64 * kGateWaves, lds, st>>>(x, Wg, bias, N, H, E, m, renorm, ids, w, probs, pop, second);
    FATE_HIP(hipGetLastError());
    return FATE_OK;
}

static fate_status launch_route_mfma(hipStream_t st, const void* x, const void* Wg, const float* bias, int N, int H,
                                     int E, int m, bool renorm, int32_t* ids, float* w, float* probs, int32_t* pop,
                                     RouteSecond second, int ngates) {
    const int ntok = route_mfma_ntok(N);
    const dim3 grid((N + ntok - 1) / ntok, ngates);
    const uint16_t *xs = static_cast<const uint16_t*>(x), *ws = static_cast<const uint16_t*>(Wg);
#define FATE_GATE(TOK, NE) return launch_route_mfma_v<TOK, NE>(st, grid, xs, ws, bias, N, H, E, m, renorm, ids, w, probs, pop, second)
#define FATE_GATE_E(TOK)                          \
    if (E <= 64) FATE_GATE(TOK, 1);               \
    else if (E <= 128) FATE_GATE(TOK, 2);         \
    else FATE_GATE(TOK, 4);
    if (ntok == 8) { FATE_GATE_E(8) }
    else if (ntok == 16) { FATE_GATE_E(16) }
    else { FATE_GATE_E(32) }
#undef FATE_GATE_E
#undef FATE_GATE
}

static fate_status launch_route_rows(hipStream_t st, const void* x, const void* Wg, const float* bias, int N,
                                     int H, int E, int m, int renorm, int32_t* ids, float* w, float* probs,
                                     int32_t* pop) {
    auto xs = static_cast<const uint16_t*>(x);
    auto ws = static_cast<const uint16_t*>(Wg);
    if (N >= 64 && H % 1024 == 0)     // prefill-sized batches: gate GEMM on the matrix cores
        return launch_route_mfma(st, x, Wg, bias, N, H, E, m, renorm, ids, w, probs, pop, RouteSecond{}, 1);
    // four tokens per workgroup share the gate rows once one token each would be several rounds of workgroups
#define FATE_ROWS(TPW, NW) \
    route_rows_kernel<TPW, NW><<<(N + TPW - 1) / TPW, 64 * NW, 0, st>>>(xs, ws, bias, N, H, E, m, renorm, ids, w, probs, pop)
    // 16 waves while the device holds all workgroups at once (two per compute unit); beyond that workgroups of four waves,
    // of which none idles while the tokens' selections are taken (E = 60, H = 1920: 1024 tokens 11.9 us with 16 waves, 19.5
    // with 4; 1023 tokens, a workgroup each, 28.5 and 18.3; 5000 tokens 52 and 41; 20000 tokens 208 and 137)
    const int groups = N >= 1024 ? (N + 3) / 4 : N;
    if (N >= 1024 && groups > 512) FATE_ROWS(4, 4);
    else if (N >= 1024) FATE_ROWS(4, kTokWaves);
    else if (groups > 512) FATE_ROWS(1, 4);
    else FATE_ROWS(1, kTokWaves);
#undef FATE_ROWS
    FATE_HIP(hipGetLastError());
    return FATE_OK;
}

}  // namespace fate

using namespace fate;

extern "C" fate_status fate_gate_route(void* stream, const void* x_bf16, const void* Wg_bf16, const float* bias,
                                       int N, int H, int E, int k, int renorm, int32_t* topk_ids, float* topk_w,
                                       float* probs) {
    fate_status s = check_route_args(x_bf16, Wg_bf16, bias, N, H, E, k, k, topk_ids, topk_w);
    if (s != FATE_OK) return s;
    FATE_CHECK_PTR_OPT(probs);
    if (N == 0) return FATE_OK;
    return launch_route_rows(static_cast<hipStream_t>(stream), x_bf16, Wg_bf16, bias, N, H, E, k, renorm != 0,
                             topk_ids, topk_w, probs, nullptr);
}

extern "C" fate_status fate_cross_layer_predict(void* stream, const void* x_bf16, const void* Wg_next_bf16,
                                                const float* bias_next, int N, int H, int E, int k, int m,
                                                int32_t* pred_ids, float* pred_w, int32_t* pred_pop) {
    fate_status s = check_route_args(x_bf16, Wg_next_bf16, bias_next, N, H, E, k, m, pred_ids, pred_w);
    if (s != FATE_OK) return s;
    if (pred_pop == nullptr) FATE_FAIL(FATE_EINVAL, "pred_pop is NULL");
    hipStream_t st = static_cast<hipStream_t>(stream);
    fill_i32_kernel<<<(E + 255) / 256, 256, 0, st>>>(pred_pop, E, 0);
    FATE_HIP(hipGetLastError());
    if (N == 0) return FATE_OK;
    return launch_route_rows(st, x_bf16, Wg_next_bf16, bias_next, N, H, E, m, 0, pred_ids, pred_w, nullptr,
                             pred_pop);
}

extern "C" fate_status fate_permute(void* stream, const int32_t* topk_ids, int N, int k, int E, int32_t* counts,
                                    int32_t* offsets, int32_t* perm, int32_t* inv_perm, int32_t* expert_order) {
    if (N < 0 || k < 1) FATE_FAIL(FATE_EINVAL, "need N >= 0 and k >= 1 (N = %d, k = %d)", N, k);
    if (E < 1 || E > kMaxE) FATE_FAIL(FATE_ESHAPE, "E = %d outside [1, %d]", E, kMaxE);
    if ((long long)N * k > 0x7fffffffLL) FATE_FAIL(FATE_ESHAPE, "N*k overflows int32");
    if (counts == nullptr || offsets == nullptr || expert_order == nullptr)
        FATE_FAIL(FATE_EINVAL, "counts, offsets and expert_order must not be NULL");
    if (N > 0 && (topk_ids == nullptr || perm == nullptr || inv_perm == nullptr))
        FATE_FAIL(FATE_EINVAL, "topk_ids, perm and inv_perm must not be NULL when N > 0");
    permute_kernel<<<1, 64 * perm_waves(N * k, E), 0, static_cast<hipStream_t>(stream)>>>(topk_ids, N * k, E, counts,
                                                                                           offsets, perm, inv_perm, expert_order);
    FATE_HIP(hipGetLastError());
    return FATE_OK;
}

extern "C" fate_status fate_route_fused_workspace(int N, int E, size_t* bytes) {
    if (bytes == nullptr) FATE_FAIL(FATE_EINVAL, "bytes is NULL");
    if (N < 0 || E < 1 || E > kMaxE) FATE_FAIL(FATE_EINVAL, "bad N or E");
    *bytes = 256 + (size_t)2 * (size_t)(N > 0 ? N : 1) * E * sizeof(float);
    return FATE_OK;
}

extern "C" fate_status fate_route_fused(void* stream, const void* x_bf16, const void* Wg_bf16, const float* bias,
                                        const void* Wg_next_bf16, const float* bias_next, int N, int H, int E,
                                        int k, int m, int renorm, int32_t* topk_ids, float* topk_w,
                                        int32_t* pred_ids, float* pred_w, int32_t* pred_pop, int32_t* counts,
                                        int32_t* offsets, int32_t* perm, int32_t* inv_perm,
                                        int32_t* expert_order, void* workspace, size_t workspace_bytes) {
    fate_status s = check_route_args(x_bf16, Wg_bf16, bias, N, H, E, k, m, topk_ids, topk_w);
    if (s != FATE_OK) return s;
    const bool big = N >= 64 && H % 1024 == 0;     // both gate products in one launch on the matrix cores
    if (N < 1 || (N > kFusedMaxN && !big))
        FATE_FAIL(FATE_ESHAPE, "fused routing needs 1 <= N <= %d, or N >= 64 with H a multiple of 1024 (N = %d, H = %d)",
                  kFusedMaxN, N, H);
    if (Wg_next_bf16) {
        FATE_CHECK_PTR(Wg_next_bf16);
        FATE_CHECK_PTR_OPT(bias_next);
        if (!pred_ids || !pred_w || !pred_pop) FATE_FAIL(FATE_EINVAL, "pred outputs must not be NULL");
    }
    if (!counts || !offsets || !perm || !inv_perm || !expert_order)
        FATE_FAIL(FATE_EINVAL, "permutation outputs must not be NULL");
    size_t need = 0;
    fate_route_fused_workspace(N, E, &need);
    if (workspace == nullptr || workspace_bytes < need)
        FATE_FAIL(FATE_EWORKSPACE, "workspace of %zu bytes needed, %zu given", need, workspace_bytes);
    FATE_CHECK_PTR(workspace);
    if (big) {
        hipStream_t st = static_cast<hipStream_t>(stream);
        // the workgroups' counts go through the workspace and are added up by the permutation
        // kernel: no zeroing launch, no atomics on the device-wide histogram
        const int ntok = route_mfma_ntok(N), nparts = (N + ntok - 1) / ntok;
        int32_t* cnt_part = reinterpret_cast<int32_t*>(static_cast<char*>(workspace) + 256);
        int32_t* pop_part = cnt_part + (size_t)nparts * E;         // (nparts <= N / 8 + 1: the logits' room holds both)
        s = launch_route_mfma(st, x_bf16, Wg_bf16, bias, N, H, E, k, renorm != 0, topk_ids, topk_w, nullptr, nullptr,
                              RouteSecond{static_cast<const uint16_t*>(Wg_next_bf16), bias_next, m, pred_ids, pred_w,
                                          pred_pop, pop_part, cnt_part},
                              Wg_next_bf16 ? 2 : 1);
        if (s != FATE_OK) return s;
        permute_parts_kernel<<<nparts, 256, 0, st>>>(topk_ids, N * k, ntok * k, E, nparts, cnt_part,
                                                     Wg_next_bf16 ? pop_part : nullptr, counts, offsets, perm, inv_perm,
                                                     expert_order, pred_pop);
        FATE_HIP(hipGetLastError());
        return FATE_OK;
    }
    FusedRouteArgs a{static_cast<const uint16_t*>(x_bf16), static_cast<const uint16_t*>(Wg_bf16), bias,
                     static_cast<const uint16_t*>(Wg_next_bf16), bias_next, N, H, E, k, m, renorm != 0,
                     topk_ids, topk_w, pred_ids, pred_w, pred_pop, counts, offsets, perm, inv_perm, expert_order};
    route_fused_kernel<<<dim3(N, Wg_next_bf16 ? 2 : 1), 64 * kTokWaves, 0, static_cast<hipStream_t>(stream)>>>(
        a, static_cast<int32_t*>(workspace));
    FATE_HIP(hipGetLastError());
    return FATE_OK;
}
