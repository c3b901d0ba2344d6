// Shared between the FFN translation units.
#pragma once
#include <hip/hip_fp16.h>
#include "common.h"

namespace fate {

struct DecodeArgs {
    const uint16_t* x;
    int N, H, E, k;
    const fate_qexpert* experts;
    const fate_qexpert* shared;
    int n_shared;
    const int32_t* counts;
    const int32_t* offsets;
    const int32_t* perm;
    const int32_t* inv_perm;
    const int32_t* order;
    const float* topk_w;
    const uint16_t* shared_gate;
    int nact;            // routed expert slots in the grid: min(E, N*k)
    int rb_r, rb_s;      // 32-row blocks per routed / shared expert (up kernel)
    int bits_r, group_r, bits_s, group_s;
    __half* h_r; int ldh_r;   // [P][I_max] fp16, rows in sorted pair order
    __half* h_s; int ldh_s;   // [n_shared*N][I_shared_max] fp16
    float* part_r;            // [P][nchunk_r][H] fp32: weighted partial outputs, rows in sorted pair order
    float* part_s;            // [n_shared][nchunk_s][N][H] fp32 (gated)
    int32_t* status;
    int nchunk_r, nchunk_s, cg_r, cg_s;   // reduction chunks of the down kernel
    int lds_rows;        // activation rows staged in LDS per pass, plus one zero row
};

// Pair order of the GEMMs' activations (xh, h_r, h_s) inside every 32 columns: column 8d + 2j + i lies at place
// 8j + 2d + i.  The 16 bytes of piece j are then columns 2j, 2j + 1 of every 8, which is what one mask takes out of the
// four dwords (one per 8 columns) of a lane's 4-bit codes.
__host__ __device__ inline int pair_place(int col) { return (col & ~31) + ((col & 7) >> 1) * 8 + ((col & 31) >> 3) * 2 + (col & 1); }
#ifdef __HIPCC__
// the fp16 columns 8c .. 8c + 7 of a row go to their places
__device__ __forceinline__ void store_pairs(void* row, int c, uint4 v) {
    uint32_t* o = static_cast<uint32_t*>(row) + (c >> 2) * 16 + (c & 3);
    o[0] = v.x; o[4] = v.y; o[8] = v.z; o[12] = v.w;
}
#endif

struct MfmaScratch {
    __half* xh;        // [N,H] fp16 copy of x, pair order
    float* sgate;      // [N] shared gate values
    int4* tab_up;      // [E + n_shared + 1] segments of the up GEMM: first tile, expert, first row, rows
    int4* tab_down;    // same for the down GEMM
    void* yp_r;        // [kp_r][P,H] per-pair outputs of the down GEMM, mfma_out_bytes() each
    void* yp_s;        // [kp_s][n_shared*N,H]
};

struct FfnWorkspace {
    int32_t* status;
    __half* h_r;
    __half* h_s;
    float* part_r;   // decode path: partial outputs of the down kernel, summed in a fixed order by a last launch
    float* part_s;
    MfmaScratch ms;  // MFMA path only
    size_t bytes;
};

fate_status check_decode_groups(const fate_ffn_desc& d);
fate_status launch_ffn_decode(hipStream_t st, const fate_ffn_desc& d, DecodeArgs a, void* y_out);
// reduction chunks (of at most 16 groups) of the decode down kernel for an intermediate size of G groups
inline int decode_down_chunks(int G) { return G > 0 ? (G + 15) / 16 : 1; }
// Piece of a layer (matrix-core path): the routed experts of `mask` (bit e), the shared experts and
// the preparation of x with the first piece, the per-token combination with the last one.
struct PartSel {
    unsigned long long mask[4];
    int first, last;
};
__host__ __device__ inline PartSel part_all() { return PartSel{{~0ull, ~0ull, ~0ull, ~0ull}, 1, 1}; }

// parts of the reduction dimension of the down GEMM of routed / shared experts
void mfma_k_parts(const fate_ffn_desc& d, int* kp_r, int* kp_s);
// bytes per element of its outputs: fp16 only for a whole sum, and not in the decode-sized form
inline size_t mfma_out_bytes(bool exact, int kp) { return exact || kp > 1 ? 4 : 2; }
// Routing of a decode layer inside its up GEMM's launch, from the logits (at most 64 pairs): every workgroup
// selects for itself, the first one writes the outputs.
struct LayerOut {
    const float* z;                    // [gates][N][E] logits
    int N, k, m, E, renorm;
    int32_t* ids; float* w;
    int32_t* pids; float* pw;          // pids NULL: no prediction
    int32_t *counts, *offsets, *perm, *inv_perm, *order, *pop;
    int32_t* calls;                    // counts the calls
};

// How launch_ffn_mfma runs: phase 0 = whole FFN, 1 = prep + up GEMM only, 2 = down GEMM + combine only (timing
// aid); exact = the decode-sized form of the GEMMs (at most 16 tokens); layer = inside a decode layer (at most 8
// tokens, exact): the logits, x and the shared gate are there, nothing else of the routing is, and entries of
// another format than the descriptor's, or with zero-points, count as absent.
struct MfmaMode {
    int phase = 0;
    bool exact = false;
    const LayerOut* layer = nullptr;
};
fate_status launch_ffn_mfma(hipStream_t st, const fate_ffn_desc& d, DecodeArgs da, const MfmaScratch& ms,
                            void* y_out, const PartSel& sel, const MfmaMode& mode);

// Column blocks per segment of the two GEMMs' tile tables, K parts of the down GEMM included, and the most rows of
// a tile of routed / shared experts (1 << rows_r, rows_s).
struct TileBlocks {
    int r_up, s_up, r_down, s_down, rows_r, rows_s;
};
TileBlocks mfma_tile_blocks(const fate_ffn_desc& d, bool exact);
constexpr int kTileRowsLog2 = 7;          // prefill: 128 rows
// 64 where the nominal width is not 4 bits: a workgroup takes its rows 64 at a time there, and two workgroups are
// faster than two passes of one (8-bit, H = 256, I = 512, E = 8, 300 tokens: 32 us with
// tiles of 128 rows, 24 with these; E = 64, k = 6, H = 2048, I = 1408 with two shared experts, 2048 tokens: 506 and 464).
constexpr int kTileRowsLog2Wide = 6;
constexpr int kExactTileRowsLog2 = 4;     // decode-sized form: 16 rows (an expert has more if tokens name it repeatedly)

// The decode kernels' job done by the GEMM's decode-sized form (exact weights, fp32 per-pair outputs):
// up to 16 tokens, sizes that are multiples of 128, and at least half a device of its 128-neuron
// workgroups.  Below that the decode kernels' 32-neuron workgroups spread the weights further (two
// int8 layers of H = 256, I = 512, E = 8 at 16 tokens: 49 us with them, 56 with the GEMMs).
inline bool decode_by_gemm(const fate_ffn_desc& d) {
    if (d.N > 16 || d.H % 128 || d.I_max % 128 || (d.n_shared && d.I_shared_max % 128)) return false;
    const long long experts = (long long)d.N * d.k < d.E ? (long long)d.N * d.k : d.E;
    return experts * (d.I_max / 128) + d.n_shared * ((d.n_shared ? d.I_shared_max : 0) / 128) >= 128;
}

}  // namespace fate
