// Launch interface of the prompt (prefill) kernels (ls_prefill.hip).
#pragma once
#include "ls_gemm.h"

namespace ls {

constexpr int kPrefillRowsMax = 2048;   // prompt rows one prefill pass carries (buffers of a handle are sized for it)

// The fp32 state of prompt rows: [row tile][group of 4 columns][16 rows][4]; element (m, k), k a multiple of 4
__device__ __forceinline__ size_t prefill_state(int m, int k, int h) {
    return ((size_t)(m / 16) * (h / 4) + k / 4) * 64 + (m % 16) * 4;
}

// A launch over M consecutive prompt positions of one sequence: row m is
// position p0 + m.  Buffers hold whole row tiles (M rounded up to 16).
struct PrefillGemm {
    Geo g;
    int M, p0, seq;
    const void* A;         // [M][K] operand order
    const float* SSQ;      // QKV, SWIGLU: [M][h/16] sums of squares of A's fp32 state
    int K;
    const void* Wp;        // packed weights (launch_pack)
    int tile0, tiles;      // 16-feature tiles tile0 .. tile0 + tiles - 1 of the packed matrix
    int N_mat;
    const float* Xin;      // RESID: residual in and out (prefill_state order); rounded copy (operand order) and
                           // tile sums of squares [M][h/16] of the result
    float* Xout;
    void* XBout;
    float* SSQout;
    void* act;             // SWIGLU: [M][F] operand order
    void* q;               // QKV: [M][h] rotated queries, compute dtype, row-major
    void* kvc;             // QKV: committed cache
    int table;             // QKV: key/value table of the block at this depth
    const float* rope;
};

hipError_t prefill_prepare();   // allow the kernels' LDS sizes
hipError_t launch_prefill_gemm(const PrefillGemm& p, int epi, bool bf16, hipStream_t st);

// Causal attention of the rows of a 16-bit model's prompt pass over positions
// 0 .. p0 + m of their table in the committed cache.
struct PrefillAttn {
    Geo g;
    int M, p0, seq, table;
    const void* q;         // [M][h] row-major
    const void* kvc;
    void* out;             // [M][h] operand order
};
hipError_t launch_prefill_attn(const PrefillAttn& p, hipStream_t st);

// X[m] = E[tok[m]], its rounded copy and tile sums of squares, for M prompt rows
hipError_t launch_prefill_embed(const Geo& g, const int32_t* tok, int M, const void* E, bool bf16, float* X,
                                PassBuf pb, hipStream_t st);

// row m of a prompt state, row-major
hipError_t launch_prefill_row(const Geo& g, const float* X, int m, float* out, hipStream_t st);

}  // namespace ls
