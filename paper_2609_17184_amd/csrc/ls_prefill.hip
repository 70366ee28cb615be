// Prompt (prefill) kernels: the block GEMMs over up to kPrefillRowsMax
// consecutive positions of one sequence, and the prompt's embedding.
//
// A prompt pass multiplies M rows with every weight matrix, so unlike the
// decode's weight stream it is a contraction bound by the matrix cores and by
// how often the operands are re-read on chip.
//
// Both operands lie in memory in MFMA operand order (fragments of 16 rows x
// one k step, a lane's 16 bytes at lane * 16): the weights packed when they are
// bound, the activations because every prompt kernel writes them that way
// (opd_elem).  A wave's load is 1 KB of consecutive bytes: in row-major
// order the 16 rows of a fragment lie a multiple of 4 KB apart (K = 2048), on
// one L2 channel.  The product is formed transposed (weights as the MFMA's A operand): a lane ends with four
// consecutive features of one row.  Partials meet in
// LDS and the epilogue takes them from there in the order that its global
// accesses want.  A workgroup is four waves and two workgroups share a CU (two
// waves per SIMD: one wave alone draws only half of the LDS read rate), so one
// workgroup's prologue and epilogue run under the other's products.
//
// k_prefill_tile: 128 rows x 128 features, for launches with enough tiles to
// fill the chip; 64 x 64 per wave.  Activations go through LDS in fragment
// order (no bank conflicts on either side).
//
// k_prefill_slice: 64 rows x 64 features, for the launches that would leave
// CUs idle at 128 x 128.  Every wave takes a quarter of k for the whole tile
// and loads both operands straight into registers: no LDS and no barrier
// until the partials meet.
//
// Measured by kernel trace inside a prompt (us per launch, and the rate in
// TFLOP/s).  h = 2048, F = 5632, 512 rows: QKV 31 (415), O 12.6 (340), gate/up 48
// (490), down 25 (465); 2048 rows: 75 (685), 31 (560), 131 (720), 65 (725).  h = 5280,
// F = 17920, 320 rows: 110 (485), 45 (400), 212 (570), 133 (455); 1024 rows: 230
// (745), 107 (535), 485 (800), 313 (620).  Back-to-back MFMAs reach 2100; the
// decode's 64-row launches took eight times 30, 18, 38 and 32 us for 512 rows of
// the first shape.  What bounds them now: the CU's L1 (64 B a clock, both
// operands once per workgroup and the weights once more for the second row
// half), and at 512 rows the weights' way from HBM, the first loads and the
// epilogue.
#include "ls_prefill.h"

#include <algorithm>

#include "ls_opd_dev.h"

namespace ls {

// The workgroup's tile from NP partials in LDS ([NP][BM][NMAT * BN + 4] fp32,
// summed in order) through the epilogue of its kind: BM rows from m0, feature
// tiles t0 .. of the packed matrix (BN / 16 of them; gate/up: the columns of
// gate, then of up).  A thread takes one row of one tile at a time.  Rows run
// fastest over the lanes where the output is in operand order (runs of 256
// bytes); tiles do for QKV, whose outputs and RoPE table are row-major.
template <typename WT, int EPI, int NMAT, int BM, int BN, int NP>
__device__ __forceinline__ void prefill_finish(const PrefillGemm& p, int m0, int t0, const float* part, const float* rinv) {
    constexpr int LD = NMAT * BN + 4, TPB = BN / kTile, N = BM * TPB, ITER = (N + 255) / 256;
    const int tid = threadIdx.x;
    auto sum = [&](int row, int col, float (&o)[16]) {
#pragma unroll
        for (int e = 0; e < 16; e += 4) {
            f32x4 v = *(const f32x4*)(part + (size_t)row * LD + col + e);
#pragma unroll
            for (int k = 1; k < NP; ++k) v += *(const f32x4*)(part + ((size_t)k * BM + row) * LD + col + e);
            o[e] = v[0];
            o[e + 1] = v[1];
            o[e + 2] = v[2];
            o[e + 3] = v[3];
        }
    };
#pragma unroll
    for (int i = 0; i < ITER; ++i) {
        const int u = i * 256 + tid, r = EPI == EPI_QKV ? u / TPB : u % BM, c = EPI == EPI_QKV ? u % TPB : u / BM;
        const int m = m0 + r, tl = t0 + c, tg = p.tile0 + tl;
        if (u >= N || m >= p.M || tl >= p.tiles) continue;
        float o[16];
        if constexpr (EPI == EPI_RESID) {
            f32x4 x[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) x[e] = *(const f32x4*)(p.Xin + prefill_state(m, tg * kTile + e * 4, p.g.h));
            sum(r, c * kTile, o);
            float sq = 0.f;
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                o[e] += x[e >> 2][e & 3];
                sq = fmaf(o[e], o[e], sq);
            }
#pragma unroll
            for (int e = 0; e < 4; ++e)
                *(f32x4*)(p.Xout + prefill_state(m, tg * kTile + e * 4, p.g.h)) =
                    f32x4{o[e * 4], o[e * 4 + 1], o[e * 4 + 2], o[e * 4 + 3]};
            store_act16<WT>(p.XBout, m, tg * kTile, p.g.h, o);
            p.SSQout[(size_t)m * p.g.ssq_tiles + tg] = sq;
        } else if constexpr (EPI == EPI_SWIGLU) {
            float up[16];
            sum(r, c * kTile, o);
            sum(r, BN + c * kTile, up);
            const float ri = rinv[r];
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const float a = o[e] * ri;
                o[e] = a / (1.0f + expf(-a)) * (up[e] * ri);
            }
            store_act16<WT>(p.act, m, tg * kTile, p.N_mat, o);
        } else {
            // a tile holds the RoPE pairs (i, i + dh/2) of eight i in columns k and k + 8
            const int tph = p.g.h / kTile, tpd = p.g.dh / kTile, half = p.g.dh / 2;
            const int mat = tg / tph, lt = tg - mat * tph, head = lt / tpd, i0 = (lt - head * tpd) * 8;
            sum(r, c * kTile, o);
            const float ri = rinv[r];
#pragma unroll
            for (int e = 0; e < 16; ++e) o[e] *= ri;
            if (mat < 2) {
                const f32x4* rp = (const f32x4*)(p.rope + ((size_t)(p.p0 + m) * half + i0) * 2);
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float cs = rp[e >> 1][(e & 1) * 2], sn = rp[e >> 1][(e & 1) * 2 + 1];
                    const float a = o[e], b = o[e + 8];
                    o[e] = a * cs - b * sn;
                    o[e + 8] = b * cs + a * sn;
                }
            }
#pragma unroll
            for (int hf = 0; hf < 2; ++hf) {
                const int d = i0 + hf * half;
                WT* dst = mat == 0 ? (WT*)p.q + (size_t)m * p.g.h + head * p.g.dh + d
                                   : (WT*)p.kvc + kvc_index(p.g, p.seq, p.table, mat - 1, head, p.p0 + m) + d;
#pragma unroll
                for (int e = 0; e < 8; e += WTraits<WT>::VEC) *(u32x4*)(dst + e) = pack16<WT>(o + hf * 8 + e);
            }
        }
    }
}

// 1/rms of rows m0 .. m0 + BM - 1 from their tile sums of squares, 16 lanes per row
template <int BM>
__device__ __forceinline__ void prefill_rinv(const PrefillGemm& p, int m0, float* rinv) {
    const int T = p.g.ssq_tiles, tid = threadIdx.x;
#pragma unroll
    for (int i = 0; i < BM / 16; ++i) {
        const int r = i * 16 + (tid >> 4), m = m0 + r;
        float s = 0.f;
        if (m < p.M) {
#pragma unroll 8
            for (int t = tid & 15; t < T; t += 16) s += p.SSQ[(size_t)m * T + t];
        }
        s = group_sum<16>(s);
        if ((tid & 15) == 0) rinv[r] = 1.0f / sqrtf(s / (float)p.g.h + p.g.eps);
    }
}

// Workgroups are dealt to the 8 XCDs in turn: each XCD takes a contiguous run
// of (feature block, row block) pairs, row blocks fastest, so the row blocks
// that share weights run on one XCD at a time and read them through its L2.
__device__ __forceinline__ void prefill_block(int mb, int* nblk, int* mblk) {
    const int total = gridDim.x, xcd = blockIdx.x & 7, q = total >> 3, r = total & 7;
    const int id = xcd * q + min(xcd, r) + (blockIdx.x >> 3);
    *nblk = id / mb;
    *mblk = id - *nblk * mb;
}

// A wave's packed feature tile t (of the launch): its fragments, k step by k step
template <int NMAT>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t prefill_weights(const PrefillGemm& p, int t, int ns) {
    const size_t tb = (size_t)ns * NMAT * 1024;
    const bool ok = t < p.tiles;
    return buf_rsrc((const char*)p.Wp + (ok ? (size_t)(p.tile0 + t) * tb : 0), ok ? (uint32_t)tb : 0u);
}

template <typename WT, int EPI, int NMAT>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) k_prefill_tile(PrefillGemm p) {
    constexpr int KSTEP = WTraits<WT>::KSTEP, ES = sizeof(WT);
    constexpr int BM = 128, BN = 128 / NMAT, FT = 4 / NMAT, PF = 2, NS = 4;
    extern __shared__ __align__(16) char smem[];
    u32x4* const lds = (u32x4*)(smem + BM * 4);           // [3 buffers][2 steps][8 row tiles][64]
    float* const rinv = (float*)smem;
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wr = wv >> 1, wf = wv & 1;
    const int j = lane & 15, grp = lane >> 4;
    int nblk, mblk;
    prefill_block((p.M + BM - 1) / BM, &nblk, &mblk);
    const int m0 = mblk * BM, t0 = nblk * (BN / 16);
    const int ns = p.K / KSTEP, stages = (ns + 1) / 2;     // k steps, stages of two
    __amdgpu_buffer_rsrc_t rw[FT];
#pragma unroll
    for (int f = 0; f < FT; ++f) rw[f] = prefill_weights<NMAT>(p, t0 + wf * FT + f, ns);
    // the block's row tiles (those past the last row's lie beyond the range: zeros)
    const int rts = min(BM / 16, (p.M - m0 + 15) / 16);
    const __amdgpu_buffer_rsrc_t ra = buf_rsrc((const char*)p.A + (size_t)m0 * p.K * ES, (uint32_t)(rts * ns * 1024));
    const int vw = lane * 16;

    u32x4 w[PF][2][FT][NMAT], a[2][NS], x0[4], x1[4];
    // (steps past the end multiply zero activations)
    auto load_w = [&](int ks, u32x4 (&r)[FT][NMAT]) {
#pragma unroll
        for (int f = 0; f < FT; ++f)
#pragma unroll
            for (int q = 0; q < NMAT; ++q) r[f][q] = buf_load16<0>(rw[f], vw, (ks * NMAT + q) * 1024);
    };
    // the four waves stage the 2 x 8 fragments of a stage: row tiles wv, wv + 4 of each step
    auto load_a = [&](int s, u32x4 (&r)[NS]) {
#pragma unroll
        for (int i = 0; i < NS; ++i) {
            const int ks = s * 2 + (i >> 1), tf = wv + 4 * (i & 1);
            r[i] = buf_load16<0>(ra, ks < ns ? vw : kOutOfRange, (tf * ns + ks) * 1024);
        }
    };
    auto put_a = [&](int buf, const u32x4 (&r)[NS]) {
#pragma unroll
        for (int i = 0; i < NS; ++i) lds[(buf * 16 + (i >> 1) * 8 + wv + 4 * (i & 1)) * 64 + lane] = r[i];
    };
    auto get_x = [&](int buf, int k, u32x4 (&x)[4]) {
#pragma unroll
        for (int t = 0; t < 4; ++t) x[t] = lds[(buf * 16 + k * 8 + wr * 4 + t) * 64 + lane];
    };
    f32x4 acc[FT][NMAT][4];
#pragma unroll
    for (int f = 0; f < FT; ++f)
#pragma unroll
        for (int q = 0; q < NMAT; ++q)
#pragma unroll
            for (int t = 0; t < 4; ++t) acc[f][q][t] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto mul = [&](const u32x4 (&r)[FT][NMAT], const u32x4 (&x)[4]) {
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int f = 0; f < FT; ++f)
#pragma unroll
                for (int q = 0; q < NMAT; ++q) mfma_one<WT>(r[f][q], x[t], acc[f][q][t]);
    };

    load_a(0, a[0]);
    load_a(1, a[1]);
#pragma unroll
    for (int u = 0; u < PF; ++u)
#pragma unroll
        for (int k = 0; k < 2; ++k) load_w(u * 2 + k, w[u][k]);
    if constexpr (EPI != EPI_RESID) prefill_rinv<BM>(p, m0, rinv);
    // A stage s: read its second step's fragments; multiply the first's;
    // barrier; store the rows of stage s + 2 (into the buffer every wave left
    // before the barrier); read the first fragments of stage s + 1 (stored
    // before it); multiply the second step's: every LDS read is a step ahead
    // of its use.  Stages run in groups of PF; those past the end multiply zeros.
    put_a(0, a[0]);
    load_a(2, a[0]);
    put_a(1, a[1]);
    load_a(3, a[1]);
    __syncthreads();
    get_x(0, 0, x0);
    int b0 = 0;                                           // buffer of the current stage
    for (int s0 = 0; s0 < stages; s0 += PF) {
#pragma unroll
        for (int u = 0; u < PF; ++u) {
            const int s = s0 + u, b1 = b0 == 2 ? 0 : b0 + 1, b2 = b0 == 0 ? 2 : b0 - 1;
            get_x(b0, 1, x1);
            __builtin_amdgcn_sched_barrier(0);
            mul(w[u][0], x0);
            load_w((s + PF) * 2, w[u][0]);
            __builtin_amdgcn_sched_barrier(0);
            __syncthreads();
            put_a(b2, a[u & 1]);
            load_a(s + 4, a[u & 1]);
            get_x(b1, 0, x0);
            __builtin_amdgcn_sched_barrier(0);
            mul(w[u][1], x1);
            load_w((s + PF) * 2 + 1, w[u][1]);
            __builtin_amdgcn_sched_barrier(0);
            b0 = b1;
        }
    }
    // the tile: [row][feature] over the staging buffers
    constexpr int LD = NMAT * BN + 4;
    float* const part = (float*)(smem + BM * 4);
    __syncthreads();
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int f = 0; f < FT; ++f)
#pragma unroll
            for (int q = 0; q < NMAT; ++q)
                *(f32x4*)(part + (size_t)(wr * 64 + t * 16 + j) * LD + q * BN + (wf * FT + f) * 16 + grp * 4) =
                    acc[f][q][t];
    __syncthreads();
    prefill_finish<WT, EPI, NMAT, BM, BN, 1>(p, m0, t0, part, rinv);
}

template <typename WT, int EPI, int NMAT>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) k_prefill_slice(PrefillGemm p) {
    constexpr int KSTEP = WTraits<WT>::KSTEP, ES = sizeof(WT);
    constexpr int BM = 64, BN = 64 / NMAT, FT = 4 / NMAT, PF = 4, LD = NMAT * BN + 4;
    extern __shared__ __align__(16) char smem[];
    float* const rinv = (float*)smem;
    float* const part = (float*)(smem + BM * 4);
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int j = lane & 15, grp = lane >> 4;
    int nblk, mblk;
    prefill_block((p.M + BM - 1) / BM, &nblk, &mblk);
    const int m0 = mblk * BM, t0 = nblk * (BN / 16);
    const int ns = p.K / KSTEP, k0 = ns * wv / 4, n = ns * (wv + 1) / 4 - k0;
    __amdgpu_buffer_rsrc_t rw[FT];
#pragma unroll
    for (int f = 0; f < FT; ++f) rw[f] = prefill_weights<NMAT>(p, t0 + f, ns);
    // the block's row tiles (those past the last row's lie beyond the range: zeros)
    const int rts = min(BM / 16, (p.M - m0 + 15) / 16);
    const __amdgpu_buffer_rsrc_t ra = buf_rsrc((const char*)p.A + (size_t)m0 * p.K * ES, (uint32_t)(rts * ns * 1024));
    const int vw = lane * 16;
    u32x4 w[PF][FT][NMAT], x[PF][4];
    // (steps past the wave's share are loaded but not used)
    auto load = [&](int i, u32x4 (&r)[FT][NMAT], u32x4 (&y)[4]) {
#pragma unroll
        for (int f = 0; f < FT; ++f)
#pragma unroll
            for (int q = 0; q < NMAT; ++q) r[f][q] = buf_load16<0>(rw[f], vw, ((k0 + i) * NMAT + q) * 1024);
#pragma unroll
        for (int t = 0; t < 4; ++t) y[t] = buf_load16<0>(ra, vw, (t * ns + k0 + i) * 1024);
    };
    f32x4 acc[FT][NMAT][4];
#pragma unroll
    for (int f = 0; f < FT; ++f)
#pragma unroll
        for (int q = 0; q < NMAT; ++q)
#pragma unroll
            for (int t = 0; t < 4; ++t) acc[f][q][t] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto mul = [&](const u32x4 (&r)[FT][NMAT], const u32x4 (&y)[4]) {
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int f = 0; f < FT; ++f)
#pragma unroll
                for (int q = 0; q < NMAT; ++q) mfma_one<WT>(r[f][q], y[t], acc[f][q][t]);
    };
#pragma unroll
    for (int u = 0; u < PF; ++u) load(u, w[u], x[u]);
    if constexpr (EPI != EPI_RESID) prefill_rinv<BM>(p, m0, rinv);
    int i = 0;
    for (; i + PF <= n; i += PF) {
#pragma unroll
        for (int u = 0; u < PF; ++u) {
            mul(w[u], x[u]);
            load(i + u + PF, w[u], x[u]);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
#pragma unroll
    for (int u = 0; u < PF - 1; ++u)
        if (i + u < n) mul(w[u], x[u]);
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int f = 0; f < FT; ++f)
#pragma unroll
            for (int q = 0; q < NMAT; ++q)
                *(f32x4*)(part + ((size_t)wv * BM + t * 16 + j) * LD + q * BN + f * 16 + grp * 4) = acc[f][q][t];
    __syncthreads();
    prefill_finish<WT, EPI, NMAT, BM, BN, 4>(p, m0, t0, part, rinv);
}

// LDS of a workgroup: 1/rms of its rows, then the partials (which the staging buffers share)
constexpr size_t kTileLds = 128 * 4 + (size_t)128 * 132 * 4;
constexpr size_t kSliceLds = 64 * 4 + (size_t)4 * 64 * 68 * 4;
static_assert(3 * 16 * 1024 <= 128 * 132 * 4, "staging buffers fit the partials' area");

template <typename WT, int EPI, int NMAT>
static hipError_t launch_shape(const PrefillGemm& p, hipStream_t st) {
    const int tb = ((p.tiles * NMAT + 7) / 8) * ((p.M + 127) / 128), sb = ((p.tiles * NMAT + 3) / 4) * ((p.M + 63) / 64);
    // Slices fill the CUs with a quarter of the work per workgroup, tiles read
    // half as much per flop.  us per launch inside a prompt (h = 2048, F = 5632),
    // tiles / slices, at so many tiles: 48 QKV 31 / 15; 128 O 27 / 21, down 60 / 45;
    // 192 QKV 31 / 30, O 29 / 34, down 62 / 71; 208 to 240 O
    // 30 / 48, down 64 / 105, QKV 31 / 37; from 256 on tiles win by 1.2 to 2.  fp32
    // (a quarter of the arithmetic rate, so the chip's idle part weighs more):
    // 192 gate/up 80 / 62, 216 QKV 79 / 90, 256 gate/up 81 / 90, 264 QKV 136 / 110.
    const bool tile = tb >= (sizeof(WT) == 2 ? 200 : 256);
    const void* f = tile ? (const void*)k_prefill_tile<WT, EPI, NMAT> : (const void*)k_prefill_slice<WT, EPI, NMAT>;
    PrefillGemm q = p;
    void* args[] = {(void*)&q};
    return hipLaunchKernel(f, dim3(tile ? tb : sb), dim3(256), args, tile ? kTileLds : kSliceLds, st);
}

// ---------------------------------------------------------------------------
// Causal attention of prompt rows over the committed cache (16-bit models):
// one workgroup per (head, 64 NQ queries), 16 NQ queries per wave, keys and
// values in tiles of 64 positions.  As in the decode's attention, a weight is
// rounded to fp16 against the largest of its own 64 keys and the tiles are
// combined in fp32: the sums are brought to each tile's maximum, up or
// down, before its products are added to them, and the query's own position
// joins at the end, unrounded.  (One reference for the whole row, the largest
// score so far, rounds the largest weight of every other tile too and leaves
// small ones no bits: off from 64 bits by 1.5e-4 instead of 0.8e-4 over 6000
// keys with scores of deviation 2, and by 40 % instead of 5 % where one key of
// no value lies 15 above the others.)
//
// Both products are formed transposed, S^T = K Q^T and O^T = V^T P^T: a lane
// then holds the scores of one query (column l % 16) against keys 4 (l / 16)
// + v of each 16-key tile, so maxima and sums cross lanes twice per 64 keys,
// and those same registers, rounded to fp16, are the second product's operand
// without any exchange: its k index may run over the keys in any order, and
// the values are staged in that order (slot (g, e) of a 32-key step: key 4 g +
// e of its first 16-key tile for e < 4, of its second for e >= 4).  Staging
// turns four keys x eight dimensions per thread in registers.  Keys and
// values are read from memory once per workgroup, not once per row, and the
// next tile's loads are in flight under the current one's products.
//
// Measured (16 heads x 128, us per launch): 14.3 at 512 positions, 61 at 2048
// (280 TFLOP/s of the causal products), 202 for 2048 rows behind 4096 positions
// (425); one workgroup per (row, head), the decode's arrangement, took 145,
// 1190 and 4240.  What bounds it: the exponentials and the packing of the
// weights (VALU) next to the two products, and at 512 positions the 128
// workgroups, one on every other CU.
//
// A masked key of a loaded tile has the weight 0, and 0 times an infinite
// value is NaN: a position that is not finite makes the rows of its key tile
// before it so too.  (The last position of such a prompt is not finite either
// way, and the call fails.)
// ---------------------------------------------------------------------------
template <int DH, int NQ>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) k_prefill_attn(PrefillAttn p) {
    constexpr int KD = (DH + 31) / 32, DT = DH / 16, QB = 64 * NQ, VS = 65;   // (a value fragment is padded to 65 x 16 bytes)
    __shared__ __align__(16) u32x4 kl[2][4 * KD * 64];
    __shared__ __align__(16) u32x4 vl[2][2 * DT * VS];
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int j = lane & 15, grp = lane >> 4;
    // heads dealt to the XCDs (their keys and values stay in one L2), the long query blocks first
    int head, qb;
    const int nqb = (p.M + QB - 1) / QB;
    prefill_block(nqb, &head, &qb);
    qb = nqb - 1 - qb;
    const int q0 = qb * QB + wv * 16 * NQ;                 // this wave's first row
    const int last = min(p.M, qb * QB + QB) - 1, nt = (p.p0 + last) / 64 + 1;
    const uint32_t range = (uint32_t)(p.p0 + p.M) * DH * 2;
    const __amdgpu_buffer_rsrc_t rk = buf_rsrc((const uint16_t*)p.kvc + kvc_index(p.g, p.seq, p.table, 0, head, 0), range);
    const __amdgpu_buffer_rsrc_t rv = buf_rsrc((const uint16_t*)p.kvc + kvc_index(p.g, p.seq, p.table, 1, head, 0), range);
    // queries: row q0 + 16 n + j, dimensions 32 kd + 8 grp .. + 7 (rows past the last one repeat it)
    u32x4 q[NQ][KD];
    int pos[NQ];
#pragma unroll
    for (int n = 0; n < NQ; ++n) {
        const int m = min(q0 + n * 16 + j, p.M - 1);
        pos[n] = p.p0 + m;
#pragma unroll
        for (int kd = 0; kd < KD; ++kd) {
            const int d = kd * 32 + grp * 8;
            q[n][kd] = d < DH ? *(const u32x4*)((const uint16_t*)p.q + (size_t)m * p.g.h + head * DH + d)
                              : u32x4{0u, 0u, 0u, 0u};
        }
    }
    const int wmin = p.p0 + min(q0, p.M - 1), wmax = p.p0 + min(q0 + 16 * NQ, p.M) - 1;   // (wave-uniform)
    u32x4 kr[KD], vr[4];
    const int d8 = j;                                       // values: dimensions 8 d8 .. + 7 of keys 4 grp .. + 3
    auto load_kv = [&](int it) {
        const int key0 = it * 64 + wv * 16;                 // this wave stages key tile wv
#pragma unroll
        for (int kd = 0; kd < KD; ++kd) {
            const int d = kd * 32 + grp * 8;
            kr[kd] = buf_load16<0>(rk, d < DH ? ((key0 + j) * DH + d) * 2 : kOutOfRange, 0);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
            vr[i] = buf_load16<0>(rv, d8 * 8 < DH ? ((key0 + grp * 4 + i) * DH + d8 * 8) * 2 : kOutOfRange, 0);
    };
    auto put_kv = [&](int buf) {
#pragma unroll
        for (int kd = 0; kd < KD; ++kd) kl[buf][(wv * KD + kd) * 64 + lane] = kr[kd];
        if (d8 * 8 < DH) {
            uint2* dst = (uint2*)(vl[buf] + ((d8 >> 1) * 2 + (wv >> 1)) * VS + grp * 16 + (d8 & 1) * 8) + (wv & 1);
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                dst[4 * c] = make_uint2(__builtin_amdgcn_perm(vr[1][c], vr[0][c], 0x05040100u),
                                        __builtin_amdgcn_perm(vr[3][c], vr[2][c], 0x05040100u));
                dst[4 * c + 2] = make_uint2(__builtin_amdgcn_perm(vr[1][c], vr[0][c], 0x07060302u),
                                            __builtin_amdgcn_perm(vr[3][c], vr[2][c], 0x07060302u));
            }
        }
    };
    // o, l: weighted values and weights against the reference ref; top: the
    // largest score so far; so: the own position's score, in the lane that holds it
    f32x4 o[NQ][DT];
    float ref[NQ], top[NQ], l[NQ], so[NQ];
#pragma unroll
    for (int n = 0; n < NQ; ++n) {
        ref[n] = top[n] = -1e30f;
        l[n] = so[n] = 0.f;
#pragma unroll
        for (int t = 0; t < DT; ++t) o[n][t] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    const float sl2 = p.g.attn_scale * 1.4426950408889634f;   // (the softmax runs in base 2)
    load_kv(0);
    put_kv(0);
    load_kv(1);
    __syncthreads();
    for (int it = 0; it < nt; ++it) {
        const int cur = it & 1, key0 = it * 64;
        if (key0 <= wmax) {
            f32x4 s[NQ][4];
#pragma unroll
            for (int n = 0; n < NQ; ++n)
#pragma unroll
                for (int t = 0; t < 4; ++t) s[n][t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int kd = 0; kd < KD; ++kd) {
                    const u32x4 kf = kl[cur][(t * KD + kd) * 64 + lane];
#pragma unroll
                    for (int n = 0; n < NQ; ++n) mfma_one<uint16_t>(kf, q[n][kd], s[n][t]);
                }
            u32x4 pr[NQ][2];
#pragma unroll
            for (int n = 0; n < NQ; ++n) {
                if (key0 + 63 >= wmin) {                    // keys at and behind the queries (wave-uniform)
#pragma unroll
                    for (int t = 0; t < 4; ++t)
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            const int d = key0 + t * 16 + grp * 4 + v - pos[n];
                            if (d == 0) so[n] = s[n][t][v];
                            if (d >= 0) s[n][t][v] = -INFINITY;
                        }
                }
                float m = -INFINITY;
#pragma unroll
                for (int t = 0; t < 4; ++t)
#pragma unroll
                    for (int v = 0; v < 4; ++v) m = fmaxf(m, s[n][t][v]);
                m = fmaxf(m, __shfl_xor(m, 16));
                m = fmaxf(m, __shfl_xor(m, 32)) * sl2;
                // the tile's maximum becomes the reference, or 2^-64 of the
                // largest weight so far: what lies below that does not show in
                // an fp16 output (o stays below 2^64 x 2^17 keys x 2^16)
                top[n] = fmaxf(top[n], m);
                const float rn = fmaxf(m, top[n] - 64.f), a = __builtin_amdgcn_exp2f(ref[n] - rn);
                ref[n] = rn;
                l[n] *= a;
#pragma unroll
                for (int t = 0; t < DT; ++t) o[n][t] *= a;
                // weights rounded to fp16, and summed as rounded
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        const f32x4& x = s[n][2 * h + (c >> 1)];
                        const int v = (c & 1) * 2;
                        const uint32_t w = pack_h2(__builtin_amdgcn_exp2f(fmaf(x[v], sl2, -rn)), __builtin_amdgcn_exp2f(fmaf(x[v + 1], sl2, -rn)));
                        pr[n][h][c] = w;
                        l[n] = __builtin_amdgcn_fdot2(__builtin_bit_cast(f16x2, w),
                                                      f16x2{(_Float16)1.f, (_Float16)1.f}, l[n], false);
                    }
            }
#pragma unroll
            for (int t = 0; t < DT; ++t)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const u32x4 vf = vl[cur][(t * 2 + h) * VS + lane];
#pragma unroll
                    for (int n = 0; n < NQ; ++n) mfma_one<uint16_t>(vf, pr[n][h], o[n][t]);
                }
        }
        put_kv(cur ^ 1);                                    // (its readers passed the last barrier)
        load_kv(it + 2);
        __syncthreads();
    }
#pragma unroll
    for (int n = 0; n < NQ; ++n) {
        float z = l[n], own = so[n];
        z += __shfl_xor(z, 16);
        z += __shfl_xor(z, 32);
        own += __shfl_xor(own, 16);
        own += __shfl_xor(own, 32);
        own *= sl2;
        const int m = q0 + n * 16 + j;
        if (m >= p.M) continue;
        // the own position joins in fp32
        const float big = fmaxf(ref[n], own), a = __builtin_amdgcn_exp2f(ref[n] - big), b = __builtin_amdgcn_exp2f(own - big);
        const float r = 1.0f / fmaf(z, a, b), ra = a * r, rb = b * r;
        const uint16_t* vo = (const uint16_t*)p.kvc + kvc_index(p.g, p.seq, p.table, 1, head, pos[n]) + grp * 4;
#pragma unroll
        for (int t = 0; t < DT; ++t) {
            const uint2 w = *(const uint2*)(vo + t * 16);
            const f16x2 lo = __builtin_bit_cast(f16x2, w.x), hi = __builtin_bit_cast(f16x2, w.y);
            const float v[4] = {(float)lo.x * rb, (float)lo.y * rb, (float)hi.x * rb, (float)hi.y * rb};
            *(uint2*)((uint16_t*)p.out + opd_elem<uint16_t>(m, head * DH + t * 16 + grp * 4, p.g.h)) =
                make_uint2(pack_h2(fmaf(o[n][t][0], ra, v[0]), fmaf(o[n][t][1], ra, v[1])),
                           pack_h2(fmaf(o[n][t][2], ra, v[2]), fmaf(o[n][t][3], ra, v[3])));
        }
    }
}

template <int DH>
static hipError_t launch_attn_dh(const PrefillAttn& p, hipStream_t st) {
    // 32 queries per wave read each key tile half as often but leave half the
    // workgroups: they pay where those still are three per CU and the keys go
    // far back.  us per launch, 32 / 16 queries, 2048 rows behind 0 / 4096 / 8192
    // positions: 55 heads of 96 (880 workgroups of 128 queries) 137 / 137, 415 / 435,
    // 666 / 728; 16 heads of 128 (256) 66 / 64, 204 / 202, 310 / 304; 16 of 64 47 / 42,
    // 133 / 125, 219 / 198; 8 of 96 (128) 56 / 40, 155 / 112, 253 / 183.
    const int n2 = p.g.H * ((p.M + 127) / 128), n1 = p.g.H * ((p.M + 63) / 64);
    if (n2 >= 768 && p.p0 >= 4096)
        hipLaunchKernelGGL((k_prefill_attn<DH, 2>), dim3(n2), dim3(256), 0, st, p);
    else
        hipLaunchKernelGGL((k_prefill_attn<DH, 1>), dim3(n1), dim3(256), 0, st, p);
    return hipGetLastError();
}

hipError_t launch_prefill_attn(const PrefillAttn& p, hipStream_t st) {
    switch (p.g.dh) {
        case 16: return launch_attn_dh<16>(p, st);
        case 32: return launch_attn_dh<32>(p, st);
        case 64: return launch_attn_dh<64>(p, st);
        case 96: return launch_attn_dh<96>(p, st);
        case 128: return launch_attn_dh<128>(p, st);
    }
    return hipErrorInvalidValue;
}

template <typename WT, int EPI, int NMAT>
static hipError_t allow_lds() {
    const hipError_t e = hipFuncSetAttribute((const void*)k_prefill_tile<WT, EPI, NMAT>,
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)kTileLds);
    return e != hipSuccess ? e
                           : hipFuncSetAttribute((const void*)k_prefill_slice<WT, EPI, NMAT>,
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)kSliceLds);
}

hipError_t prefill_prepare() {
    hipError_t e;
    if ((e = allow_lds<uint16_t, EPI_QKV, 1>()) != hipSuccess || (e = allow_lds<uint16_t, EPI_RESID, 1>()) != hipSuccess ||
        (e = allow_lds<uint16_t, EPI_SWIGLU, 2>()) != hipSuccess || (e = allow_lds<float, EPI_QKV, 1>()) != hipSuccess ||
        (e = allow_lds<float, EPI_RESID, 1>()) != hipSuccess)
        return e;
    return allow_lds<float, EPI_SWIGLU, 2>();
}

template <typename WT>
static hipError_t launch_epi(const PrefillGemm& p, int epi, hipStream_t st) {
    switch (epi) {
        case EPI_QKV: return launch_shape<WT, EPI_QKV, 1>(p, st);
        case EPI_RESID: return launch_shape<WT, EPI_RESID, 1>(p, st);
        case EPI_SWIGLU: return launch_shape<WT, EPI_SWIGLU, 2>(p, st);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_prefill_gemm(const PrefillGemm& p, int epi, bool bf16, hipStream_t st) {
    if (p.M < 1 || p.tiles < 1 || p.M > kPrefillRowsMax) return hipErrorInvalidValue;
    return bf16 ? launch_epi<uint16_t>(p, epi, st) : launch_epi<float>(p, epi, st);
}

// ---------------------------------------------------------------------------
// H^(0) = E[x] of the prompt rows, with the pass buffers of their first block:
// one 16-column tile per thread at a time
// ---------------------------------------------------------------------------
template <typename WT>
__global__ void __launch_bounds__(256) k_prefill_embed(Geo g, const int32_t* tok, const WT* E, float* X, PassBuf pb) {
    const int m = blockIdx.x;
    const WT* e = E + (size_t)tok[m] * g.h;
    for (int t = threadIdx.x; t < g.ssq_tiles; t += blockDim.x) {
        float v[16];
#pragma unroll
        for (int c = 0; c < 16; ++c)
            v[c] = sizeof(WT) == 2 ? bf2f(((const uint16_t*)e)[t * 16 + c]) : ((const float*)e)[t * 16 + c];
#pragma unroll
        for (int c = 0; c < 16; c += 4)
            *(f32x4*)(X + prefill_state(m, t * 16 + c, g.h)) = f32x4{v[c], v[c + 1], v[c + 2], v[c + 3]};
        store_act16<WT>(pb.XB, m, t * 16, g.h, v);
        pb.SSQR[(size_t)m * g.ssq_tiles + t] = ssq16(v);
    }
}

hipError_t launch_prefill_embed(const Geo& g, const int32_t* tok, int M, const void* E, bool bf16, float* X,
                                PassBuf pb, hipStream_t st) {
    if (bf16)
        hipLaunchKernelGGL(k_prefill_embed<uint16_t>, dim3(M), dim3(256), 0, st, g, tok, (const uint16_t*)E, X, pb);
    else
        hipLaunchKernelGGL(k_prefill_embed<float>, dim3(M), dim3(256), 0, st, g, tok, (const float*)E, X, pb);
    return hipGetLastError();
}

// One row of a prompt pass's state, row-major (the prompt's last position goes on as a single row)
__global__ void __launch_bounds__(256) k_prefill_row(Geo g, const float* X, int m, float* out) {
    const int k = blockIdx.x * 256 + threadIdx.x;
    if (k < g.h) out[k] = X[prefill_state(m, k & ~3, g.h) + (k & 3)];
}

hipError_t launch_prefill_row(const Geo& g, const float* X, int m, float* out, hipStream_t st) {
    hipLaunchKernelGGL(k_prefill_row, dim3((g.h + 255) / 256), dim3(256), 0, st, g, X, m, out);
    return hipGetLastError();
}

}  // namespace ls
