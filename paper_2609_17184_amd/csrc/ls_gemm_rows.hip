// Weight-streaming GEMM for decode passes of 17 to 64 rows (handles with more
// than 16 branch slots).
//
// A launch streams one packed matrix once and multiplies it with up to NT row
// tiles of 16 activations, so it is bound by HBM as long as the activations,
// which every workgroup needs, come cheaply: they lie in MFMA operand order
// (opd_elem), 1 KB of consecutive bytes per fragment, and come from the L2.
//
// A workgroup is four waves that split k, for FT feature tiles (of each
// matrix) and all rows; each wave loads both operands straight into
// registers, PF steps ahead, with no barrier until the partials meet in LDS,
// where they are summed in wave order.  Row tiles past the live ones are neither
// read nor multiplied.  A row's result depends on nothing but its own values:
// the split of k is fixed by K, and every row tile is summed in the same order
// whatever the depth.
//
// Measured by kernel trace inside a decode, us per launch (TB/s of weights).
// Raven width, 8 live rows / 24 / 48: QKV 29 (5.7) / 35 (4.8) / 46, O 16 (3.4) /
// 21 (2.6) / 28, gate/up 62 (6.1) / 77 (4.9) / 108, down 48 (3.9) / 63 (3.0) / 80,
// LM head at 8 to 24 rows 108 (6.4).  h = 2048, F = 5120, 24 / 48: QKV 11.4 / 15.5,
// O 6.6 / 8.3, gate/up 14.2 / 17.0, down 11.4 / 14.9.  Bound by HBM and the
// loads in flight (a weight fragment takes 3.4 us to arrive under load); down
// and O (330 workgroups for 256 CUs) by the ragged last CUs; past 32 rows by the
// activations, four fragments for one or two of weights.
#include "ls_opd_dev.h"

namespace ls {

// The wave's share of k for NT row tiles, PF steps ahead: its partial of the
// workgroup's tile into part[row][LD].  `between` runs under the first loads.
template <typename WT, int NMAT, int FT, int NT, int PF, int LD, typename F>
__device__ __forceinline__ void rows_stream(const __amdgpu_buffer_rsrc_t (&rw)[FT], __amdgpu_buffer_rsrc_t ra, int ns, int k0,
                                            int n, int ntl, float* part, F between) {
    const int lane = threadIdx.x & 63, j = lane & 15, grp = lane >> 4, vw = lane * 16;
    u32x4 w[PF][FT][NMAT], x[PF][NT];
    // (steps past the wave's share are loaded but not used, row tiles past the live ones read as zeros)
    auto load = [&](int i, u32x4 (&r)[FT][NMAT], u32x4 (&y)[NT]) {
#pragma unroll
        for (int f = 0; f < FT; ++f)
#pragma unroll
            for (int q = 0; q < NMAT; ++q) r[f][q] = buf_load16<2>(rw[f], vw, ((k0 + i) * NMAT + q) * 1024);
#pragma unroll
        for (int t = 0; t < NT; ++t) y[t] = buf_load16<0>(ra, t < ntl ? vw : kOutOfRange, (t * ns + k0 + i) * 1024);
    };
    f32x4 acc[FT][NMAT][NT];
#pragma unroll
    for (int f = 0; f < FT; ++f)
#pragma unroll
        for (int q = 0; q < NMAT; ++q)
#pragma unroll
            for (int t = 0; t < NT; ++t) acc[f][q][t] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto mul = [&](const u32x4 (&r)[FT][NMAT], const u32x4 (&y)[NT]) {
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            if (t >= ntl) break;
#pragma unroll
            for (int f = 0; f < FT; ++f)
#pragma unroll
                for (int q = 0; q < NMAT; ++q) mfma_one<WT>(r[f][q], y[t], acc[f][q][t]);
        }
    };
#pragma unroll
    for (int u = 0; u < PF; ++u) load(u, w[u], x[u]);
    between();
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
    for (int t = 0; t < NT; ++t) {
        if (t >= ntl) break;
#pragma unroll
        for (int f = 0; f < FT; ++f)
#pragma unroll
            for (int q = 0; q < NMAT; ++q)
                *(f32x4*)(part + (size_t)(t * 16 + j) * LD + (q * FT + f) * 16 + grp * 4) = acc[f][q][t];
    }
}

// k steps ahead for NT live row tiles
constexpr int rows_depth(bool deep, int nt) { return nt <= 2 || deep ? 6 : 4; }

template <typename WT, int EPI, int NMAT, int FT, int NT, bool DEEP>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) k_gemm_rows(GemmParams p) {
    constexpr int BN = FT * 16, LD = NMAT * BN + 4, ROWS = 16 * NT;
    constexpr int UI = (ROWS * FT * 4 + 255) / 256;       // epilogue units per thread
    __shared__ __align__(16) float part[4 * ROWS * LD];
    __shared__ float rinv[ROWS];
    __shared__ int xr[ROWS], pos[ROWS], slot[ROWS], seq[ROWS], dep[ROWS];
    const int M = min(ld_uniform(p.nrows), ROWS);
    if (M <= 0) return;
    const int tid = threadIdx.x, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ntl = (M + 15) / 16, t0 = blockIdx.x * FT;
    const int ns = p.K / WTraits<WT>::KSTEP, k0 = ns * wv / 4, n = ns * (wv + 1) / 4 - k0;
    const size_t tb = (size_t)ns * NMAT * 1024;
    __amdgpu_buffer_rsrc_t rw[FT];
#pragma unroll
    for (int f = 0; f < FT; ++f) {
        const bool ok = t0 + f < p.tiles;
        rw[f] = buf_rsrc((const char*)p.Wp + (ok ? (size_t)(t0 + f) * tb : 0), ok ? (uint32_t)tb : 0u);
    }
    const __amdgpu_buffer_rsrc_t ra = buf_rsrc(EPI == EPI_RESID ? p.abuf : p.XB, (uint32_t)ntl * ns * 1024);
    // a thread's units of the epilogue: four features (quarter q4) of one row of one tile
    const int q4 = tid & 3;
    const int tpd = p.g.dh / kTile, half = p.g.dh / 2, tph = p.g.h / kTile;
    f32x4 pre[UI][2];
    auto between = [&]() __attribute__((always_inline)) {
        // the rows' 1/rms (16 lanes per row) and epilogue fields, then the units' operands
        if constexpr (EPI != EPI_RESID) {
            const int T = p.g.ssq_tiles;
            for (int m = tid >> 4; m < M; m += 16) {
                float s = 0.f;
#pragma unroll 8
                for (int t = tid & 15; t < T; t += 16) s += p.SSQR[(size_t)m * T + t];
                s = group_sum<16>(s);
                if ((tid & 15) == 0) rinv[m] = 1.0f / sqrtf(s / (float)p.g.h + p.g.eps);
            }
        }
        if (EPI == EPI_RESID || EPI == EPI_QKV) {
            if (tid < M) {
                const Row& r = p.rows[tid];
                xr[tid] = r.xrow;
                pos[tid] = r.pos;
                slot[tid] = r.slot;
                seq[tid] = r.seq;
                dep[tid] = r.depth;
            }
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < UI; ++i) {
            const int u = (i * 256 + tid) >> 2, c = u % FT, m = u / FT, t = t0 + c;
            pre[i][0] = pre[i][1] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (m >= M || t >= p.tiles) continue;
            if (EPI == EPI_RESID) pre[i][0] = *(const f32x4*)(p.X + (size_t)xr[m] * p.g.h + t * kTile + q4 * 4);
            if (EPI == EPI_QKV && t / tph < 2) {
                const int sub = t % tph % tpd;
                const f32x4* rp = (const f32x4*)(p.rope + ((size_t)pos[m] * half + sub * 8 + (q4 & 1) * 4) * 2);
                pre[i][0] = rp[0];
                pre[i][1] = rp[1];
            }
        }
    };
    float* const mine = part + (size_t)wv * ROWS * LD;
    if (NT == 2 || ntl <= 2)
        rows_stream<WT, NMAT, FT, 2, rows_depth(DEEP, 2), LD>(rw, ra, ns, k0, n, ntl, mine, between);
    else
        rows_stream<WT, NMAT, FT, NT, rows_depth(DEEP, NT), LD>(rw, ra, ns, k0, n, ntl, mine, between);
    __syncthreads();
    auto sum = [&](int row, int col) {
        f32x4 v = *(const f32x4*)(part + (size_t)row * LD + col);
#pragma unroll
        for (int k = 1; k < 4; ++k) v += *(const f32x4*)(part + (size_t)(k * ROWS + row) * LD + col);
        return v;
    };
    auto put_act = [&](void* base, int m, int k, int K, const f32x4& v) {   // four columns in operand order
        const size_t e = opd_elem<WT>(m, k, K);
        if constexpr (sizeof(WT) == 2)
            *(uint2*)((uint16_t*)base + e) = make_uint2(pack_h2(v[0], v[1]), pack_h2(v[2], v[3]));
        else
            *(f32x4*)((float*)base + e) = v;
    };
#pragma unroll
    for (int ui = 0; ui < UI; ++ui) {
        // (the four lanes of a row's tile take the same branches)
        const int u = (ui * 256 + tid) >> 2, c = u % FT, m = u / FT, t = t0 + c, col = t * kTile + q4 * 4;
        if (m >= M || t >= p.tiles) continue;
        f32x4 o = sum(m, c * 16 + q4 * 4);
        if constexpr (EPI == EPI_RESID) {
            o += pre[ui][0];
            *(f32x4*)(p.X + (size_t)xr[m] * p.g.h + col) = o;
            put_act(p.XBout, m, col, p.g.h, o);
            const float sq = group_sum<4>(fmaf(o[3], o[3], fmaf(o[2], o[2], fmaf(o[1], o[1], o[0] * o[0]))));
            if (q4 == 0) p.SSQRout[(size_t)m * p.g.ssq_tiles + t] = sq;
        } else if constexpr (EPI == EPI_SWIGLU) {
            const f32x4 up = sum(m, BN + c * 16 + q4 * 4);
            const float r = rinv[m];
            f32x4 a;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const float gt = o[v] * r;
                a[v] = gt / (1.0f + expf(-gt)) * (up[v] * r);
            }
            put_act(p.act, m, col, p.N_mat, a);
        } else if constexpr (EPI == EPI_QKV) {
            // quarters 0, 1 hold the first halves of eight RoPE pairs, quarters 2, 3 their partners
            const int mat = t / tph, lt = t % tph, head = lt / tpd, i0 = lt % tpd * 8 + (q4 & 1) * 4;
            o *= rinv[m];
            if (mat < 2) {
                const f32x4 a = pre[ui][0], b = pre[ui][1];
                const float cs[4] = {a[0], a[2], b[0], b[2]}, sn[4] = {a[1], a[3], b[1], b[3]};
                const float sign = q4 < 2 ? -1.f : 1.f;
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const float other = dpp_mov<0x4E>(o[v]);      // quad_perm [2,3,0,1]
                    o[v] = o[v] * cs[v] + sign * (other * sn[v]);
                }
            }
            const int d = i0 + (q4 >> 1) * half;
            if (mat == 0) {
                *(f32x4*)(p.qout + (size_t)m * p.g.h + head * p.g.dh + d) = o;
            } else {
                const int tab = kv_table(p.g, p.stack, p.layer, dep[m]);
                WT* dst = (slot[m] >= 0 ? (WT*)p.kvs + kvs_index(p.g, slot[m], tab, mat - 1) + head * p.g.dh
                                        : (WT*)p.kvc + kvc_index(p.g, seq[m], tab, mat - 1, head, pos[m])) + d;
                if constexpr (sizeof(WT) == 2)
                    *(uint2*)dst = make_uint2(pack_h2(o[0], o[1]), pack_h2(o[2], o[3]));
                else
                    *(f32x4*)dst = o;
            }
        } else {
            o *= rinv[m];
            // the tile's maximum over its live columns, ties to the lowest id
            float best = -INFINITY;
            int bi = -1;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                if (col + v >= p.N_mat) continue;
                p.logits[(size_t)m * p.N_mat + col + v] = o[v];
                if (!(fabsf(o[v]) <= 3.0e38f)) atomicOr(p.err, 1);
                if (bi < 0 || o[v] > best) {
                    best = o[v];
                    bi = col + v;
                }
            }
#pragma unroll
            for (int s = 1; s <= 2; s <<= 1) {
                const float ob = __shfl_xor(best, s);
                const int oi = __shfl_xor(bi, s);
                if (oi >= 0 && (bi < 0 || ob > best || (ob == best && oi < bi))) {
                    best = ob;
                    bi = oi;
                }
            }
            if (q4 == 0) {
                p.tmax[(size_t)m * p.tiles + t] = best;
                p.targ[(size_t)m * p.tiles + t] = bi;
            }
        }
    }
}

template <typename WT, int EPI, int NMAT, int FT, int NT>
static hipError_t launch_ft(const GemmParams& p, hipStream_t st) {
    GemmParams q = p;
    void* args[] = {(void*)&q};
    // Gate/up reads two weight fragments a step and so has the most to gain
    // from six steps ahead instead of four behind more than two row tiles
    // (two row tiles always have six), at the registers of the third workgroup
    // of a CU.  33 to 64 live rows, fp16, workgroups / k steps: 130 / 64 13.2 ->
    // 10.2 us, 272 / 64 19.0 -> 16.7, 384 / 128 43.7 -> 35.8, 480 / 192 63.8 -> 53.7;
    // up to 32 rows the same time.  Past 512 workgroups those rows miss the
    // third one (770 / 128: 47.6 -> 48.0 us at 24 rows, 65.3 -> 56.9 at 40), and with
    // shorter shares the first loads weigh more (276 / 48: 16.1 -> 17.2).  fp32
    // steps hold half of the columns: 272 / 96 27.0 -> 27.7 us, 304 / 128 34.2 ->
    // 36.8, 368 / 176 48.2 -> 44.2, 432 / 256 80.3 -> 78.7.  (QKV, O and down lose
    // up to 7 % so and gain at most 5 %; 10 or 16 steps ahead for two row tiles lose 10 %
    // of all of them.)
    const int wgs = (p.tiles + FT - 1) / FT, ns = p.K / WTraits<WT>::KSTEP;
    const void* f = (const void*)k_gemm_rows<WT, EPI, NMAT, FT, NT, false>;
    if constexpr (NMAT == 2 && NT == 4)
        if (wgs <= 512 && ns >= (sizeof(WT) == 2 ? 64 : 160)) f = (const void*)k_gemm_rows<WT, EPI, NMAT, FT, NT, true>;
    return ls_launch(f, dim3(wgs), dim3(256), args, 0, st);
}

template <typename WT, int EPI, int NMAT, int NT>
static hipError_t launch_nt(const GemmParams& p, hipStream_t st) {
    // two feature tiles per workgroup where that still leaves three workgroups
    // per two CUs: the rows are read half as often
    if (NMAT == 1 && p.tiles >= 768) return launch_ft<WT, EPI, NMAT, NMAT == 1 ? 2 : 1, NT>(p, st);
    return launch_ft<WT, EPI, NMAT, 1, NT>(p, st);
}

template <typename WT, int NT>
static hipError_t launch_epi(const GemmParams& p, int epi, hipStream_t st) {
    switch (epi) {
        case EPI_QKV: return launch_nt<WT, EPI_QKV, 1, NT>(p, st);
        case EPI_RESID: return launch_nt<WT, EPI_RESID, 1, NT>(p, st);
        case EPI_SWIGLU: return launch_nt<WT, EPI_SWIGLU, 2, NT>(p, st);
        case EPI_LOGITS: return launch_nt<WT, EPI_LOGITS, 1, NT>(p, st);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_gemm_rows(const GemmParams& p, int epi, bool bf16, int rows_cap, hipStream_t st) {
    if (rows_cap > kMaxRows) return hipErrorInvalidValue;
    if (rows_cap <= 32) return bf16 ? launch_epi<uint16_t, 2>(p, epi, st) : launch_epi<float, 2>(p, epi, st);
    return bf16 ? launch_epi<uint16_t, 4>(p, epi, st) : launch_epi<float, 4>(p, epi, st);
}

}  // namespace ls
