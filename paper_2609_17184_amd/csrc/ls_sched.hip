// Device-resident LoopSpec scheduler and the kernels that feed it.
//
// The scheduler carries out the bookkeeping of Alg. 1 between two batched
// recurrent passes, entirely on the GPU so a whole decode step can be replayed
// as one graph with no host round trip:
//   * every branch of the pass advanced one depth;
//   * the root that reached R commits the token chosen by Verify (readout
//     kernels decided it) and the set is re-rooted at the chosen child
//     (Reroot: keep c* and its descendants, free the rest); its KV for every
//     depth moves to the committed cache at its position;
//   * a branch that reached d1 spawns a child on X || x1; a branch that reached
//     d2 with an open gate spawns a second child on X || x2 (Spawn);
//   * the row lists of the next pass are rebuilt: every live branch (B rows),
//     the branches whose next depth is a readout depth (C rows), and the
//     freshly spawned branches (P rows, for prelude blocks).
// Verification and re-rooting are applied before the proposals of the same
// step; a child spawned this step inside a pruned subtree would be dropped in
// the same step, so skipping it gives the same branch set (Alg. 1 order).
#include "ls_sched.h"

#include <algorithm>

namespace ls {

// ---------------------------------------------------------------------------
// scheduler: one wave, lane x for slot x (the tree holds at most 64 branches)
//
// The bookkeeping is a chain of small dependent reads and writes, so what
// bounds it is the latency of the tables: they come into LDS in one round trip
// at the start (every load of the launch is issued before any is waited for)
// and leave in one at the end.  The steps of Alg. 1 run in every lane alike (a
// table entry that all lanes write gets the same value from each); what ranges
// over slots -- pruning, free slots, the row lists of the next pass -- runs one
// slot per lane.  With one thread on the tables in memory a step took 10 us
// for one sequence and up to 73 us for a tree of 28 slots.
// ---------------------------------------------------------------------------
static_assert(kMaxRows <= 64, "a slot per lane");

struct SchedTree {
    int active[64], seq[64], pos[64], tok[64], depth[64], parent[64], c1[64], c2[64], x1[64], x2[64], gate[64];
    int root[64], tdone[64], ncommit[64], target[64], state[64], last_tok[64], last_src[64];
    int r_slot[64], r_seq[64], r_pos[64], r_depth[64], ro_tok[64], ro_aux[64];   // readout rows of the step
    int js[128];
};

// LDS written by some lanes is read by others after this
__device__ __forceinline__ void lds_sync() { __syncthreads(); }

__device__ __forceinline__ int alloc_slot(const SchedTree& t, int S, int lane) {
    const unsigned long long m = __ballot(lane < S && !t.active[lane]);
    return m ? (int)__builtin_ctzll(m) : -1;
}

__device__ __forceinline__ void init_slot(SchedTree& t, int c, int q, int pos, int tok, int parent) {
    t.active[c] = 1;
    t.seq[c] = q;
    t.pos[c] = pos;
    t.tok[c] = tok;
    t.depth[c] = 0;
    t.parent[c] = parent;
    t.c1[c] = -1;
    t.c2[c] = -1;
    t.x1[c] = -1;
    t.x2[c] = -1;
    t.gate[c] = 0;
    lds_sync();
}

__device__ __forceinline__ bool in_subtree(const SchedTree& t, int S, int x, int c) {
    if (c < 0) return false;
    for (int k = 0; x >= 0 && k <= S; ++k) {
        if (x == c) return true;
        x = t.parent[x];
    }
    return false;
}

// Row of slot x at `depth` into *r
__device__ __forceinline__ void put_row(const SchedTree& t, int x, int depth, int xrow, Row* r, int32_t* err) {
    const int tdone = t.tdone[t.seq[x]], pos = t.pos[x];
    r->xrow = xrow;
    r->slot = x;
    r->seq = t.seq[x];
    r->pos = pos;
    r->depth = depth;
    r->tdone = tdone;
    r->src = x;                                        // copy source for readout rows
    r->pad = 0;
    int y = t.parent[x];
    for (int p = pos - 1; p >= tdone; --p) {
        if (p - tdone >= kChainMax || y < 0) {         // inconsistent tree: never index out of range
            atomicOr(err, ERR_SLOTS);
            break;
        }
        r->anc[p - tdone] = y;
        y = t.parent[y];
    }
}

__device__ static bool is_readout(const Sched& s, int mode, int d) {
    if (mode == MODE_FORCED) return d >= 1 && d <= s.R;
    if (mode == MODE_VANILLA) return d == s.R;
    return d == s.d1 || (s.d2 > 0 && d == s.d2) || d == s.R;
}

__global__ void __launch_bounds__(64) k_sched(Sched s, int op, int op_seq, int op_pos, const int32_t* op_tok) {
    __shared__ SchedTree t;
    __shared__ long long st[ST_N];                     // what this step adds to the statistics
    const int lane = threadIdx.x, S = s.g.S, Q = s.max_seqs, ctx = s.g.max_ctx;
    // ---- the tables (rows past the lists' lengths are read and not used)
    const int mode = *s.mode, nB0 = *s.nB, nC0 = *s.nC;
    const int tok0 = op == OP_INIT ? op_tok[0] : -1;
    int32_t* const slot_g[] = {s.s_active, s.s_seq, s.s_pos, s.s_tok, s.s_depth, s.s_parent,
                               s.s_c1, s.s_c2, s.s_x1, s.s_x2, s.s_gate};
    int* const slot_l[] = {t.active, t.seq, t.pos, t.tok, t.depth, t.parent, t.c1, t.c2, t.x1, t.x2, t.gate};
    int32_t* const seq_g[] = {s.q_root, s.q_tdone, s.q_ncommit, s.q_target, s.q_state, s.q_last_tok, s.q_last_src};
    int* const seq_l[] = {t.root, t.tdone, t.ncommit, t.target, t.state, t.last_tok, t.last_src};
    int v[11], w[7], b_slot = 0, c[6] = {0, 0, 0, 0, 0, 0};
    const bool has_slot = lane < S, has_seq = lane < Q;
#pragma unroll
    for (int i = 0; i < 11; ++i) v[i] = has_slot ? slot_g[i][lane] : 0;
#pragma unroll
    for (int i = 0; i < 7; ++i) w[i] = has_seq ? seq_g[i][lane] : 0;
    if (op == OP_STEP && has_slot) {
        b_slot = s.rowsB[lane].slot;
        const Row& r = s.rowsC[lane];
        c[0] = r.slot;
        c[1] = r.seq;
        c[2] = r.pos;
        c[3] = r.depth;
        c[4] = s.ro_tok[lane];
        c[5] = s.ro_aux[lane];
    }
#pragma unroll
    for (int i = 0; i < 11; ++i) slot_l[i][lane] = v[i];
#pragma unroll
    for (int i = 0; i < 7; ++i) seq_l[i][lane] = w[i];
    t.r_slot[lane] = c[0];
    t.r_seq[lane] = c[1];
    t.r_pos[lane] = c[2];
    t.r_depth[lane] = c[3];
    t.ro_tok[lane] = c[4];
    t.ro_aux[lane] = c[5];
    for (int i = lane; i < ST_N; i += 64) st[i] = 0;
    lds_sync();
    int njc = 0, njs = 0;
    // (all lanes write the same values, so a statement's reads and writes need no order between lanes)
    auto spawn = [&](int slot, int tok) {
        t.js[2 * njs] = slot;
        t.js[2 * njs + 1] = tok;
        ++njs;
    };
    auto error = [&](int bit) {
        if (lane == 0) atomicOr(s.err, bit);
    };
    // statistics: lane 0 keeps them
    auto count = [&](int k, long long n) {
        if (lane == 0) st[k] += n;
    };

    if (op == OP_STEP) {
        const int nB = min(nB0, S), nC = min(nC0, S);
        if (lane < nB) t.depth[b_slot] += 1;           // (the rows of a pass are distinct slots)
        if (nB > 0) {
            count(ST_STEPS, 1);
            count(ST_SUM_M, nB);
            count(ST_HIST + (nB < 64 ? nB : 64), 1);
        }
        t.last_tok[lane] = -1;
        t.last_src[lane] = -1;
        lds_sync();
        // ---- gate statistics: Alg. 1 evaluates the gate of every branch that
        //      reaches d2 this step, before the root's verification prunes any
        if (mode == MODE_LOOPSPEC && s.d2 > 0) {
            const bool at = lane < nC && t.r_depth[lane] == s.d2;
            count(ST_GATE_EVAL, __popcll(__ballot(at)));
            count(ST_GATE_OPEN, __popcll(__ballot(at && t.ro_aux[lane] != 0)));
        }
        // ---- roots at depth R: commit, re-root, prune -----------------------
        for (int i = 0; i < nC; ++i) {
            if (t.r_depth[i] != s.R) continue;
            const int q = t.r_seq[i], b = t.r_slot[i], np = t.r_pos[i] + 1;
            int tok = t.ro_tok[i], src = t.ro_aux[i];
            if (mode == MODE_FORCED) {
                tok = s.forced[(size_t)q * ctx + np];
                src = 0;
            } else if (mode == MODE_VANILLA) {
                src = 0;
            }
            if (lane == 0) {
                s.Y[(size_t)q * ctx + np] = tok;
                s.jc[3 * njc] = q;
                s.jc[3 * njc + 1] = b;
                s.jc[3 * njc + 2] = np - 1;
            }
            ++njc;
            const int nc = t.ncommit[q] + 1;
            t.ncommit[q] = nc;
            t.last_tok[q] = tok;
            t.last_src[q] = src;
            count(ST_COMMITTED, 1);
            if (mode == MODE_LOOPSPEC) count(src == 1 ? ST_ACC1 : src == 2 ? ST_ACC2 : ST_RESTART, 1);
            // greedy: TV between one-hot readouts is the argmax mismatch (the
            // argmax at d2 is kept in x2 whether or not its branch was
            // spawned; the sampled readout adds its TV sums itself)
            if (mode == MODE_LOOPSPEC && s.greedy && t.x1[b] >= 0) {
                const int x1 = t.x1[b], a2 = t.x2[b] >= 0 ? t.x2[b] : x1;
                count(ST_TVN, 1);
                if (x1 != tok) count(ST_TV1, 1LL << 32);
                if (s.d2 > 0 && a2 != tok) count(ST_TV2, 1LL << 32);
            }
            int k = src == 1 ? t.c1[b] : src == 2 ? t.c2[b] : -1;
            const bool drop = has_slot && t.active[lane] && t.seq[lane] == q && !in_subtree(t, S, lane, k);
            lds_sync();
            if (drop) t.active[lane] = 0;
            t.tdone[q] = np;
            lds_sync();
            if (np >= ctx - 1) {                       // no room for another position
                error(ERR_CTX);
                t.state[q] = SEQ_PAUSED;
                t.root[q] = -1;
                if (has_slot && t.seq[lane] == q) t.active[lane] = 0;
                lds_sync();
                continue;
            }
            if (k < 0) {
                k = alloc_slot(t, S, lane);
                if (k < 0) {                           // cannot happen: the old root was just freed
                    error(ERR_SLOTS);
                    t.state[q] = SEQ_PAUSED;
                    t.root[q] = -1;
                    lds_sync();
                    continue;
                }
                init_slot(t, k, q, np, tok, -1);
                spawn(k, tok);
            }
            t.parent[k] = -1;
            t.root[q] = k;
            if (nc >= t.target[q]) t.state[q] = SEQ_PAUSED;
            lds_sync();
        }
        // ---- proposals at d1 / d2 -----------------------------------------------
        if (mode == MODE_LOOPSPEC) {
            for (int i = 0; i < nC; ++i) {
                const int b = t.r_slot[i], q = t.r_seq[i], pos = t.r_pos[i], dep = t.r_depth[i];
                // the branch must still hold this slot: a slot pruned above may
                // already carry a new root (depth 0) of the same step.  A
                // sequence that reached its commit target in this step still
                // records its drafts (it resumes from this tree on the next
                // call); one whose tree was dropped has no active slot left.
                if (!t.active[b] || t.seq[b] != q || t.pos[b] != pos || t.depth[b] != dep || t.root[q] < 0) continue;
                const int x = t.ro_tok[i];
                if (dep == s.d1) {
                    t.x1[b] = x;
                    t.c2[b] = -1;
                    t.gate[b] = 0;
                    const int k = pos + 1 < ctx - 1 ? alloc_slot(t, S, lane) : -1;
                    t.c1[b] = k;
                    lds_sync();
                    if (k < 0) {
                        count(ST_REFUSED, 1);
                        continue;
                    }
                    init_slot(t, k, q, pos + 1, x, b);
                    spawn(k, x);
                } else if (s.d2 > 0 && dep == s.d2) {
                    if (s.greedy) t.x2[b] = x;         // verification reads it only with the gate open
                    lds_sync();
                    if (!t.ro_aux[i]) continue;
                    const int k = pos + 1 < ctx - 1 ? alloc_slot(t, S, lane) : -1;
                    if (k < 0) {                       // no room: the gate stays closed
                        count(ST_REFUSED, 1);
                        continue;
                    }
                    t.gate[b] = 1;
                    t.x2[b] = x;
                    t.c2[b] = k;
                    init_slot(t, k, q, pos + 1, x, b);
                    spawn(k, x);
                }
            }
        }
    } else if (op == OP_RESET) {
        // new proposal depths: drop every speculative branch of the sequence
        // and its root's drafts.  A root below the new d1 keeps the depths it
        // has computed (they do not depend on d1, d2); one at or past it
        // restarts at depth 0 from its embedding, so that it drafts at the new
        // d1 (its hidden states and slot keys / values are recomputed)
        const int q = op_seq, r = t.root[q];
        if (r >= 0) {
            if (has_slot && lane != r && t.active[lane] && t.seq[lane] == q) t.active[lane] = 0;
            const int depth = t.depth[r], pos = t.pos[r], tok = t.tok[r];
            lds_sync();
            init_slot(t, r, q, pos, tok, -1);
            if (depth < s.d1)
                t.depth[r] = depth;
            else
                spawn(r, tok);
        }
    } else if (op == OP_INIT) {
        const int q = op_seq, n = op_pos;
        if (has_slot && t.seq[lane] == q) t.active[lane] = 0;
        lds_sync();
        const int k = alloc_slot(t, S, lane);
        if (k < 0) {
            error(ERR_SLOTS);
        } else {
            init_slot(t, k, q, n, tok0, -1);
            t.root[q] = k;
            t.tdone[q] = n;
            t.ncommit[q] = 1;
            t.state[q] = SEQ_PAUSED;
            if (lane == 0) s.Y[(size_t)q * ctx + n] = tok0;
            spawn(k, tok0);
        }
    }
    lds_sync();

    // ---- next pass: rows of every live branch, grouped by sequence, slots ascending
    const int q = has_slot ? t.seq[lane] : -1;
    const bool live = has_slot && t.active[lane] && q >= 0 && q < Q && t.state[q] == SEQ_LIVE;
    const int dn = has_slot ? t.depth[lane] + 1 : 0;
    const bool ro = live && is_readout(s, mode, dn);
    const unsigned long long below = (1ull << lane) - 1;
    int nB = 0, nC = 0, ib = 0, ic = 0;
    for (int k = 0; k < Q; ++k) {
        const unsigned long long mb = __ballot(live && q == k), mc = __ballot(ro && q == k);
        if (q == k) {
            ib = nB + __popcll(mb & below);
            ic = nC + __popcll(mc & below);
        }
        nB += __popcll(mb);
        nC += __popcll(mc);
    }
    // steps until a live branch reads out: to its next readout depth, at or past the next pass's
    int quiet = 0x7FFFFFFF;
    if (live)
        quiet = mode == MODE_FORCED ? 0
                                    : (mode == MODE_VANILLA || dn > (s.d2 > 0 ? s.d2 : s.d1) ? s.R : dn <= s.d1 ? s.d1 : s.d2) - dn;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) quiet = min(quiet, __shfl_xor(quiet, o));
    if (live) put_row(t, lane, dn, lane, s.rowsB + ib, s.err);
    if (ro) put_row(t, lane, dn, s.coda_xrow0 >= 0 ? s.coda_xrow0 + ic : lane, s.rowsC + ic, s.err);
    if (lane < njs) put_row(t, t.js[2 * lane], 0, t.js[2 * lane], s.rowsP + lane, s.err);
    // ---- the tables back
    for (int i = lane; i < 2 * njs; i += 64) s.js[i] = t.js[i];
#pragma unroll
    for (int i = 0; i < 11; ++i)
        if (has_slot) slot_g[i][lane] = slot_l[i][lane];
    // (targets are the host's)
#pragma unroll
    for (int i = 0; i < 7; ++i)
        if (has_seq && i != 3) seq_g[i][lane] = seq_l[i][lane];
    if (op == OP_STEP)
        for (int i = lane; i < ST_N; i += 64) {
            if (i == ST_MAX_M) {
                if (nB0 > s.stats[i]) s.stats[i] = nB0;
            } else if (st[i]) {
                s.stats[i] += st[i];
            }
        }
    if (lane == 0) {
        *s.nB = nB;
        *s.nC = nC;
        *s.nP = njs;
        *s.njc = njc;
        *s.njs = njs;
        *s.quiet = nB ? max(quiet, 0) : 0;
    }
}

hipError_t launch_sched(const Sched& s, int op, int op_seq, int op_pos, const int32_t* op_tok, hipStream_t st) {
    hipLaunchKernelGGL(k_sched, dim3(1), dim3(64), 0, st, s, op, op_seq, op_pos, op_tok);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// greedy readout: arg-max over the per-tile maxima, then the step's decision
// for the row (draft at d1, gate + second proposal at d2, cascade at R)
// ---------------------------------------------------------------------------
__device__ __forceinline__ bool better(float v, int i, float bv, int bi) {
    return v > bv || (v == bv && i < bi) || bi < 0;
}

__global__ void __launch_bounds__(256) k_finalize_greedy(Sched s, int fin_op, const float* tmax,
                                                          const int32_t* targ, int tiles) {
    const int i = blockIdx.x;
    if (i >= *s.nC) return;
    __shared__ float sv[256];
    __shared__ int si[256];
    float bv = -INFINITY;
    int bi = -1;
    for (int t = threadIdx.x; t < tiles; t += 256) {
        const float v = tmax[(size_t)i * tiles + t];
        const int id = targ[(size_t)i * tiles + t];
        if (better(v, id, bv, bi)) {
            bv = v;
            bi = id;
        }
    }
    sv[threadIdx.x] = bv;
    si[threadIdx.x] = bi;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (threadIdx.x < o) {
            const float v = sv[threadIdx.x + o];
            const int id = si[threadIdx.x + o];
            if (id >= 0 && better(v, id, sv[threadIdx.x], si[threadIdx.x])) {
                sv[threadIdx.x] = v;
                si[threadIdx.x] = id;
            }
        }
        __syncthreads();
    }
    if (threadIdx.x != 0) return;
    const int a = si[0];
    const Row row = s.rowsC[i];
    const int mode = *s.mode;
    int aux = 0;
    if (fin_op == FIN_STEP && mode == MODE_LOOPSPEC) {
        const int b = row.slot;
        if (row.depth == s.d2 && s.d2 > 0) {
            aux = a != s.s_x1[b];                               // greedy gate: argmax q2~ != x1
        } else if (row.depth == s.R) {
            aux = a == s.s_x1[b] ? 1 : (s.s_gate[b] && a == s.s_x2[b]) ? 2 : 0;
        }
    }
    s.ro_tok[i] = a;
    s.ro_aux[i] = aux;
}

// ---------------------------------------------------------------------------
// P for Ouro-style models: H^(0) = E[x]
// ---------------------------------------------------------------------------
template <typename WT>
__device__ __forceinline__ void embed_job(const Geo& g, const int32_t* jobs, int j, const WT* E, float* X) {
    const int xrow = jobs[2 * j], tok = jobs[2 * j + 1];
    const WT* e = E + (size_t)tok * g.h;
    float* x = X + (size_t)xrow * g.h;
    for (int k = threadIdx.x; k < g.h; k += blockDim.x)
        x[k] = sizeof(WT) == 2 ? bf2f(((const uint16_t*)e)[k]) : ((const float*)e)[k];
}

template <typename WT>
__global__ void __launch_bounds__(256) k_embed(Geo g, const int32_t* jobs, const int32_t* njobs, const WT* E,
                                               float* X) {
    const int j = blockIdx.x;
    if (j >= *njobs) return;
    embed_job<WT>(g, jobs, j, E, X);
}

hipError_t launch_embed(const Geo& g, const int32_t* jobs, const int32_t* njobs, int jobs_cap, const void* E,
                        bool bf16, float* X, hipStream_t st) {
    if (bf16)
        hipLaunchKernelGGL(k_embed<uint16_t>, dim3(jobs_cap), dim3(256), 0, st, g, jobs, njobs,
                           (const uint16_t*)E, X);
    else
        hipLaunchKernelGGL(k_embed<float>, dim3(jobs_cap), dim3(256), 0, st, g, jobs, njobs, (const float*)E, X);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// pass buffers: the rounded hidden state and its RMSNorm statistics, in the
// row order of the pass (the partials are the ones the residual epilogue writes)
// ---------------------------------------------------------------------------
template <typename WT>
__global__ void __launch_bounds__(256) k_gather(Geo g, const Row* rows, const int32_t* nrows, const float* X,
                                                PassBuf pb, int opd) {
    const int m = blockIdx.x;
    if (m >= *nrows) return;
    const float* x = X + (size_t)rows[m].xrow * g.h;
    for (int t = threadIdx.x; t < g.ssq_tiles; t += blockDim.x) {
        float v[16];
#pragma unroll
        for (int c = 0; c < 16; ++c) v[c] = x[t * 16 + c];
        pb.SSQR[(size_t)m * g.ssq_tiles + t] = ssq16(v);
#pragma unroll
        for (int c = 0; c < 16; ++c) {
            const size_t i = opd ? opd_elem<WT>(m, t * 16 + c, g.h) : (size_t)m * g.h + t * 16 + c;
            if (sizeof(WT) == 2)
                ((uint16_t*)pb.XB)[i] = f2h(v[c]);
            else
                ((float*)pb.XB)[i] = v[c];
        }
    }
}

hipError_t launch_gather(const Geo& g, const Row* rows, const int32_t* nrows, int rows_cap, const float* X,
                         PassBuf pb, bool bf16, bool opd, hipStream_t st) {
    if (bf16)
        hipLaunchKernelGGL(k_gather<uint16_t>, dim3(rows_cap), dim3(128), 0, st, g, rows, nrows, X, pb, (int)opd);
    else
        hipLaunchKernelGGL(k_gather<float>, dim3(rows_cap), dim3(128), 0, st, g, rows, nrows, X, pb, (int)opd);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// KV commit: the verified root's keys/values of every depth move to the
// committed cache at its position (they are needed by every later position)
// ---------------------------------------------------------------------------
// commit job j, table t (of g.T), keys (kv = 0) or values (kv = 1)
__device__ __forceinline__ void commit_job(const Sched& s, int j, int t, int kv, char* kvc, const char* kvs,
                                           int wbytes) {
    const int q = s.jc[3 * j], b = s.jc[3 * j + 1], pos = s.jc[3 * j + 2];
    const u32x4* src = (const u32x4*)(kvs + kvs_index(s.g, b, t, kv) * wbytes);
    const int per_head = s.g.dh * wbytes / 16;        // 16-byte vectors per head slice
    const int n = s.g.H * per_head;
    for (int k = threadIdx.x; k < n; k += blockDim.x) {
        const int head = k / per_head, i = k - head * per_head;
        u32x4* dst = (u32x4*)(kvc + kvc_index(s.g, q, t, kv, head, pos) * wbytes);
        dst[i] = src[k];
    }
}

// The two independent tails of a decode step in one launch: rows y <
// max_seqs of the grid copy the committed roots' keys and values, row y =
// max_seqs embeds the spawned branches' tokens (as k_embed); x covers
// max(2 T, slots).
template <typename WT>
__global__ void __launch_bounds__(256) k_commit_embed(Sched s, char* kvc, const char* kvs, int wbytes, const WT* E,
                                                      float* X) {
    const int y = blockIdx.y, x = blockIdx.x;
    if (y < s.max_seqs) {
        if (y < *s.njc && x < 2 * s.g.T) commit_job(s, y, x >> 1, x & 1, kvc, kvs, wbytes);
    } else if (x < *s.njs) {
        embed_job<WT>(s.g, s.js, x, E, X);
    }
}

hipError_t launch_commit_embed(const Sched& s, void* kvc, const void* kvs, int wbytes, const void* E, bool bf16,
                               float* X, hipStream_t st) {
    const dim3 grid(std::max(2 * s.g.T, s.g.S), s.max_seqs + 1);
    if (bf16)
        hipLaunchKernelGGL(k_commit_embed<uint16_t>, grid, dim3(256), 0, st, s, (char*)kvc, (const char*)kvs, wbytes,
                           (const uint16_t*)E, X);
    else
        hipLaunchKernelGGL(k_commit_embed<float>, grid, dim3(256), 0, st, s, (char*)kvc, (const char*)kvs, wbytes,
                           (const float*)E, X);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// readout copies for coda blocks: X[row.xrow] = X[row.src]; the coda transforms
// a copy so the branch's own hidden state keeps recurring
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_copy_rows(Geo g, const Row* rows, const int32_t* nrows, float* X) {
    const int i = blockIdx.x;
    if (i >= *nrows) return;
    const int dst = rows[i].xrow, src = rows[i].src;
    for (int k = threadIdx.x; k < g.h; k += blockDim.x) X[(size_t)dst * g.h + k] = X[(size_t)src * g.h + k];
}

hipError_t launch_copy_rows(const Geo& g, const Row* rows, const int32_t* nrows, int rows_cap, float* X,
                            hipStream_t st) {
    hipLaunchKernelGGL(k_copy_rows, dim3(rows_cap), dim3(256), 0, st, g, rows, nrows, X);
    return hipGetLastError();
}

hipError_t launch_finalize_greedy(const Sched& s, int fin_op, const float* tmax, const int32_t* targ, int tiles,
                                  int rows_cap, hipStream_t st) {
    hipLaunchKernelGGL(k_finalize_greedy, dim3(rows_cap), dim3(256), 0, st, s, fin_op, tmax, targ, tiles);
    return hipGetLastError();
}

}  // namespace ls
