// The all-pairs energy path (Algorithms 3 and 4 without a cell list): it streams
// the particle records in chunks, one chunk per workgroup, with a fixed-order
// second pass.
#include "gcmc_internal.h"

namespace gcmc {

constexpr int kBlk = 256;

__device__ __forceinline__ double block_sum(double v, double* red) {
    v = wave_sum(v);
    const int w = threadIdx.x / kWave;
    __syncthreads();
    if ((threadIdx.x & (kWave - 1)) == 0) red[w] = v;
    __syncthreads();
    double t = 0.0;
    const int nw = blockDim.x / kWave;
    for (int i = 0; i < nw; ++i) t += red[i];
    return t;
}

// Constants of an energy pass held in registers for the whole kernel (read
// once from the descriptor: the compiler would otherwise reload them from
// memory inside the candidate loop), the species tables in LDS.
struct PassConst {
    double L[3], hL[3], rc2, e4, s2;
};

__device__ __forceinline__ PassConst pass_const(const DevBox& B) {
    PassConst c;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        c.L[a] = unid(B.L[a]);
        c.hL[a] = unid(B.hL[a]);
    }
    c.rc2 = unid(B.rc2);
    c.e4 = unid(B.eps4[0]);
    c.s2 = unid(B.sig2[0]);
    return c;
}

// Squared minimum-image distance with the pass constants (the same
// operations, in the same order, as dist2).
__device__ __forceinline__ double pass_dist2(const PassConst& K, double px, double py, double pz, double qx, double qy,
                                             double qz) {
    const double dx = nearest_image(qx - px, K.L[0], K.hL[0]);
    const double dy = nearest_image(qy - py, K.L[1], K.hL[1]);
    const double dz = nearest_image(qz - pz, K.L[2], K.hL[2]);
    return (dx * dx + dy * dy) + dz * dz;
}

// --------------------------------------------------------- all-pairs total
template <bool MIX>
__global__ __launch_bounds__(kBlk) void k_total_allpairs(const DevBox* __restrict__ boxp, double* e_out,
                                                          double* partial) {
    __shared__ double4 tile[kBlk];
    __shared__ double red[kBlk / kWave];
    const DevBox& B = *boxp;
    const PassConst K = pass_const(B);
    const int ns = uni(B.ns);
    const int64_t n = B.st->n;
    const int64_t i = (int64_t)blockIdx.x * kBlk + threadIdx.x;
    const bool own = i < n;
    const double4 me = gload(B.pos + (own ? i : 0));
    const int sa = meta_species(me.w);
    double ei = 0.0;
    for (int64_t j0 = 0; j0 < n; j0 += kBlk) {
        const int64_t j = j0 + threadIdx.x;
        __syncthreads();
        tile[threadIdx.x] = gload(B.pos + (j < n ? j : 0));
        __syncthreads();
        const int lim = (n - j0) < kBlk ? (int)(n - j0) : kBlk;
        for (int q = 0; q < lim; ++q) {
            const double4 o = tile[q];
            if (own && j0 + q != i) {
                const double r2 = pass_dist2(K, me.x, me.y, me.z, o.x, o.y, o.z);
                if (MIX) {
                    const int qq = sa * ns + meta_species(o.w);
                    ei += lj_from_r2(r2, K.rc2, B.eps4[qq], B.sig2[qq]);
                } else {
                    ei += lj_from_r2(r2, K.rc2, K.e4, K.s2);
                }
            }
        }
    }
    if (own && e_out) e_out[i] = ei;
    const double s = block_sum(ei, red);
    if (threadIdx.x == 0) partial[blockIdx.x] = 0.5 * s;
}

// ------------------------------------------------------ all-pairs moves
// The trial of move m of the all-pairs chain, or of a caller-given move.
struct APTrial {
    int type, npos, sp;
    int64_t idx;
    double p[2][3];
    bool valid;
};

__device__ __forceinline__ void ap_chunk_sums(const DevBox& B, const APTrial& T, int64_t n, int64_t j0,
                                              int64_t j1, bool mix, double& sa, double& sb, double& wa, double& wb) {
    sa = 0.0;
    sb = 0.0;
    wa = 0.0;
    wb = 0.0;
    const PassConst K = pass_const(B);
    const int ns = uni(B.ns);
    for (int64_t j = j0 + threadIdx.x; j < j1; j += blockDim.x) {
        if (j == T.idx) continue;
        const double4 o = gload(B.pos + j);
        int q = 0;
        if (mix) q = T.sp * ns + meta_species(o.w);
        const double e4 = mix ? B.eps4[q] : K.e4, s2 = mix ? B.sig2[q] : K.s2;
        const double r2a = pass_dist2(K, T.p[0][0], T.p[0][1], T.p[0][2], o.x, o.y, o.z);
        sa += lj_uw_from_r2(r2a, K.rc2, e4, s2, wa);
        if (T.npos == 2) {
            const double r2b = pass_dist2(K, T.p[1][0], T.p[1][1], T.p[1][2], o.x, o.y, o.z);
            sb += lj_uw_from_r2(r2b, K.rc2, e4, s2, wb);
        }
    }
}

__device__ __forceinline__ APTrial ap_trial_from_move(const DevBox& B, const gcmc_move& mv, int64_t n) {
    APTrial T;
    T.valid = true;
    T.type = mv.type;
    T.idx = -1;
    T.npos = 1;
    T.sp = 0;
    if (mv.type == GCMC_MOVE_INSERT) {
        T.valid = mv.species >= 0 && mv.species < B.ns;
        T.sp = mv.species;
        T.p[0][0] = mv.x; T.p[0][1] = mv.y; T.p[0][2] = mv.z;
        return T;
    }
    if ((mv.type != GCMC_MOVE_DISPLACE && mv.type != GCMC_MOVE_DELETE) || mv.index < 0 || mv.index >= n) {
        T.valid = false;
        return T;
    }
    T.idx = mv.index;
    const double4 pi = gload(B.pos + T.idx);
    T.sp = meta_species(pi.w);
    T.p[0][0] = pi.x; T.p[0][1] = pi.y; T.p[0][2] = pi.z;
    if (mv.type == GCMC_MOVE_DISPLACE) {
        T.npos = 2;
        T.p[1][0] = mv.x; T.p[1][1] = mv.y; T.p[1][2] = mv.z;
    }
    return T;
}

// grid (chunks, moves): scratch[(m * chunks + chunk) * 4 + {0,1,2,3}] (energy old/new, virial old/new)
__global__ __launch_bounds__(kBlk) void k_delta_ap_partial(const DevBox* __restrict__ boxp, const gcmc_move* moves,
                                                            int64_t chunk, double* scratch) {
    __shared__ double red[kBlk / kWave];
    const DevBox& B = *boxp;
    const int64_t n = B.st->n;
    const int64_t m = blockIdx.y;
    const APTrial T = ap_trial_from_move(B, moves[m], n);
    const int64_t j0 = (int64_t)blockIdx.x * chunk;
    int64_t j1 = j0 + chunk;
    if (j1 > n) j1 = n;
    double sa = 0.0, sb = 0.0, wa = 0.0, wb = 0.0;
    if (T.valid) ap_chunk_sums(B, T, n, j0, j1, B.ns > 1, sa, sb, wa, wb);
    sa = block_sum(sa, red);
    sb = block_sum(sb, red);
    wa = block_sum(wa, red);
    wb = block_sum(wb, red);
    if (threadIdx.x == 0) {
        double* o = scratch + (m * gridDim.x + blockIdx.x) * 4;
        o[0] = sa;
        o[1] = sb;
        o[2] = wa;
        o[3] = wb;
    }
}

__global__ __launch_bounds__(kBlk) void k_delta_ap_finish(const DevBox* __restrict__ boxp, const gcmc_move* moves,
                                                           int64_t nchunks, const double* scratch, double* dU_pair,
                                                           double* dU_tail, double* dW_pair) {
    __shared__ double red[kBlk / kWave];
    const DevBox& B = *boxp;
    const int64_t n = B.st->n;
    const int64_t m = blockIdx.x;
    const APTrial T = ap_trial_from_move(B, moves[m], n);
    double sa = 0.0, sb = 0.0, wa = 0.0, wb = 0.0;
    for (int64_t q = threadIdx.x; q < nchunks; q += kBlk) {
        const double* o = scratch + (m * nchunks + q) * 4;
        sa += o[0];
        sb += o[1];
        wa += o[2];
        wb += o[3];
    }
    sa = block_sum(sa, red);
    sb = block_sum(sb, red);
    wa = block_sum(wa, red);
    wb = block_sum(wb, red);
    if (threadIdx.x == 0) {
        int64_t nsp[kMaxSpecies];
        for (int s = 0; s < kMaxSpecies; ++s) nsp[s] = B.st->nsp[s];
        double p, t, w;
        if (!T.valid) {
            p = __builtin_nan("");
            t = __builtin_nan("");
            w = __builtin_nan("");
        } else if (T.type == GCMC_MOVE_DISPLACE) {
            p = sb - sa;
            t = 0.0;
            w = wb - wa;
        } else if (T.type == GCMC_MOVE_INSERT) {
            p = sa;
            t = tail_change(B, nsp, T.sp, +1);
            w = wa;
        } else {
            p = -sa;
            t = tail_change(B, nsp, T.sp, -1);
            w = -wa;
        }
        dU_pair[m] = p;
        if (dU_tail) dU_tail[m] = t;
        if (dW_pair) dW_pair[m] = w;
    }
}

// ------------------------------------------------ all-pairs chain (A12)
// Device-side chain bookkeeping of the all-pairs path.
struct APChain {
    uint64_t counter;   // next move counter
    uint64_t ctr0;      // first counter of this call
    int64_t att[3], acc[3];
    double sum_n, sum_u, sum_n2, sum_w;
    int64_t moves_done;
    int64_t candidates, pair_evals;
};

__device__ __forceinline__ APTrial ap_trial_from_draws(const DevBox& B, const U8& u, int64_t n) {
    APTrial T;
    T.valid = true;
    T.sp = 0;
    T.type = (u.u[0] < B.p_disp) ? GCMC_MOVE_DISPLACE : ((u.u[1] < 0.5) ? GCMC_MOVE_DELETE : GCMC_MOVE_INSERT);
    T.idx = -1;
    T.npos = 1;
    if (T.type == GCMC_MOVE_INSERT) {
        for (int a = 0; a < 3; ++a) T.p[0][a] = wrap_into_box(B.L[a] * u.u[4 + a], B.L[a]);
        return T;
    }
    if (n == 0) {
        T.valid = false;
        return T;
    }
    const int64_t i = pick_particle(u.u[2], u.u[7], n);
    T.idx = i;
    const double4 pi = gload(B.pos + i);
    T.p[0][0] = pi.x; T.p[0][1] = pi.y; T.p[0][2] = pi.z;
    if (T.type == GCMC_MOVE_DISPLACE) {
        T.npos = 2;
        for (int a = 0; a < 3; ++a)
            T.p[1][a] = wrap_into_box(T.p[0][a] + B.max_disp * (2.0 * u.u[4 + a] - 1.0), B.L[a]);
    }
    return T;
}

__global__ __launch_bounds__(kBlk) void k_ap_chain_eval(const DevBox* __restrict__ boxp, const APChain* ch,
                                                         int64_t chunk, double* scratch) {
    __shared__ double red[kBlk / kWave];
    const DevBox& B = *boxp;
    if (B.st->error != GCMC_OK) return;
    const int64_t n = B.st->n;
    const U8 u = move_uniforms(B.seed, ch->counter, B.box_id);
    const APTrial T = ap_trial_from_draws(B, u, n);
    const int64_t j0 = (int64_t)blockIdx.x * chunk;
    int64_t j1 = j0 + chunk;
    if (j1 > n) j1 = n;
    double sa = 0.0, sb = 0.0, wa = 0.0, wb = 0.0;
    if (T.valid) ap_chunk_sums(B, T, n, j0, j1, false, sa, sb, wa, wb);
    sa = block_sum(sa, red);
    sb = block_sum(sb, red);
    wa = block_sum(wa, red);
    wb = block_sum(wb, red);
    if (threadIdx.x == 0) {
        double* o = scratch + blockIdx.x * 4;
        o[0] = sa;
        o[1] = sb;
        o[2] = wa;
        o[3] = wb;
    }
}

__device__ int commit_ap(const DevBox& B, const APTrial& T, const double4& meta_rec, int64_t n, int32_t& maxc);

__global__ __launch_bounds__(kBlk) void k_ap_chain_decide(const DevBox* __restrict__ boxp, APChain* ch,
                                                           int64_t nchunks, const double* scratch, gcmc_log* log) {
    __shared__ double red[kBlk / kWave];
    const DevBox& B = *boxp;
    BoxState* st = B.st;
    if (st->error != GCMC_OK) return;
    const int64_t n = st->n;
    const uint64_t ctr = ch->counter;
    const U8 u = move_uniforms(B.seed, ctr, B.box_id);
    const APTrial T = ap_trial_from_draws(B, u, n);
    double sa = 0.0, sb = 0.0, wa = 0.0, wb = 0.0;
    for (int64_t q = threadIdx.x; q < nchunks; q += kBlk) {
        sa += scratch[q * 4];
        sb += scratch[q * 4 + 1];
        wa += scratch[q * 4 + 2];
        wb += scratch[q * 4 + 3];
    }
    sa = block_sum(sa, red);
    sb = block_sum(sb, red);
    wa = block_sum(wa, red);
    wb = block_sum(wb, red);
    if (threadIdx.x != 0) return;
    const int64_t m = (int64_t)(ctr - ch->ctr0);
    const double tk = B.tailK[0];
    ch->att[T.type] += 1;
    gcmc_log r;
    r.type = T.type;
    r.flags = 0;
    r.accepted = 0;
    r.dU_pair = 0.0;
    r.dU_tail = 0.0;
    r.arg = 0.0;
    r.dW_pair = 0.0;
    r.x = r.y = r.z = 0.0;
    int64_t n_after = n;
    if (!T.valid) {
        r.index = -1;
        r.flags = 1;
    } else {
        double dUp, dUt, dWp;
        if (T.type == GCMC_MOVE_DISPLACE) {
            dUp = sb - sa;
            dUt = 0.0;
            dWp = wb - wa;
        } else if (T.type == GCMC_MOVE_INSERT) {
            dUp = sa;
            dUt = tk * (2.0 * (double)n + 1.0);
            dWp = wa;
        } else {
            dUp = -sa;
            dUt = tk * (1.0 - 2.0 * (double)n);
            dWp = -wa;
        }
        r.dW_pair = dWp;
        const double dU = dUp + dUt;
        const double arg = accept_log_ratio(B, T.type, dU, n);
        const bool ok = metropolis(arg, dU, u.u[3]);
        r.index = (T.type == GCMC_MOVE_INSERT) ? (int32_t)n : (int32_t)T.idx;
        r.dU_pair = dUp;
        r.dU_tail = dUt;
        r.arg = arg;
        const int w = (T.type == GCMC_MOVE_DISPLACE) ? 1 : 0;
        r.x = T.p[w][0]; r.y = T.p[w][1]; r.z = T.p[w][2];
        const int64_t others = (T.idx >= 0) ? n - 1 : n;
        ch->candidates += others;
        ch->pair_evals += others * T.npos;
        if (ok) {
            int32_t mc = st->maxcount;
            const double4 rec = (T.idx >= 0) ? gload(B.pos + T.idx) : make_double4(0, 0, 0, 0);
            const int e = commit_ap(B, T, rec, n, mc);
            if (e != GCMC_OK) {
                ch->att[T.type] -= 1;
                st->error = e;
                st->error_move = (int64_t)ctr;
                return;
            }
            st->maxcount = mc;
            n_after = n + ((T.type == GCMC_MOVE_INSERT) ? 1 : ((T.type == GCMC_MOVE_DELETE) ? -1 : 0));
            st->n = n_after;
            st->nsp[0] = n_after;
            st->u_pair += dUp;
            st->w_pair += dWp;
            ch->acc[T.type] += 1;
            r.accepted = 1;
        }
    }
    if (log) log[m] = r;
    ch->sum_n += (double)n_after;
    ch->sum_n2 += (double)n_after * (double)n_after;
    ch->sum_u += st->u_pair + tk * (double)n_after * (double)n_after;
    ch->sum_w += st->w_pair;
    ch->moves_done = m + 1;
    ch->counter = ctr + 1;
}

__global__ void k_ap_chain_begin(const DevBox* __restrict__ boxp, APChain* ch, uint64_t ctr0) {
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        if (ctr0 == GCMC_COUNTER_CONTINUE) ctr0 = (uint64_t)boxp->st->counter;
        ch->counter = ctr0;
        ch->ctr0 = ctr0;
        for (int t = 0; t < 3; ++t) ch->att[t] = ch->acc[t] = 0;
        ch->sum_n = ch->sum_u = ch->sum_n2 = ch->sum_w = 0.0;
        ch->moves_done = 0;
        ch->candidates = ch->pair_evals = 0;
    }
}

__global__ void k_ap_chain_end(const DevBox* __restrict__ boxp, const APChain* ch, gcmc_stats* stats) {
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    const DevBox& B = *boxp;
    ChainSums L;
    L.moves = ch->moves_done;
    for (int t = 0; t < 3; ++t) {
        L.att[t] = ch->att[t];
        L.acc[t] = ch->acc[t];
    }
    L.sum_n = ch->sum_n;
    L.sum_n2 = ch->sum_n2;
    L.sum_u = ch->sum_u;
    L.sum_w = ch->sum_w;
    B.st->counter = (int64_t)ch->counter;
    // in_cutoff is not counted on the all-pairs path (-1)
    finish_launch(B, B.st, L, B.st->n, B.st->u_pair, B.st->w_pair, ch->moves_done, ch->candidates, ch->pair_evals,
                  -1, stats);
}

// The all-pairs chain keeps the cell list up to date as well (same commit).
__device__ int commit_ap(const DevBox& B, const APTrial& T, const double4& rec, int64_t n, int32_t& maxc) {
    const int cap = B.cap;
    auto cell_of = [&](const double* p) {
        const int32_t cx = axis_cell(p[0], B.invS[0], B.M[0]);
        const int32_t cy = axis_cell(p[1], B.invS[1], B.M[1]);
        const int32_t cz = axis_cell(p[2], B.invS[2], B.M[2]);
        return ((int64_t)cz * B.M[1] + cy) * B.M[0] + cx;
    };
    auto remove = [&](int64_t c, int64_t loc) {
        const int32_t nc = gload(B.count + c);
        const int64_t last = c * cap + nc - 1;
        if (loc != last) {
            const double4 e = gload(B.ent + last);
            gstore(B.ent + loc, e);
            gstore_w(B.pos + (meta_low(e.w)), pack_meta(meta_species(e.w), (int32_t)loc));
        }
        gstore(B.count + c, nc - 1);
    };
    if (T.type == GCMC_MOVE_DISPLACE) {
        const int64_t c0 = cell_of(T.p[0]), c1 = cell_of(T.p[1]);
        const int64_t loc = meta_low(rec.w);
        if (c0 == c1) {
            gstore(B.ent + loc, make_double4(T.p[1][0], T.p[1][1], T.p[1][2], pack_meta(T.sp, (int32_t)T.idx)));
            gstore(B.pos + T.idx, make_double4(T.p[1][0], T.p[1][1], T.p[1][2], rec.w));
            return GCMC_OK;
        }
        const int32_t nc = gload(B.count + c1);
        if (nc >= cap) return GCMC_ERR_CELL_OVERFLOW;
        remove(c0, loc);
        const int64_t nl = c1 * cap + nc;
        gstore(B.ent + nl, make_double4(T.p[1][0], T.p[1][1], T.p[1][2], pack_meta(T.sp, (int32_t)T.idx)));
        gstore(B.count + c1, nc + 1);
        gstore(B.pos + T.idx, make_double4(T.p[1][0], T.p[1][1], T.p[1][2], pack_meta(T.sp, (int32_t)nl)));
        if (nc + 1 > maxc) maxc = nc + 1;
        return GCMC_OK;
    }
    if (T.type == GCMC_MOVE_INSERT) {
        if (n >= B.max_n) return GCMC_ERR_CAPACITY;
        const int64_t c0 = cell_of(T.p[0]);
        const int32_t nc = gload(B.count + c0);
        if (nc >= cap) return GCMC_ERR_CELL_OVERFLOW;
        const int64_t nl = c0 * cap + nc;
        gstore(B.ent + nl, make_double4(T.p[0][0], T.p[0][1], T.p[0][2], pack_meta(T.sp, (int32_t)n)));
        gstore(B.count + c0, nc + 1);
        gstore(B.pos + n, make_double4(T.p[0][0], T.p[0][1], T.p[0][2], pack_meta(T.sp, (int32_t)nl)));
        if (nc + 1 > maxc) maxc = nc + 1;
        return GCMC_OK;
    }
    const int64_t c0 = cell_of(T.p[0]);
    remove(c0, meta_low(rec.w));
    if (T.idx != n - 1) {
        const double4 last = gload(B.pos + (n - 1));
        gstore(B.pos + T.idx, last);
        gstore_w(B.ent + (meta_low(last.w)), pack_meta(meta_species(last.w), (int32_t)T.idx));
    }
    return GCMC_OK;
}

// ------------------------------------------------------------ launchers
int launch_total(const DevBox& hb, const DevBox* d_box, bool all_pairs, double* e_out, double* partial,
                 int64_t partial_len, double* U, hipStream_t s, int64_t n, int32_t maxcount) {
    if (!all_pairs) return launch_total_cells(hb, d_box, e_out, partial, partial_len, U, s, n, maxcount);
    const int64_t nb = n > 0 ? (n + kBlk - 1) / kBlk : 1;
    if (nb > partial_len) return -1;
    auto f = hb.ns > 1 ? k_total_allpairs<true> : k_total_allpairs<false>;
    hipLaunchKernelGGL(f, dim3((unsigned)nb), dim3(kBlk), 0, s, d_box, e_out, partial);
    launch_total_finish(d_box, partial, nb, U, s);
    return 0;
}

int64_t total_partials_needed(const DevBox& hb, bool all_pairs, int64_t n) {
    return all_pairs ? (n + kBlk - 1) / kBlk + 1 : pass_partials(hb, n);
}

int64_t ap_chunk_len() { return 8 * kBlk; }

int launch_delta_allpairs(const DevBox* d_box, int64_t n, const gcmc_move* moves, int64_t n_moves, double* scratch,
                          double* dp, double* dt, double* dw, hipStream_t s) {
    const int64_t chunk = ap_chunk_len();
    int64_t nch = (n + chunk - 1) / chunk;
    if (nch < 1) nch = 1;
    if (n_moves > 65535) return -1;
    hipLaunchKernelGGL(k_delta_ap_partial, dim3((unsigned)nch, (unsigned)n_moves), dim3(kBlk), 0, s, d_box, moves,
                       chunk, scratch);
    hipLaunchKernelGGL(k_delta_ap_finish, dim3((unsigned)n_moves), dim3(kBlk), 0, s, d_box, moves, nch, scratch, dp,
                       dt, dw);
    return 0;
}

size_t ap_chain_state_bytes() { return sizeof(APChain); }

void launch_ap_chain_begin(const DevBox* d_box, void* ch, uint64_t ctr0, hipStream_t s) {
    hipLaunchKernelGGL(k_ap_chain_begin, dim3(1), dim3(64), 0, s, d_box, (APChain*)ch, ctr0);
}

void launch_ap_chain_move(const DevBox* d_box, void* ch, int64_t nch, double* scratch, gcmc_log* log,
                          hipStream_t s) {
    hipLaunchKernelGGL(k_ap_chain_eval, dim3((unsigned)nch), dim3(kBlk), 0, s, d_box, (const APChain*)ch,
                       ap_chunk_len(), scratch);
    hipLaunchKernelGGL(k_ap_chain_decide, dim3(1), dim3(kBlk), 0, s, d_box, (APChain*)ch, nch, scratch, log);
}

void launch_ap_chain_end(const DevBox* d_box, const void* ch, gcmc_stats* stats, hipStream_t s) {
    hipLaunchKernelGGL(k_ap_chain_end, dim3(1), dim3(64), 0, s, d_box, (const APChain*)ch, stats);
}

}  // namespace gcmc
