// Host-driven move kernels: energy deltas of caller-given trial moves, the
// commit of one accepted move, and the neighbour-candidate gather (for checking
// the cell list).
#include <type_traits>

#include "cell_pass.h"
#include "trial.h"

namespace gcmc {

// Energy and virial changes of caller-given moves, one wavefront per move: the
// stencil of each position through the rows of cell_pass.h (the counters in one
// round trip, the candidates' records in the next), the pairs inside the cutoff
// queued in LDS and evaluated 64 at a time.  A displacement inside its cell tests
// both positions against the same candidates (Sec. 3.2.4).  Bound by vector issue.
// Four wavefronts per move with a slot for every place of the fullest cell spent
// most lanes on empty slots: 16,384 moves of 262,144 particles 103 -> 45 us, one
// move of 4,000 5.3 -> 4.1 us.  W > 1: a few moves of wide stencils, where the rows of
// one wavefront would be a serial chain: W wavefronts a move, each a share of the rows.
constexpr int kDeltaRows = 4;
constexpr int kDeltaQueue = kWave + 2 * kDeltaRows * kWave;
constexpr int kDeltaWide = 8;

template <bool MIX, int W>
__global__ __launch_bounds__(kWave* W) void k_delta(const DevBox* __restrict__ boxp, const gcmc_move* __restrict__ moves,
                                                 int64_t n_moves, double* dU_pair, double* dU_tail, double* dW_pair) {
    __shared__ PassRows rows_w[W];
    __shared__ double q_w[W][kDeltaQueue];
    __shared__ uint8_t qp_w[W][MIX ? kDeltaQueue : 1];
    __shared__ double te4[kMaxSpecies * kMaxSpecies], ts2[kMaxSpecies * kMaxSpecies];
    __shared__ double sum_w[W][2];
    const DevBox& B = *boxp;
    const PassBox P = pass_box(B);
    const int lane = threadIdx.x & (kWave - 1), wv = W > 1 ? uni((int32_t)threadIdx.x / kWave) : 0;
    PassRows& rows_s = rows_w[wv];
    double* const q = q_w[wv];
    uint8_t* const qp = qp_w[wv];
    const int ns = uni(B.ns);
    if (MIX && threadIdx.x < kMaxSpecies * kMaxSpecies) {
        te4[threadIdx.x] = B.eps4[threadIdx.x];
        ts2[threadIdx.x] = B.sig2[threadIdx.x];
    }
    if (W > 1) __syncthreads();
    const double e4 = unid(B.eps4[0]), s2 = unid(B.sig2[0]);
    const int64_t n = B.st->n;
    for (int64_t m = blockIdx.x; m < n_moves; m += gridDim.x) {
        const gcmc_move mv = moves[m];
        Trial T;
        const bool ok = trial_from_move(B, mv, n, T);
        double su = 0.0, sw = 0.0;   // the new position's sums minus the old one's for a displacement
        if (__builtin_amdgcn_readfirstlane(ok ? 1 : 0) != 0) {
            const int type = uni(T.type), spn = uni(T.sp) * ns;
            const int32_t excl = uni((int32_t)T.idx);
            const bool disp = type == GCMC_MOVE_DISPLACE, both = disp && uni(T.same) != 0;
            uint32_t tail = 0;
            auto drain = [&](uint32_t from, uint32_t cnt) {
                wave_lds_sync();
                if ((uint32_t)lane < cnt) {
                    const double v = q[from + lane];   // the sign bit marks a displacement's old position
                    const int k = MIX ? qp[from + lane] : 0;
                    double w = 0.0;
                    const double u = lj_uw_from_r2(__builtin_fabs(v), P.rc2, MIX ? te4[k] : e4, MIX ? ts2[k] : s2, w);
                    su += __builtin_copysign(1.0, v) * u;
                    sw += __builtin_copysign(1.0, v) * w;
                }
                wave_lds_sync();
            };
            // the stencil of position `which`; BOTH: its candidates meet the two positions
            auto stencil = [&](int which, auto both_t) {
                constexpr bool BOTH = decltype(both_t)::value;
                const int32_t c[3] = {uni(T.c[which][0]), uni(T.c[which][1]), uni(T.c[which][2])};
                const int32_t cl = (c[2] * B.M[1] + c[1]) * B.M[0] + c[0];
                const bool inside = uni(pass_inside(B, c[0], c[1], c[2]) ? 1 : 0) != 0;
                const bool neg = disp && which == 0;
                const double4 p = make_double4(unid(T.p[which][0]), unid(T.p[which][1]), unid(T.p[which][2]), 0.0);
                const double4 p1 = make_double4(unid(T.p[1][0]), unid(T.p[1][1]), unid(T.p[1][2]), 0.0);
                stencil_rows<kDeltaRows, false, true, W>(
                    B, P, rows_s, cl, c[0], c[1], c[2],
                    [&](const double3* e, const double* mw, int rows, int32_t rel, uint32_t own) {
                        auto test = [&](auto wrap_t, auto rows_t) {
                            constexpr bool WRAP = decltype(wrap_t)::value;
                            constexpr int R = decltype(rows_t)::value;
                            double ra[R], rb[R];
#pragma unroll
                            for (int r = 0; r < R; ++r) {
                                ra[r] = pass_r2<WRAP>(P, e[r], p);
                                if (BOTH) rb[r] = pass_r2<WRAP>(P, e[r], p1);
                            }
#pragma unroll
                            for (int r = 0; r < R; ++r) {
                                const uint64_t other = __ballot(meta_low(mw[r]) != excl);   // not itself
                                auto push = [&](double r2, double v) {
                                    const uint64_t mk = __ballot(r2 < P.rc2) & other;
                                    if (__builtin_amdgcn_inverse_ballot_w64(mk)) {
                                        const uint32_t at = lanes_below(mk, tail);
                                        q[at] = v;
                                        if (MIX) qp[at] = (uint8_t)(spn + meta_species(mw[r]));
                                    }
                                    tail += (uint32_t)__builtin_popcountll(mk);
                                };
                                push(ra[r], neg ? -ra[r] : ra[r]);
                                if (BOTH) push(rb[r], rb[r]);
                            }
                            tail = (uint32_t)uni((int32_t)tail);
                            while (tail >= (uint32_t)kWave) {
                                tail -= kWave;
                                drain(tail, kWave);
                            }
                        };
                        pass_dispatch<kDeltaRows>(inside, rows, test);
                    }, (uint32_t)wv);
            };
            if (both) {
                stencil(0, std::true_type{});
            } else {
                stencil(0, std::false_type{});
                if (disp) stencil(1, std::false_type{});
            }
            if (tail) drain(0, tail);
            su = wave_sum(su);
            sw = wave_sum(sw);
        }
        if (W > 1) {
            __syncthreads();   // the last move's sums have been read
            if (lane == 0) {
                sum_w[wv][0] = su;
                sum_w[wv][1] = sw;
            }
            __syncthreads();
            su = sw = 0.0;
            for (int v = 0; v < W; ++v) {
                su += sum_w[v][0];
                sw += sum_w[v][1];
            }
        }
        if (threadIdx.x == 0) {
            double p, t, w;
            if (!ok) {
                p = t = w = __builtin_nan("");
            } else {
                const bool del = T.type == GCMC_MOVE_DELETE;
                p = del ? -su : su;
                w = del ? -sw : sw;
                t = 0.0;
                if (T.type != GCMC_MOVE_DISPLACE) {
                    int64_t nsp[kMaxSpecies];
#pragma unroll
                    for (int s = 0; s < kMaxSpecies; ++s) nsp[s] = B.st->nsp[s];
                    t = tail_change(B, nsp, T.sp, del ? -1 : +1);
                }
            }
            dU_pair[m] = p;
            if (dU_tail) dU_tail[m] = t;
            if (dW_pair) dW_pair[m] = w;
        }
    }
}

__global__ void k_commit(const DevBox* __restrict__ boxp, const gcmc_move* move, const double* dU_pair,
                         const double* dW_pair) {
    const DevBox& B = *boxp;
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    BoxState* st = B.st;
    if (st->error != GCMC_OK) return;
    const int64_t n = st->n;
    const gcmc_move mv = *move;
    Trial T;
    if (!trial_from_move(B, mv, n, T)) {
        st->error = GCMC_ERR_INVALID_ARG;
        st->error_move = -1;
        return;
    }
    int32_t mc = st->maxcount;
    const int e = commit_trial(B, T, n, mc);
    if (e != GCMC_OK) {
        st->error = e;
        st->error_move = -1;
        return;
    }
    st->maxcount = mc;
    if (T.type == GCMC_MOVE_INSERT) {
        st->n = n + 1;
        st->nsp[T.sp] += 1;
    } else if (T.type == GCMC_MOVE_DELETE) {
        st->n = n - 1;
        st->nsp[T.sp] -= 1;
    }
    st->u_pair += *dU_pair;
    st->w_pair = dW_pair ? st->w_pair + *dW_pair : __builtin_nan("");
}

// Candidate ids of points (a slot for every place of the fullest cell).
__global__ __launch_bounds__(256) void k_neighbors(const DevBox* __restrict__ boxp, const double* pts,
                                                   const int32_t* excl, int64_t n, int32_t max_ids, int32_t* ids,
                                                   int32_t* counts) {
    __shared__ uint32_t tab[kMaxStencil];
    __shared__ int32_t fill;
    const DevBox& B = *boxp;
    load_stencil(B, tab);
    const int lg = log2_ceil(B.st->maxcount);
    const int NS = B.nstencil << lg;
    const int gmask = (1 << lg) - 1;
    for (int64_t m = blockIdx.x; m < n; m += gridDim.x) {
        if (threadIdx.x == 0) fill = 0;
        __syncthreads();
        Trial T;
        T.p[0][0] = pts[m]; T.p[0][1] = pts[n + m]; T.p[0][2] = pts[2 * n + m];
        locate(B, T, 0);
        const int32_t ex = excl ? excl[m] : -1;
        for (int s = threadIdx.x; s < NS; s += blockDim.x) {
            const int t = s >> lg, k = s & gmask;
            const int64_t c = stencil_cell(B, tab[t], T.c[0][0], T.c[0][1], T.c[0][2]);
            if (k < gload(B.count + c) && k < B.cap) {
                const int32_t id = meta_low(gload(B.ent + (c * B.cap + k)).w);
                if (id != ex) {
                    const int32_t at = atomicAdd(&fill, 1);
                    if (at < max_ids) ids[m * max_ids + at] = id;
                }
            }
        }
        __syncthreads();
        if (threadIdx.x == 0) counts[m] = fill;
        __syncthreads();
    }
}

// ---------------------------------------------------------- dispatch
// Eight wavefronts a move where the stencil may hold 64 rows and the moves alone would not fill the chip.
// Calls in us, four wavefronts each with a slot for every place (the mapping before k_delta) / one / eight:
// 30,000 particles in 27 cells, 1 move 136 / 153 / 78, 256 moves 230 / 284 / 131, 1,024 moves 371 / 300 / 248;
// 262,144 at a cutoff of 20, 256 moves 1,574 / 2,974 / 856; 4,000 in 27 cells, 64 moves 93 / 91 / 63.  Each
// wavefront numbers the candidates of the whole stencil: with several groups of 64 cells that is worth it for
// fewer moves (600 cells, 256 moves 73 / 66 / 64, 1,024 moves 84 / 72 / 93).
int launch_delta(const DevBox& hb, const DevBox* d_box, int64_t n_moves, const gcmc_move* moves, double* dp, double* dt,
                 double* dw, hipStream_t s) {
    const unsigned g = (unsigned)(n_moves < 65536 ? n_moves : 65536);
    const bool mix = hb.ns > 1;
    if (n_moves <= (hb.nstencil <= kWave ? 1024 : 256) && (int64_t)hb.nstencil * hb.cap >= 64 * kWave) {
        auto f = mix ? k_delta<true, kDeltaWide> : k_delta<false, kDeltaWide>;
        hipLaunchKernelGGL(f, dim3(g), dim3(kWave * kDeltaWide), 0, s, d_box, moves, n_moves, dp, dt, dw);
        return 0;
    }
    auto f = mix ? k_delta<true, 1> : k_delta<false, 1>;
    hipLaunchKernelGGL(f, dim3(g), dim3(kWave), 0, s, d_box, moves, n_moves, dp, dt, dw);
    return 0;
}

void launch_commit(const DevBox* d_box, const gcmc_move* move, const double* dU, const double* dW, hipStream_t s) {
    hipLaunchKernelGGL(k_commit, dim3(1), dim3(64), 0, s, d_box, move, dU, dW);
}

void launch_neighbors(const DevBox* d_box, const double* pts, const int32_t* excl, int64_t n, int32_t max_ids,
                      int32_t* ids, int32_t* counts, hipStream_t s) {
    const int64_t g64 = n < 65536 ? n : 65536;
    hipLaunchKernelGGL(k_neighbors, dim3((int)(g64 < 1 ? 1 : g64)), dim3(256), 0, s, d_box, pts, excl, n, max_ids,
                       ids, counts);
}

}  // namespace gcmc
