// The persistent chain of Algorithm 1 for a small box held in local memory.
//
// In a box of a few hundred to a couple of thousand particles the 27-cell
// stencil covers most or all of the box, so the cell list prunes little, and a move
// of the global-memory kernels costs a chain of dependent memory round trips of
// about a microsecond each.  Here one workgroup copies the box's coordinates
// into LDS once per launch and runs every move against that copy.
//
// Rounds of W moves: wavefront w evaluates move m + w against every other
// particle of the state at the start of the round (the energy of a move is the
// sum over all particles inside the cutoff, Eq. 1 with the strict cutoff: the
// same pairs the cell list finds), and wavefront 0 decides the moves in order.
// A move whose particle an earlier accepted move of the round changed, or
// whose pick at the current N is another particle, ends the round and is
// evaluated again in the next.  Every other move is used with its energy and
// virial corrected for the earlier accepted moves of the round: removing a
// particle at a and adding one at b changes the move's sums by f(b) - f(a),
// f(r) the pair terms of r with the move's new position minus those with its
// old one, prepared by the move's own wavefront.  An overlap's term taken away again would leave
// its rounding in place of the sums' digits (4 (sigma / r)^12 is 1e16 at r = 0.05), so the terms of
// particles that overlap the move's positions and that an earlier move would take away are kept apart
// from its sums and added while their particles are there.
//
// Lane k of wavefront 0 holds move k of the round and its decision at the current
// state, so the rejections up to the next accepted or stale move take one ballot,
// and only an accepted move (about one in eight) costs a serial step: N, the
// running sums and the LDS copy change, and the later lanes add its corrections and
// decide again.  Deciding move by move took 0.85 us each, two thirds of a round:
// 512 particles 1.63 -> 0.83 us per move, 1,536 particles 2.4 -> 1.3 (waves = 8).  What bounds
// it now is the latency of one wavefront's evaluation (rows of 64 particles taken
// two to four at a time) and about 1 us of decision per round.
// Particles with an index of kResCap or more (a box that grows past it) are read
// from and written to global memory instead: correct, slower.
//
// The cells are not maintained during the launch.  At its end the workgroup
// writes the coordinates back and rebuilds the box's cell list in the layout
// of gcmc_cell_build (entries of a cell in particle-id order, back-pointers in
// the records), so every other kernel and call finds the box as it expects.
#include <type_traits>

#include "cell_pass.h"
#include "spec_eval.h"

namespace gcmc {

constexpr int kResCap = 2048;   // particles whose coordinates live in LDS
constexpr int kResRing = 64;    // moves prepared at once
// (r / sigma)^2 below which a term is kept apart from the sums: there it passes 256 well depths, where
// (sigma / r)^6 = 1 / 2 + sqrt(64.25), and its rounding 3e-14 of them
constexpr double kApart2 = 0.49;

// What a move needs from its draws, prepared for kResRing moves at a time:
// the type, ln A, the 53 bits of the pick fields as an integer, the floor
// fallback's uniform, and the displacement (or the inserted position).
struct ResMove {
    int32_t type;
    uint32_t klo, khi;
    double u2, lnA;
    double q[3];
};

// Pairs of one wavefront waiting for their energies: at most 63 left over and four
// rows of 64 more between two looks (four rows for one position, or two for two).
constexpr int kResQueue = kWave + 4 * kWave;

// The particle a displacement or deletion picks among n (the rule of
// pick_particle with the spare draw's 53 bits given as an integer), every lane on
// its own move or its own n.
__device__ __forceinline__ int32_t res_pick(uint32_t klo, uint32_t khi, double u2, int32_t n) {
    if (n <= 1) return 0;
    const uint64_t k = ((uint64_t)khi << 32) | (uint64_t)klo;
    const int b = 32 - __clz(n - 1);
    const uint32_t mask = (1u << b) - 1u;
    int32_t idx = -1;
    for (int sh = 53 - b; sh >= 0 && idx < 0; sh -= b) {
        const uint32_t v = (uint32_t)(k >> sh) & mask;
        if (v < (uint32_t)n) idx = (int32_t)v;
    }
    if (idx < 0) {
        const int32_t i = (int32_t)floor(u2 * (double)n);
        idx = i > n - 1 ? n - 1 : i;
    }
    return idx;
}

// Squared minimum-image distance, the bits of dist2 (coordinates in [0, L)): the
// magnitude of a minimum image is the smaller of |d| and L - |d|.
__device__ __forceinline__ double res_dist2(const double* L, double px, double py, double pz, const double3& e) {
    const double dx = image_abs(e.x - px, L[0]), dy = image_abs(e.y - py, L[1]), dz = image_abs(e.z - pz, L[2]);
    return (dx * dx + dy * dy) + dz * dz;
}

// Pair energy and virial, the operations of lj_uw_from_r2 with selects for branches.
__device__ __forceinline__ double res_pair(double r2, double rc2, double eps4, double sig2, double& w) {
    const double sr2 = sig2 / r2;
    const double s6 = sr2 * sr2 * sr2;
    const double s12 = s6 * s6;
    const bool in = r2 < rc2 && eps4 != 0.0, over = r2 == 0.0;
    w = in ? (over ? __builtin_inf() : 6.0 * eps4 * (2.0 * s12 - s6)) : 0.0;
    return in ? (over ? __builtin_inf() : eps4 * (s12 - s6)) : 0.0;
}

// W moves at a time, S wavefronts for each; OCC: wavefronts a SIMD must have room for
// (the register bound).
template <int W, int S, int OCC>
__global__ __launch_bounds__(kWave* W* S, OCC) void k_chain_resident(const DevBox* __restrict__ boxes,
                                                              const int32_t* __restrict__ order, int64_t n_moves,
                                                              uint64_t ctr0, gcmc_stats* stats, gcmc_log* trace) {
    __shared__ double px[kResCap], py[kResCap], pz[kResCap];
    __shared__ DrawRing<kResRing> dring;
    __shared__ ResMove mv[kResRing];
    // log acceptance prefactors for N = lbase + t: insertion V / (Lambda^3 (N + 1)), deletion
    // Lambda^3 N / V (the moves prepared together change N by at most one each)
    __shared__ double lpi[2 * kResRing + 1], lpd[2 * kResRing + 1];
    __shared__ double pq[W * S][kResQueue];   // each wavefront's queue of in-cutoff pairs
    // move k's evaluation by each of its wavefronts: pair energy and virial change against the
    // round's start, pairs inside the cutoff, and bit o: its pick at N_round - (W - 1) + o is the
    // particle it evaluated; bit 16 + j: the terms of the particle that move j takes away are in
    // apart[j][k], not in its sums
    __shared__ double ev_u[S][W], ev_w[S][W];
    __shared__ int32_t ev_in[S][W];
    __shared__ uint32_t ev_pick[W];
    __shared__ double apart_e[W][W], apart_w[W][W];
    // corr[j][k]: the change of move k's pair energy and virial if move j < k of the round is
    // accepted (move j's removed and added positions against move k's positions)
    __shared__ double corr_e[W][W], corr_w[W][W];
    __shared__ int32_t ready[W * S];      // round whose evaluation wavefront w has published
    // the state after a round, by round parity (a wavefront may still read the last round's)
    __shared__ int4 sh_state[2];   // N, moves decided, error
    __shared__ int32_t wred[W * S];
    __shared__ int32_t sh_flag;
    const int bi = order ? order[blockIdx.x] : (int)blockIdx.x;
    const DevBox B = hot_copy(boxes[blockIdx.x]);
    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane(tid / kWave);
    BoxState* st = B.st;

    if (ctr0 == GCMC_COUNTER_CONTINUE) ctr0 = (uint64_t)st->counter;
    int32_t N = uni((int32_t)st->n);   // below 2^31
    double U = st->u_pair;      // running energy and virial: kept by wavefront 0
    double Wvir = st->w_pair;
    int32_t err = uni(st->error);
    int64_t err_move = st->error_move;
    const double tk = B.tailK[0];
    const double rc2 = B.rc2, eps4 = B.eps4[0], sig2 = B.sig2[0];
    const int32_t spin_cap = wait_bound(B.wait_limit);
    const double apart2 = eps4 != 0.0 ? fmin(kApart2 * sig2, rc2) : 0.0;
    // wavefront wv takes part `part` of move `own` of a round: every parts-th group of rows (a bound
    // that lets nobody wait leaves a move to one wavefront)
    const int parts = spin_cap < 0 ? 1 : S, part = wv / W, own = wv - part * W;
    // statistics of wavefront 0, lane k's sums over the moves it decided as move k of a round (counts as
    // doubles, exact below 2^53): in local memory, as registers they would be spilled through the rounds
    enum { kAtt, kAcc = 3, kSumN = 6, kSumN2, kSumU, kSumW, kCand, kEvals, kIncut, kStats };
    __shared__ double acc_s[kStats][W];
    for (int t = tid; t < kStats * W; t += blockDim.x) (&acc_s[0][0])[t] = 0.0;

    auto get = [&](int32_t j) -> double3 {
        if (j < kResCap) return make_double3(px[j], py[j], pz[j]);
        return gload_xyz(B.pos + j);
    };
    auto put = [&](int32_t j, double x, double y, double z) {
        if (j < kResCap) {
            px[j] = x;
            py[j] = y;
            pz[j] = z;
        } else {
            gstore(B.pos + j, make_double4(x, y, z, 0.0));
        }
    };

    {
        const int32_t nl = N < kResCap ? N : kResCap;
        for (int32_t j = tid; j < nl; j += blockDim.x) {
            const double4 r = gload(B.pos + j);
            px[j] = r.x;
            py[j] = r.y;
            pz[j] = r.z;
        }
    }
    if (tid == 0) sh_flag = 0;
    if (tid < W * S) ready[tid] = -1;
    if (err == GCMC_OK && B.ns != 1) {
        err = GCMC_ERR_UNSUPPORTED;
        err_move = (int64_t)ctr0;
    }
    __syncthreads();
    int64_t m = 0;
    int64_t prep_end = 0;   // moves m' < prep_end have their draws prepared (with the tables)
    int32_t lbase = 0;
    int32_t rnd = 0;
    while (err == GCMC_OK && m < n_moves) {
        rnd = rnd == INT32_MAX ? 1 : rnd + 1;
        if (m + W > prep_end) {
            // moves m .. m + kResRing - 1: Philox block t & 3 of move m + t / 4 per thread, the
            // prefactor tables for every N those moves can meet, then one thread per move derives
            // what the move needs
            const uint64_t ctr = ctr0 + (uint64_t)m;
            for (int t = tid; t < 4 * kResRing; t += blockDim.x)
                draw_block(B, &dring, ctr + (uint64_t)(t >> 2), t & 3);
            lbase = N - kResRing;
            for (int t = tid; t < 2 * (2 * kResRing + 1); t += blockDim.x) {
                const bool del = t > 2 * kResRing;
                const int32_t n = lbase + (del ? t - (2 * kResRing + 1) : t);
                if (n >= 0) {
                    const double x = del ? (B.lambda3 * (double)n) / B.V : B.V / (B.lambda3 * (double)(n + 1));
                    if (del) lpd[t - (2 * kResRing + 1)] = log(x);
                    else lpi[t] = log(x);
                }
            }
            __syncthreads();
            if (tid < kResRing) {
                const int sl = (int)((ctr + (uint64_t)tid) & (uint64_t)(kResRing - 1));
                ResMove r;
                r.type = dring.type[sl];
                const uint64_t k = (uint64_t)(dring.u7[sl] * 9007199254740992.0);
                r.klo = (uint32_t)k;
                r.khi = (uint32_t)(k >> 32);
                r.u2 = dring.u2[sl];
                r.lnA = dring.lnA[sl];
                const double ud[3] = {dring.px[sl], dring.py[sl], dring.pz[sl]};
#pragma unroll
                for (int a = 0; a < 3; ++a)
                    r.q[a] = r.type == GCMC_MOVE_INSERT ? wrap_into_box(B.L[a] * ud[a], B.L[a])
                                                        : B.max_disp * (2.0 * ud[a] - 1.0);
                mv[sl] = r;
            }
            prep_end = m + kResRing;
            __syncthreads();
        }
        const int kend = (n_moves - m) < W ? (int)(n_moves - m) : W;
        if (own < kend && part < parts) {
            // ---------------------------------------- the round's moves, lane k: move m + k
            int32_t type = GCMC_MOVE_INSERT, idx = -1;
            double u2 = 0.0, lnA = 0.0;
            uint32_t klo = 0, khi = 0;
            double ax = 0.0, ay = 0.0, az = 0.0;   // the position it takes away (displacement, deletion)
            double bx = 0.0, by = 0.0, bz = 0.0;   // the position it adds (displacement, insertion)
            if (lane < kend) {
                const ResMove& R = mv[(int)((ctr0 + (uint64_t)(m + lane)) & (uint64_t)(kResRing - 1))];
                type = R.type;
                u2 = R.u2;
                lnA = R.lnA;
                klo = R.klo;
                khi = R.khi;
                bx = R.q[0];
                by = R.q[1];
                bz = R.q[2];
                if (type != GCMC_MOVE_INSERT && N > 0) {
                    idx = res_pick(klo, khi, u2, N);
                    const double3 o = get(idx);
                    ax = o.x;
                    ay = o.y;
                    az = o.z;
                    if (type == GCMC_MOVE_DISPLACE) {
                        bx = wrap_into_box(ax + bx, B.L[0]);
                        by = wrap_into_box(ay + by, B.L[1]);
                        bz = wrap_into_box(az + bz, B.L[2]);
                    }
                }
            }
            // ---------------------------------------- evaluate move m + own, or part of it
            const int mt = __builtin_amdgcn_readlane(type, own);
            const int32_t mi = __builtin_amdgcn_readlane(idx, own);
            if (mt == GCMC_MOVE_INSERT || N > 0) {
                const bool disp = mt == GCMC_MOVE_DISPLACE, ins = mt == GCMC_MOVE_INSERT;
                const double p0x = read_lane(ins ? bx : ax, own), p0y = read_lane(ins ? by : ay, own),
                             p0z = read_lane(ins ? bz : az, own);
                const double p1x = read_lane(bx, own), p1y = read_lane(by, own), p1z = read_lane(bz, own);
                double* q = pq[wv];
                uint32_t tail = 0;
                int32_t n_in = 0;
                double su = 0.0, sw = 0.0;   // new position minus old (displacement), else the one position
                uint32_t first = 0;          // earlier moves whose particle's terms are kept apart (each particle once)
                int rp = part, rs = parts;   // its share of the rows
                auto drain = [&](uint32_t from, uint32_t cnt) {
                    wave_lds_sync();
                    if ((uint32_t)lane < cnt) {
                        const double v = q[from + lane];   // the sign bit marks a displacement's old position
                        double w = 0.0;
                        const double u = lj_uw_from_r2(__builtin_fabs(v), rc2, eps4, sig2, w);
                        su += __builtin_copysign(1.0, v) * u;
                        sw += __builtin_copysign(1.0, v) * w;
                    }
                    wave_lds_sync();
                };
                auto push = [&](double r2, double v) {
                    const uint64_t mk = __ballot(r2 < rc2);
                    if (__builtin_amdgcn_inverse_ballot_w64(mk)) q[lanes_below(mk, tail)] = v;
                    tail += (uint32_t)__builtin_popcountll(mk);
                };
                // rows of 64 particles, RB at a time (independent chains); x = 1e300: no candidate
                auto rows = [&](auto two_t) {
                    constexpr bool TWO = decltype(two_t)::value;
                    constexpr int RB = TWO ? 2 : 4;
                    for (int32_t j0 = rp * RB * kWave; j0 < N; j0 += rs * RB * kWave) {
                        double3 e[RB];
#pragma unroll
                        for (int r = 0; r < RB; ++r) {
                            const int32_t j = j0 + r * kWave + lane;
                            e[r] = make_double3(1e300, 0.0, 0.0);
                            if (j0 + r * kWave < kResCap) {
                                // (reads past the particles stay inside the arrays)
                                const double3 o = make_double3(px[j], py[j], pz[j]);
                                if (j < N && j != mi) e[r] = o;
                            } else if (j < N && j != mi) {
                                e[r] = gload_xyz(B.pos + j);
                            }
                            for (uint32_t l = first; l; l &= l - 1u)
                                if (j == __builtin_amdgcn_readlane(idx, (int)__builtin_ctz(l))) e[r].x = 1e300;
                        }
                        double ra[RB], rb[RB];
#pragma unroll
                        for (int r = 0; r < RB; ++r) {
                            ra[r] = res_dist2(B.L, p0x, p0y, p0z, e[r]);
                            if (TWO) rb[r] = res_dist2(B.L, p1x, p1y, p1z, e[r]);
                        }
                        const uint32_t t0 = tail;
#pragma unroll
                        for (int r = 0; r < RB; ++r) {
                            push(ra[r], TWO ? -ra[r] : ra[r]);
                            if (TWO) push(rb[r], rb[r]);
                        }
                        tail = (uint32_t)uni((int32_t)tail);
                        n_in += (int32_t)(tail - t0);
                        while (tail >= (uint32_t)kWave) {
                            tail -= kWave;
                            drain(tail, kWave);
                        }
                    }
                };
                if (disp) rows(std::true_type{});
                else rows(std::false_type{});
                if (tail) drain(0, tail);
                tail = 0;
                // the correction if the earlier move j of the round is accepted: f(b_j) - f(a_j), f(r) the
                // pair terms of r with this move's new position minus those with its old one; lane
                // 16 g + j takes one of the four terms: (new, b), (old, b), (new, a), (old, a)
                if (own > 0 && part == parts - 1) {
                    const int j = lane & 15, g = lane >> 4;
                    const int32_t tc = __shfl(type + (idx == mi ? 4 : 0), j, kWave), tj = tc & 3;
                    const double jax = __shfl(ax, j, kWave), jay = __shfl(ay, j, kWave), jaz = __shfl(az, j, kWave);
                    const double jbx = __shfl(bx, j, kWave), jby = __shfl(by, j, kWave), jbz = __shfl(bz, j, kWave);
                    const bool b_side = g < 2, new_side = (g & 1) == 0;
                    const bool has = j < own && (b_side ? tj != GCMC_MOVE_DELETE : tj != GCMC_MOVE_INSERT) &&
                                     (new_side ? mt != GCMC_MOVE_DELETE : !ins) && (tj == GCMC_MOVE_INSERT || N > 0) &&
                                     (b_side || tc < 4);   // (moves of its own particle, accepted, make it stale)
                    const bool second = new_side && disp;
                    double u = 0.0, w = 0.0, r2 = rc2;
                    if (has) {
                        r2 = res_dist2(B.L, second ? p1x : p0x, second ? p1y : p0y, second ? p1z : p0z,
                                       make_double3(b_side ? jbx : jax, b_side ? jby : jay, b_side ? jbz : jaz));
                        u = res_pair(r2, rc2, eps4, sig2, w);
                    }
                    const uint64_t close = __ballot(!b_side && r2 < apart2);
                    if (close) {
                        // (seldom) the sums again, without the particles that would be taken away from that close
                        const uint32_t apart = (uint32_t)((close >> 32) | (close >> 48)) & 0xFFFFu;
                        const double du = u - __shfl_down(u, 16, kWave), dw = w - __shfl_down(w, 16, kWave);
                        for (uint32_t l = apart; l; l &= l - 1u) {
                            const int a = (int)__builtin_ctz(l);
                            const uint64_t same = __ballot(idx == __builtin_amdgcn_readlane(idx, a)) & apart;
                            if ((int)__builtin_ctzll(same) == a) first |= 1u << a;
                        }
                        if (g == 2 && ((first >> j) & 1u)) {
                            apart_e[j][own] = du;
                            apart_w[j][own] = dw;
                        }
                        if (!b_side && ((apart >> j) & 1u)) u = w = 0.0;
                        const int32_t pairs = n_in;
                        su = sw = 0.0;
                        rp = 0;
                        rs = 1;
                        if (disp) rows(std::true_type{});
                        else rows(std::false_type{});
                        if (tail) drain(0, tail);
                        n_in = pairs;
                    }
                    // (new - old) at b, minus (new - old) at a
                    u -= __shfl_down(u, 16, kWave);
                    w -= __shfl_down(w, 16, kWave);
                    u -= __shfl_down(u, 32, kWave);
                    w -= __shfl_down(w, 32, kWave);
                    if (lane < own) {
                        corr_e[lane][own] = u;
                        corr_w[lane][own] = w;
                    }
                }
                // the pick at every N the move can meet (lane o: N - (W - 1) + o)
                uint32_t pm = 0xFFFFFFFFu;
                if (!ins && part == parts - 1) {
                    const uint32_t olo = __builtin_amdgcn_readlane(klo, own), ohi = __builtin_amdgcn_readlane(khi, own);
                    const double ou2 = read_lane(u2, own);
                    const int32_t np = N - (W - 1) + lane;
                    const int32_t at = res_pick(olo, ohi, ou2, np > 0 ? np : 0);
                    pm = (uint32_t)__ballot(lane < 2 * W - 1 && np >= 0 && at == mi);
                }
                su = wave_sum_uniform(su);
                sw = wave_sum_uniform(sw);
                if (lane == 0) {
                    ev_u[part][own] = mt == GCMC_MOVE_DELETE ? -su : su;
                    ev_w[part][own] = mt == GCMC_MOVE_DELETE ? -sw : sw;
                    ev_in[part][own] = n_in;
                    if (part == parts - 1) ev_pick[own] = (pm & 0xFFFFu) | first << 16;
                }
            }
            if (wv != 0) {
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
                if (lane == 0) __hip_atomic_store(&ready[wv], rnd, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            } else {
                // ------------------------------------ decide in order, lane k: move m + k
                // Every lane keeps its move's decision at the current state.  The moves up to the
                // first accepted or stale one are rejections; an accepted one changes N and the
                // corrections of the later lanes, which decide again.
                int kw = kend;   // moves whose evaluation arrived
                if (spin_cap < 0) {
                    kw = 1;
                } else {
                    int32_t spins = 0;
                    for (;;) {
                        const bool wait = lane > 0 && lane < W * S && lane % W < kend &&
                                          __hip_atomic_load(&ready[lane & (W * S - 1)], __ATOMIC_ACQUIRE,
                                                            __HIP_MEMORY_SCOPE_WORKGROUP) != rnd;
                        const uint64_t late = __ballot(wait);
                        if (late == 0) break;
                        __builtin_amdgcn_s_sleep(1);
                        if (++spins > spin_cap) {
                            for (uint64_t l = late; l; l &= l - 1ull) {
                                const int q = (int)__builtin_ctzll(l) % W;   // the first move not whole
                                kw = q < kw ? q : kw;
                            }
                            break;
                        }
                    }
                }
                kw = uni(kw);
                wave_lds_sync();
                const bool mine = lane < kw;
                const bool disp = type == GCMC_MOVE_DISPLACE, ins = type == GCMC_MOVE_INSERT;
                const bool empty = !ins && N == 0;   // a displacement or deletion in an empty box
                double dUp = 0.0, dWp = 0.0;
                uint32_t pick = 0;   // and, from bit 16 on, the moves whose particle's terms are kept apart
                int32_t n_in = 0;
                if (mine && !empty) {
                    pick = ev_pick[lane];
                    for (int q = 0; q < parts; ++q) {
                        // (the sums without the particles kept apart were taken by one wavefront)
                        const bool use = pick < 0x10000u || q == parts - 1;
                        dUp += use ? ev_u[q][lane] : 0.0;
                        dWp += use ? ev_w[q][lane] : 0.0;
                        n_in += ev_in[q][lane];
                    }
                }
                const int32_t n_round = N;
                bool stale = false;
                // sums with the terms kept apart of the particles that are still there, the sums without in
                // ev_u[0], ev_w[0] from here on
                const bool any_apart = __ballot(pick >= 0x10000u) != 0;
                auto with_apart = [&]() {
                    dUp = ev_u[0][lane];
                    dWp = ev_w[0][lane];
                    for (uint32_t l = pick >> 16; l; l &= l - 1u) {
                        dUp += apart_e[__builtin_ctz(l)][lane];
                        dWp += apart_w[__builtin_ctz(l)][lane];
                    }
                };
                if (any_apart && mine) {
                    ev_u[0][lane] = dUp;
                    ev_w[0][lane] = dWp;
                    with_apart();
                }
                double dUt = 0.0, arg = 0.0;
                double aft_n = 0.0, aft_u = 0.0, aft_w = 0.0;
                uint64_t accbits = 0;
                int k = 0;
                while (k < kw) {
                    const uint64_t todo = ((1ull << kw) - 1ull) & ~((1ull << k) - 1ull);
                    // (branch-free: every lane's move, the others masked out below)
                    const double lp = ins ? lpi[N - lbase] : lpd[N - lbase], n2 = 2.0 * (double)N;
                    const double t_now = disp ? 0.0 : tk * (ins ? n2 + 1.0 : 1.0 - n2);
                    const double dU = dUp + t_now;
                    const double now = spec_arg(B.beta, disp ? 0.0 : B.mu, ins ? 1ull << 63 : 0ull, dU, disp ? 0.0 : lp);
                    const bool ok = !empty & (dU == dU) & (lnA < now);
                    // the empty-box rejection holds only while the box is still empty
                    const bool bad = empty ? N != 0 : !ins & (stale | (((pick >> (N - n_round + W - 1)) & 1u) == 0));
                    arg = lane >= k ? now : arg;
                    dUt = lane >= k ? t_now : dUt;
                    const uint64_t bads = __ballot(bad) & todo;
                    const uint64_t stop = bads | (__ballot(ok) & todo);
                    const int f = stop ? (int)__builtin_ctzll(stop) : kw;
                    if (lane >= k && lane < f) {   // rejected: the state after them is the current one
                        aft_n = (double)N;
                        aft_u = U;
                        aft_w = Wvir;
                    }
                    k = f;
                    if (f == kw || ((bads >> f) & 1ull)) break;
                    // ---- move f is accepted
                    const int32_t tf = __builtin_amdgcn_readlane(type, f), fi = __builtin_amdgcn_readlane(idx, f);
                    const bool fins = tf == GCMC_MOVE_INSERT, fdel = tf == GCMC_MOVE_DELETE;
                    if (fins && N >= B.max_n) {
                        err = GCMC_ERR_CAPACITY;
                        err_move = (int64_t)(ctr0 + (uint64_t)(m + f));
                        break;
                    }
                    // into the LDS copy: every evaluation of the round has been read
                    if (lane == f) {
                        if (!fdel) {
                            put(fins ? N : fi, bx, by, bz);
                        } else if (fi != N - 1) {
                            const double3 l = get(N - 1);
                            put(fi, l.x, l.y, l.z);
                        }
                    }
                    // the indices whose particle changed: the moved or deleted one, the inserted one,
                    // and the last one a deletion relabels
                    stale = stale || idx == (fins ? N : fi) || (fdel && idx == N - 1);
                    if (lane > f && lane < kw) {
                        dUp += corr_e[f][lane];
                        dWp += corr_w[f][lane];
                    }
                    N += fins ? 1 : (fdel ? -1 : 0);
                    U += read_lane(dUp, f);
                    Wvir += read_lane(dWp, f);
                    if (any_apart) {   // (seldom)
                        const uint32_t gone = fins ? 0u : (uint32_t)__ballot(idx == fi) << 16;
                        if (lane > f && lane < kw) {
                            pick &= ~gone;
                            ev_u[0][lane] += corr_e[f][lane];
                            ev_w[0][lane] += corr_w[f][lane];
                            with_apart();
                        }
                    }
                    if (lane == f) {
                        aft_n = (double)N;
                        aft_u = U;
                        aft_w = Wvir;
                    }
                    accbits |= 1ull << f;
                    k = f + 1;
                }
                if (err == GCMC_OK && k == kw && kw < kend) {
                    err = GCMC_ERR_INTERNAL;   // move kw's evaluation did not arrive
                    err_move = (int64_t)(ctr0 + (uint64_t)(m + kw));
                }
                // ---- statistics and log of the k moves decided, lane by lane
                const bool done = lane < k;
                const bool acc = done && ((accbits >> lane) & 1ull) != 0;
                if (done) {
                    auto add = [&](int what, double v) {   // (an LDS instruction nobody waits for)
                        __hip_atomic_fetch_add(&acc_s[what][lane], v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
                    };
                    add(kAtt + type, 1.0);
                    if (acc) add(kAcc + type, 1.0);
                    add(kSumN, aft_n);
                    add(kSumN2, aft_n * aft_n);
                    add(kSumU, aft_u + tk * aft_n * aft_n);
                    add(kSumW, aft_w);
                    const double c = empty ? 0.0 : (double)(n_round - (ins ? 0 : 1));
                    add(kCand, c);
                    add(kEvals, disp ? 2.0 * c : c);
                    add(kIncut, (double)n_in);
                    if (trace) {
                        gcmc_log r;
                        r.type = type;
                        const double dn = acc ? (ins ? 1.0 : (disp ? 0.0 : -1.0)) : 0.0;
                        r.index = empty ? -1 : (ins ? (int32_t)(aft_n - dn) : idx);
                        r.accepted = acc ? 1 : 0;
                        r.flags = empty ? 1 : 0;
                        r.dU_pair = dUp;
                        r.dU_tail = empty ? 0.0 : dUt;
                        const bool del = type == GCMC_MOVE_DELETE;
                        r.x = empty ? 0.0 : (del ? ax : bx);
                        r.y = empty ? 0.0 : (del ? ay : by);
                        r.z = empty ? 0.0 : (del ? az : bz);
                        r.arg = empty ? 0.0 : arg;
                        r.dW_pair = dWp;
                        trace[(size_t)bi * n_moves + (m + lane)] = r;
                    }
                }
                if (lane == 0) sh_state[rnd & 1] = make_int4(N, k, err, 0);
            }
        }
        __syncthreads();   // the new state visible to every wavefront
        const int4 after = sh_state[rnd & 1];
        N = uni(after.x);
        m += uni(after.y);
        err = uni(after.z);   // (its move is known to wavefront 0, which reports it)
    }
    // ---------------------------------------------------- coordinates back, cells rebuilt
    // (after any move; a launch that ran none changed nothing)
    __syncthreads();
    const int64_t n_cells = m > 0 ? B.ncells : 0;
    const int64_t n_bin = m > 0 ? N : 0;
    for (int64_t c = tid; c < n_cells; c += blockDim.x) gstore(B.count + c, 0);
    __syncthreads();
    const int cap = B.cap;
    bool over = false;
    for (int64_t j = tid; j < n_bin; j += blockDim.x) {
        const double3 p = get(j);
        // every coordinate goes back, also a particle whose cell overflows (its back-pointer
        // is set with its slot below)
        gstore(B.pos + j, make_double4(p.x, p.y, p.z, 0.0));
        const int64_t c = cell_of_point(B, p.x, p.y, p.z);
        const int32_t k = atomicAdd(&B.count[c], 1);
        if (k < cap) gstore(B.ent + (c * cap + k), make_double4(p.x, p.y, p.z, pack_meta(0, (int32_t)j)));
        else over = true;
    }
    if (over) atomicOr(&sh_flag, 1);
    __syncthreads();
    int32_t maxc = 0;
    if (cap <= kWave) {
        // one wavefront per cell: an entry's slot is the number of the cell's entries with a smaller id
        for (int64_t c = wv; c < n_cells; c += W * S) {
            // the counters were raised by other wavefronts' atomics: read them where those happened
            int32_t cnt = __hip_atomic_load(B.count + c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            cnt = __builtin_amdgcn_readfirstlane(cnt > cap ? cap : cnt);
            if (cnt == 0) continue;
            double4 v = make_double4(0.0, 0.0, 0.0, 0.0);
            int32_t id = INT32_MAX;
            if (lane < cnt) {
                v = gload(B.ent + (c * cap + lane));
                id = meta_low(v.w);
            }
            int32_t rank = 0;
            for (int q = 0; q < cnt; ++q) rank += (__builtin_amdgcn_readlane(id, q) < id) ? 1 : 0;
            if (lane < cnt) {
                const int32_t slot = (int32_t)(c * cap + rank);
                gstore(B.ent + slot, v);
                gstore(B.pos + id, make_double4(v.x, v.y, v.z, pack_meta(0, slot)));
            }
            maxc = cnt > maxc ? cnt : maxc;
        }
    } else {
        for (int64_t c = tid; c < n_cells; c += blockDim.x) {
            int32_t cnt = __hip_atomic_load(B.count + c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (cnt > cap) cnt = cap;
            double4* e = B.ent + c * cap;
            for (int32_t a = 1; a < cnt; ++a) {
                const double4 v = e[a];
                const int32_t id = meta_low(v.w);
                int32_t b = a - 1;
                while (b >= 0 && meta_low(e[b].w) > id) {
                    e[b + 1] = e[b];
                    --b;
                }
                e[b + 1] = v;
            }
            for (int32_t a = 0; a < cnt; ++a) {
                const double4 v = e[a];
                gstore(B.pos + meta_low(v.w), make_double4(v.x, v.y, v.z, pack_meta(0, (int32_t)(c * cap + a))));
            }
            maxc = cnt > maxc ? cnt : maxc;
        }
    }
    maxc = wave_max_i32_uniform(maxc);
    if (lane == 0) wred[wv] = maxc;
    __syncthreads();
    double t[kStats];
    if (wv == 0)
        for (int what = 0; what < kStats; ++what) t[what] = wave_sum_vec(lane < W ? acc_s[what][lane] : 0.0);
    if (tid == 0) {
        int32_t mx = 0;
        for (int v = 0; v < W * S; ++v) mx = wred[v] > mx ? wred[v] : mx;
        if (err == GCMC_OK && sh_flag) {
            // a cell of the rebuilt list overflowed: the chain itself is complete; a rebuild with a
            // larger capacity (gcmc_cell_build) restores the cells and clears the error
            err = GCMC_ERR_CELL_OVERFLOW;
            err_move = (int64_t)(ctr0 + (uint64_t)m);
        }
        st->n = N;
        st->u_pair = U;
        st->w_pair = Wvir;
        st->maxcount = mx > st->maxcount ? mx : st->maxcount;
        st->nsp[0] = N;
        st->counter = (int64_t)(ctr0 + (uint64_t)m);
        if (err != GCMC_OK && st->error == GCMC_OK) {
            st->error = err;
            st->error_move = err_move;
        }
        ChainSums L;
        L.moves = m;
        for (int k = 0; k < 3; ++k) {
            L.att[k] = (int64_t)t[kAtt + k];
            L.acc[k] = (int64_t)t[kAcc + k];
        }
        L.sum_n = t[kSumN];
        L.sum_n2 = t[kSumN2];
        L.sum_u = t[kSumU];
        L.sum_w = t[kSumW];
        finish_launch(B, st, L, N, U, Wvir, 0, (int64_t)t[kCand], (int64_t)t[kEvals], (int64_t)t[kIncut],
                      stats ? stats + bi : nullptr);
    }
}

using resident_fn = void (*)(const DevBox*, const int32_t*, int64_t, uint64_t, gcmc_stats*, gcmc_log*);

bool resident_cfg_exists(int waves) { return waves == 4 || waves == 8; }

// waves = 4: four moves at a time by two wavefronts each, in 128 registers (one
// spilled), so that a compute unit holds two boxes, or one beside a speculative one.
// One wavefront a move left the SIMDs waiting (a wavefront issues an instruction every
// eight cycles or so): 200 to 512 boxes of up to 1,024 particles 1.95 ms per 1,000 moves,
// 1.75 with two; one box of 1,536 particles 2.20 and 1.83 (1.67 since).  waves = 8: one wavefront
// a move and as many registers as the kernel takes (512 particles, 1,000 moves: 0.91 ms,
// 0.96 with two, 0.83 with one since; from 1,000 particles on two would be 2 to 6 % faster).
int launch_chain_resident(const DevBox* d_boxes, const int32_t* d_order, int n_boxes, int waves, int64_t n_moves,
                          uint64_t ctr0, gcmc_stats* stats, gcmc_log* log, hipStream_t s) {
    if (!resident_cfg_exists(waves)) return -1;
    resident_fn f = waves == 4 ? k_chain_resident<4, 2, 4> : k_chain_resident<8, 1, 2>;
    hipLaunchKernelGGL(f, dim3(n_boxes), dim3(kWave * (waves == 4 ? 8 : 8 * 1)), 0, s, d_boxes, d_order, n_moves, ctr0,
                       stats, log);
    return 0;
}

}  // namespace gcmc
