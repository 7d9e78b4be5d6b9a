// Evaluation of one chain move against the current state by one wavefront,
// shared by the speculative kernels (rounds of W moves, and the pipeline of a
// committer and evaluators).  The wavefront counts the insertions (I) and
// deletions (D) among the moves that precede its move and are not yet decided (N
// at the move's decision lies in [N - D, N + I]), and picks at the N expected
// from the chain's running acceptance rates; spec_sums then forms the pair sums
// over the stencils of the move's position(s).
//
// The draws (move type, pick, position, ln A) come either from a ring of
// draws in LDS that the round kernel fills for the moves it may take next, or are
// computed here (the pipelined kernel).
#pragma once
#include <type_traits>

#include "cell_pass.h"
#include "trial.h"

namespace gcmc {

constexpr int kSpecOwn = 8192;       // flattened candidates per wavefront of the 32-cell path
constexpr int kSpecRecWin = 1024;    // record indices per window of the microcell path
// A wavefront's owner buffer in LDS.  The 32-cell path keeps 64 cell bases and one start mask per 64
// flattened candidates (a second stencil begins a row of its own), written by 64-bit atomics;
// the microcell path a window of record indices.
template <int NG>
struct SpecOwn {
    uint32_t rec[kSpecRecWin];
};
template <>
struct SpecOwn<0> {
    uint32_t base[kWave];
    uint64_t starts[kSpecOwn / 64 + 1];
};
constexpr int kSpecGroups = 16;      // groups of 64 stencil cells: stencils of up to 512 cells (two for a displacement)
constexpr int kSpecMaxStencil = kSpecGroups * kWave / 2;
constexpr int kSpecGroupsSmall = 4;  // the instantiation for stencils of up to 128 cells (fewer registers)
constexpr int kSpecQueue = kWave + 4 * kWave;   // queued in-cutoff pairs per wavefront: 63 left over, 4 rows more

// Draws of the moves a round may take, one slot per move (slot = move counter
// mod RING, RING a power of two): move type, pick draw, ln A, and the three
// position draws (insertion point, or the displacement).
template <int RING>
struct DrawRing {
    double u2[RING], u7[RING], lnA[RING], px[RING], py[RING], pz[RING];
    int32_t type[RING];
};

// Philox block `b` of move `ctr` into its ring slot (one lane per block:
// block 0 gives the type, 1 the pick draw and ln A, 2 and 3 the position
// draws and the pick fields).
template <int RING>
__device__ __forceinline__ void draw_block(const DevBox& B, DrawRing<RING>* dr, uint64_t ctr, int b) {
    uint32_t c0 = (uint32_t)ctr, c1 = (uint32_t)(ctr >> 32), c2 = B.box_id, c3 = (uint32_t)b;
    philox_block(c0, c1, c2, c3, (uint32_t)B.seed, (uint32_t)(B.seed >> 32));
    const double ua = to_unit(c0, c1), ub = to_unit(c2, c3);
    const int s = (int)(ctr & (uint64_t)(RING - 1));
    if (b == 0) {
        dr->type[s] = (ua < B.p_disp) ? GCMC_MOVE_DISPLACE : ((ub < 0.5) ? GCMC_MOVE_DELETE : GCMC_MOVE_INSERT);
    } else if (b == 1) {
        dr->u2[s] = ua;
        dr->lnA[s] = log(ub);
    } else if (b == 2) {
        dr->px[s] = ua;
        dr->py[s] = ub;
    } else {
        dr->pz[s] = ua;
        dr->u7[s] = ub;
    }
}

// The coordinates of a 32-byte record (its fourth word, the id, is not
// needed: a move's own particle is excluded by its slot).
__device__ __forceinline__ double3 gload_xyz(const double4* p) {
    typedef double gcmc_d2v __attribute__((ext_vector_type(2)));
    const GCMC_GLOBAL_AS double* q = (const GCMC_GLOBAL_AS double*)p;
    const gcmc_d2v xy = *(const GCMC_GLOBAL_AS gcmc_d2v*)q;
    return make_double3(xy.x, xy.y, q[2]);
}

struct SpecRec {
    // what the in-order commit reads for every move, first
    int32_t type, flags;
    uint32_t pickmask;   // bit o: the pick still valid at N = N_round - (W - 1) + o
    int64_t idx;
    int32_t c0[3], c1[3];
    // what it reads for an accepted move
    int32_t two, cnt0, cnt1, cl0, cl1, pad;
    double dUp, dWp, lnA, u2, u7;   // pair energy change, pair virial change, ln A, pick draws
    double p0[3], p1[3];
    double4 rec, elast;
    int32_t cand, evals, incut, pad2;
};

__device__ __forceinline__ int spec_type(const DevBox& B, const U8& u) {
    return (u.u[0] < B.p_disp) ? GCMC_MOVE_DISPLACE : ((u.u[1] < 0.5) ? GCMC_MOVE_DELETE : GCMC_MOVE_INSERT);
}

__device__ __forceinline__ int64_t spec_pick(double u2, double u7, int64_t n) { return pick_particle(u2, u7, n); }

__device__ __forceinline__ int32_t spec_axis_cell(double x, double invS, int32_t M) {
    return __builtin_amdgcn_readfirstlane(axis_cell(x, invS, M));
}

// Is cell (x, y, z) inside the stencil of centre cell c?
__device__ __forceinline__ bool in_stencil(const DevBox& B, int32_t x, int32_t y, int32_t z, const int32_t* c) {
    const int32_t v[3] = {x, y, z};
    bool in = true;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        int32_t d = v[a] - c[a];
        d = d < 0 ? -d : d;
        const int32_t e = B.M[a] - d;
        d = e < d ? e : d;
        in = in && (B.full[a] || d <= B.k[a]);
    }
    return in;
}

// What the evaluation of a move returns besides the move itself.
struct SpecSums {
    double su, sw;   // pair energy and virial, the new position's minus the old one's for a displacement (every lane)
    int32_t cand, evals, incut;   // candidate records, pair distances, pairs inside the cutoff
    int32_t cnt0, cnt1;           // occupancies of the centre cells
    double4 elast;                // last entry of the first centre cell
};

// Pair sums of a move over the stencils of its position(s) by one wavefront: p0 the
// old, inserted or deleted position in cell c0 (linear cl0), p1 a displacement's
// new one in c1 (cl1); `two`: the displacement leaves its cell and has two stencils,
// else its positions share the candidates.  excl_slot: the moving particle's own
// record (never a candidate of itself).  NG: 0 for the 32-cell path, else the number
// of groups of 64 stencil cells the microcell path provides.
//
// The candidates are flattened, 64 per row, a second stencil starting a row of its
// own, so a row meets one position (or both, for a displacement inside its cell).
// Up to CR rows are requested at once; the squared distances of two to four rows
// are formed together (independent chains), and the pairs inside the cutoff, about
// one in seven, wait in LDS until 64 of them are evaluated, one per lane (the sign
// bit marks a displacement's old position, whose terms are subtracted).  mid() runs
// once while the counters are on their way.
//
// FEW: a block of at most two rows is taken by code of its own, one row after the other.
// In a gas a stencil fills a part of one row, and in the pipelined chain, where a move
// evaluated again holds up every later one, the instructions for CR rows showed (waves = 4, 20,000
// particles at density 0.02 2,610 -> 2,360 us per 1,000 moves, at 0.1 2,758 -> 2,465; at
// 0.67 2,125 -> 2,030; a cutoff of 4.25 4,110 -> 4,200).  Rounds of moves wait for their slowest
// wavefront and keep the shorter code.
template <int CR, int NG, bool FEW, typename Mid>
__device__ __forceinline__ SpecSums spec_sums(const DevBox& B, const uint32_t* tab, const int32_t* offs, SpecOwn<NG>& ownbuf,
                                              double* q, int type, int two, const double* p0, const double* p1,
                                              const int32_t* c0, const int32_t* c1, int32_t cl0, int32_t cl1,
                                              int32_t excl_slot, bool no_full, const Mid& mid) {
    const int lane = threadIdx.x & (kWave - 1);
    const int nst = B.nstencil;
    const int ncs = two ? 2 * nst : nst;
    const bool disp = type == GCMC_MOVE_DISPLACE;
    const bool fast = __builtin_amdgcn_readfirstlane(
                          (no_full && c0[0] >= B.k[0] && c0[0] <= B.M[0] - 1 - B.k[0] && c0[1] >= B.k[1] &&
                           c0[1] <= B.M[1] - 1 - B.k[1] && c0[2] >= B.k[2] && c0[2] <= B.M[2] - 1 - B.k[2] &&
                           (!two || (c1[0] >= B.k[0] && c1[0] <= B.M[0] - 1 - B.k[0] && c1[1] >= B.k[1] &&
                                     c1[1] <= B.M[1] - 1 - B.k[1] && c1[2] >= B.k[2] &&
                                     c1[2] <= B.M[2] - 1 - B.k[2])))
                              ? 1
                              : 0) != 0;
    // candidates need the minimum image unless the stencils stay inside the box with room to spare (every
    // candidate then lies within (k + 1) cells of the position along each axis, half a cell short of
    // L/2 at least, where the minimum image is the difference itself, bit for bit)
    const bool wrap = !(fast && B.M[0] >= 2 * B.k[0] + 3 && B.M[1] >= 2 * B.k[1] + 3 && B.M[2] >= 2 * B.k[2] + 3);
    SpecSums out;
    out.su = out.sw = 0.0;
    out.cand = out.evals = out.incut = 0;
    out.elast = make_double4(0, 0, 0, 0);
    uint32_t tail = 0;   // queued pairs (wave-uniform; the last ones are taken first)
    auto drain = [&](uint32_t from, uint32_t cnt) {
        wave_lds_sync();
        if ((uint32_t)lane < cnt) {
            const double v = q[from + lane];
            double w = 0.0;
            const double u = lj_uw_from_r2(__builtin_fabs(v), B.rc2, B.eps4[0], B.sig2[0], w);
            out.su += __builtin_copysign(1.0, v) * u;
            out.sw += __builtin_copysign(1.0, v) * w;
        }
        wave_lds_sync();
    };
    auto push = [&](double r2, double v) {
        const uint64_t m = __ballot(r2 < B.rc2);
        if (__builtin_amdgcn_inverse_ballot_w64(m)) q[lanes_below(m, tail)] = v;
        tail += (uint32_t)__builtin_popcountll(m);
    };
    // rows base / 64 ... of the candidates e (x = 1e300: none); rows from flattened position
    // `second` on belong to the second stencil
    auto consume = [&](const double3* e, int base, int end, int second, auto wrap_t, auto both_t, auto few_t) {
        constexpr bool WRAP = decltype(wrap_t)::value, BOTH = decltype(both_t)::value;
        constexpr int R = decltype(few_t)::value ? 2 : CR;
        constexpr int G = decltype(few_t)::value ? 1 : (CR < (BOTH ? 2 : 4) ? CR : (BOTH ? 2 : 4));
        auto dist2 = [&](const double* p, const double3& c) {
            double dx = c.x - p[0], dy = c.y - p[1], dz = c.z - p[2];
            if (WRAP) {
                dx = image_abs(dx, B.L[0]);
                dy = image_abs(dy, B.L[1]);
                dz = image_abs(dz, B.L[2]);
            }
            return (dx * dx + dy * dy) + dz * dz;
        };
#pragma unroll
        for (int g = 0; g < R; g += G) {
            if (base + g * kWave < end) {
                double ra[G], rb[G];
                bool neg[G];
#pragma unroll
                for (int r = 0; r < G; ++r) {
                    const bool sec = !BOTH && base + (g + r) * kWave >= second;   // wave-uniform
                    neg[r] = disp && !sec;
                    const double p[3] = {sec ? p1[0] : p0[0], sec ? p1[1] : p0[1], sec ? p1[2] : p0[2]};
                    ra[r] = dist2(p, e[g + r]);
                    if (BOTH) rb[r] = dist2(p1, e[g + r]);
                }
                const uint32_t t0 = tail;
#pragma unroll
                for (int r = 0; r < G; ++r) {
                    push(ra[r], neg[r] ? -ra[r] : ra[r]);
                    if (BOTH) push(rb[r], rb[r]);
                }
                tail = (uint32_t)uni((int32_t)tail);
                out.incut += (int32_t)(tail - t0);
                while (tail >= (uint32_t)kWave) {
                    tail -= kWave;
                    drain(tail, kWave);
                }
            }
        }
    };
    auto dispatch = [&](const double3* e, int base, int end, int second, auto few_t) {
        if (disp && !two) {
            if (wrap) consume(e, base, end, second, std::true_type{}, std::true_type{}, few_t);
            else consume(e, base, end, second, std::false_type{}, std::true_type{}, few_t);
        } else {
            if (wrap) consume(e, base, end, second, std::true_type{}, std::false_type{}, few_t);
            else consume(e, base, end, second, std::false_type{}, std::false_type{}, few_t);
        }
    };
    int32_t first2 = INT32_MAX, gap_end = INT32_MAX;   // flattened end of the first stencil, start of the second
    int32_t n_all = 0, n_own = 0;                      // candidates, of those the moving particle itself
    if constexpr (NG == 0) {
        const int wh = lane >= nst ? 1 : 0;
        const int t = lane - wh * nst;
        const bool cell_lane = lane < ncs;
        int32_t cell = cl0;
        if (cell_lane) {
            if (fast) {
                cell = (wh ? cl1 : cl0) + offs[t];
            } else {
                cell = (int32_t)stencil_cell(B, tab[t], wh ? c1[0] : c0[0], wh ? c1[1] : c0[1], wh ? c1[2] : c0[2]);
            }
        }
        const int32_t cnt = cell_lane ? gload(B.count + cell) : 0;
        mid();
        const int32_t incl = pass_scan(cnt);
        n_all = __builtin_amdgcn_readlane(incl, 63);
        int32_t pre = incl - cnt, total = n_all;
        if (two) {
            first2 = __builtin_amdgcn_readlane(incl, nst - 1);
            gap_end = (first2 + kWave - 1) & ~(kWave - 1);
            pre += wh ? gap_end - first2 : 0;
            total += gap_end - first2;
        }
        // lanes of the two centre cells (each appears once in its stencil)
        const int tc = (int)__builtin_ctzll(__ballot(cell_lane && !wh && cell == cl0));
        const int tc1 = two ? (int)__builtin_ctzll(__ballot(cell_lane && wh && cell == cl1)) : tc;
        out.cnt0 = __builtin_amdgcn_readlane(cnt, tc);
        out.cnt1 = __builtin_amdgcn_readlane(cnt, tc1);
        // ---- owner of each flattened candidate: the nonempty cells, in lane order, are numbered
        // k = 0, 1, ...; cbk[k] = the cell's record index minus its first flattened position,
        // and bit q of the row masks marks a flattened position q where a nonempty cell begins,
        // so the owner of q is the number of marks at or below q, minus one
        uint32_t* cbk = ownbuf.base;
        uint64_t* smask = ownbuf.starts;
        const int nrows = (total + kWave - 1) / kWave;
        for (int r = lane; r < nrows; r += kWave) smask[r] = 0;
        wave_lds_sync();
        {
            const bool nonempty = cnt > 0;
            const uint64_t nzm = __ballot(nonempty);
            if (nonempty) {
                cbk[lanes_below(nzm, 0u)] = (uint32_t)(cell * B.cap - pre);
                __hip_atomic_fetch_or(&smask[pre >> 6], 1ull << (pre & 63), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
            }
        }
        wave_lds_sync();
        uint32_t starts = 0;   // nonempty cells beginning before the current row (wave-uniform)
        // last entry of the old centre cell (removal by swap-with-last)
        if (out.cnt0 > 0) out.elast = gload(B.ent + ((size_t)(uint32_t)cl0 * (uint32_t)B.cap + (out.cnt0 - 1)));
        // ---- candidates
        auto block = [&](int base, auto few_t) {
            constexpr int R = decltype(few_t)::value ? 2 : CR;
            double3 e[R];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int row = (base >> 6) + r;
                e[r] = make_double3(1e300, 0.0, 0.0);
                if (row < nrows) {
                    const int at = row * kWave + lane;
                    const uint64_t m = smask[row];
                    const uint32_t k = lanes_below(m, starts) + (uint32_t)((m >> lane) & 1ull) - 1u;
                    starts += (uint32_t)__builtin_popcountll(m);
                    const bool in = at < total && !(at >= first2 && at < gap_end);
                    const int32_t ri = in ? (int32_t)cbk[k & (kWave - 1)] + at : cl0 * B.cap;
                    const bool own = in && ri == excl_slot;
                    n_own += __builtin_popcountll(__ballot(own));
                    if (in && !own) e[r] = gload_xyz(B.ent + (size_t)(uint32_t)ri);
                }
            }
            dispatch(e, base, total, two ? gap_end : INT32_MAX, few_t);
        };
        for (int base = 0; base < total; base += kWave * CR) {
            if (FEW && total - base <= 2 * kWave) block(base, std::true_type{});
            else block(base, std::false_type{});
        }
    } else {
        // ---- microcell stencils: groups of 64 cells, one lane per cell
        const int G = (ncs + kWave - 1) / kWave;
        int32_t cellg[NG], cntg[NG], preg[NG];
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            cellg[g] = cl0;
            cntg[g] = 0;
            if (g < G) {
                const int f = g * kWave + lane;
                const int wh = f >= nst ? 1 : 0;
                const int t = f - wh * nst;
                if (f < ncs)
                    cellg[g] = fast ? (wh ? cl1 : cl0) + offs[t]
                                    : (int32_t)stencil_cell(B, tab[t], wh ? c1[0] : c0[0], wh ? c1[1] : c0[1],
                                                            wh ? c1[2] : c0[2]);
                cntg[g] = f < ncs ? gload(B.count + cellg[g]) : 0;
            }
        }
        mid();
        out.cnt0 = out.cnt1 = 0;
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            preg[g] = 0;
            if (g < G) {
                const int f = g * kWave + lane;
                const bool on = f < ncs;
                const int wh = f >= nst ? 1 : 0;
                const int32_t incl = pass_scan(cntg[g]);
                preg[g] = n_all + incl - cntg[g];
                if (two && (nst - 1) / kWave == g) first2 = n_all + __builtin_amdgcn_readlane(incl, (nst - 1) & (kWave - 1));
                n_all += __builtin_amdgcn_readlane(incl, 63);
                // the centre cells (each appears once in its stencil)
                const uint64_t b0 = __ballot(on && !wh && cellg[g] == cl0);
                if (b0) out.cnt0 = __builtin_amdgcn_readlane(cntg[g], (int)__builtin_ctzll(b0));
                const uint64_t b1 = __ballot(on && wh && cellg[g] == cl1);
                if (b1) out.cnt1 = __builtin_amdgcn_readlane(cntg[g], (int)__builtin_ctzll(b1));
            }
        }
        int32_t total = n_all;
        if (two) {
            gap_end = (first2 + kWave - 1) & ~(kWave - 1);
            total += gap_end - first2;
#pragma unroll
            for (int g = 0; g < NG; ++g) preg[g] += (g * kWave + lane) >= nst ? gap_end - first2 : 0;
        } else {
            out.cnt1 = out.cnt0;
        }
        if (out.cnt0 > 0) out.elast = gload(B.ent + ((size_t)(uint32_t)cl0 * (uint32_t)B.cap + (out.cnt0 - 1)));
        // ---- record indices of the flattened candidates, window by window
        uint32_t* recw = ownbuf.rec;
        for (int w0 = 0; w0 < total; w0 += kSpecRecWin) {
            const int w1 = (total - w0) < kSpecRecWin ? total : w0 + kSpecRecWin;
#pragma unroll
            for (int g = 0; g < NG; ++g) {
                if (g < G) {
                    const uint32_t rb = (uint32_t)cellg[g] * (uint32_t)B.cap;
                    const int kmax = wave_max_i32_uniform(cntg[g]);
                    for (int kk = 0; kk < kmax; ++kk) {
                        const int at = preg[g] + kk;
                        if (kk < cntg[g] && at >= w0 && at < w1) recw[at - w0] = rb + (uint32_t)kk;
                    }
                }
            }
            wave_lds_sync();   // the indices other lanes of this wavefront wrote, visible to every lane
            for (int base = w0; base < w1; base += kWave * CR) {
                double3 e[CR];
#pragma unroll
                for (int r = 0; r < CR; ++r) {
                    const int at = base + r * kWave + lane;
                    e[r] = make_double3(1e300, 0.0, 0.0);
                    if (base + r * kWave < w1) {
                        const bool in = at < w1 && !(at >= first2 && at < gap_end);
                        const int32_t ri = in ? (int32_t)recw[at - w0] : cl0 * B.cap;
                        const bool own = in && ri == excl_slot;
                        n_own += __builtin_popcountll(__ballot(own));
                        if (in && !own) e[r] = gload_xyz(B.ent + (size_t)(uint32_t)ri);
                    }
                }
                dispatch(e, base, w1, two ? gap_end : INT32_MAX, std::false_type{});
            }
            wave_lds_sync();   // every lane has read this window before the next overwrites it
        }
    }
    if (tail) drain(0, tail);   // the pairs still queued
    out.su = wave_sum_uniform(out.su);
    out.sw = wave_sum_uniform(out.sw);
    out.cand = n_all - n_own;
    out.evals = disp && !two ? 2 * out.cand : out.cand;
    return out;
}

// The caller's work that needs only the move's type, draws and pick, run by
// the evaluation while the picked record is being loaded (none by default).
struct SpecNoEarly {
    __device__ __forceinline__ void operator()(int, double, double, int64_t) const {}
};

// The caller's work once the record holds everything but the sums (none by default).
struct SpecNoPub {
    __device__ __forceinline__ void operator()() const {}
};

// Wavefront k evaluates move ctr_round + k against the current state.  NG:
// 0 for the 32-cell path, else the number of groups of 64 stencil cells the
// microcell path provides (see above).  RING > 0: the draws come from `dr`
// (the moves ctr_round .. ctr_round + k must be in it); RING = 0: computed
// here, for k < 16.  pq: this wavefront's pair queue (kSpecQueue doubles of
// LDS).
template <int CR, int NG, int RING, typename Early = SpecNoEarly, typename Pub = SpecNoPub>
__device__ __forceinline__ void spec_eval(const DevBox& B, const uint32_t* tab, const int32_t* offs, SpecOwn<NG>& ownbuf,
                                          double* pq, const DrawRing<RING>* dr, uint64_t ctr_round, int k, int64_t N,
                                          bool no_full, double a_ins, double a_del, SpecRec* out,
                                          const Early& early = Early(), const Pub& pub = Pub()) {
    const int lane = threadIdx.x & (kWave - 1);
    int type;
    double u2, u7, lnA, ux, uy, uz;
    int64_t D, I;
    if constexpr (RING > 0) {
        // the round's draws from the ring; lane j < k reads the type of the j-th earlier move
        const int s = (int)((ctr_round + (uint64_t)k) & (uint64_t)(RING - 1));
        type = uni(dr->type[s]);
        u2 = dr->u2[s];
        u7 = dr->u7[s];
        lnA = dr->lnA[s];
        ux = dr->px[s];
        uy = dr->py[s];
        uz = dr->pz[s];
        const int tj = lane < k ? dr->type[(int)((ctr_round + (uint64_t)lane) & (uint64_t)(RING - 1))] : -1;
        D = __popcll(__ballot(tj == GCMC_MOVE_DELETE));
        I = __popcll(__ballot(tj == GCMC_MOVE_INSERT));
    } else {
        // draws of the round's moves: lane 4j + b computes Philox block b of move ctr_round + j
        double ua, ub;
        {
            const uint64_t c = ctr_round + (uint64_t)(lane >> 2);
            uint32_t c0 = (uint32_t)c, c1 = (uint32_t)(c >> 32), c2 = B.box_id, c3 = (uint32_t)(lane & 3);
            philox_block(c0, c1, c2, c3, (uint32_t)B.seed, (uint32_t)(B.seed >> 32));
            ua = to_unit(c0, c1);
            ub = to_unit(c2, c3);
        }
        U8 u;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            u.u[2 * q] = read_lane(ua, 4 * k + q);
            u.u[2 * q + 1] = read_lane(ub, 4 * k + q);
        }
        type = __builtin_amdgcn_readfirstlane(spec_type(B, u));
        u2 = u.u[2];
        u7 = u.u[7];
        lnA = log(u.u[3]);
        ux = u.u[4];
        uy = u.u[5];
        uz = u.u[6];
        // insertions (I) and deletions (D) among the earlier moves of the round: N at this
        // move's commit lies in [N - D, N + I]
        const int tj = (ua < B.p_disp) ? GCMC_MOVE_DISPLACE : ((ub < 0.5) ? GCMC_MOVE_DELETE : GCMC_MOVE_INSERT);
        const bool earlier = (lane & 3) == 0 && (lane >> 2) < k;
        D = __popcll(__ballot(earlier && tj == GCMC_MOVE_DELETE));
        I = __popcll(__ballot(earlier && tj == GCMC_MOVE_INSERT));
    }
    const double ud[3] = {ux, uy, uz};
    if (type != GCMC_MOVE_INSERT && N == 0) {
        if (lane == 0) {
            out->type = type;
            out->flags = 1;
            out->lnA = 0.0;
            out->u2 = u2;
            out->u7 = u7;
            out->cand = out->evals = out->incut = 0;
        }
        pub();
        return;
    }
    int64_t idx = -1;
    double4 rec = make_double4(0, 0, 0, 0);
    double p0[3], p1[3];
    if (type == GCMC_MOVE_INSERT) {
#pragma unroll
        for (int a = 0; a < 3; ++a) p0[a] = wrap_into_box(B.L[a] * ud[a], B.L[a]);
        early(type, u2, u7, idx);
    } else {
        // the pick at the N expected at commit from the running acceptance rates
        const int64_t n_lo = (N - D) > 1 ? (N - D) : 1, n_hi = N + I;
        int64_t n_c = (int64_t)floor((double)N + (double)I * a_ins - (double)D * a_del + 0.5);
        n_c = uni64(n_c < n_lo ? n_lo : (n_c > n_hi ? n_hi : n_c));
        idx = spec_pick(u2, u7, n_c);
        // (an index past N names a particle an earlier insertion of the round may add: read inside the array,
        // used only if that insertion is decided first)
        rec = gload(B.pos + (idx < B.max_n ? idx : B.max_n - 1));
        early(type, u2, u7, idx);   // the caller's work that needs only the pick, while the record loads
        p0[0] = rec.x; p0[1] = rec.y; p0[2] = rec.z;
    }
    int32_t c0[3], c1[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) c0[a] = spec_axis_cell(p0[a], B.invS[a], B.M[a]);
    const int32_t cl0 = (c0[2] * B.M[1] + c0[1]) * B.M[0] + c0[0];
    int32_t cl1 = cl0;
    int same = 1;
    if (type == GCMC_MOVE_DISPLACE) {
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            p1[a] = wrap_into_box(p0[a] + B.max_disp * (2.0 * ud[a] - 1.0), B.L[a]);
            c1[a] = spec_axis_cell(p1[a], B.invS[a], B.M[a]);
        }
        cl1 = (c1[2] * B.M[1] + c1[1]) * B.M[0] + c1[0];
        same = __builtin_amdgcn_readfirstlane(cl1 == cl0 ? 1 : 0);
    } else {
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            p1[a] = p0[a];
            c1[a] = c0[a];
        }
    }
    const int two = (type == GCMC_MOVE_DISPLACE && !same) ? 1 : 0;
    const int32_t excl_slot = type == GCMC_MOVE_INSERT ? -1 : meta_low(rec.w);
    // everything of the record but the sums, written while the counters are loaded
    auto mid = [&]() {
        if (lane == 0) {
            out->lnA = lnA;
            out->u2 = u2;
            out->u7 = u7;
            out->type = type;
            out->flags = 0;
            out->two = two;
            out->idx = idx;
            out->rec = rec;
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                out->p0[a] = p0[a];
                out->p1[a] = p1[a];
                out->c0[a] = c0[a];
                out->c1[a] = c1[a];
            }
            out->cl0 = cl0;
            out->cl1 = cl1;
        }
        pub();
    };
    const SpecSums S = spec_sums<CR, NG, RING == 0>(B, tab, offs, ownbuf, pq, type, two, p0, p1, c0, c1, cl0, cl1,
                                                    excl_slot, no_full, mid);
    const double dUp = type == GCMC_MOVE_DELETE ? -S.su : S.su;
    const double dWp = type == GCMC_MOVE_DELETE ? -S.sw : S.sw;
    if (lane == 0) {
        out->dUp = dUp;
        out->dWp = dWp;
        out->elast = S.elast;
        out->cnt0 = S.cnt0;
        out->cnt1 = S.cnt1;
        out->cand = S.cand;
        out->evals = S.evals;
        out->incut = S.incut;
    }
}

// Log acceptance ratio of a move (Eqs. 3-5) from its energy change and its log prefactor (0 for a
// displacement), without a branch on its type: sign holds the sign bit for an insertion, mu is 0 for a
// displacement.
__device__ __forceinline__ double spec_arg(double beta, double mu, uint64_t sign, double dU, double lpref) {
    const double y = beta * (mu + __builtin_bit_cast(double, __builtin_bit_cast(uint64_t, dU) ^ sign));
    return lpref - __builtin_bit_cast(double, __builtin_bit_cast(uint64_t, y) ^ sign);
}

}  // namespace gcmc
