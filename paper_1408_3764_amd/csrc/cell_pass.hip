// Whole-box passes over the cell list: total energy, per-particle energies, the
// pair virial (Sec. 3.1.1 computes each unique pair once; so do the totals here)
// and the gradient, with the pair loop of cell_pass.h.  Sums are taken in an order that
// depends on the configuration and the launch alone.
#include <algorithm>

#include "cell_pass.h"

namespace gcmc {

// f(c, i0, i1) for the items of this workgroup (one wavefront): a home cell and the
// share [i0, i1) of its nc particles, [part nc / parts, (part + 1) nc / parts).
// Workgroups go to the 8 XCDs in turn (the grid is a multiple of 8); XCD x takes the
// chunks x, x + 8, ... of `span` cells, so that neighbouring home cells find their stencils in
// the same L2 (how many chunks: pass_grid).
// The counters of 64 items are read at once, so that empty cells cost little.
template <typename F>
__device__ __forceinline__ void pass_items(const PassBox& P, int32_t parts, int32_t span, const F& f) {
    const uint32_t lane = threadIdx.x & (kWave - 1), x = blockIdx.x & 7u, stride = gridDim.x >> 3;
    for (uint32_t j0 = blockIdx.x >> 3;; j0 += kWave * stride) {
        const uint32_t j = j0 + lane * stride, k = j / (uint32_t)parts, part = j - k * (uint32_t)parts;
        const uint32_t q = k / (uint32_t)span, c = (q * 8u + x) * (uint32_t)span + (k - q * (uint32_t)span);
        const bool in = c < (uint32_t)P.ncells;
        int32_t nc = in ? gload(P.count + c) : 0;
        nc = nc > P.cap ? P.cap : nc;
        const int32_t i0 = (int32_t)((uint64_t)nc * part / (uint32_t)parts);
        const int32_t i1 = (int32_t)((uint64_t)nc * (part + 1) / (uint32_t)parts);
        for (uint64_t todo = __ballot(i0 < i1); todo; todo &= todo - 1ull) {
            const int l = (int)__builtin_ctzll(todo);
            f(__builtin_amdgcn_readlane((int32_t)c, l), __builtin_amdgcn_readlane(i0, l),
              __builtin_amdgcn_readlane(i1, l));
        }
        if (__ballot(in) != ~0ull) break;   // c grows with j
    }
}

// ------------------------------------------------------------- totals
// Rows of candidates a wavefront holds at once.  Half a stencil of 27 cells at
// liquid densities has 105-235 particles: two to four rows.
constexpr int kTotalRows = 4;
constexpr int kTotalQueue = kWave * kTotalRows + kWave;   // at most 63 left over and 4 x 64 new

// partial[block] = the block's sum of pair energies (VIR: of pair virials), each
// pair once.  Item = home cell x part: part p of `parts` takes the home
// particles [p n / parts, (p + 1) n / parts).  69 to 73 VGPRs and 3 to 3.6 KB of LDS
// per wavefront leave room for 6 or 7 wavefronts per SIMD.
template <bool MIX, bool VIR>
__global__ __launch_bounds__(kWave) void k_pair_total(const DevBox* __restrict__ boxp, int32_t parts, int32_t span,
                                                      double* partial) {
    __shared__ PassRows rows_s;
    __shared__ double qr[kTotalQueue];
    __shared__ uint8_t qp[MIX ? kTotalQueue : 1];
    __shared__ double te4[kMaxSpecies * kMaxSpecies], ts2[kMaxSpecies * kMaxSpecies];
    const DevBox& B = *boxp;
    const PassBox P = pass_box(B);
    const int lane = threadIdx.x;
    const int ns = uni(B.ns);
    if (MIX) {
        if (threadIdx.x < kMaxSpecies * kMaxSpecies) {
            te4[threadIdx.x] = B.eps4[threadIdx.x];
            ts2[threadIdx.x] = B.sig2[threadIdx.x];
        }
        __syncthreads();
    }
    const double e4 = unid(B.eps4[0]), s2 = unid(B.sig2[0]);
    uint32_t tail = 0;   // queued pairs (wave-uniform; the last ones are taken first)
    double acc = 0.0;
    auto drain = [&](uint32_t from, uint32_t cnt) {
        wave_lds_sync();
        if ((uint32_t)lane < cnt) {
            const double r2 = qr[from + lane];
            const int q = MIX ? qp[from + lane] : 0;
            const double a = MIX ? te4[q] : e4, b = MIX ? ts2[q] : s2;
            acc += VIR ? lj_virial_from_r2(r2, P.rc2, a, b) : lj_from_r2(r2, P.rc2, a, b);
        }
        wave_lds_sync();
    };
    pass_items(P, parts, span, [&](int32_t c, int32_t i0, int32_t i1) {
        const int32_t cz = c / P.M01, cy = (c - cz * P.M01) / P.M0, cx = c - cz * P.M01 - cy * P.M0;
        const double4* he = P.ent + (size_t)c * (uint32_t)P.cap;
        const bool inside = uni(pass_inside(B, cx, cy, cz) ? 1 : 0) != 0;
        stencil_rows<kTotalRows, true, MIX>(
            B, P, rows_s, c, cx, cy, cz,
            [&](const double3* e, const double* mw, int rows, int32_t rel, uint32_t own) {
                auto test = [&](auto wrap_t, auto rows_t) {
                    constexpr bool WRAP = decltype(wrap_t)::value;
                    constexpr int R = decltype(rows_t)::value;
                    double4 nx = sload4(he + i0);
                    for (int32_t i = i0; i < i1; ++i) {
                        const double4 h = nx;
                        nx = sload4(he + (i + 1 < i1 ? i + 1 : i));
                        const int sa = MIX ? meta_species(h.w) * ns : 0;
                        double r2[R];
                        uint64_t m[R];
#pragma unroll
                        for (int r = 0; r < R; ++r) {
                            r2[r] = pass_r2<WRAP>(P, e[r], h);
                            m[r] = __ballot(r2[r] < P.rc2);
                        }
#pragma unroll
                        for (int r = 0; r < R; ++r) {
                            // in the home cell, only the particles after this one
                            if (own & (1u << r)) m[r] &= __ballot((uint32_t)(rel + r * kWave) > (uint32_t)i);
                            if (__builtin_amdgcn_inverse_ballot_w64(m[r])) {
                                const uint32_t at = lanes_below(m[r], tail);
                                qr[at] = r2[r];
                                if (MIX) qp[at] = (uint8_t)(sa + meta_species(mw[r]));
                            }
                            tail += (uint32_t)__builtin_popcountll(m[r]);
                        }
                        tail = (uint32_t)uni((int32_t)tail);
                        while (tail >= (uint32_t)kWave) {
                            tail -= kWave;
                            drain(tail, kWave);
                        }
                    }
                };
                pass_dispatch<kTotalRows>(inside, rows, test);
            });
    });
    if (tail) drain(0, tail);
    acc = wave_sum(acc);
    if (lane == 0) partial[blockIdx.x] = acc;
}

// ----------------------------------------------------- per-particle energies
// e_i of every particle over its full stencil, and partial[block] = half their
// sum over the block's particles.  The queue holds the pair's home particle too,
// whose sum is an LDS accumulator; home particles go in batches of 64.
constexpr int kEachRows = 4;
constexpr int kEachQueue = kWave * kEachRows + kWave;

template <bool MIX>
__global__ __launch_bounds__(kWave) void k_pair_each(const DevBox* __restrict__ boxp, int32_t parts, int32_t span,
                                                     double* e_out, double* partial) {
    __shared__ PassRows rows_s;
    __shared__ double qr[kEachQueue];
    __shared__ uint16_t qm[kEachQueue];   // home particle of the batch | species pair << 8
    __shared__ double ae[kWave];
    __shared__ double te4[kMaxSpecies * kMaxSpecies], ts2[kMaxSpecies * kMaxSpecies];
    const DevBox& B = *boxp;
    const PassBox P = pass_box(B);
    const int lane = threadIdx.x;
    const int ns = uni(B.ns);
    if (MIX) {
        if (threadIdx.x < kMaxSpecies * kMaxSpecies) {
            te4[threadIdx.x] = B.eps4[threadIdx.x];
            ts2[threadIdx.x] = B.sig2[threadIdx.x];
        }
        __syncthreads();
    }
    const double e4 = unid(B.eps4[0]), s2 = unid(B.sig2[0]);
    double tot = 0.0;
    auto drain = [&](uint32_t from, uint32_t cnt) {
        wave_lds_sync();
        if ((uint32_t)lane < cnt) {
            const double r2 = qr[from + lane];
            const int mt = qm[from + lane], q = mt >> 8;
            const double a = MIX ? te4[q] : e4, b = MIX ? ts2[q] : s2;
            atomicAdd(&ae[mt & 0xFF], lj_from_r2(r2, P.rc2, a, b));
        }
        wave_lds_sync();
    };
    pass_items(P, parts, span, [&](int32_t c, int32_t p0, int32_t p1) {
        const int32_t cz = c / P.M01, cy = (c - cz * P.M01) / P.M0, cx = c - cz * P.M01 - cy * P.M0;
        const double4* he = P.ent + (size_t)c * (uint32_t)P.cap;
        const bool inside = uni(pass_inside(B, cx, cy, cz) ? 1 : 0) != 0;
        for (int32_t i0 = p0; i0 < p1; i0 += kWave) {
            const int32_t i1 = p1 - i0 < kWave ? p1 : i0 + kWave;
            uint32_t tail = 0;
            ae[lane] = 0.0;
            wave_lds_sync();
            stencil_rows<kEachRows, false, MIX>(
                B, P, rows_s, c, cx, cy, cz,
                [&](const double3* e, const double* mw, int rows, int32_t rel, uint32_t own) {
                    auto test = [&](auto wrap_t, auto rows_t) {
                        constexpr bool WRAP = decltype(wrap_t)::value;
                        constexpr int R = decltype(rows_t)::value;
                        double4 nx = sload4(he + i0);
                        for (int32_t i = i0; i < i1; ++i) {
                            const double4 h = nx;
                            nx = sload4(he + (i + 1 < i1 ? i + 1 : i));
                            const int sa = MIX ? meta_species(h.w) * ns : 0;
                            double r2[R];
                            uint64_t m[R];
#pragma unroll
                            for (int r = 0; r < R; ++r) {
                                r2[r] = pass_r2<WRAP>(P, e[r], h);
                                m[r] = __ballot(r2[r] < P.rc2);
                            }
#pragma unroll
                            for (int r = 0; r < R; ++r) {
                                if (own & (1u << r)) m[r] &= __ballot(rel + r * kWave != i);   // not itself
                                if (__builtin_amdgcn_inverse_ballot_w64(m[r])) {
                                    const uint32_t at = lanes_below(m[r], tail);
                                    qr[at] = r2[r];
                                    qm[at] = (uint16_t)((i - i0) | (MIX ? (sa + meta_species(mw[r])) << 8 : 0));
                                }
                                tail += (uint32_t)__builtin_popcountll(m[r]);
                            }
                            tail = (uint32_t)uni((int32_t)tail);
                            while (tail >= (uint32_t)kWave) {
                                tail -= kWave;
                                drain(tail, kWave);
                            }
                        }
                    };
                    pass_dispatch<kEachRows>(inside, rows, test);
                });
            if (tail) drain(0, tail);
            if (lane < i1 - i0) {
                const double ei = ae[lane];
                e_out[meta_low(gload(he + i0 + lane).w)] = ei;
                tot += ei;
            }
            wave_lds_sync();
        }
    });
    tot = wave_sum(tot);
    if (lane == 0) partial[blockIdx.x] = 0.5 * tot;
}

// ------------------------------------------------------------- gradient
// Per particle: dU/dr_i = sum_j (24 eps / r^2)(2 s12 - s6) d_ij over its full
// stencil, written by particle id; parameter sums per ordered species pair, each
// pair met from both ends and contributing half from each.
//
// The candidates of up to kGradRows rows and the home particles of the batch are
// kept in LDS too: the queue holds only which two particles a pair joins (4 bytes),
// and the evaluation, 64 pairs at a time, forms the distance again and adds the
// force to the home particle's sums with LDS atomics.  Neighbouring entries
// mostly belong to one home particle, so it has four copies of its sums.  Bound by
// vector issue (66 million instructions for 262,144 particles, half of them in
// the evaluation) and the LDS pipeline (0.4 of the time) together.  A mixture of
// 262,144 particles: 350 -> 190 us, 500 particles 139 -> 12 us, against one lane per
// home particle.  Rows held: 203 us with one, 192 with two, 190 with three, 202 with
// four; two copies of the sums 230, eight 204.
constexpr int kGradRows = 3;
constexpr int kGradBatch = 32;   // home particles at a time
constexpr int kGradCopies = 4;
constexpr int kGradQueue = kWave * kGradRows + kWave;

// The minimum image of a coordinate difference with its sign (the bits of
// nearest_image for |d| < L).
__device__ __forceinline__ double image_signed(double d, double L, double hL) {
    const double t = d - __builtin_copysign(L, d);
    return __builtin_fabs(d) > hL ? t : d;
}

// The wavefront's sums for the eps and sigma derivatives of each species pair q, v1 = s12 - s6 and
// v2 = 2 s12 - s6: in registers per unordered pair for up to two species, else in LDS;
// partial[(2 q + v) * gridDim.x + block].
template <int S>
__device__ __forceinline__ void pass_param_sums(const double* v1, const double* v2, const double* pv, int ns,
                                                double* partial) {
    constexpr bool REGS = S <= 2;
    const int lane = threadIdx.x;
    wave_lds_sync();
#pragma unroll
    for (int q = 0; q < S * S; ++q) {
        if (q < ns * ns) {
            double s1, s2q;
            if (REGS) {
                const int k = S == 1 ? 0 : (q + 1) / 2;
                s1 = wave_sum(v1[REGS ? k : 0]) * (q == 1 || q == 2 ? 0.5 : 1.0);
                s2q = wave_sum(v2[REGS ? k : 0]) * (q == 1 || q == 2 ? 0.5 : 1.0);
            } else {
                s1 = (pv[8 * q] + pv[8 * q + 1]) + (pv[8 * q + 2] + pv[8 * q + 3]);
                s2q = (pv[8 * q + 4] + pv[8 * q + 5]) + (pv[8 * q + 6] + pv[8 * q + 7]);
            }
            if (lane == 0) {
                partial[(size_t)(2 * q) * gridDim.x + blockIdx.x] = s1;
                partial[(size_t)(2 * q + 1) * gridDim.x + blockIdx.x] = s2q;
            }
        }
    }
}

// S: a bound on the number of species (1, 2 or kMaxSpecies).  PARAMS: also the
// sums for the eps and sigma derivatives of each species pair q: v1 = s12 - s6 and
// v2 = 2 s12 - s6, in registers for up to two species, else in LDS;
// partial[(2 q + v) * gridDim.x + block].
template <int S, bool PARAMS>
__global__ __launch_bounds__(kWave, 5) void k_pair_grad(const DevBox* __restrict__ boxp, int32_t parts, int32_t span, int64_t n,
                                                      double* grad, double* partial) {
    constexpr bool MIX = S > 1;
    constexpr int Q = S * S;
    constexpr bool REGS = S <= 2;
    __shared__ PassRows rows_s;
    __shared__ double cx_s[kGradRows * kWave], cy_s[kGradRows * kWave], cz_s[kGradRows * kWave];
    __shared__ double hx_s[kGradBatch], hy_s[kGradBatch], hz_s[kGradBatch];
    __shared__ double ax[kGradBatch * kGradCopies], ay[kGradBatch * kGradCopies], az[kGradBatch * kGradCopies];
    __shared__ uint32_t qm[kGradQueue];   // candidate | home particle of the batch << 8 | species pair << 16
    __shared__ double te4[Q], ts2[Q];
    __shared__ double pv[REGS || !PARAMS ? 1 : 2 * Q * 4];
    const DevBox& B = *boxp;
    const PassBox P = pass_box(B);
    const int lane = threadIdx.x;
    const int ns = uni(B.ns);
    if (MIX && lane < Q) {
        te4[lane] = B.eps4[lane];
        ts2[lane] = B.sig2[lane];
    }
    if (!REGS && PARAMS)
        for (int t = lane; t < 2 * Q * 4; t += kWave) pv[t] = 0.0;
    const double e4 = unid(B.eps4[0]), s2 = unid(B.sig2[0]);
    const double hL[3] = {unid(B.hL[0]), unid(B.hL[1]), unid(B.hL[2])};
    // up to two species: a sum per unordered pair, both orders of a pair add the same terms
    constexpr int K = S == 1 ? 1 : 3;
    double v1[K], v2[K];
#pragma unroll
    for (int k = 0; k < K; ++k) v1[k] = v2[k] = 0.0;

    auto drain = [&](auto wrap_t, uint32_t from, uint32_t cnt) {
        constexpr bool WRAP = decltype(wrap_t)::value;
        wave_lds_sync();
        if ((uint32_t)lane < cnt) {
            const uint32_t mt = qm[from + lane];
            const int j = mt & 0xFF, i = (mt >> 8) & 0xFF, q = MIX ? (int)(mt >> 16) : 0;
            double dx = cx_s[j] - hx_s[i], dy = cy_s[j] - hy_s[i], dz = cz_s[j] - hz_s[i];
            if (WRAP) {
                dx = image_signed(dx, P.L[0], hL[0]);
                dy = image_signed(dy, P.L[1], hL[1]);
                dz = image_signed(dz, P.L[2], hL[2]);
            }
            const double r2 = (dx * dx + dy * dy) + dz * dz;
            if (r2 != 0.0) {   // (overlapping particles: no direction, no term)
                const double ir2 = 1.0 / r2;
                const double sr2 = (MIX ? ts2[q] : s2) * ir2;
                const double s6 = sr2 * sr2 * sr2;
                const double s12 = s6 * s6;
                const double w = 2.0 * s12 - s6;
                const double coef = (6.0 * (MIX ? te4[q] : e4) * ir2) * w;
                if (grad) {
                    const int at = i * kGradCopies + (lane & (kGradCopies - 1));
                    atomicAdd(&ax[at], coef * dx);
                    atomicAdd(&ay[at], coef * dy);
                    atomicAdd(&az[at], coef * dz);
                }
                if (PARAMS) {
                    if (REGS) {
#pragma unroll
                        for (int k = 0; k < K; ++k) {   // pairs 00, 01 and 10, 11
                            const bool mine = K == 1 || (k == 0 ? q == 0 : (k == 2 ? q == 3 : q == 1 || q == 2));
                            v1[k] += mine ? s12 - s6 : 0.0;
                            v2[k] += mine ? w : 0.0;
                        }
                    } else {
                        atomicAdd(&pv[(2 * q) * 4 + (lane & 3)], s12 - s6);
                        atomicAdd(&pv[(2 * q + 1) * 4 + (lane & 3)], w);
                    }
                }
            }
        }
        wave_lds_sync();
    };

    pass_items(P, parts, span, [&](int32_t c, int32_t p0, int32_t p1) {
        const int32_t cz = c / P.M01, cy = (c - cz * P.M01) / P.M0, cx = c - cz * P.M01 - cy * P.M0;
        const double4* he = P.ent + (size_t)c * (uint32_t)P.cap;
        const bool inside = uni(pass_inside(B, cx, cy, cz) ? 1 : 0) != 0;
        for (int32_t i0 = p0; i0 < p1; i0 += kGradBatch) {
            const int32_t i1 = p1 - i0 < kGradBatch ? p1 : i0 + kGradBatch;
            int32_t id = 0;
            wave_lds_sync();
            if (lane < i1 - i0) {
                const double4 h = gload(he + i0 + lane);
                hx_s[lane] = h.x;
                hy_s[lane] = h.y;
                hz_s[lane] = h.z;
                id = meta_low(h.w);
            }
            for (int t = lane; t < kGradBatch * kGradCopies; t += kWave) ax[t] = ay[t] = az[t] = 0.0;
            wave_lds_sync();
            stencil_rows<kGradRows, false, MIX>(
                B, P, rows_s, c, cx, cy, cz,
                [&](const double3* e, const double* mw, int rows, int32_t rel, uint32_t own) {
#pragma unroll
                    for (int r = 0; r < kGradRows; ++r) {
                        cx_s[r * kWave + lane] = e[r].x;
                        cy_s[r * kWave + lane] = e[r].y;
                        cz_s[r * kWave + lane] = e[r].z;
                    }
                    auto test = [&](auto wrap_t, auto rows_t) {
                        constexpr bool WRAP = decltype(wrap_t)::value;
                        constexpr int R = decltype(rows_t)::value;
                        uint32_t tail = 0;
                        double4 nx = sload4(he + i0);
                        for (int32_t i = i0; i < i1; ++i) {
                            const double4 h = nx;
                            nx = sload4(he + (i + 1 < i1 ? i + 1 : i));
                            const uint32_t mi = ((uint32_t)(i - i0) << 8) + (MIX ? (uint32_t)(meta_species(h.w) * ns) << 16 : 0u);
                            uint64_t m[R];
#pragma unroll
                            for (int r = 0; r < R; ++r) m[r] = __ballot(pass_r2<WRAP>(P, e[r], h) < P.rc2);
#pragma unroll
                            for (int r = 0; r < R; ++r) {
                                if (own & (1u << r)) m[r] &= __ballot(rel + r * kWave != i);   // not itself
                                if (__builtin_amdgcn_inverse_ballot_w64(m[r]))
                                    qm[lanes_below(m[r], tail)] =
                                        (uint32_t)(r * kWave + lane) + (MIX ? (uint32_t)meta_species(mw[r]) << 16 : 0u) + mi;
                                tail += (uint32_t)__builtin_popcountll(m[r]);
                            }
                            tail = (uint32_t)uni((int32_t)tail);
                            while (tail >= (uint32_t)kWave) {
                                tail -= kWave;
                                drain(wrap_t, tail, kWave);
                            }
                        }
                        // the rows' coordinates leave LDS with this block: nothing stays queued
                        if (tail) drain(wrap_t, 0u, tail);
                    };
                    pass_dispatch<kGradRows>(inside, rows, test);
                });
            if (grad && lane < i1 - i0) {
                double f[3] = {0.0, 0.0, 0.0};
#pragma unroll
                for (int k = 0; k < kGradCopies; ++k) {
                    f[0] += ax[lane * kGradCopies + k];
                    f[1] += ay[lane * kGradCopies + k];
                    f[2] += az[lane * kGradCopies + k];
                }
#pragma unroll
                for (int a = 0; a < 3; ++a) grad[a * n + id] = f[a];
            }
        }
    });
    if (PARAMS) pass_param_sums<S>(v1, v2, pv, ns, partial);
}

// ------------------------------------------------------- sparse boxes
// The same passes for a vapour.  With a particle or two in a cell a wavefront of the
// kernels above gathers the candidates of a whole stencil (some 400 instructions) for one or two
// home particles.  Here each lane has a home particle of its own and walks its stencil: a
// wavefront reads the counters of 64 cells at once, lists their particles in LDS and takes 64
// of the list at a time.  A total meets each pair from one side, as above; energies and forces
// take the full stencil.  Bound by the latency of the counters and records, so the next
// counter and two records are requested ahead.  262,144 particles at a density of 0.02, calls of
// total energy / energies / gradient: 264, 332 and 399 us with the kernels above and empty cells one
// by one, 170, 174 and 255 with the counters of 64 cells at once, 76, 90 and 98 so.
constexpr int kSparseStep = 8;     // places of a cell listed at once
constexpr int kSparseAtOnce = 2;   // records requested together (one: 3 to 9 % slower, four level)
constexpr int kSparseHome = kWave - 1 + kWave * kSparseStep;
enum { kPairU, kPairW, kPairEach, kPairGrad };

// out: the energies (kPairEach) or gradients (kPairGrad, may be NULL) by particle id; partial as in the
// kernels above (S, PARAMS: as in k_pair_grad).
template <int S, int MODE, bool PARAMS>
__global__ __launch_bounds__(kWave) void k_pair_sparse(const DevBox* __restrict__ boxp, int32_t span, int64_t n,
                                                       double* out, double* partial) {
    constexpr bool MIX = S > 1, HALF = MODE <= kPairW;
    constexpr int Q = S * S, K = S == 1 ? 1 : 3;
    constexpr bool REGS = S <= 2;
    __shared__ uint32_t home[kSparseHome];
    __shared__ double te4[Q], ts2[Q];
    __shared__ double pv[REGS || !PARAMS ? 1 : 2 * Q * 4];
    const DevBox& B = *boxp;
    const PassBox P = pass_box(B);
    const int lane = threadIdx.x;
    const int ns = uni(B.ns);
    if (MIX && lane < Q) {
        te4[lane] = B.eps4[lane];
        ts2[lane] = B.sig2[lane];
    }
    if (!REGS && PARAMS)
        for (int t = lane; t < 2 * Q * 4; t += kWave) pv[t] = 0.0;
    const double e4 = unid(B.eps4[0]), s2 = unid(B.sig2[0]);
    const double hL[3] = {unid(B.hL[0]), unid(B.hL[1]), unid(B.hL[2])};
    double acc = 0.0;   // energies or virials of this lane's pairs
    double v1[K], v2[K];
#pragma unroll
    for (int k = 0; k < K; ++k) v1[k] = v2[k] = 0.0;

    // home particle h meets o: ei and f are its energy and force so far
    auto pair = [&](const double4& h, const double4& o, int sa, double& ei, double* f) {
        const double dx = image_signed(o.x - h.x, P.L[0], hL[0]), dy = image_signed(o.y - h.y, P.L[1], hL[1]),
                     dz = image_signed(o.z - h.z, P.L[2], hL[2]);
        const double r2 = (dx * dx + dy * dy) + dz * dz;
        if (!(r2 < P.rc2)) return;
        const int q = MIX ? sa + meta_species(o.w) : 0;
        const double a = MIX ? te4[q] : e4, b = MIX ? ts2[q] : s2;
        if (MODE == kPairU) acc += lj_from_r2(r2, P.rc2, a, b);
        if (MODE == kPairW) acc += lj_virial_from_r2(r2, P.rc2, a, b);
        if (MODE == kPairEach) ei += lj_from_r2(r2, P.rc2, a, b);
        if (MODE == kPairGrad && r2 != 0.0) {   // (overlapping particles: no direction, no term)
            const double ir2 = 1.0 / r2;
            const double sr2 = b * ir2;
            const double s6 = sr2 * sr2 * sr2;
            const double s12 = s6 * s6;
            const double w = 2.0 * s12 - s6;
            const double coef = (6.0 * a * ir2) * w;
            f[0] += coef * dx;
            f[1] += coef * dy;
            f[2] += coef * dz;
            if (PARAMS && REGS) {
#pragma unroll
                for (int m = 0; m < K; ++m) {   // pairs 00, 01 and 10, 11
                    const bool mine = K == 1 || (m == 0 ? q == 0 : (m == 2 ? q == 3 : q == 1 || q == 2));
                    v1[m] += mine ? s12 - s6 : 0.0;
                    v2[m] += mine ? w : 0.0;
                }
            }
            if (PARAMS && !REGS) {
                atomicAdd(&pv[(2 * q) * 4 + (lane & 3)], s12 - s6);
                atomicAdd(&pv[(2 * q + 1) * 4 + (lane & 3)], w);
            }
        }
    };
    // the listed particles from .. from + cnt - 1, one per lane
    auto batch = [&](uint32_t from, uint32_t cnt) {
        wave_lds_sync();
        if ((uint32_t)lane < cnt) {
            const uint32_t slot = home[from + lane];
            const double4 h = gload(P.ent + slot);
            const int32_t c = (int32_t)(slot / (uint32_t)P.cap), own = (int32_t)slot - c * P.cap;
            const int32_t cz = c / P.M01, cy = (c - cz * P.M01) / P.M0, cx = c - cz * P.M01 - cy * P.M0;
            const int sa = MIX ? meta_species(h.w) * ns : 0;
            double f[3] = {0.0, 0.0, 0.0}, ei = 0.0;
            // (the next cell's counter is on its way while this one's particles are met)
            auto counter = [&](int t, int32_t& nb) {
                nb = (int32_t)stencil_cell(B, gload(P.stab + t), cx, cy, cz);
                bool take = true;
                if (HALF && nb != c) {
                    int32_t d = nb - c;
                    d += d < 0 ? P.ncells : 0;
                    const uint32_t d2 = 2u * (uint32_t)d;
                    take = d2 < (uint32_t)P.ncells || (d2 == (uint32_t)P.ncells && c < nb);
                }
                return take ? gload(P.count + nb) : 0;
            };
            int32_t next = c, after = counter(0, next);
            for (int t = 0; t < P.nst; ++t) {
                const int32_t nb = next, nc = after > P.cap ? P.cap : after;
                if (t + 1 < P.nst) after = counter(t + 1, next);
                const double4* e = P.ent + (size_t)nb * (uint32_t)P.cap;
                const int32_t skip = nb == c ? own : -1;
                for (int32_t k0 = HALF ? skip + 1 : 0; k0 < nc; k0 += kSparseAtOnce) {
                    double4 o[kSparseAtOnce];
#pragma unroll
                    for (int u = 0; u < kSparseAtOnce; ++u)
                        if (k0 + u < nc) o[u] = gload(e + k0 + u);
#pragma unroll
                    for (int u = 0; u < kSparseAtOnce; ++u) {
                        if (k0 + u >= nc || (!HALF && k0 + u == skip)) continue;
                        pair(h, o[u], sa, ei, f);
                    }
                }
            }
            const int32_t id = meta_low(h.w);
            if (MODE == kPairEach) {
                out[id] = ei;
                acc += 0.5 * ei;
            }
            if (MODE == kPairGrad && out) {
#pragma unroll
                for (int a = 0; a < 3; ++a) out[a * n + id] = f[a];
            }
        }
        wave_lds_sync();
    };
    uint32_t tail = 0;   // listed particles (wave-uniform; the last ones are taken first)
    const uint32_t x = blockIdx.x & 7u;
    for (uint32_t j = blockIdx.x >> 3;; j += gridDim.x >> 3) {
        const uint32_t q = j / (uint32_t)span, b = (q * 8u + x) * (uint32_t)span + (j - q * (uint32_t)span);
        if ((uint64_t)b * kWave >= (uint64_t)P.ncells) break;   // b grows with j
        const int32_t c = (int32_t)(b * kWave) + lane;
        int32_t nc = c < P.ncells ? gload(P.count + c) : 0;
        nc = nc > P.cap ? P.cap : nc;
        for (int32_t k0 = 0; __ballot(k0 < nc); k0 += kSparseStep) {
            const int32_t left = nc - k0, m = left < 0 ? 0 : (left > kSparseStep ? kSparseStep : left);
            const int32_t incl = pass_scan(m);
            for (int32_t k = 0; k < m; ++k)
                home[tail + (uint32_t)(incl - m + k)] = (uint32_t)c * (uint32_t)P.cap + (uint32_t)(k0 + k);
            tail += (uint32_t)__builtin_amdgcn_readlane(incl, kWave - 1);
            while (tail >= (uint32_t)kWave) {
                tail -= kWave;
                batch(tail, kWave);
            }
        }
    }
    if (tail) batch(0u, tail);
    if (MODE != kPairGrad) {
        acc = wave_sum(acc);
        if (lane == 0) partial[blockIdx.x] = acc;
    }
    if (PARAMS) pass_param_sums<S>(v1, v2, pv, ns, partial);
}

// ------------------------------------------------------------ finishes
constexpr int kFinish = 1024;

__device__ __forceinline__ double finish_sum(const double* partial, int64_t np, double* red) {
    // at most 16 x 1024 partials from a cell pass: eight loads in flight per thread
    double s = 0.0;
    for (int64_t q0 = threadIdx.x; q0 < np; q0 += 8 * kFinish) {
        double v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = q0 + u * kFinish < np ? partial[q0 + u * kFinish] : 0.0;
#pragma unroll
        for (int u = 0; u < 8; ++u) s += v[u];
    }
    s = wave_sum(s);
    if ((threadIdx.x & (kWave - 1)) == 0) red[threadIdx.x / kWave] = s;
    __syncthreads();
    double t = 0.0;
    for (int w = 0; w < kFinish / kWave; ++w) t += red[w];
    return t;
}

// U_pair = sum of the partials in a fixed order; U_tail from the species
// counts; the running pair energy is reset to U_pair.
__global__ __launch_bounds__(kFinish) void k_pair_total_finish(const DevBox* __restrict__ boxp, const double* partial,
                                                                int64_t np, double* U) {
    __shared__ double red[kFinish / kWave];
    const DevBox& B = *boxp;
    const double up = finish_sum(partial, np, red);
    if (threadIdx.x == 0) {
        double ut = 0.0;
        for (int a = 0; a < B.ns; ++a)
            for (int b = 0; b < B.ns; ++b)
                ut += (double)B.st->nsp[a] * (double)B.st->nsp[b] * B.tailK[a * B.ns + b];
        U[0] = up;
        U[1] = ut;
        if (B.st->error == GCMC_OK) B.st->u_pair = up;
    }
}

// The virial W = sum over pairs inside the cutoff of -r du/dr (in a fixed order)
// and the pressure P = N / (beta V) + W / (3V) + P_tail, P_tail the pressure of
// the full potential beyond r_c: (16 pi / (3 V^2)) sum_ab N_a N_b eps_ab
// sigma_ab^3 [(2/3) q^9 - q^3], q = sigma_ab / r_c.
__global__ __launch_bounds__(kFinish) void k_pair_virial_finish(const DevBox* __restrict__ boxp,
                                                                 const double* partial, int64_t np, double* out) {
    __shared__ double red[kFinish / kWave];
    const DevBox& B = *boxp;
    const double W = finish_sum(partial, np, red);
    if (threadIdx.x == 0) {
        double pt = 0.0;
        for (int a = 0; a < B.ns; ++a)
            for (int b = 0; b < B.ns; ++b)
                pt += (double)B.st->nsp[a] * (double)B.st->nsp[b] * B.ptailK[a * B.ns + b];
        out[0] = W;
        out[1] = (double)B.st->n / (B.beta * B.V) + W / (3.0 * B.V) + pt;
        if (B.st->error == GCMC_OK) B.st->w_pair = W;
    }
}

// Block q: the parameter sums of species pair q in a fixed order, and the
// tail-correction terms: dU/d eps = 4 sum (s12 - s6), dU/d sigma = (24 eps / sigma) sum
// (2 s12 - s6) over the pairs of the box, half of it from each end of a pair.
__global__ __launch_bounds__(kFinish) void k_pair_grad_finish(const DevBox* __restrict__ boxp, const double* partial,
                                                               int64_t np, double* deps, double* dsig) {
    __shared__ double red[kFinish / kWave];
    const DevBox& B = *boxp;
    const int ns = B.ns, q = (int)blockIdx.x, a = q / ns, b = q % ns;
    const double s1 = finish_sum(partial + (size_t)(2 * q) * np, np, red);
    __syncthreads();
    const double s2 = finish_sum(partial + (size_t)(2 * q + 1) * np, np, red);
    if (threadIdx.x == 0) {
        const double pre = (8.0 * M_PI / (3.0 * B.V)) * (double)B.st->nsp[a] * (double)B.st->nsp[b];
        const double e = 0.25 * B.eps4[q], s = sqrt(B.sig2[q]);
        const double x = s / sqrt(B.rc2), x3 = x * x * x, x9 = x3 * x3 * x3;
        if (deps) deps[q] = 2.0 * s1 + pre * (s * s * s) * (x9 / 3.0 - x3);
        if (dsig) dsig[q] = (3.0 * B.eps4[q] / s) * s2 + pre * e * (s * s) * (4.0 * x9 - 6.0 * x3);
    }
}

// ------------------------------------------------------------ launchers
// How a box of n particles is cut.  Parts per home cell: enough for four
// wavefronts on every SIMD of the 256 compute units, and at most 24 particles each
// (uneven last rounds otherwise); a part keeps at least two particles, below
// which gathering the candidates costs more than the pairs.  4,000 particles in
// 512 cells: 10.2 us with one part, 7.7 with two, 6.9 with three; 32,768
// in 2,744 cells: 15.9, 14.6 with two, 16.4 with three; 262,144 in 15,625: 75 with one,
// 81 with two.  At most 16,384 workgroups, each striding over its XCD's items.
//
// Chunks of cells: one range for each XCD where the particles are everywhere (the fullest cell holds at most
// half as many again as the mean and 8), which reads the least into each L2: with sixteen, 48,000 particles of three
// species in 2,744 cells 92 us for total energy and virial against 83, 65,000 of two in 4,096 131 against 122,
// 4,000 to 262,144 of one level.  Sixteen where they fill a part of the box, which all XCDs share then: a slab of 1.5
// million, total energy 294 us against 510, gradient 651 against 1,167; a drop of 200,000 in a box of 512,000
// cells 88 against 207 (with four 102).
constexpr int kPassChunks = 8 * 16;

struct PassGrid {
    int32_t parts, span;
    unsigned blocks;
    bool sparse;
};

// The most items that an XCD has: with a wavefront for each, none comes round for a second item beside
// others that had one (an eighth of all can be fewer; the passes of the 2,744 cells in sixteen chunks: 92 us
// so, 89 with this).
static int64_t xcd_items(int64_t items, int32_t span) { return ((items + span - 1) / span + 7) / 8 * span; }

static PassGrid pass_grid(const DevBox& hb, int64_t n, int32_t maxcount) {
    const int64_t cells = hb.ncells > 0 ? hb.ncells : 1;
    const int64_t mean = n / cells;
    PassGrid g;
    // One lane per particle: fewer particles than cells and enough of them that a wavefront per cell would
    // come round several times, or up to two a cell in a large box, and no dense part (a drop, a slab), where a
    // lane would walk full cells.  us, wavefront per cell against lane per particle, gradient: 32,768 particles
    // at a mean of 0.3 80 and 60, of 0.8 64 and 73; 65,536 at 0.8 90 and 80; 262,144 at 0.8 227 and 106, at 1.6
    // 174 and 174 (energies 123 and 169); 524,288 at 1.6 300 and 222 (207 and 210).
    g.sparse = ((n >= 65536 && n < cells) || (n >= 524288 && n < 2 * cells)) && maxcount <= 16;
    if (g.sparse) {
        // groups of 64 cells in place of cells; half a listful of particles for each wavefront (one batch then
        // takes them, twice the wavefronts are in flight), a whole one where the wavefronts would run out
        const int64_t groups = (cells + kWave - 1) / kWave, half = n / (kWave / 2);
        const int64_t waves = std::min(groups, half <= 16384 ? half : n / kWave);
        g.parts = 1;
        g.span = (int32_t)((groups + kPassChunks - 1) / kPassChunks);
        g.blocks = 8u * (unsigned)std::min<int64_t>(waves == groups ? xcd_items(groups, g.span) : (waves + 7) / 8, 2048);
        return g;
    }
    int64_t parts = std::max<int64_t>((4096 + cells - 1) / cells, (mean + 23) / 24);
    parts = std::max<int64_t>(1, std::min(parts, mean / 2));
    g.parts = (int32_t)parts;
    const int chunks = maxcount <= mean + mean / 2 + 8 ? 8 : kPassChunks;
    g.span = (int32_t)((cells + chunks - 1) / chunks);
    g.blocks = 8u * (unsigned)std::min<int64_t>(xcd_items(cells, g.span) * parts, 2048);
    return g;
}

void launch_total_finish(const DevBox* d_box, const double* partial, int64_t np, double* U, hipStream_t s) {
    hipLaunchKernelGGL(k_pair_total_finish, dim3(1), dim3(kFinish), 0, s, d_box, partial, np, U);
}

int64_t pass_partials(const DevBox& hb, int64_t n) { return pass_grid(hb, n, INT32_MAX).blocks; }   // (sparse: fewer)

template <int MODE>
static void launch_sparse(const DevBox& hb, const DevBox* d_box, const PassGrid& g, int64_t n, double* out,
                          double* partial, hipStream_t s) {
    auto f = hb.ns > 1 ? k_pair_sparse<kMaxSpecies, MODE, false> : k_pair_sparse<1, MODE, false>;
    hipLaunchKernelGGL(f, dim3(g.blocks), dim3(kWave), 0, s, d_box, g.span, n, out, partial);
}

int launch_total_cells(const DevBox& hb, const DevBox* d_box, double* e_out, double* partial, int64_t partial_len,
                       double* U, hipStream_t s, int64_t n, int32_t maxcount) {
    const PassGrid g = pass_grid(hb, n, maxcount);
    if (g.blocks > partial_len) return -1;
    const bool mix = hb.ns > 1;
    if (g.sparse) {
        if (e_out) launch_sparse<kPairEach>(hb, d_box, g, n, e_out, partial, s);
        else launch_sparse<kPairU>(hb, d_box, g, n, nullptr, partial, s);
    } else if (e_out) {
        auto f = mix ? k_pair_each<true> : k_pair_each<false>;
        hipLaunchKernelGGL(f, dim3(g.blocks), dim3(kWave), 0, s, d_box, g.parts, g.span, e_out, partial);
    } else {
        auto f = mix ? k_pair_total<true, false> : k_pair_total<false, false>;
        hipLaunchKernelGGL(f, dim3(g.blocks), dim3(kWave), 0, s, d_box, g.parts, g.span, partial);
    }
    launch_total_finish(d_box, partial, g.blocks, U, s);
    return 0;
}

int launch_virial(const DevBox& hb, const DevBox* d_box, double* partial, int64_t partial_len, double* out,
                  hipStream_t s, int64_t n, int32_t maxcount) {
    const PassGrid g = pass_grid(hb, n, maxcount);
    if (g.blocks > partial_len) return -1;
    if (g.sparse) {
        launch_sparse<kPairW>(hb, d_box, g, n, nullptr, partial, s);
    } else {
        auto f = hb.ns > 1 ? k_pair_total<true, true> : k_pair_total<false, true>;
        hipLaunchKernelGGL(f, dim3(g.blocks), dim3(kWave), 0, s, d_box, g.parts, g.span, partial);
    }
    hipLaunchKernelGGL(k_pair_virial_finish, dim3(1), dim3(kFinish), 0, s, d_box, partial, (int64_t)g.blocks, out);
    return 0;
}

int64_t grad_partials_needed(const DevBox& hb, int64_t n) { return 2 * hb.ns * hb.ns * pass_partials(hb, n); }

template <int S>
static void launch_grad_of(const DevBox* d_box, const PassGrid& g, int64_t n, bool params, double* grad, double* partial,
                           hipStream_t s) {
    if (g.sparse) {
        auto f = params ? k_pair_sparse<S, kPairGrad, true> : k_pair_sparse<S, kPairGrad, false>;
        hipLaunchKernelGGL(f, dim3(g.blocks), dim3(kWave), 0, s, d_box, g.span, n, grad, partial);
    } else {
        auto f = params ? k_pair_grad<S, true> : k_pair_grad<S, false>;
        hipLaunchKernelGGL(f, dim3(g.blocks), dim3(kWave), 0, s, d_box, g.parts, g.span, n, grad, partial);
    }
}

int launch_grad(const DevBox& hb, const DevBox* d_box, double* grad, double* partial, double* deps, double* dsig,
                hipStream_t s, int64_t n, int32_t maxcount) {
    const PassGrid g = pass_grid(hb, n, maxcount);
    const bool params = deps || dsig;
    if (hb.ns > 2) launch_grad_of<kMaxSpecies>(d_box, g, n, params, grad, partial, s);
    else if (hb.ns == 2) launch_grad_of<2>(d_box, g, n, params, grad, partial, s);
    else launch_grad_of<1>(d_box, g, n, params, grad, partial, s);
    if (params)
        hipLaunchKernelGGL(k_pair_grad_finish, dim3(hb.ns * hb.ns), dim3(kFinish), 0, s, d_box, partial,
                           (int64_t)g.blocks, deps, dsig);
    return 0;
}

}  // namespace gcmc
