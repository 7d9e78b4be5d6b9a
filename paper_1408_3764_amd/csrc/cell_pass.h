// The pair loop of the whole-box passes over the cell list (total energy,
// virial, per-particle energies, gradient).
//
// One wavefront takes one home cell (or an equal share of its particles, a
// "part").  The particles of its stencil are flattened in cell order, 64 per
// row: the counters come back one lane per stencil cell, a prefix sum gives
// each nonempty cell its range, one bit per flattened position marks where a
// cell begins, so the owner of a position is the number of marks at or below it.
// Lane l holds candidate l of up to CR rows in registers, and the home
// particles are read one after the other through the scalar cache, so a pair
// test loads nothing: three subtractions, the squared distance and a compare.
// The pairs inside the cutoff (about one in six) are queued in LDS and
// evaluated 64 at a time, one per lane.
//
// What bounds it: vector issue (80 % busy in steady state; per row of 64 pairs 9
// FP64 instructions for the test, 15 where the stencil crosses the periodic
// boundary, about 8 to queue its hits, and 30 per 64 pairs evaluated).  The
// mapping before it (one lane per home particle, each walking its own stencil)
// waited on 27 dependent counter and record loads, one after the other.  Total
// energy or virial kernel, before -> now: 262,144 particles of a mixture 180 -> 72 us,
// 32,768 particles 95 -> 14 us, 4,000 67 -> 6.7 us, 500 128 -> 9.0 us.
#pragma once
#include <type_traits>

#include "gcmc_internal.h"

namespace gcmc {

constexpr int kPassRowWin = 32;  // rows of 64 flattened candidates per window of start marks

// A record through the scalar cache: the address is the same for every lane and
// nothing writes the records while a pass runs.
__device__ __forceinline__ double4 sload4(const double4* p) {
    typedef const __attribute__((address_space(4))) gcmc_d4v* cptr;
    const gcmc_d4v v = *(cptr)(uintptr_t)p;
    return make_double4(v.x, v.y, v.z, v.w);
}

// Box constants of a pass in scalar registers.
struct PassBox {
    const double4* ent;
    const int32_t* count;
    const uint32_t* stab;
    int32_t cap, nst;
    int32_t ncells, M0, M01;   // cells, cells per x row, cells per xy plane
    double L[3], rc2;
};

__device__ __forceinline__ PassBox pass_box(const DevBox& B) {
    PassBox P;
    P.ent = unip(B.ent);
    P.count = unip(B.count);
    P.stab = unip(B.stab);
    P.cap = uni(B.cap);
    P.nst = uni(B.nstencil);
    P.ncells = uni((int32_t)B.ncells);
    P.M0 = uni(B.M[0]);
    P.M01 = uni(B.M[0]) * uni(B.M[1]);
#pragma unroll
    for (int a = 0; a < 3; ++a) P.L[a] = unid(B.L[a]);
    P.rc2 = unid(B.rc2);
    return P;
}

// LDS of one wavefront's candidate rows.
struct PassRows {
    uint32_t base[kWave];           // of the k-th nonempty cell: record index minus first flattened position
    uint64_t starts[kPassRowWin];   // bit q of row r: a nonempty cell begins at flattened position 64 r + q
};

// Does the stencil of cell (cx, cy, cz) stay clear of the periodic wrap with room
// to spare?  Then every candidate lies within (k + 1) S < L/2 of the home
// particle along each axis (at least 2k + 3 cells per axis: half a cell of
// margin, far above the rounding of the cell assignment), and the minimum
// image of a coordinate difference is the difference itself, bit for bit.
__device__ __forceinline__ bool pass_inside(const DevBox& B, int32_t cx, int32_t cy, int32_t cz) {
    const int32_t c[3] = {cx, cy, cz};
    bool in = true;
#pragma unroll
    for (int a = 0; a < 3; ++a)
        in = in && B.M[a] >= 2 * B.k[a] + 3 && c[a] >= B.k[a] && c[a] <= B.M[a] - 1 - B.k[a];
    return in;
}

// |minimum image| of a coordinate difference with |d| < L: the same bits as
// |nearest_image(d)| (L - |d| rounds once either way, and rounding is monotone,
// so the smaller of the two is |d| exactly when |d| <= L/2), in two
// instructions instead of eight.
__device__ __forceinline__ double image_abs(double d, double L) {
    const double a = __builtin_fabs(d);
    return __builtin_fmin(a, L - a);
}

// Squared distance of a candidate to a home particle, the operations and order
// of dist2.
template <bool WRAP>
__device__ __forceinline__ double pass_r2(const PassBox& P, const double3& e, const double4& h) {
    double dx = e.x - h.x, dy = e.y - h.y, dz = e.z - h.z;
    if (WRAP) {
        dx = image_abs(dx, P.L[0]);
        dy = image_abs(dy, P.L[1]);
        dz = image_abs(dz, P.L[2]);
    }
    return (dx * dx + dy * dy) + dz * dz;
}

// Inclusive prefix sum over the wavefront's lanes (DPP row shifts, then the
// row broadcasts carry each row's total into the next rows).
__device__ __forceinline__ int32_t pass_scan(int32_t v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);   // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);   // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);   // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);   // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);   // row_bcast:15
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);   // row_bcast:31
    return v;
}

__device__ __forceinline__ uint32_t lanes_below(uint64_t m, uint32_t add) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, add));
}

__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
}

// Call f(e, mw, rows, rel, own) for every block of up to CR rows of candidates
// of home cell c at (cx, cy, cz): e[r] the coordinates of this lane's candidate
// in row r (x = 1e300 past the last candidate: outside any cutoff), mw[r] its
// packed species and id (META only), rows the rows in use, rel the position of this lane's row-0
// candidate relative to the home cell's first particle, bit r of own set when
// row r holds particles of the home cell.
//
// HALF: each pair of cells from one side only.  With d = c' - c modulo the number
// of cells, c takes c' when 2 d < cells (c < c' at equality): d and cells - d
// belong to the two sides, so exactly one of them takes the pair, whatever the
// stencil (axes it covers whole included; a stencil is symmetric and names a cell
// once).  SHARES > 1: only every SHARES-th block, from the `share`-th on.
template <int CR, bool HALF, bool META, int SHARES = 1, typename F>
__device__ __forceinline__ void stencil_rows(const DevBox& B, const PassBox& P, PassRows& W, int32_t c, int32_t cx,
                                             int32_t cy, int32_t cz, const F& f, uint32_t share = 0) {
    const int lane = threadIdx.x & (kWave - 1);
    uint32_t block = 0;
    for (int g0 = 0; g0 < P.nst; g0 += kWave) {
        const int t = g0 + lane;
        const bool on = t < P.nst;
        int32_t nb = c;
        if (on) nb = (int32_t)stencil_cell(B, gload(P.stab + t), cx, cy, cz);
        bool take = on;
        if (HALF && nb != c) {
            int32_t d = nb - c;
            d += d < 0 ? P.ncells : 0;
            const uint32_t d2 = 2u * (uint32_t)d;
            take = on && (d2 < (uint32_t)P.ncells || (d2 == (uint32_t)P.ncells && c < nb));
        }
        int32_t cnt = take ? gload(P.count + nb) : 0;
        cnt = cnt > P.cap ? P.cap : cnt;
        const int32_t incl = pass_scan(cnt);
        const int32_t pre = incl - cnt;
        const int32_t total = __builtin_amdgcn_readlane(incl, kWave - 1);
        const uint64_t hm = __ballot(on && nb == c);
        // the home cell's flattened range in this group of cells (none: far beyond every position)
        const int32_t hl = hm ? (int32_t)__builtin_ctzll(hm) : 0;
        const int32_t ph = hm ? __builtin_amdgcn_readlane(pre, hl) : INT32_MAX;
        const int32_t pe = hm ? ph + __builtin_amdgcn_readlane(cnt, hl) : INT32_MAX;
        const uint64_t nz = __ballot(cnt > 0);
        wave_lds_sync();   // the previous group's rows have been read
        if (cnt > 0) W.base[lanes_below(nz, 0u)] = (uint32_t)nb * (uint32_t)P.cap - (uint32_t)pre;
        uint32_t begun = 0;   // nonempty cells beginning before the current row (wave-uniform)
        for (int w0 = 0; w0 < total; w0 += kPassRowWin * kWave) {
            const int w1 = total - w0 < kPassRowWin * kWave ? total : w0 + kPassRowWin * kWave;
            wave_lds_sync();
            if (lane < kPassRowWin) W.starts[lane] = 0;
            wave_lds_sync();
            if (cnt > 0 && pre >= w0 && pre < w1)
                __hip_atomic_fetch_or(&W.starts[(pre - w0) >> 6], 1ull << (pre & 63), __ATOMIC_RELAXED,
                                      __HIP_MEMORY_SCOPE_WAVEFRONT);
            wave_lds_sync();
            for (int b0 = w0; b0 < w1; b0 += CR * kWave) {
                double3 e[CR];
                double mw[CR];
                const int left = (w1 - b0 + kWave - 1) / kWave;
                const int rows = left < CR ? left : CR;
                if (SHARES > 1 && block++ % SHARES != share) {
                    for (int r = 0; r < rows; ++r) begun += (uint32_t)__builtin_popcountll(W.starts[((b0 - w0) >> 6) + r]);
                    continue;
                }
                uint32_t own = 0;
#pragma unroll
                for (int r = 0; r < CR; ++r) {
                    e[r] = make_double3(1e300, 0.0, 0.0);
                    mw[r] = 0.0;
                    if (r < rows) {
                        const int q0 = b0 + r * kWave, q = q0 + lane;
                        const uint64_t m = W.starts[(q0 - w0) >> 6];
                        const uint32_t k = lanes_below(m, begun) + (uint32_t)((m >> lane) & 1ull) - 1u;
                        begun += (uint32_t)__builtin_popcountll(m);
                        if (q < w1) {
                            const double4* p = P.ent + (size_t)(W.base[k & (kWave - 1)] + (uint32_t)q);
                            if (META) {
                                const double4 v = gload(p);
                                e[r] = make_double3(v.x, v.y, v.z);
                                mw[r] = v.w;
                            } else {
                                const GCMC_GLOBAL_AS double* s = (const GCMC_GLOBAL_AS double*)(const double*)p;
                                typedef double d2v __attribute__((ext_vector_type(2)));
                                const d2v xy = *(const GCMC_GLOBAL_AS d2v*)s;
                                e[r] = make_double3(xy.x, xy.y, s[2]);
                            }
                        }
                        if (q0 < pe && q0 + kWave > ph) own |= 1u << r;
                    }
                }
                f(e, mw, rows, b0 + lane - ph, own);
            }
        }
    }
}

// test(wrap, rows) with both as compile-time constants: the squared distances of
// all rows are independent chains that the compiler interleaves (one row at a
// time left a wavefront waiting for its own results).
template <int CR, typename F>
__device__ __forceinline__ void pass_dispatch(bool inside, int rows, const F& test) {
    if constexpr (CR > 1) {
        if (rows < CR) {
            pass_dispatch<CR - 1>(inside, rows, test);
            return;
        }
    }
    if (inside) test(std::false_type{}, std::integral_constant<int, CR>{});
    else test(std::true_type{}, std::integral_constant<int, CR>{});
}

}  // namespace gcmc
