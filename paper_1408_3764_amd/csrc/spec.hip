// Speculative evaluation of consecutive moves of one chain, committed in order
// (the exact chain of Algorithm 1; not the "keep the first accepted" scheme the
// paper lists as future work, which would change the sampled distribution).
//
// A round takes the next W moves.  Wavefront w < W evaluates move m + w against
// the state at the start of the round:
//   * its draws, type and trial positions (a displacement or deletion picks among
//     the N expected at its commit: the round's earlier insertions and deletions
//     times the chain's running acceptance rates);
//   * the counters of its stencil cells, the candidates' records, the pair sums
//     (spec_sums: one memory round trip for each of the picked record, the
//     counters and the records);
//   * a bit for every N the move can be decided at: is its pick still the particle
//     it evaluated?
//
// The last wavefront decides.  While the others evaluate it prepares the next round
// (draws, acceptance prefactors), loads the records of particles N - W .. N - 1 and,
// once every move is known but for its sums, finds what each would add to the later
// ones if it is accepted (the pair terms with the position taken away and the one
// added, which come within the cutoff of few); then lane k holds move k of the round
// and its decision at the current state.  The rejections up to the next accepted or
// stale move take one ballot; an accepted move is committed (stores only: what it
// needs came back with its evaluation) and changes N and the later lanes:
//   * a later move whose particle it touched, or one of whose centre cells it
//     changed (the slots and counts that move would commit with), is stale: it
//     ends the round and is evaluated again in the next;
//   * so is one with a pair term so large (an overlap, beyond 64 times the well depth's
//     four) that adding and taking it away again would cost its sums digits;
//   * any other later move has its energy and virial corrected by those pair terms.
// So every move is decided on exactly the state the sequential chain would have, up
// to the rounding of its sums.
//
// The deciding wavefront is one of its own, not one that also evaluates: the
// state of the commit then takes no registers from the evaluation, whose scalar
// values were spilled and reloaded inside the candidate loop (evaluation alone: 142
// vector registers and 26 scalar spills; one kernel for both took 256 and 160).
// When eight moves a round were decided so first, a round of the 1.5-million-particle slab
// took 7.6 us (12.5 with the decisions in the first evaluating wavefront, 8.1 with the pair
// terms computed after each accepted move): the slowest evaluation 6 (three dependent
// memory round trips and the arithmetic; a wavefront issues an instruction every eight
// cycles or so, so more of them side by side cost little), the decision 0.8 and 0.8 per
// accepted move.  Per move, waves = 8, with the decisions in an evaluating wavefront and
// now: slab 1.35 -> 0.72 us, 4,000 particles 1.41 -> 0.73, cutoff 4.25 on microcells 2.5 -> 1.6.
//
// An accepted move is a serial step of that one wavefront (an instruction every eight cycles, so every
// instruction counts): N and the number of awaited moves are passed through readfirstlane, or
// the compiler keeps the whole loop under execution masks with N in vector registers (24 of them
// and 40 to 50 spills more), and the decision itself has no branch.  In a vapour, where three moves in
// four are accepted, waves = 8 took 1.83 us a move without, 1.42 with (1.60 with eight moves a round
// decided by the first evaluating wavefront); 4,000 particles 0.88 and 0.73.
//
// NG > 0: stencils of more than 32 cells (microcells, Sec. 3.3) go through
// the evaluation's path with NG groups of 64 cells; the round and the commit
// are the same.
#include "spec_eval.h"

namespace gcmc {

// Log acceptance prefactors at N = base + t: insertion V / (Lambda^3 (N + 1)),
// deletion Lambda^3 N / V (entries at N < 0 are never read).  Filled by one wavefront.
constexpr int kSpecPref = 128;
constexpr int32_t kSpecAgain = INT32_MIN;   // in place of a pair count: evaluate the later move again
__device__ __attribute__((noinline)) void spec_prefactors(double V, double lambda3, double* lpi, double* lpd, int32_t base) {
    const int lane = threadIdx.x & (kWave - 1);
    for (int t = lane; t < kSpecPref; t += kWave) {
        const double n = (double)(base + t);
        lpi[t] = log(V / (lambda3 * (n + 1.0)));
        lpd[t] = log((lambda3 * n) / V);
    }
}

// Squared minimum-image distance of two positions, the bits of dist2.
__device__ __forceinline__ double spec_r2(const DevBox& B, double px, double py, double pz, double qx, double qy,
                                          double qz) {
    const double dx = image_abs(qx - px, B.L[0]), dy = image_abs(qy - py, B.L[1]), dz = image_abs(qz - pz, B.L[2]);
    return (dx * dx + dy * dy) + dz * dz;
}

// Is cell v one of the kept stencil cells of centre cell c?  (Within the half-widths,
// and on the axes not covered whole the squared gaps between the cells sum to at most
// rc^2 (1 + 1e-9), the rule the stencil was built by; side: the cell edges.)
__device__ __forceinline__ bool kept_in_stencil(const DevBox& B, const double* side, const int32_t* v, const int32_t* c) {
    bool in = true;
    double g2 = 0.0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        int32_t d = v[a] - c[a];
        d = d < 0 ? -d : d;
        const int32_t e = B.M[a] - d;
        d = e < d ? e : d;
        in = in && (B.full[a] || d <= B.k[a]);
        const double g = d > 1 && !B.full[a] ? (double)(d - 1) * side[a] : 0.0;
        g2 += g * g;
    }
    return in && !(g2 > B.rc2 * (1.0 + 1e-9));
}

// draw_block, not inlined: the constants of log and of the generator would be kept in
// registers through the whole decision loop otherwise (177 -> 160 vector registers).
template <int RING>
__device__ __attribute__((noinline)) void spec_draws(DrawRing<RING>* ring, uint64_t ctr, uint64_t seed, uint32_t box_id, double p_disp, int b) {
    DevBox B;
    B.seed = seed; B.box_id = box_id; B.p_disp = p_disp;
    draw_block(B, ring, ctr, b);
}
// W evaluating wavefronts and one that decides.
template <int W, int CR, int NG>
__global__ __launch_bounds__(kWave*(W + 1), W == 2 ? 3 : (W == 3 || W == 7 ? 4 : 1)) void k_chain_spec(const DevBox* __restrict__ boxes,
                                                               const int32_t* __restrict__ order, int64_t n_moves,
                                                               uint64_t ctr0, gcmc_stats* stats, gcmc_log* trace) {
    constexpr int kOffs = NG ? NG * kWave / 2 : 64;    // stencil slots with a precomputed linear offset
    // forms with more than 128 registers have room for what saves an accepted move latency (in the others it
    // spills: 5 to 15 % slower there, 2 to 9 % faster here)
    constexpr bool kRoomy = W == 2 || W == 11;
    constexpr int RING = W > 8 ? 32 : (W > 4 ? 16 : (W > 2 ? 8 : 4));   // a power of two, at least 2 W
    __shared__ uint32_t tab[kMaxStencil];
    __shared__ int32_t offs[kOffs];
    __shared__ SpecRec recs_s[2][W];            // the round's evaluations, by round parity
    __shared__ SpecOwn<NG> own[W];              // cell bases and start masks, or record indices
    __shared__ double4 top[2 * W];              // records of particles base .. base + 2W - 1
    __shared__ double lpi[kSpecPref], lpd[kSpecPref];   // the deciding wavefront's prefactors
    // its statistics, lane k's sums over the moves it decided as move k of a round (counts as doubles, exact
    // below 2^53)
    enum { kAtt, kAcc = 3, kSumN = 6, kSumN2, kSumU, kSumW, kStencils, kCand, kEvals, kIncut, kStats };
    __shared__ double acc_s[kStats][W];
    __shared__ DrawRing<RING> dring;            // draws of moves m .. m + 2W - 1
    __shared__ double pq[W][kSpecQueue];    // each wavefront's queue of in-cutoff pairs
    __shared__ int32_t ready[W];            // round whose evaluation wavefront w has published
    __shared__ int32_t known[W];                // round whose move w is known but for its sums
    // what move j of the round adds to move k's energy and virial changes if it is accepted, and to its pairs
    __shared__ double corr_u[W][W], corr_w[W][W];
    __shared__ int32_t corr_n[W][W];
    // the state after a round, by round parity (a wavefront may still read the last round's)
    __shared__ int4 sh_state[2];                // N, moves decided, error
    __shared__ double2 sh_acc[2];               // running acceptance of insertions and deletions
    const int bi = order ? order[blockIdx.x] : (int)blockIdx.x;
    const DevBox B = hot_copy(boxes[blockIdx.x]);
    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane(tid / kWave);
    BoxState* st = B.st;

    if (ctr0 == GCMC_COUNTER_CONTINUE) ctr0 = (uint64_t)st->counter;
    int32_t N = uni((int32_t)st->n);   // below 2^31
    int32_t err = uni(st->error);
    const bool no_full = !(B.full[0] | B.full[1] | B.full[2]);
    for (int t = tid; t < B.nstencil; t += blockDim.x) {
        const uint32_t pk = gload(B.stab + t);
        const int tx = pk & 0x3FF, ty = (pk >> 10) & 0x3FF, tz = pk >> 20;
        tab[t] = pk;
        if (t < kOffs) offs[t] = ((tz - B.k[2]) * B.M[1] + (ty - B.k[1])) * B.M[0] + (tx - B.k[0]);
    }
    if (tid < W) ready[tid] = -1;
    if (tid < W) known[tid] = -1;
    // draws of the first 2W moves
    for (int t = tid; t < 8 * W; t += blockDim.x) draw_block(B, &dring, ctr0 + (uint64_t)(t >> 2), t & 3);
    __syncthreads();
    const bool wrong = err == GCMC_OK && B.ns != 1;
    if (wrong) err = GCMC_ERR_UNSUPPORTED;
    int64_t m = 0;
    int32_t rnd = 0;                   // rounds begun
    if (wv < W) {
        // ================================================ evaluate move m + wv of every round
        double a_ins = 0.5, a_del = 0.5;   // running acceptance of insertions and deletions
        while (err == GCMC_OK && m < n_moves) {
            rnd = rnd == INT32_MAX ? 1 : rnd + 1;   // round numbers stay positive (a flag starts at -1)
            SpecRec* recs = recs_s[rnd & 1];
            if (m + wv < n_moves) {
                // is the pick at every N the move can meet (lane o: N - (W - 1) + o) the evaluated one? (found
                // while the picked record is loaded)
                const int32_t np = N - (W - 1) + lane;
                uint64_t pm = 0;
                auto early = [&](int type, double u2, double u7, int64_t idx) {
                    pm = __ballot(lane < 2 * W - 1 && np >= 0 &&
                                  (type == GCMC_MOVE_INSERT || spec_pick(u2, u7, np) == idx));
                };
                auto pub = [&]() {
                    if (lane == 0) recs[wv].pickmask = (uint32_t)pm;
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
                    if (lane == 0) __hip_atomic_store(&known[wv], rnd, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                };
                spec_eval<CR, NG, RING>(B, tab, offs, own[wv], pq[wv], &dring, ctr0 + (uint64_t)m, wv, N, no_full, a_ins,
                                        a_del, &recs[wv], early, pub);
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
                if (lane == 0) __hip_atomic_store(&ready[wv], rnd, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
            __syncthreads();   // commit stores done and visible; the new state published
            const int4 after = sh_state[rnd & 1];
            const double2 a = sh_acc[rnd & 1];
            N = uni(after.x);
            m += uni(after.y);
            err = uni(after.z);
            a_ins = a.x;
            a_del = a.y;
        }
        return;
    }
    // ==================================================== decide and commit (wavefront W)
    int64_t err_move = st->error_move;
    if (wrong) err_move = (int64_t)ctr0;
    double U = st->u_pair;
    double Wvir = st->w_pair;
    int32_t maxc = st->maxcount;
    const double tk = B.tailK[0];
    const int cap = B.cap;
    // the arrays a commit stores to, in vector registers: as scalars they are spilled and read back word by word
    double4 *cpos = B.pos, *cent = B.ent;
    int32_t* ccount = B.count;
    if constexpr (kRoomy) asm("" : "+v"(cpos), "+v"(cent), "+v"(ccount));
    const int32_t spin_cap = wait_bound(B.wait_limit);
    const double side[3] = {B.L[0] / (double)B.M[0], B.L[1] / (double)B.M[1], B.L[2] / (double)B.M[2]};
    double n_ins = 0.0, n_del = 0.0, y_ins = 0.0, y_del = 0.0;   // insertions and deletions, and those accepted
    for (int t = lane; t < kStats * W; t += kWave) (&acc_s[0][0])[t] = 0.0;
    int32_t lbase = N - kSpecPref / 2;
    spec_prefactors(B.V, B.lambda3, lpi, lpd, lbase);
    while (err == GCMC_OK && m < n_moves) {
        rnd = rnd == INT32_MAX ? 1 : rnd + 1;
        const int32_t base = N - W;
        const int kend = (n_moves - m) < W ? (int)(n_moves - m) : W;
        const SpecRec* recs = recs_s[rnd & 1];
        // ------------------------------------------ while the others evaluate
        // the records of particles N - W .. N - 1; the draws of moves m + W .. m + 2W - 1 (the next round
        // takes moves m + k .. m + k + W - 1 with 1 <= k <= W; the others are in the ring already); the
        // prefactors, when N has drifted towards an end of their table
        const bool has_top = lane < W && base + lane >= 0;
        const double4 tv = gload(B.pos + (has_top ? base + lane : 0));
        if (lane < 4 * W) spec_draws<RING>(&dring, ctr0 + (uint64_t)(m + W) + (uint64_t)(lane >> 2), B.seed, B.box_id, B.p_disp, lane & 3);
        if (N < lbase + W || N > lbase + kSpecPref - 1 - W) {
            lbase = N - kSpecPref / 2;
            spec_prefactors(B.V, B.lambda3, lpi, lpd, lbase);
        }
        if (has_top) top[lane] = tv;
        // ------------------------------------------ the evaluations
        int kw = spin_cap < 0 ? 0 : kend;   // moves whose evaluation arrived
        int32_t spins = 0;
        auto wait_for = [&](const int32_t* flag) {   // lane's flag, of move m + lane
            while (kw > 0) {
                const bool wait = lane < kw && __hip_atomic_load(flag, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) != rnd;
                const uint64_t late = __ballot(wait);
                if (late == 0) break;
                __builtin_amdgcn_s_sleep(1);
                if (++spins > spin_cap) {
                    kw = (int)__builtin_ctzll(late);
                    break;
                }
            }
            kw = uni(kw);
            wave_lds_sync();
        };
        // the moves but for their sums; meanwhile what each would change in the later ones
        wait_for(&known[lane < W ? lane : 0]);
        for (int t = lane; t < W * W; t += kWave) {
            const int j = t / W, k = t - j * W;
            if (j < k && k < kw) {
                const SpecRec& F = recs[j];
                const SpecRec& G = recs[k];
                double u = 0.0, w = 0.0;
                int32_t n = 0;
                bool big = false;   // a term that would take digits from the sum it is added to
                if (((F.flags | G.flags) & 1) == 0) {
                    const bool fdel = F.type == GCMC_MOVE_DELETE, fins = F.type == GCMC_MOVE_INSERT;
                    const bool has_new = G.type != GCMC_MOVE_DELETE, has_old = G.type != GCMC_MOVE_INSERT;
                    const double* fb = F.p1;   // the position added (an insertion's is in p0 and p1)
                    const double* gn = G.p1;   // the new position
                    const double out = B.rc2;   // outside the cutoff: no term
                    // new position minus old one, with the position added (b) and the one taken away (a)
                    double r_nb = out, r_ob = out, r_na = out, r_oa = out;
                    if (!fdel) {
                        if (has_new) r_nb = spec_r2(B, gn[0], gn[1], gn[2], fb[0], fb[1], fb[2]);
                        if (has_old) r_ob = spec_r2(B, G.p0[0], G.p0[1], G.p0[2], fb[0], fb[1], fb[2]);
                    }
                    if (!fins) {
                        if (has_new) r_na = spec_r2(B, gn[0], gn[1], gn[2], F.p0[0], F.p0[1], F.p0[2]);
                        if (has_old) r_oa = spec_r2(B, G.p0[0], G.p0[1], G.p0[2], F.p0[0], F.p0[1], F.p0[2]);
                    }
                    auto term = [&](double r2, double sign, int32_t pairs) {
                        if (r2 < out) {   // (at most a handful of the round's pairs)
                            double tw = 0.0;
                            const double tu = lj_uw_from_r2(r2, B.rc2, B.eps4[0], B.sig2[0], tw);
                            u += sign * tu;
                            w += sign * tw;
                            n += pairs;
                            big = big || !(__builtin_fabs(tu) <= 64.0 * B.eps4[0]);
                        }
                    };
                    term(r_nb, 1.0, 1);
                    term(r_ob, -1.0, 1);
                    term(r_na, -1.0, -1);
                    term(r_oa, 1.0, -1);
                }
                corr_u[j][k] = u;
                corr_w[j][k] = w;
                corr_n[j][k] = big ? kSpecAgain : n;
            }
        }
        const bool known_k = lane < kw;
        const SpecRec& R = recs[known_k ? lane : 0];
        const int32_t type = known_k ? R.type : GCMC_MOVE_INSERT;
        const bool empty = known_k && (R.flags & 1) != 0;   // a displacement or deletion in an empty box
        const uint32_t pick = R.pickmask;
        const int32_t idx = known_k && !empty ? (int32_t)R.idx : -1;
        const int32_t cl0 = R.cl0, cl1 = R.cl1;
        const double lnA = R.lnA;
        const bool disp = type == GCMC_MOVE_DISPLACE, ins = type == GCMC_MOVE_INSERT;
        const double p0x = R.p0[0], p0y = R.p0[1], p0z = R.p0[2];   // old, inserted or deleted position
        const double p1x = R.p1[0], p1y = R.p1[1], p1z = R.p1[2];   // a displacement's new position
        const int32_t two = known_k ? R.two : 0;
        const int32_t loc = meta_low(R.rec.w);                       // slot of its particle's record
        // the log prefactor (lp) and the tail energy change at the current N (none of a displacement)
        double lpref = 0.0, dUt = 0.0;
        auto pref = [&](int32_t n) { return ins ? lpi[n - lbase] : lpd[n - lbase]; };
        auto at_n = [&](double lp) {
            const double n2 = 2.0 * (double)N;
            lpref = kRoomy && disp ? 0.0 : lp;
            dUt = kRoomy && disp ? 0.0 : tk * (ins ? n2 + 1.0 : 1.0 - n2);
        };
        if (kRoomy || !disp) at_n(pref(N));
        // the sums
        wait_for(&ready[lane < W ? lane : 0]);
        __builtin_amdgcn_s_setprio(3);
        const bool mine = lane < kw;
        double dUp = mine && !empty ? R.dUp : 0.0, dWp = mine && !empty ? R.dWp : 0.0;
        const int32_t cnt0 = R.cnt0, cnt1 = R.cnt1;                  // occupancies of its centre cells
        const int32_t id_end = meta_low(R.elast.w);                  // particle of its first cell's last entry
        int32_t r_in = R.incut;
        const int32_t n_round = N;
        bool stale = false;
        double arg = 0.0;
        const double mu = disp ? 0.0 : B.mu;
        const uint64_t sign = ins ? 1ull << 63 : 0ull;
        double aft_n = 0.0, aft_u = 0.0, aft_w = 0.0;
        uint64_t accbits = 0;
        int k = 0;
        while (k < kw) {
            const uint64_t todo = ((1ull << kw) - 1ull) & ~((1ull << k) - 1ull);
            // (branch-free: every lane's move, the others masked out below)
            const double dU = dUp + dUt;
            const double now = spec_arg(B.beta, mu, sign, dU, lpref);
            const bool ok = dU == dU && lnA < now && !empty;
            // the empty-box rejection holds only while the box is still empty
            const bool bad = empty ? N != 0 : (stale | (!ins & (((pick >> (N - n_round + W - 1)) & 1u) == 0)));
            arg = lane >= k ? now : arg;
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
            // ---------------------------------- move f is accepted: commit it (lane f holds it)
            auto of = [&](int32_t v) { return (int32_t)__builtin_amdgcn_readlane(v, f); };
            const int32_t tf = of(type), fi = of(idx), ftwo = of(two), c0 = of(cl0), c1 = of(cl1);
            const bool fdisp = tf == GCMC_MOVE_DISPLACE, fins = tf == GCMC_MOVE_INSERT, fdel = tf == GCMC_MOVE_DELETE;
            const int32_t fcnt0 = of(cnt0), fcnt1 = of(cnt1), floc = of(loc);
            // what it adds to the later moves, and their prefactors after it: requested before the commit
            const int32_t n_next = N + (fins ? 1 : (fdel ? -1 : 0));
            double add_u = 0.0, add_w = 0.0, lp = 0.0;
            int32_t add_n = 0;
            auto request = [&](int col) {
                add_u = corr_u[f][col];
                add_w = corr_w[f][col];
                add_n = corr_n[f][col];
                lp = pref(n_next);
            };
            if constexpr (kRoomy) request(lane < W ? lane : W - 1);
            int e = GCMC_OK;
            if (fins) {
                if (N >= B.max_n) e = GCMC_ERR_CAPACITY;
                else if (fcnt0 >= cap) e = GCMC_ERR_CELL_OVERFLOW;
            } else if (fdisp && ftwo) {
                if (fcnt1 >= cap) e = GCMC_ERR_CELL_OVERFLOW;
            }
            if (e != GCMC_OK) {
                err = e;
                err_move = (int64_t)(ctr0 + (uint64_t)(m + f));
                break;
            }
            // slot and cell indices fit 32 bits (cells x capacity < 2^31 for this kernel)
            const bool removes = fdel || (fdisp && ftwo);
            const bool swap = removes && floc != c0 * cap + fcnt0 - 1;
            const int32_t id_last = swap ? of(id_end) : -1;
            // the record of particle N - 1 as of now, and its cell when a deletion gives it another id
            double4 rl = make_double4(0.0, 0.0, 0.0, 0.0);
            int32_t c2 = c0;
            if (fdel && fi != N - 1) {
                rl = top[N - 1 - base];
                if (id_last != N - 1) c2 = uni((int32_t)cell_of_point(B, rl.x, rl.y, rl.z));
            }
            if (lane == f) {
                // every store to pos[j] for j in the round's window is mirrored in top[]
                if (swap) {
                    const double4 el = R.elast;
                    gstore(cent + loc, el);
                    const double w = pack_meta(meta_species(el.w), loc);
                    gstore_w(cpos + id_end, w);
                    const int32_t t = id_end - base;
                    if (t >= 0 && t < 2 * W) top[t].w = w;
                }
                if (removes) gstore(ccount + cl0, cnt0 - 1);
                double4 nr;
                int32_t j = -1;
                if (fdel) {
                    if (fi != N - 1) {
                        if (id_last == N - 1) rl.w = pack_meta(meta_species(rl.w), loc);
                        nr = rl;
                        gstore_w(cent + meta_low(rl.w), pack_meta(meta_species(rl.w), fi));
                        j = fi;
                    }
                } else {
                    // a displacement inside its cell keeps its slot; else the slot after the cell's last
                    const bool stay = fdisp && !ftwo;
                    const int32_t cn = fdisp ? cl1 : cl0, nn = fdisp ? cnt1 : cnt0;
                    const int32_t slot = stay ? loc : cn * cap + nn;
                    j = fins ? N : fi;
                    const double x = fdisp ? p1x : p0x, y = fdisp ? p1y : p0y, z = fdisp ? p1z : p0z;
                    gstore(cent + slot, make_double4(x, y, z, pack_meta(0, j)));
                    if (!stay) gstore(ccount + cn, nn + 1);
                    nr = make_double4(x, y, z, pack_meta(0, slot));
                }
                if (j >= 0) {
                    gstore(cpos + j, nr);
                    const int32_t t = j - base;
                    if (t >= 0 && t < 2 * W) top[t] = nr;
                }
            }
            if (fdisp && ftwo && fcnt1 + 1 > maxc) maxc = fcnt1 + 1;
            if (fins && fcnt0 + 1 > maxc) maxc = fcnt0 + 1;
            // ---------------------------------- what it means for the later moves of the round
            if (mine && lane > f && !empty) {
                // its slots, counts or record: the particle it touched, or one of its centre cells changed
                stale = stale || idx == (fins ? N : fi) || (swap && idx == id_last) || (fdel && idx == N - 1) ||
                        cl0 == c0 || cl0 == c2 || (fdisp && ftwo && cl0 == c1) ||
                        (two && (cl1 == c0 || cl1 == c2 || (fdisp && ftwo && cl1 == c1)));
                // its pairs with the position taken away and the one added
                if constexpr (!kRoomy) request(lane);
                dUp += add_u;
                dWp += add_w;
                r_in += add_n;
                stale = stale || add_n == kSpecAgain;
            }
            N = n_next;
            if (kRoomy) {
                if (lane > f) at_n(lp);
            } else if (!disp && lane > f) {
                at_n(pref(N));
            }
            U += read_lane(dUp, f);
            Wvir += read_lane(dWp, f);
            if (lane == f) {
                aft_n = (double)N;
                aft_u = U;
                aft_w = Wvir;
            }
            accbits |= 1ull << f;
            k = f + 1;
            wave_lds_sync();   // the mirror's new records, seen by every lane
        }
        if (err == GCMC_OK && k == kw && kw < kend) {
            err = GCMC_ERR_INTERNAL;   // move kw's evaluation did not arrive
            err_move = (int64_t)(ctr0 + (uint64_t)(m + kw));
        }
        const bool done = lane < k;
        const bool acc = done && ((accbits >> lane) & 1ull) != 0;
        n_ins += (double)__builtin_popcountll(__ballot(done && ins));
        y_ins += (double)__builtin_popcountll(__ballot(acc && ins));
        n_del += (double)__builtin_popcountll(__ballot(done && type == GCMC_MOVE_DELETE));
        y_del += (double)__builtin_popcountll(__ballot(acc && type == GCMC_MOVE_DELETE));
        if (lane == 0) {
            sh_state[rnd & 1] = make_int4(N, k, err, 0);
            sh_acc[rnd & 1] = make_double2((y_ins + 1.0) / (n_ins + 2.0), (y_del + 1.0) / (n_del + 2.0));
        }
        __builtin_amdgcn_s_setprio(0);
        __syncthreads();   // commit stores done and visible; the new state published
        // ------------------------------------------ statistics and log of the k moves decided, lane by lane
        // (the next round's evaluations run meanwhile).  The candidates of a move are those of the state
        // it was decided on: each earlier accepted move of the round that took a particle out of, or put
        // one into, one of its stencils changes their number.
        int32_t r_cand = R.cand;
        for (uint64_t left = accbits & ((1ull << k) - 1ull); left; left &= left - 1ull) {
            const int f = (int)__builtin_ctzll(left);
            const int32_t tf = __builtin_amdgcn_readlane(type, f), ftwo = __builtin_amdgcn_readlane(two, f);
            if (tf == GCMC_MOVE_DISPLACE && !ftwo) continue;   // stays in its cell
            const SpecRec& F = recs[f];
            const int32_t* a = F.c0;                                  // the cell a particle left
            const int32_t* b = tf == GCMC_MOVE_INSERT ? F.c0 : F.c1;   // the one it entered
            if (lane > f && done && !empty) {
#pragma unroll 1
                for (int q = 0; q < 4; ++q) {
                    const bool gone = q < 2, second = (q & 1) != 0;
                    if ((gone ? tf == GCMC_MOVE_INSERT : tf == GCMC_MOVE_DELETE) || (second && !two)) continue;
                    if (kept_in_stencil(B, side, gone ? a : b, second ? R.c1 : R.c0)) r_cand += gone ? -1 : 1;
                }
            }
        }
        if (done) {
            auto add = [&](int what, double v) { acc_s[what][lane] += v; };
            add(kAtt + type, 1.0);
            if (acc) add(kAcc + type, 1.0);
            add(kSumN, aft_n);
            add(kSumN2, aft_n * aft_n);
            add(kSumU, aft_u + tk * aft_n * aft_n);
            add(kSumW, aft_w);
            if (!empty) {
                add(kStencils, two ? 2.0 : 1.0);
                add(kCand, (double)r_cand);
                add(kEvals, (double)(disp && !two ? 2 * r_cand : r_cand));
                add(kIncut, (double)r_in);
            }
            if (trace) {
                gcmc_log r;
                const double dn = acc ? (ins ? 1.0 : (disp ? 0.0 : -1.0)) : 0.0;
                r.type = type;
                r.index = empty ? -1 : (ins ? (int32_t)(aft_n - dn) : idx);
                r.accepted = acc ? 1 : 0;
                r.flags = empty ? 1 : 0;
                r.dU_pair = dUp;
                r.dU_tail = empty ? 0.0 : dUt;
                r.x = empty ? 0.0 : (disp ? p1x : p0x);
                r.y = empty ? 0.0 : (disp ? p1y : p0y);
                r.z = empty ? 0.0 : (disp ? p1z : p0z);
                r.arg = empty ? 0.0 : arg;
                r.dW_pair = dWp;
                trace[(size_t)bi * n_moves + m + lane] = r;
            }
        }
        m += k;
    }
    wave_lds_sync();
    // sums over the moves of a round in a fixed order
    auto total = [&](int what) {
        double v = 0.0;
        for (int j = 0; j < W; ++j) v += acc_s[what][j];
        return v;
    };
    if (lane == 0) {
        st->n = N;
        st->u_pair = U;
        st->w_pair = Wvir;
        st->maxcount = maxc;
        st->nsp[0] = N;
        st->counter = (int64_t)(ctr0 + (uint64_t)m);
        if (err != GCMC_OK && st->error == GCMC_OK) {
            st->error = err;
            st->error_move = err_move;
        }
        ChainSums L;
        L.moves = m;
        for (int t = 0; t < 3; ++t) {
            L.att[t] = (int64_t)total(kAtt + t);
            L.acc[t] = (int64_t)total(kAcc + t);
        }
        L.sum_n = total(kSumN);
        L.sum_n2 = total(kSumN2);
        L.sum_u = total(kSumU);
        L.sum_w = total(kSumW);
        finish_launch(B, st, L, N, U, Wvir, (int64_t)total(kStencils), (int64_t)total(kCand), (int64_t)total(kEvals),
                      (int64_t)total(kIncut), stats ? stats + bi : nullptr);
    }
}

using spec_fn = void (*)(const DevBox*, const int32_t*, int64_t, uint64_t, gcmc_stats*, gcmc_log*);

struct SpecCfg {
    int key;   // the waves value of gcmc_box_set_launch that selects it
    int w;     // moves evaluated at once
    int ng;    // groups of 64 stencil cells of the microcell path, 0 for the 32-cell path
    spec_fn f;
};

// What waves selects: how many moves are evaluated at once, the deciding wavefront
// beside them.  More moves hide each other's latencies and share the decision, but
// an accepted move makes more of them stale, and a wavefront has fewer registers.
// 2: three in 128 registers, so that a compute unit holds four such boxes: 1,024 boxes of
// 1,024 to 8,192 particles, 300 moves 1.19 ms, with two moves in 160 registers 2.07 (1.74 with two
// wavefronts that did both); one box of 4,000 particles 1.74 and 2.42 us a move.  On microcells
// two.  4: seven in 128 registers, so that a compute unit holds two such boxes, or
// one and an LDS-held one: 300 moves of 64 boxes of 128 to 1,024 particles 0.47 ms, with three moves
// 0.78; of 512 boxes 0.68 and 0.99; of 1,024 boxes 1.12 and 1.02, of 1,024 to 8,192 particles 1.08 and
// 1.19.  8: eleven, the most that leave 160 registers: the slab's 10,000 moves take 9.1 ms with
// eight, 7.2 with eleven, 7.4 with 13 (128 registers) and 6.9 with 15, but at a density of 0.3, where
// one move in four is accepted, 1,000 moves 1.06 ms with eleven and 1.19 with 15, and a box of 128
// particles 1.37 and 1.76.  On microcells, where the evaluation is longer,
// 15: 4,000 moves at a cutoff of 4.25 take 8.6 ms with eight, 7.0 with eleven, 6.9 with 13 and
// 6.4 with 15.  16: 15, a workgroup having 16 wavefronts at most.
static const SpecCfg kSpecCfgs[] = {
    {2, 3, 0, k_chain_spec<3, 4, 0>},
    {4, 7, 0, k_chain_spec<7, 4, 0>},
    {8, 11, 0, k_chain_spec<11, 8, 0>},
    {16, 15, 0, k_chain_spec<15, 4, 0>},
    {2, 2, kSpecGroupsSmall, k_chain_spec<2, 8, kSpecGroupsSmall>},
    {4, 7, kSpecGroupsSmall, k_chain_spec<7, 4, kSpecGroupsSmall>},
    {8, 15, kSpecGroupsSmall, k_chain_spec<15, 4, kSpecGroupsSmall>},
    {16, 15, kSpecGroupsSmall, k_chain_spec<15, 4, kSpecGroupsSmall>},
    {2, 2, kSpecGroups, k_chain_spec<2, 8, kSpecGroups>},
    {4, 7, kSpecGroups, k_chain_spec<7, 4, kSpecGroups>},
    {8, 15, kSpecGroups, k_chain_spec<15, 4, kSpecGroups>},
    {16, 15, kSpecGroups, k_chain_spec<15, 4, kSpecGroups>},
};

// Groups of 64 cells the box's stencils need: 0 (the 32-cell path) for
// stencils of at most 32 cells whose candidates fit the owner table, else the
// smallest instantiation of the microcell path that holds both stencils of a
// displacement.
static int spec_groups(const DevBox& hb) {
    if (hb.nstencil <= 32 && (int64_t)2 * hb.nstencil * hb.cap <= kSpecOwn) return 0;
    return 2 * hb.nstencil <= kSpecGroupsSmall * kWave ? kSpecGroupsSmall : kSpecGroups;
}

// The speculative kernel handles one species and stencils of at most 512
// cells (32-bit cell slots).
bool spec_supported(const DevBox& hb) {
    return hb.ns == 1 && hb.nstencil <= kSpecMaxStencil && hb.ncells * (int64_t)hb.cap < ((int64_t)1 << 31);
}

bool spec_cfg_exists(int waves) {
    for (const SpecCfg& c : kSpecCfgs)
        if (c.key == waves) return true;
    return false;
}

// A batch launches the path with the most groups any of its boxes needs (the
// microcell path serves any stencil that fits it).
int launch_chain_spec(const DevBox* d_boxes, const int32_t* d_order, int n_boxes, int waves, int64_t n_moves,
                      uint64_t ctr0, gcmc_stats* stats, gcmc_log* log, hipStream_t s, int ng) {
    for (const SpecCfg& c : kSpecCfgs) {
        if (c.key == waves && c.ng == ng) {
            hipLaunchKernelGGL(c.f, dim3(n_boxes), dim3(kWave * (c.w + 1)), 0, s, d_boxes, d_order, n_moves, ctr0, stats,
                               log);
            return 0;
        }
    }
    return -1;
}

int spec_needs_groups(const DevBox& hb) { return spec_groups(hb); }

}  // namespace gcmc
