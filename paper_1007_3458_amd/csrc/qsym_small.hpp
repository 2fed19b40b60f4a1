// qsym_small.hpp -- whole steps of small systems in one launch: one
// workgroup per system, the state in LDS, every phase of the step separated
// by workgroup barriers instead of kernel boundaries.
#pragma once
#include "qsym_kernels.hpp"
#include "qsym_route.hpp"

namespace qsym {

// ------------------------------------------------------------------------
// What bounds a small context is its launches: eight kernels a step, 4 to 5
// us each from dispatch to completion however little they do.  Here a launch
// takes up to kSmallSteps steps of every system, and what bounds it is the
// latency of the chains of one step: at 104 bodies 86k cycles, of them 38k
// in the two kicks, 21k in Kepler's equation (the slowest body's iterations),
// 12k in a two-body set's Hermite.  Measured per step, in us, the step's own
// kernels and this: 8 systems of four planets 46 and 19, 16 of 100 bodies 71
// and 40, 256 of 100 102 and 41, 512 of 250 bodies 190 and 165.  Which contexts
// take it: small_route.
//
// The arithmetic, its order and its results are those of the step's kernels
// over full-matrix kick shapes bit for bit: the same device functions,
// partial sums over the same j-chunks added in the same order, the momentum
// over the same 64-body chunks.
//
// Up to kSmallMax bodies a system: a kick then is at most 128 pair terms a
// thread (two chunks of 128 over 512 threads), and no set can need the
// Hermite's grid phase.
// ------------------------------------------------------------------------
constexpr int kSmallThreads = 512;   // as k_hermite, whose set functions run here
constexpr int kSmallSteps = 256;     // steps per launch
constexpr int kSmallQ = 1024;        // queued pairs under the crude bound, and candidates kept in LDS
constexpr int kSmallEnc = kSmallMax * 4 + 64;   // encounter pairs of one system (its segment)

// words of the launch's own counters (zero between launches)
enum SmallWord {
    SW_TICKET = 0,   // workgroups done
    SW_OVF,          // kSmallSteps - (first step that overflowed), 0: none
    SW_CAND,         // last step: candidates, sets and members placed so far
    SW_NSETS,
    SW_NU,
    SW_STEP0,        // [kSmallSteps] candidates of every step over all systems
    SW_COUNT = SW_STEP0 + kSmallSteps
};

// figures each workgroup leaves for the last one to add up
enum SmallStat {
    SS_ENC = 0, SS_MAXSET, SS_SUB, SS_TENC, SS_TSUB, SS_WHOLE, SS_STATUS, SS_HIST,
    SS_KIT = SS_HIST + kHist, SS_KMAX, SS_KRS, SS_COUNT
};

struct SmallArgs {
    Dev d;
    unsigned long long *w;     // [SW_COUNT]
    unsigned long long *st;    // [nsys][SS_COUNT]
    HermArgs h;                // tau, G, epsH, eta, eta_s, max_substeps
    double aE, aH, cs, planet_mass;
    double r2seed, c158, c32;
    long long cap;             // candidate capacity
    int jc[2];                 // j-chunk of the plain and of the crude kick
    int hill_mode, kepler_mode;
    int nsys, nsteps;
    int first;                 // 1: the first launch of a call
    int redo;                  // 1: after a launch in which a system overflowed (see below)
};

// state of the workgroup's system in LDS
struct SmallLds {
    double x[kSmallMax], y[kSmallMax], z[kSmallMax], vx[kSmallMax], vy[kSmallMax], vz[kSmallMax];
    double m[kSmallMax], h[kSmallMax], A[kSmallMax], ch[kSmallMax], cv[kSmallMax];
    double x0[kSmallMax], y0[kSmallMax], z0[kSmallMax];
    double vx0[kSmallMax], vy0[kSmallMax], vz0[kSmallMax];
    double bk[6][kSmallMax];                    // the step's start
    double4 sj[kSmallMax];                      // x, y, z, G m of the kick
    double part[3][kSmallMax];                  // kick accelerations
    double pm[kSmallMax / 64][3];               // momentum partials of the 64-body chunks
    double smax[3][kSmallMax / 64];
    unsigned long long large[kSmallMax / 64];   // bodies left out of the crude maxima
    unsigned q[kSmallQ];                        // pairs i << 16 | j
    unsigned cand[kSmallQ];
    unsigned enc[kSmallEnc];
    unsigned nq, ncand, nenc;
    int bad;
    // set partition
    unsigned lab[kSmallMax];                    // union-find labels, then roots
    int uq[kSmallMax], mem[kSmallMax], sid[kSmallMax];
    int sstart[kSmallMax / 2 + 1], scount[kSmallMax / 2 + 1];
    unsigned long long rcb[kSmallMax / 2 + 1];
    unsigned long long inenc[kSmallMax / 64], root[kSmallMax / 64];
    int planets[kSmallMax / 2 + 1];
    int whole, nsets, nu, maxset, sub, hfail;
    // Hermite staging (x, y, z, u, v, w, m); between the sets the kick's tile
    // and, at the end, the waves' shares of the figures: one array for all
    double stage[8][kHermLds];
    double hr[6 * kCoopMin];
    double red[kHermThreads / 64 + 1];
    unsigned hist[kHist];
    unsigned long long kit;
    unsigned kmax, krs;
    int base_cand, base_set, base_mem, last;
};

// momentum of the system from the chunk partials: the value system_momentum's
// butterfly over the lanes gives (at most four of them hold a partial)
__device__ __forceinline__ void small_momentum(const SmallLds &L, int nch, double P[3])
{
    static_assert(kSmallMax <= 4 * 64, "at most four chunks");
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        double p[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) p[c] = c < nch ? 0.0 + L.pm[c][k] : 0.0;
        P[k] = (p[0] + p[1]) + (p[2] + p[3]);
    }
}

// per-system upper bound of a body's crude limit, either Hill form
__device__ __forceinline__ double small_bound(const KickArgs &ka, double hi, double Ai, double vi,
                                              double hj, double Aj, double vj)
{
    return ka.hill_mode == 0 ? pair_bound<1>(ka, hi, Ai, vi, hj, Aj, vj)
                             : pair_bound<2>(ka, hi, Ai, vi, hj, Aj, vj);
}

// All-pairs kick in tiles of T bodies j, two phases each.  First every thread
// forms G m_j r^-3 of eight pairs (body i = t mod NB, NB = 64, 128 or 256, and
// every NG-th j of the tile, NG = 512 / NB, T = 8 NG) into LDS: eight chains
// side by side.  Then a thread per body and component (two components where
// 512 threads are short of three a body) adds the tile's terms in ascending
// j, the chain that fixes the result's bits: one difference and one fma a
// term.  A thread per body doing both, four pair terms at a time, took 22k
// cycles at 104 bodies, this 17k.  acc is valid on threads below n.  CRUDE:
// pairs i < j under the crude bound are queued in q (as k_kick).  Called by
// the whole workgroup.
template <int LG, bool CRUDE, int PREC>
__device__ __forceinline__ void small_kick_tiles(SmallLds &L, const KickArgs &ka, int n, int jc,
                                                 double th2)
{
    constexpr int NB = 1 << LG, NG = kSmallThreads >> LG, T = 8 * NG;
    const int t = threadIdx.x;
    const int i = t & (NB - 1), g = __builtin_amdgcn_readfirstlane(t >> LG);
    const bool ok = i < n;
    const int ii = ok ? i : 0;
    const double xi = L.x[ii], yi = L.y[ii], zi = L.z[ii];
    auto push = [&](int j) {
        const unsigned k = atomicAdd(&L.nq, 1u);
        if (k < (unsigned)kSmallQ) L.q[k] = ((unsigned)i << 16) | (unsigned)j;
    };
    if constexpr (CRUDE) {
        // the bodies left out of the maxima (as in k_kick), by the first
        // thread of each body
        if (ok && g == 0) {
            const double hi = L.ch[ii], Ai = L.A[ii], vi = L.cv[ii];
            for (int w = 0; w < (NB >> 6); ++w)
                for (unsigned long long m = L.large[w]; m; m &= m - 1) {
                    const int j = 64 * w + __builtin_ctzll(m);
                    if (j <= i) continue;
                    const double dx = L.sj[j].x - xi, dy = L.sj[j].y - yi, dz = L.sj[j].z - zi;
                    const double r2 = fma(dz, dz, fma(dy, dy, fma(dx, dx, r2_seed<PREC>(ka))));
                    if (!(r2 < th2) && r2 < small_bound(ka, hi, Ai, vi, L.ch[j], L.A[j], L.cv[j]))
                        push(j);
                }
        }
    }
    double *const ms = &L.stage[0][0] + i;   // [T][NB] over the Hermite's staging
    static_assert(sizeof(L.stage) >= T * NB * sizeof(double), "the tile fits the staging");
    // components of this thread in the second phase
    constexpr bool three = NG >= 3;
    const int c0 = three ? g : (g == 0 ? 0 : 2);
    const bool two = !three && g == 0;
    const double *const sc = reinterpret_cast<const double *>(L.sj) + c0;
    const double p0 = c0 == 0 ? xi : (c0 == 1 ? yi : zi), p1 = yi;
    double s0 = 0.0, s1 = 0.0, a0 = 0.0, a1 = 0.0;
    int cnext = jc;   // end of the current chunk
    for (int jt = 0; jt < n; jt += T) {
        const int nt = min(T, n - jt);
        // a row of j past the tile's end repeats its last j and is not used;
        // a tile of one row forms that row only
        auto factors = [&](auto rows) {
            constexpr int Q = decltype(rows)::value;
            double dx[Q], dy[Q], dz[Q], gm[Q], r2[Q], m[Q];
            unsigned hits = 0u;
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const double4 pj = L.sj[jt + min(g + NG * q, nt - 1)];
                dx[q] = pj.x;
                dy[q] = pj.y;
                dz[q] = pj.z;
                gm[q] = pj.w;
            }
            __builtin_amdgcn_sched_barrier(0);   // all of a row's reads first
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                dx[q] = dx[q] - xi;
                dy[q] = dy[q] - yi;
                dz[q] = dz[q] - zi;
            }
            pair_factors<Q, PREC>(gm, dx, dy, dz, ka.r2seed, ka.c158, ka.c32, r2, m);
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                ms[(g + NG * q) * NB] = m[q];
                if constexpr (CRUDE) {
                    const int jl = g + NG * q;
                    hits |= (ok && r2[q] < th2 && jt + jl > i && jl < nt) ? 1u << q : 0u;
                }
            }
            if constexpr (CRUDE)
                for (; hits; hits &= hits - 1) push(jt + g + NG * __builtin_ctz(hits));
        };
        if (nt > NG) factors(std::integral_constant<int, 8>{});
        else factors(std::integral_constant<int, 1>{});
        __syncthreads();
        // blocks of eight terms requested before any is added; in a block
        // past the tile's or the chunk's end, terms of zero
        auto add = [&](auto both) {
            constexpr bool B = decltype(both)::value;
            for (int jl = 0; jl < nt;) {
                const int je = min(nt, cnext - jt);
                for (; jl < je; jl += 8) {
                    const double *pm = ms + jl * NB, *pc = sc + 4 * (jt + jl);
                    double m[8], u[8], v[8];
                    if (jl + 8 <= je) {
#pragma unroll
                        for (int q = 0; q < 8; ++q) {
                            m[q] = pm[q * NB];
                            u[q] = pc[4 * q];
                            if constexpr (B) v[q] = pc[4 * q + 1];
                        }
                    } else {
#pragma unroll
                        for (int q = 0; q < 8; ++q) {
                            const int k = min(q, je - 1 - jl);
                            m[q] = q == k ? pm[k * NB] : 0.0;
                            u[q] = pc[4 * k];
                            if constexpr (B) v[q] = pc[4 * k + 1];
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int q = 0; q < 8; ++q) {
                        s0 = fma(m[q], u[q] - p0, s0);
                        if constexpr (B) s1 = fma(m[q], v[q] - p1, s1);
                    }
                }
                jl = je;
                if (jt + je == cnext || jt + je == n) {
                    // the chunks' sums in slot order
                    a0 += s0;
                    a1 += s1;
                    s0 = s1 = 0.0;
                    cnext += jc;
                }
            }
        };
        if constexpr (three) {
            if (g < 3) add(std::false_type{});
        } else {
            if (two) add(std::true_type{});
            else add(std::false_type{});
        }
        __syncthreads();
    }
    if (ok && (!three || g < 3)) {
        L.part[c0][i] = a0;
        if (two) L.part[1][i] = a1;
    }
}

template <bool CRUDE, int PREC>
__device__ __forceinline__ void small_kick(SmallLds &L, const KickArgs &ka, int n, int jc,
                                           double acc[3])
{
    const int t = threadIdx.x;
    const int nb = (n + 63) & ~63;
    if (t < n) L.sj[t] = make_double4(L.x[t], L.y[t], L.z[t], ka.G * L.m[t]);
    if constexpr (CRUDE) {
        if (t < kSmallMax) {
            double t0 = t < n ? L.ch[t] : 0.0, t1 = t < n ? L.A[t] : 0.0, t2 = t < n ? L.cv[t] : 0.0;
            const unsigned long long lg = ka.hill_mode == 0 ? split_large<1>(t < n, t0, t1, t2)
                                                            : split_large<2>(t < n, t0, t1, t2);
            t0 = wave_max(t0);
            t1 = wave_max(t1);
            t2 = wave_max(t2);
            if ((t & 63) == 0) {
                L.large[t >> 6] = lg;
                L.smax[0][t >> 6] = t0;
                L.smax[1][t >> 6] = t1;
                L.smax[2][t >> 6] = t2;
            }
        }
        if (t == 0) {
            L.nq = 0u;
            L.ncand = 0u;
        }
    }
    __syncthreads();
    auto bound = [&](int i) {
        double HT = L.smax[0][0], AT = L.smax[1][0], VT = L.smax[2][0];
        for (int w = 1; w < (nb >> 6); ++w) {
            HT = fmax(HT, L.smax[0][w]);
            AT = fmax(AT, L.smax[1][w]);
            VT = fmax(VT, L.smax[2][w]);
        }
        return i < n ? small_bound(ka, L.ch[i], L.A[i], L.cv[i], HT, AT, VT) : -1.0;
    };
    if (nb <= 64) small_kick_tiles<6, CRUDE, PREC>(L, ka, n, jc, CRUDE ? bound(t & 63) : 0.0);
    else if (nb <= 128) small_kick_tiles<7, CRUDE, PREC>(L, ka, n, jc, CRUDE ? bound(t & 127) : 0.0);
    else small_kick_tiles<8, CRUDE, PREC>(L, ka, n, jc, CRUDE ? bound(t & 255) : 0.0);
    __syncthreads();
    if (t < n)
        for (int k = 0; k < 3; ++k) acc[k] = L.part[k][t];
}

__device__ __forceinline__ CrudeBody small_body(const SmallLds &L, const double *X, const double *Y,
                                                const double *Z, int i)
{
    return CrudeBody{X[i], Y[i], Z[i], L.h[i], L.A[i], L.cv[i]};
}

// the exact crude test of the queued pairs (of every pair when the queue
// overflowed): the candidates, the first kSmallQ of them in LDS
__device__ __forceinline__ void small_candidates(SmallLds &L, const KickArgs &ka, int n)
{
    const int t = threadIdx.x;
    auto test = [&](int i, int j) {
        if (crude_test(ka.hill_mode, ka.aE, ka.cs, ka.tau_abs, small_body(L, L.x, L.y, L.z, i),
                       small_body(L, L.x, L.y, L.z, j))) {
            const unsigned k = atomicAdd(&L.ncand, 1u);
            if (k < (unsigned)kSmallQ) L.cand[k] = ((unsigned)i << 16) | (unsigned)j;
        }
    };
    const unsigned nq = L.nq;
    if (nq <= (unsigned)kSmallQ) {
        for (unsigned e = t; e < nq; e += kSmallThreads) test((int)(L.q[e] >> 16), (int)(L.q[e] & 0xffffu));
    } else {
        for (int i = t; i < n; i += kSmallThreads)
            for (int j = i + 1; j < n; ++j) test(i, j);
    }
}

// fine test of the candidates into L.enc (of every pair that passes the
// crude test at the snapshot when the list overflowed); nenc is the true count
__device__ __forceinline__ void small_fine(SmallLds &L, const SmallArgs &a, double m0, int n, int cap)
{
    const int t = threadIdx.x;
    auto test = [&](int i, int j) {
        const double a0[3] = {L.x0[j] - L.x0[i], L.y0[j] - L.y0[i], L.z0[j] - L.z0[i]};
        const double b0[3] = {L.vx0[j] - L.vx0[i], L.vy0[j] - L.vy0[i], L.vz0[j] - L.vz0[i]};
        const double a1[3] = {L.x[j] - L.x[i], L.y[j] - L.y[i], L.z[j] - L.z[i]};
        const double b1[3] = {L.vx[j] - L.vx[i], L.vy[j] - L.vy[i], L.vz[j] - L.vz[i]};
        double lhs, rhs;
        if (fine_pair(a.hill_mode, a.aE, m0, a.h.tau, L.m[i], L.m[j], L.h[i], L.h[j], L.A[i], L.A[j],
                      a0, b0, a1, b1, lhs, rhs)) {
            const unsigned k = atomicAdd(&L.nenc, 1u);
            if (k < (unsigned)cap) L.enc[k] = ((unsigned)i << 16) | (unsigned)j;
        }
    };
    const unsigned nc = L.ncand;
    if (nc <= (unsigned)kSmallQ) {
        for (unsigned e = t; e < nc; e += kSmallThreads)
            test((int)(L.cand[e] >> 16), (int)(L.cand[e] & 0xffffu));
    } else {
        for (int i = t; i < n; i += kSmallThreads)
            for (int j = i + 1; j < n; ++j)
                if (crude_test(a.hill_mode, a.aE, a.cs, fabs(a.h.tau),
                               small_body(L, L.x0, L.y0, L.z0, i), small_body(L, L.x0, L.y0, L.z0, j)))
                    test(i, j);
    }
}

// the sets of the ne encounter pairs (as k_sets: components ordered by their
// smallest body, members ascending, r_crit; one set of all bodies when a set
// holds two planets): nsets, sstart, scount, mem, rcb, maxset
__device__ __forceinline__ void small_sets(SmallLds &L, const SmallArgs &a, int n, int ne)
{
    const int t = threadIdx.x, lane = t & 63;
    if (t < n) L.lab[t] = 0x80000000u | (unsigned)t;   // the top bit: in no pair yet
    if (t == 0) L.whole = 0;
    __syncthreads();
    for (int k = t; k < ne; k += kSmallThreads) {
        const unsigned p = L.enc[k];
        atomicAnd(&L.lab[p >> 16], 0x7fffffffu);
        atomicAnd(&L.lab[p & 0xffffu], 0x7fffffffu);
    }
    __syncthreads();
    // union by minimum, as k_sets
    volatile unsigned *vlab = L.lab;
    for (int k = t; k < ne; k += kSmallThreads) {
        unsigned x = L.enc[k] >> 16, y = L.enc[k] & 0xffffu;
        for (;;) {
            while (vlab[x] != x) x = vlab[x];
            while (vlab[y] != y) y = vlab[y];
            if (x == y) break;
            if (x > y) {
                const unsigned s = x;
                x = y;
                y = s;
            }
            const unsigned old = atomicCAS(&L.lab[y], y, x);
            if (old == y) break;
            y = old;
        }
    }
    __syncthreads();
    unsigned r = 0xffffffffu;   // root of body t
    if (t < n && !(L.lab[t] >> 31)) {
        r = (unsigned)t;
        while (L.lab[r] != r) r = L.lab[r];
    }
    const unsigned long long in = __ballot(r != 0xffffffffu), rt = __ballot(r == (unsigned)t);
    if (lane == 0 && t < kSmallMax) {
        L.inenc[t >> 6] = in;
        L.root[t >> 6] = rt;
    }
    __syncthreads();
    auto before = [](const unsigned long long *bits, int i) {   // set bits below i
        int k = __popcll(bits[i >> 6] & ((1ull << (i & 63)) - 1ull));
        for (int w = 0; w < (i >> 6); ++w) k += __popcll(bits[w]);
        return k;
    };
    int nu = 0, nsets = 0;
    for (int w = 0; w < kSmallMax / 64; ++w) {
        nu += __popcll(L.inenc[w]);
        nsets += __popcll(L.root[w]);
    }
    for (int k = t; k < nsets; k += kSmallThreads) {
        L.scount[k] = 0;
        L.rcb[k] = 0ull;
        L.planets[k] = 0;
    }
    __syncthreads();
    int sid = -1;
    if (r != 0xffffffffu) {
        sid = before(L.root, (int)r);
        const int k = before(L.inenc, t);
        L.uq[k] = t;
        L.sid[k] = sid;
        atomicAdd(&L.scount[sid], 1);
        atomicMax(&L.rcb[sid], (unsigned long long)__double_as_longlong(L.h[t] * L.A[t]));
        if (a.planet_mass > 0.0 && L.m[t] >= a.planet_mass && atomicAdd(&L.planets[sid], 1) >= 1)
            L.whole = 1;
    }
    __syncthreads();
    if (L.whole) {
        if (t < n) L.mem[t] = t;
        if (t == 0) {
            L.sstart[0] = 0;
            L.scount[0] = n;
            L.rcb[0] = (unsigned long long)__double_as_longlong(INFINITY);
            L.nsets = 1;
            L.nu = n;
            L.maxset = n;
        }
        __syncthreads();
        return;
    }
    // starts, and each member's place among those of its set (ascending)
    for (int k = t; k < nsets; k += kSmallThreads) {
        int s = 0;
        for (int q = 0; q < k; ++q) s += L.scount[q];
        L.sstart[k] = s;
        L.rcb[k] = (unsigned long long)__double_as_longlong(a.aH * __longlong_as_double((long long)L.rcb[k]));
    }
    if (t == 0) {
        L.nsets = nsets;
        L.nu = nu;
        L.maxset = 0;
    }
    __syncthreads();
    for (int k = t; k < nsets; k += kSmallThreads) atomicMax(&L.maxset, L.scount[k]);
    for (int k = t; k < nu; k += kSmallThreads) {
        const int s = L.sid[k];
        int p = L.sstart[s];
        for (int q = 0; q < k; ++q) p += L.sid[q] == s ? 1 : 0;
        L.mem[p] = L.uq[k];
    }
    __syncthreads();
}

// corrections and Hermite of every set: the larger ones one after the other
// on the workgroup, then the small ones one per wave (as k_hermite)
__device__ __forceinline__ void small_hermite(SmallLds &L, const SmallArgs &a, double mu)
{
    const int t = threadIdx.x, lane = t & 63;
    const int w = __builtin_amdgcn_readfirstlane(t >> 6);
    const HermState hs{L.x0, L.y0, L.z0, L.vx0, L.vy0, L.vz0, L.m, L.x, L.y, L.z, L.vx, L.vy, L.vz};
    const int nsets = __builtin_amdgcn_readfirstlane(L.nsets);
    auto set_of = [&](int s) {
        return HermSet{L.mem + L.sstart[s], L.scount[s], __longlong_as_double((long long)L.rcb[s]), mu};
    };
    int nsub_b = 0, fail_b = 0;
    for (int s = 0; s < nsets; ++s) {
        if (__builtin_amdgcn_readfirstlane(L.scount[s]) <= kWaveMax) continue;
        int nsub, fail;
        hermite_set_block(a.h, hs, set_of(s),
                          SetLds{L.stage[0], L.stage[1], L.stage[2], L.stage[3], L.stage[4],
                                 L.stage[5], L.stage[6], L.hr},
                          L.red, nsub, fail);
        nsub_b += nsub;
        fail_b |= fail;
    }
    if (t == 0) {
        L.sub = nsub_b;
        L.hfail = fail_b;
    }
    __syncthreads();
    const int o = w * kWaveMax;
    const SetLds S = {L.stage[0] + o, L.stage[1] + o, L.stage[2] + o, L.stage[3] + o,
                      L.stage[4] + o, L.stage[5] + o, L.stage[6] + o};
    int nsub_w = 0, fail_w = 0, rank = 0;
    for (int s = 0; s < nsets; ++s) {
        if (__builtin_amdgcn_readfirstlane(L.scount[s]) > kWaveMax) continue;
        if (rank++ % (kSmallThreads / 64) != w) continue;
        int nsub, fail;
        hermite_set_wave(a.h, hs, set_of(s), S, lane, nsub, fail);
        nsub_w += nsub;
        fail_w |= fail;
    }
    if (lane == 0 && nsub_w > 0) atomicAdd(&L.sub, nsub_w);
    if (lane == 0 && fail_w) atomicOr(&L.hfail, 1);
    __syncthreads();
}

// figure `which` of two systems together
__device__ __forceinline__ unsigned long long small_add(int which, unsigned long long x,
                                                        unsigned long long y)
{
    if (which == SS_MAXSET || which == SS_KMAX) return x > y ? x : y;
    return which == SS_STATUS ? x | y : x + y;
}

// One launch of up to kSmallSteps steps.  A step whose encounter pairs do not
// fit a system's segment is left undone by every system of the context: with
// one system the workgroup itself goes back to that step's start; with
// several the launch only notes the first such step, nothing is published,
// and a second launch (redo; it returns at once otherwise) takes the steps
// before it again from the kept state.  The last workgroup to finish adds up
// the figures.
template <int PREC, bool SWAPPED>
__global__ __launch_bounds__(kSmallThreads) void k_small_steps(SmallArgs a)
{
    __shared__ SmallLds L;
    const Dev &d = a.d;
    const int t = threadIdx.x, lane = t & 63, s = blockIdx.x;
    const int so = d.sys_off[s], n = d.sys_off[s + 1] - so;
    const long long S = (long long)(d.y - d.x);
    unsigned long long *const st = a.st + (size_t)s * SS_COUNT;
    const bool frozen = (d.ctr[C_STATUS] & S_FREEZE) != 0;
    if (frozen) {
        // nothing is done; a new call's last step found nothing
        if (t == 0 && !a.redo) {
            if (a.first) d.sys_ecnt[s] = 0;
            if (s == 0) {
                d.ctr[C_OVERFLOW] += (unsigned long long)a.nsteps;
                if (a.first)
                    d.ctr[C_CAND] = d.ctr[C_ENC] = d.ctr[C_NSETS] = d.ctr[C_MAXSET] = d.ctr[C_SUB] =
                        d.ctr[C_NU] = 0ull;
            }
        }
        return;
    }
    const unsigned long long ovf = a.w[SW_OVF];
    if (a.redo && ovf == 0ull) return;
    // the step this launch stops in (redo), else none
    const int stop = a.redo ? kSmallSteps - (int)ovf : a.nsteps;
    const double m0 = d.sys_m0[s], mu = a.h.G * m0;
    const double tau = a.h.tau, half = tau / 2.0;
    const int segcap = d.sys_eoff[s + 1] - d.sys_eoff[s];
    const int k0 = d.sys_k0[s], nch = d.sys_k0[s + 1] - k0;
    const KickArgs ka{d, nullptr, a.h.G, a.cap, 0, 0, a.hill_mode, a.aE, a.cs, fabs(tau), a.r2seed,
                      a.c158, a.c32};
    if (t < n) {
        const int i = so + t;
        const double *b = a.redo ? d.bk + i : d.x + i;
        L.x[t] = b[0];
        L.y[t] = b[S];
        L.z[t] = b[2 * S];
        L.vx[t] = b[3 * S];
        L.vy[t] = b[4 * S];
        L.vz[t] = b[5 * S];
        L.m[t] = d.m[i];
        L.h[t] = d.h[i];
        if (!a.redo && a.nsys > 1)   // the state the second launch starts from
            for (int k = 0; k < 6; ++k) d.bk[k * S + i] = b[k * S];
    }
    if (t < kHist) L.hist[t] = 0u;
    if (t == 0) {
        L.kit = 0ull;
        L.kmax = L.krs = 0u;
        L.bad = 0;
        L.nenc = L.ncand = L.nq = 0u;
        L.nsets = L.nu = L.maxset = L.sub = 0;
    }
    __syncthreads();

    // momentum partials of the 64-body chunks (as k_momentum, k_apply_kepler)
    auto chunk_partials = [&]() {
        if (t < ((n + 63) & ~63)) {
            double p[3] = {0.0, 0.0, 0.0};
            if (t < n) {
                p[0] = L.m[t] * L.vx[t];
                p[1] = L.m[t] * L.vy[t];
                p[2] = L.m[t] * L.vz[t];
            }
            wave_sum3(p);
            if (lane == 0)
                for (int k = 0; k < 3; ++k) L.pm[t >> 6][k] = p[k];
        }
        __syncthreads();
    };
    // E_Kep(dt) of this thread's body and its statistics (as k_apply_kepler)
    auto kepler = [&](double dt) {
        int kit = -1, restart = 0;
        if (t < n) {
            int fail;
            double x = L.x[t], y = L.y[t], z = L.z[t], vx = L.vx[t], vy = L.vy[t], vz = L.vz[t];
            kit = kepler_advance(mu, a.kepler_mode, d.guess, dt, x, y, z, vx, vy, vz, fail, restart);
            L.x[t] = x;
            L.y[t] = y;
            L.z[t] = z;
            L.vx[t] = vx;
            L.vy[t] = vy;
            L.vz[t] = vz;
            if (fail) atomicOr(&L.bad, (int)S_KEPLER);
            atomicAdd(&L.hist[min(kit, kHist - 1)], 1u);
            atomicAdd(&L.kit, (unsigned long long)kit);
            atomicMax(&L.kmax, (unsigned)kit);
            if (restart) atomicAdd(&L.krs, 1u);
        }
    };
    auto finite = [&]() {
        if (t < n && !(isfinite(L.x[t]) && isfinite(L.y[t]) && isfinite(L.z[t]) && isfinite(L.vx[t]) &&
                       isfinite(L.vy[t]) && isfinite(L.vz[t])))
            atomicOr(&L.bad, (int)S_NONFINITE);
    };
    auto kick = [&](const double acc[3], double dt) {
        if (t < n) {
            L.vx[t] += dt * acc[0];
            L.vy[t] += dt * acc[1];
            L.vz[t] += dt * acc[2];
        }
    };
    auto drift = [&]() {
        double P[3];
        small_momentum(L, nch, P);
        if (t < n) {
            L.x[t] = L.x[t] + half * (P[0] / m0);
            L.y[t] = L.y[t] + half * (P[1] / m0);
            L.z[t] = L.z[t] + half * (P[2] / m0);
        }
    };
    // The momentum the first drift uses is the one the state came with: the
    // partials in global memory, which are those of its velocities
    if (t < nch)
        for (int k = 0; k < 3; ++k) L.pm[t][k] = d.pm[3 * (k0 + t) + k];
    if (a.redo) {
        __syncthreads();
        chunk_partials();
    }
    __syncthreads();

    unsigned long long tenc = 0, tsub = 0, nwhole = 0;
    int k = 0;
    bool undone = false;
    for (; k < a.nsteps; ++k) {
        if (t < n) {
            L.bk[0][t] = L.x[t];
            L.bk[1][t] = L.y[t];
            L.bk[2][t] = L.z[t];
            L.bk[3][t] = L.vx[t];
            L.bk[4][t] = L.vy[t];
            L.bk[5][t] = L.vz[t];
        }
        drift();
        double acc[3];
        if constexpr (SWAPPED) {
            kepler(half);
            finite();
            __syncthreads();
            small_kick<false, PREC>(L, ka, n, a.jc[0], acc);
            kick(acc, tau);
            kepler(half);
            finite();
            chunk_partials();
            drift();
        } else {
            // 1: per-body terms of the encounter search (as k_drift)
            if (t < n) {
                const double x = L.x[t], y = L.y[t], z = L.z[t];
                const double vx = L.vx[t], vy = L.vy[t], vz = L.vz[t];
                const double r = sqrt(x * x + y * y + z * z);
                const double inva = 2.0 / r - (vx * vx + vy * vy + vz * vz) / mu;
                const double A = (inva > 0.0) ? 1.0 / inva : r;
                L.A[t] = A;
                L.cv[t] = sqrt(2.0 * mu / r);
                L.ch[t] = (a.hill_mode == 0) ? L.h[t] : L.h[t] * A;
            }
            __syncthreads();
            // 2: kick with the crude sweep, then the candidates
            small_kick<true, PREC>(L, ka, n, a.jc[1], acc);
            small_candidates(L, ka, n);
            if (t == 0) L.nenc = 0u;
            __syncthreads();
            // 2-3: kick applied, snapshot, Kepler
            kick(acc, half);
            if (t < n) {
                L.x0[t] = L.x[t];
                L.y0[t] = L.y[t];
                L.z0[t] = L.z[t];
                L.vx0[t] = L.vx[t];
                L.vy0[t] = L.vy[t];
                L.vz0[t] = L.vz[t];
            }
            kepler(tau);
            finite();
            __syncthreads();
            // 4: fine sweep, sets
            small_fine(L, a, m0, n, min(segcap, kSmallEnc));
            if (t == 0 && L.ncand) atomicAdd(&a.w[SW_STEP0 + k], (unsigned long long)L.ncand);
            __syncthreads();
            const int ne = __builtin_amdgcn_readfirstlane((int)L.nenc);
            if (ne > segcap || k == stop) {
                undone = true;
                break;
            }
            if (t == 0) {
                L.nsets = L.nu = L.maxset = L.sub = L.hfail = 0;
                L.whole = 0;
            }
            __syncthreads();
            if (ne > 0) {
                small_sets(L, a, n, ne);
                // 5-7
                small_hermite(L, a, mu);
                tenc += (unsigned long long)ne;
                tsub += (unsigned long long)L.sub;
                nwhole += (unsigned long long)L.whole;
                if (t == 0 && L.hfail) atomicOr(&L.bad, (int)S_HERMITE);
            }
            // 9
            small_kick<false, PREC>(L, ka, n, a.jc[0], acc);
            kick(acc, half);
            finite();
            chunk_partials();
            // 10
            drift();
        }
    }
    __syncthreads();
    if (undone) {
        if (!a.redo && a.nsys > 1) {
            // another launch takes the steps before this one again
            if (t == 0) atomicMax(&a.w[SW_OVF], (unsigned long long)(kSmallSteps - k));
        } else {
            // back to the step's start
            if (t < n) {
                L.x[t] = L.bk[0][t];
                L.y[t] = L.bk[1][t];
                L.z[t] = L.bk[2][t];
                L.vx[t] = L.bk[3][t];
                L.vy[t] = L.bk[4][t];
                L.vz[t] = L.bk[5][t];
            }
            if (t == 0) L.nsets = L.nu = L.maxset = L.sub = 0;
            __syncthreads();
            chunk_partials();
        }
    }
    if (t < n) {
        const int i = so + t;
        d.x[i] = L.x[t];
        d.y[i] = L.y[t];
        d.z[i] = L.z[t];
        d.vx[i] = L.vx[t];
        d.vy[i] = L.vy[t];
        d.vz[i] = L.vz[t];
    }
    if (t < nch)
        for (int c = 0; c < 3; ++c) d.pm[3 * (k0 + t) + c] = L.pm[t][c];
    // the last step's lists
    const int ncand = SWAPPED ? 0 : (int)L.ncand, ne = SWAPPED ? 0 : (int)L.nenc;
    const int nsets = L.nsets, nu = L.nu;
    if (t == 0) {
        L.base_cand = ncand ? (int)atomicAdd(&a.w[SW_CAND], (unsigned long long)ncand) : 0;
        L.base_set = nsets ? (int)atomicAdd(&a.w[SW_NSETS], (unsigned long long)nsets) : 0;
        L.base_mem = nu ? (int)atomicAdd(&a.w[SW_NU], (unsigned long long)nu) : 0;
        d.sys_ecnt[s] = ne;
        L.nq = 0u;
    }
    __syncthreads();
    auto put_cand = [&](long long q, int i, int j) {
        if (q < a.cap) d.cand[q] = make_int2(so + i, so + j);
    };
    if (ncand <= kSmallQ) {
        for (int e = t; e < ncand; e += kSmallThreads)
            put_cand((long long)L.base_cand + e, (int)(L.cand[e] >> 16), (int)(L.cand[e] & 0xffffu));
    } else {
        for (int i = t; i < n; i += kSmallThreads)
            for (int j = i + 1; j < n; ++j)
                if (crude_test(a.hill_mode, a.aE, a.cs, fabs(tau), small_body(L, L.x0, L.y0, L.z0, i),
                               small_body(L, L.x0, L.y0, L.z0, j)))
                    put_cand((long long)L.base_cand + atomicAdd(&L.nq, 1u), i, j);
    }
    for (int e = t; e < min(ne, min(segcap, kSmallEnc)); e += kSmallThreads)
        d.enc[d.sys_eoff[s] + e] = make_int2(so + (int)(L.enc[e] >> 16), so + (int)(L.enc[e] & 0xffffu));
    for (int q = t; q < nu; q += kSmallThreads) d.set_mem[L.base_mem + q] = so + L.mem[q];
    for (int q = t; q < nsets; q += kSmallThreads) {
        d.set_start[L.base_set + q] = L.base_mem + L.sstart[q];
        d.set_count[L.base_set + q] = L.scount[q];
        d.set_rc[L.base_set + q] = __longlong_as_double((long long)L.rcb[q]);
    }
    if (t < kHist) st[SS_HIST + t] = L.hist[t];
    if (t == 0) {
        st[SS_ENC] = (unsigned long long)ne;
        st[SS_MAXSET] = (unsigned long long)L.maxset;
        st[SS_SUB] = (unsigned long long)L.sub;
        st[SS_TENC] = tenc;
        st[SS_TSUB] = tsub;
        st[SS_WHOLE] = nwhole;
        st[SS_STATUS] = (unsigned long long)L.bad;
        st[SS_KIT] = L.kit;
        st[SS_KMAX] = L.kmax;
        st[SS_KRS] = L.krs;
    }
    // the last workgroup adds the figures up: one fence and one atomic each
    __syncthreads();
    if (t == 0) {
        __threadfence();
        L.last = atomicAdd(&a.w[SW_TICKET], 1ull) == (unsigned long long)(a.nsys - 1);
    }
    __syncthreads();
    if (!L.last) return;
    __threadfence();
    const unsigned long long first = a.w[SW_OVF];
    const bool again = !a.redo && a.nsys > 1 && first != 0ull;   // the second launch publishes
    const bool froze = a.nsys == 1 ? undone : a.redo != 0;
    const int done = froze ? k : a.nsteps;   // (redo: every system stopped in the same step)
    // the figures of the systems: wave w those of every eighth system, one
    // per lane, then the waves' shares through LDS (the Hermite's staging)
    unsigned long long *const share = reinterpret_cast<unsigned long long *>(L.stage[0]);
    static_assert(SS_COUNT <= 64 && kSmallThreads <= kHermLds, "a lane per figure, a word per thread");
    {
        unsigned long long v = 0;
        if (lane < SS_COUNT)
#pragma unroll 4
            for (int q = t >> 6; q < a.nsys; q += kSmallThreads / 64)
                v = small_add(lane, v, a.st[(size_t)q * SS_COUNT + lane]);
        share[t] = v;
        // steps whose candidates would have overflowed the list: the fine
        // test does not depend on it here, the count stays
        if (t < kSmallSteps) L.lab[t] = t < a.nsteps && (long long)a.w[SW_STEP0 + t] > a.cap ? 1u : 0u;
    }
    __syncthreads();   // also: every thread has read the words that are cleared below
    if (!again && t < SS_COUNT) {
        unsigned long long v = share[t];
        for (int w = 1; w < kSmallThreads / 64; ++w) v = small_add(t, v, share[64 * w + t]);
        if (t == SS_ENC) d.ctr[C_ENC] = v;
        else if (t == SS_MAXSET) d.ctr[C_MAXSET] = v;
        else if (t == SS_SUB) d.ctr[C_SUB] = v;
        else if (t == SS_TENC) d.ctr[C_TENC] += v;
        else if (t == SS_TSUB) d.ctr[C_TSUB] += v;
        else if (t == SS_WHOLE) d.ctr[C_WHOLE] += v;
        else if (t == SS_STATUS) d.ctr[C_STATUS] |= v | (froze ? (unsigned long long)S_ENC_OVF : 0ull);
        else if (t == SS_KMAX) d.kstat[kHist + 1] = small_add(t, v, d.kstat[kHist + 1]);
        else if (t == SS_KIT) d.kstat[kHist] += v;
        else if (t == SS_KRS) d.kstat[kHist + 2] += v;
        else d.kstat[t - SS_HIST] += v;
    }
    if (!again && t == 64) {
        d.ctr[C_CAND] = a.w[SW_CAND];
        d.ctr[C_NSETS] = a.w[SW_NSETS];
        d.ctr[C_NU] = a.w[SW_NU];
        d.ctr[C_STEPS] += (unsigned long long)done;
        if (froze) d.ctr[C_OVERFLOW] += (unsigned long long)(a.nsteps - done);
        unsigned long long fb = 0;
        for (int q = 0; q < a.nsteps; ++q) fb += L.lab[q];
        d.ctr[C_FALLBACK] += fb;
    }
    __syncthreads();
    for (int q = t; q < SW_COUNT; q += kSmallThreads)
        if (q != SW_OVF || !again) a.w[q] = 0ull;
}

}  // namespace qsym
