// qsym.hip -- host side of the MI355X DH hybrid-step library: workspace
// layout, work tables, kernel launches, HIP graphs of several steps, the
// kick autotuner and the C ABI declared in include/qsym.h.
#include "qsym.h"

#include <algorithm>
#include <array>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <string>
#include <type_traits>
#include <vector>

#include "qsym_kernels.hpp"
#include "qsym_small.hpp"
#include "qsym_sweep.hpp"

using namespace qsym;

namespace {

constexpr int kPhases = 12;
enum Phase {
    P_DRIFT = 0, P_KICK1, P_APPLY1, P_FINE, P_SETS, P_HERMITE, P_KICK2, P_APPLY2, P_DRIFT2,
    P_ENERGY, P_MOMENTUM, P_OTHER
};

inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// sym: 0 full-matrix kick; 1, 2, 4, 8 symmetric kick with this many
// i-blocks per work item over j-chunks of jchunk bodies; kSymRows symmetric
// kick over balanced rows (see build_items)
constexpr int kSymRows = 16;

struct Shape {
    int ipl = 2;
    int block = 256;
    long long jchunk = 1024;
    int remap = 1;
    int sym = 0;
};

// workspace layout: byte offsets of every array
struct Layout {
    size_t off_state = 0, off_snap = 0, off_aux = 0, off_acc = 0, off_pm = 0, off_bsys = 0;
    size_t off_sysoff = 0, off_sysm0 = 0, off_sysS = 0, off_syspoff = 0, off_sysc0 = 0, off_sysk0 = 0;
    size_t off_bchunk = 0, off_kchunk = 0, off_items = 0, off_eitems = 0, off_syse0 = 0, off_cand = 0;
    size_t off_enc = 0, off_syseoff = 0, off_sysecnt = 0, off_setcount = 0, off_setstart = 0, off_setmem = 0, off_setrc = 0, off_setlist = 0;
    size_t off_sysgoff = 0, off_gsa = 0, off_bk = 0, off_krow = 0;
    long long krow_cap = 1;    // rows of the balanced-row kick shape, per kick
    long long gsa_slots = 0;   // global set-partition scratch (64-bit slots)
    size_t off_gbar = 0, off_hpart = 0;
    size_t off_swcnt = 0, off_swslot = 0, off_swrec = 0, off_swlarge = 0, off_syssw = 0,
           off_swpart = 0;
    long long sw_nb = 1;       // grid-sweep buckets
    size_t off_hw = 0, off_ctr = 0, off_kstat = 0, off_guess = 0;
    size_t off_small = 0;      // counters and figures of k_small_steps
    bool small = false;        // every system has at most kSmallMax bodies
    size_t off_erec = 0, off_ewcol = 0, off_ewrec = 0, off_sysu0 = 0, off_sysr0 = 0;
    int e_waves = 4;           // waves of k_energy_pairs (a multiple of 4)
    size_t total = 0;
    long long np = 0;          // padded body count
    long long acc_len = 0;     // doubles of kick partials
    long long nchunks = 0;     // O(N) chunks
    long long nkchunks = 0;    // Kepler-pass chunks
    long long max_items = 0;   // kick items of the finest allowed shape
    long long n_eitems = 0;
    long long cap = 0;         // candidate capacity
    long long ecap = 0;        // encounter-pair slots (sum of per-system capacities)
    long long setcap = 0;      // set slots
    long long memcap = 0;      // set-member slots
    long long jchunk_min = 128;
};

struct Tables {
    std::vector<int> sys_off, sys_S, sys_c0, sys_k0, sys_e0, sys_eoff;
    std::vector<long long> sys_poff, sys_goff;
    std::vector<long long> sys_u0, e_wcol;   // energy units per system, columns per wave
    std::vector<int> e_wrec, sys_r0;         // energy records per wave and per system
    std::vector<int4> bchunk, kchunk;
    std::vector<KickItem> eitems;
    std::vector<int> body_sys;
};

int nsys_bodies(const std::vector<long long> &off, int s) { return (int)(off[s + 1] - off[s]); }

// encounter pairs one system may append per step (its segment): four per
// body, far above any disk (the benchmark disks have well under one); a
// system with more leaves the step undone (S_ENC_OVF).  Systems whose
// segment exceeds kCapE may need the global-memory set partition.
constexpr long long kEncPerBody = 4;
long long sys_enc_cap(long long n)
{
    if (n <= 0) return 0;
    return std::min<long long>(kEncPerBody * n + 64, 1LL << 26);
}

// energy pair sum: units of 128 i x 64 j over each system's upper triangle
// (row b, i in [128 b, 128 b + 128), meets the 64-blocks of j from 2 b on),
// 64 columns each; at least 16 columns per wave where the work allows, at most
// 4096 waves (16 per compute unit).  A column is a chain of some 100 cycles;
// k_energy_pairs with 256 of them a wave (4 units) and with 16: 8 systems of 4
// bodies 25.8, 7.6 us; 1024 bodies 31.4, 8.5; 4100: 34.8, 12.5.
long long energy_units(long long n)
{
    const long long nj = (n + 63) / 64, ni = (n + 127) / 128;
    return ni * nj - ni * (ni - 1);
}

int energy_waves(const std::vector<long long> &off)
{
    long long units = 0;
    for (size_t s = 0; s + 1 < off.size(); ++s) units += energy_units(off[s + 1] - off[s]);
    const long long w = std::max<long long>(1, std::min<long long>(4 * units, 4096));
    return (int)((w + 3) / 4 * 4);
}

long long jchunk_min_for(const std::vector<long long> &off)
{
    long long nmax = 0;
    for (size_t s = 0; s + 1 < off.size(); ++s) nmax = std::max(nmax, off[s + 1] - off[s]);
    long long jm = (nmax + kSMax - 1) / kSMax;
    jm = std::max<long long>(128, (jm + 127) / 128 * 128);
    return jm;
}

// partial-sum slots of a system of n bodies: up to ceil(n / jchunk_min)
// i-side slots (one per j-chunk), and for the symmetric kick one j-side slot
// per i-range of at least 128 bodies, at most kSMax * 2 of them
long long partial_slots(long long n, long long jchunk_min)
{
    const long long si = (n + jchunk_min - 1) / jchunk_min;
    const long long sj = std::min<long long>((n + 127) / 128, 2 * kSMax);
    return si + sj;
}

Layout make_layout(const qsym_params &p, const std::vector<long long> &off)
{
    Layout L;
    const int nsys = (int)off.size() - 1;
    const long long ntot = off.back();
    L.np = std::max<long long>(256, (long long)align_up((size_t)ntot, 256));
    L.jchunk_min = jchunk_min_for(off);
    L.acc_len = 0;
    L.nchunks = 0;
    L.max_items = 0;
    L.n_eitems = 0;
    for (int s = 0; s < nsys; ++s) {
        const long long n = off[s + 1] - off[s];
        L.acc_len += 3 * partial_slots(n, L.jchunk_min) * n;
        L.nchunks += (n + kChunk - 1) / kChunk;
        L.nkchunks += (n + kChunkK - 1) / kChunkK;
        L.max_items += ((n + 127) / 128) * ((n + L.jchunk_min - 1) / L.jchunk_min);
        L.n_eitems += ((n + 255) / 256) * ((n + 1023) / 1024);
    }
    L.acc_len = std::max<long long>(L.acc_len, 3);
    L.nchunks = std::max<long long>(L.nchunks, 1);
    L.nkchunks = std::max<long long>(L.nkchunks, 1);
    L.max_items = std::max<long long>(L.max_items, 1) + 8;
    L.n_eitems = std::max<long long>(L.n_eitems, 1);
    L.cap = p.pair_capacity > 0 ? p.pair_capacity : 8 * ntot + 1024;
    L.ecap = 0;
    L.setcap = 0;
    L.gsa_slots = 0;
    for (int s = 0; s < nsys; ++s) {
        const long long n = off[s + 1] - off[s];
        L.ecap += sys_enc_cap(n);
        // a set has two members or more, or is a whole system
        if (n > 0) L.setcap += n / 2 + 1;
        if (sys_enc_cap(n) > kCapE) {
            L.gsa_slots += gs_slots(n);
        }
    }
    L.ecap = std::max<long long>(L.ecap, 1);
    L.setcap = std::max<long long>(L.setcap, 1);
    L.gsa_slots = std::max<long long>(L.gsa_slots, 1);
    // sets are disjoint: every body is a member of at most one
    L.memcap = std::max<long long>(ntot, 1);
    size_t o = 0;
    auto take = [&](size_t &field, size_t bytes) {
        o = align_up(o, 256);
        field = o;
        o += bytes;
    };
    const size_t D = sizeof(double);
    take(L.off_state, 8 * (size_t)L.np * D);
    take(L.off_snap, 6 * (size_t)L.np * D);
    take(L.off_aux, 3 * (size_t)L.np * D);
    take(L.off_acc, (size_t)L.acc_len * D);
    take(L.off_pm, 3 * (size_t)L.nkchunks * D);
    take(L.off_bsys, (size_t)L.np * sizeof(int));
    take(L.off_sysoff, (size_t)(nsys + 1) * sizeof(int));
    take(L.off_sysm0, (size_t)std::max(nsys, 1) * D);
    take(L.off_sysS, 2 * (size_t)std::max(nsys, 1) * sizeof(int4));
    take(L.off_syspoff, (size_t)std::max(nsys, 1) * sizeof(long long));
    take(L.off_sysc0, (size_t)(nsys + 1) * sizeof(int));
    take(L.off_sysk0, (size_t)(nsys + 1) * sizeof(int));
    take(L.off_bchunk, (size_t)L.nchunks * sizeof(int4));
    take(L.off_kchunk, (size_t)L.nkchunks * sizeof(int4));
    take(L.off_items, 2 * (size_t)L.max_items * sizeof(KickItem));
    take(L.off_eitems, (size_t)L.n_eitems * sizeof(KickItem));
    take(L.off_syse0, (size_t)(nsys + 1) * sizeof(int));
    take(L.off_cand, (size_t)L.cap * sizeof(int2));
    take(L.off_enc, (size_t)L.ecap * sizeof(int2));
    take(L.off_syseoff, (size_t)(nsys + 1) * sizeof(int));
    take(L.off_sysecnt, (size_t)std::max(nsys, 1) * sizeof(int));
    take(L.off_setstart, (size_t)L.setcap * sizeof(int));
    take(L.off_setcount, (size_t)L.setcap * sizeof(int));
    take(L.off_setmem, (size_t)L.memcap * sizeof(int));
    take(L.off_setrc, (size_t)L.setcap * D);
    take(L.off_setlist, (size_t)L.setcap * sizeof(int));
    take(L.off_sysgoff, (size_t)std::max(nsys, 1) * sizeof(long long));
    take(L.off_gsa, (size_t)L.gsa_slots * sizeof(unsigned long long));
    take(L.off_bk, 6 * (size_t)L.np * D);
    L.krow_cap = 1;
    for (int s = 0; s < nsys; ++s) L.krow_cap += (off[s + 1] - off[s] + 127) / 128;
    take(L.off_krow, 2 * (size_t)L.krow_cap * sizeof(int));
    take(L.off_gbar, 4 * sizeof(unsigned));
    take(L.off_hpart, 2 * (size_t)kGridMax * D);
    take(L.off_hw, (size_t)HFIELDS * L.memcap * D);
    // grid sweep: a hash table of >= 2 ntot buckets (only when selected)
    L.sw_nb = 1;
    if (p.sweep == 1)
        while (L.sw_nb < std::max<long long>(1024, 2 * ntot)) L.sw_nb <<= 1;
    const size_t swb = p.sweep == 1 ? (size_t)L.np : 1;
    take(L.off_swcnt, (size_t)L.sw_nb * sizeof(int));
    take(L.off_swslot, (size_t)L.sw_nb * kSweepCap * sizeof(int));
    take(L.off_swrec, swb * sizeof(SweepRec));
    take(L.off_swlarge, swb * sizeof(int));
    take(L.off_syssw, (size_t)std::max(nsys, 1) * sizeof(double4));
    take(L.off_swpart, 3 * (size_t)L.nchunks * D);
    take(L.off_ctr, (size_t)C_COUNT * sizeof(unsigned long long));
    take(L.off_kstat, (size_t)kStatStripes * kStatStride * sizeof(unsigned long long));
    L.small = nsys > 0;
    for (int s = 0; s < nsys; ++s) L.small = L.small && off[s + 1] - off[s] <= kSmallMax;
    take(L.off_small, L.small ? (SW_COUNT + (size_t)nsys * SS_COUNT) * sizeof(unsigned long long) : 8);
    L.e_waves = energy_waves(off);
    take(L.off_erec, (size_t)kERec * (L.e_waves + nsys) * D);
    take(L.off_ewcol, (size_t)(L.e_waves + 1) * sizeof(long long));
    take(L.off_ewrec, (size_t)L.e_waves * sizeof(int));
    take(L.off_sysu0, (size_t)(nsys + 1) * sizeof(long long));
    take(L.off_sysr0, (size_t)(nsys + 1) * sizeof(int));
    take(L.off_guess, (size_t)(kGuessWeights + 5) * sizeof(float));
    L.total = align_up(o, 256);
    return L;
}

Dev bind(char *base, const Layout &L)
{
    Dev d;
    const long long np = L.np;
    double *st = (double *)(base + L.off_state);
    d.x = st;
    d.y = st + np;
    d.z = st + 2 * np;
    d.vx = st + 3 * np;
    d.vy = st + 4 * np;
    d.vz = st + 5 * np;
    d.m = st + 6 * np;
    d.h = st + 7 * np;
    double *sn = (double *)(base + L.off_snap);
    d.x0 = sn;
    d.y0 = sn + np;
    d.z0 = sn + 2 * np;
    d.vx0 = sn + 3 * np;
    d.vy0 = sn + 4 * np;
    d.vz0 = sn + 5 * np;
    double *ax = (double *)(base + L.off_aux);
    d.A = ax;
    d.ch = ax + np;
    d.cv = ax + 2 * np;
    d.acc = (double *)(base + L.off_acc);
    d.pm = (double *)(base + L.off_pm);
    d.body_sys = (int *)(base + L.off_bsys);
    d.sys_off = (int *)(base + L.off_sysoff);
    d.sys_m0 = (double *)(base + L.off_sysm0);
    d.sys_K = (int4 *)(base + L.off_sysS);
    d.sys_poff = (long long *)(base + L.off_syspoff);
    d.sys_c0 = (int *)(base + L.off_sysc0);
    d.sys_k0 = (int *)(base + L.off_sysk0);
    d.bchunk = (int4 *)(base + L.off_bchunk);
    d.kchunk = (int4 *)(base + L.off_kchunk);
    d.items = (KickItem *)(base + L.off_items);
    d.eitems = (KickItem *)(base + L.off_eitems);
    d.sys_e0 = (int *)(base + L.off_syse0);
    d.cand = (int2 *)(base + L.off_cand);
    d.enc = (int2 *)(base + L.off_enc);
    d.sys_eoff = (int *)(base + L.off_syseoff);
    d.sys_ecnt = (int *)(base + L.off_sysecnt);
    d.set_count = (int *)(base + L.off_setcount);
    d.set_list = (int *)(base + L.off_setlist);
    d.gbar = (unsigned *)(base + L.off_gbar);
    d.hpart = (double *)(base + L.off_hpart);
    d.setcap = (int)L.setcap;
    d.sys_goff = (long long *)(base + L.off_sysgoff);
    d.gsa = (unsigned long long *)(base + L.off_gsa);
    d.bk = (double *)(base + L.off_bk);
    d.krow = (int *)(base + L.off_krow);
    d.sw_cnt = (int *)(base + L.off_swcnt);
    d.sw_slot = (int *)(base + L.off_swslot);
    d.sw_rec = (SweepRec *)(base + L.off_swrec);
    d.sw_large = (int *)(base + L.off_swlarge);
    d.sys_sw = (double4 *)(base + L.off_syssw);
    d.sw_nb = (int)L.sw_nb;
    d.sw_part = (double *)(base + L.off_swpart);
    d.memcap = (int)L.memcap;
    d.set_start = (int *)(base + L.off_setstart);
    d.set_mem = (int *)(base + L.off_setmem);
    d.set_rc = (double *)(base + L.off_setrc);
    d.hw = (double *)(base + L.off_hw);
    d.ctr = (unsigned long long *)(base + L.off_ctr);
    d.kstat = (unsigned long long *)(base + L.off_kstat);
    d.erec = (double *)(base + L.off_erec);
    d.e_wcol = (long long *)(base + L.off_ewcol);
    d.e_wrec = (int *)(base + L.off_ewrec);
    d.sys_u0 = (long long *)(base + L.off_sysu0);
    d.sys_r0 = (int *)(base + L.off_sysr0);
    d.guess = (float *)(base + L.off_guess);
    return d;
}

}  // namespace

struct qsym_ctx {
    qsym_params p{};
    int nsys = 0;
    std::vector<long long> off;
    std::vector<double> m0;
    long long ntot = 0;
    hipStream_t ustream = nullptr;  // caller's stream
    hipStream_t stream = nullptr;   // private stream (capturable)
    hipEvent_t ev_in = nullptr, ev_out = nullptr;
    Layout L;
    Dev d;
    char *base = nullptr;
    Shape shape[2];      // [0] plain kick, [1] kick with the crude sweep
    int nitems[2] = {0, 0};
    int grid_kick[2] = {0, 0};
    Tables T;
    // captured steps per kind (0 hybrid, 1 the encounter-free swapped step):
    // kGraphSteps times a step's body and the drift fused with the next
    // step's first, captured once kGraphAfter steps of this tau were taken
    struct StepGraph {
        hipGraph_t graph = nullptr;
        hipGraphExec_t exec = nullptr;
        double tau = 0.0;
        int64_t seen = 0;   // steps of this tau
        bool valid = false;
    } g[2];
    int profile = 0;   // 1: kernel timings, 2: and workgroup records
    // profiling: event pairs recorded around launches without waiting; the
    // pending pairs are read (and the events recycled) at the next flush
    std::vector<hipEvent_t> pool;
    std::vector<int> pend_phase;
    size_t pool_used = 0;
    double phase_us[kPhases] = {};
    long long phase_calls[kPhases] = {};
    int cur_phase = P_OTHER;   // phase of the Timer open around the current launch
    // workgroup records of the kick and k_hermite launches (profiling): a
    // device ring of kRecLaunches slots of rec_wg records, read at the flush
    unsigned long long *rec = nullptr;
    int rec_wg = 0;
    std::vector<std::pair<int, int>> rec_pend;   // (phase, workgroups) per used slot
    double busy_max_us[kPhases] = {};
    double busy_mean_us[kPhases] = {};
    long long busy_calls[kPhases] = {};
    int busy_units = 0;
    bool guess_loaded = false;
    int grid_blocks = 256;   // workgroups of k_hermite: the device's compute units
    int cus = 256;           // the device's compute units
    int apply_parts = 1;     // threads per body of the partial-sum reduction (1 or 4)
    double tau_crude = 0.0;  // |tau| of the crude sweep being enqueued
    int device = 0;
    // host memory that a blocking call's last kernel writes its results to
    // (the status, then each system's energy), so that they need no copy
    unsigned long long *result = nullptr;
    std::string err;
};

namespace {

// message of the last failure that had no context to hold it (creation)
thread_local std::string g_noctx_err;

}  // namespace

// the same, set from the context-free entry points of other files
void qsym_noctx_error(const char *msg) { g_noctx_err = msg ? msg : ""; }

namespace {

int fail(qsym_ctx *c, int code, const std::string &msg)
{
    if (c) c->err = msg;
    else g_noctx_err = msg;
    return code;
}

#define HIPCHK(ctx, call)                                                                    \
    do {                                                                                     \
        hipError_t e_ = (call);                                                              \
        if (e_ != hipSuccess)                                                                \
            return fail((ctx), QSYM_EHIP, std::string(#call) + ": " + hipGetErrorString(e_)); \
    } while (0)

int validate(const qsym_params *p, int32_t nsys, const int64_t *offsets, std::string &msg)
{
    if (!p || !offsets || nsys < 1) { msg = "null parameters/offsets or nsys < 1"; return QSYM_EINVAL; }
    if (offsets[0] != 0) { msg = "offsets[0] must be 0"; return QSYM_EINVAL; }
    for (int s = 0; s < nsys; ++s)
        if (offsets[s + 1] < offsets[s]) { msg = "offsets must be non-decreasing"; return QSYM_EINVAL; }
    if (offsets[nsys] >= (1LL << 30)) { msg = "too many bodies (>= 2^30)"; return QSYM_EINVAL; }
    {
        long long ecap = 0;
        for (int s = 0; s < nsys; ++s) ecap += sys_enc_cap(offsets[s + 1] - offsets[s]);
        if (ecap >= (1LL << 31)) { msg = "encounter capacity beyond 2^31 pairs"; return QSYM_EINVAL; }
    }
    if (!(p->G > 0) || !(p->aE >= 0) || !(p->aH > 0) || !(p->epsH >= 0) || !(p->eta > 0) ||
        !(p->eta_s > 0) || !(p->crude_safety >= 1.0)) {
        msg = "parameter out of range (G, aH, eta, eta_s > 0; aE, epsH >= 0; crude_safety >= 1)";
        return QSYM_EINVAL;
    }
    if (p->hill_mode < 0 || p->hill_mode > 1 || p->kepler_mode < 0 || p->kepler_mode > 2 ||
        p->precision < 0 || p->precision > 1 || p->max_substeps < 1 || p->pair_capacity < 0 ||
        !(p->planet_mass >= 0.0) || !std::isfinite(p->planet_mass) || p->sweep < 0 || p->sweep > 1) {
        msg = "mode out of range";
        return QSYM_EINVAL;
    }
    return QSYM_OK;
}

void build_tables(qsym_ctx *c)
{
    Tables &T = c->T;
    const int nsys = c->nsys;
    T.sys_off.assign(nsys + 1, 0);
    T.sys_S.assign(nsys, 0);
    T.sys_poff.assign(nsys, 0);
    T.sys_goff.assign(nsys, -1);
    T.sys_c0.assign(nsys + 1, 0);
    T.sys_k0.assign(nsys + 1, 0);
    T.sys_e0.assign(nsys + 1, 0);
    T.sys_eoff.assign(nsys + 1, 0);
    T.bchunk.clear();
    T.kchunk.clear();
    T.eitems.clear();
    T.body_sys.assign((size_t)c->L.np, 0);
    long long poff = 0;
    for (int s = 0; s < nsys; ++s) {
        const int n = nsys_bodies(c->off, s);
        T.sys_off[s] = (int)c->off[s];
        T.sys_poff[s] = poff;
        poff += 3LL * partial_slots(n, c->L.jchunk_min) * n;
        T.sys_c0[s] = (int)T.bchunk.size();
        for (int b = 0; b < n; b += kChunk)
            T.bchunk.push_back(make_int4(s, (int)c->off[s] + b, std::min(kChunk, n - b), 0));
        T.sys_k0[s] = (int)T.kchunk.size();
        for (int b = 0; b < n; b += kChunkK)
            T.kchunk.push_back(make_int4(s, (int)c->off[s] + b, std::min(kChunkK, n - b), 0));
        T.sys_e0[s] = (int)T.eitems.size();
        for (int ib = 0; ib < n; ib += 256)
            for (int jb = 0; jb < n; jb += 1024) {
                KickItem it{s, (int)c->off[s] + ib, std::min(256, n - ib), (int)c->off[s] + jb,
                            std::min(1024, n - jb), jb / 1024};
                T.eitems.push_back(it);
            }
        for (long long i = c->off[s]; i < c->off[s + 1]; ++i) T.body_sys[i] = s;
    }
    T.sys_off[nsys] = (int)c->off[nsys];
    long long goff = 0;
    for (int s = 0; s < nsys; ++s) {
        const long long n = c->off[s + 1] - c->off[s];
        T.sys_eoff[s + 1] = T.sys_eoff[s] + (int)sys_enc_cap(n);
        if (sys_enc_cap(n) > kCapE) {
            T.sys_goff[s] = goff;
            goff += gs_slots(n);
        }
    }
    T.sys_c0[nsys] = (int)T.bchunk.size();
    T.sys_k0[nsys] = (int)T.kchunk.size();
    T.sys_e0[nsys] = (int)T.eitems.size();
    // energy schedule: every wave the same number of pair columns (64 per
    // unit), and the records (one per wave and system it touches) in system
    // order, so each system's records are one contiguous run
    T.sys_u0.assign(nsys + 1, 0);
    for (int s = 0; s < nsys; ++s) T.sys_u0[s + 1] = T.sys_u0[s] + energy_units(c->off[s + 1] - c->off[s]);
    const int W = c->L.e_waves;
    const long long Ctot = 64 * T.sys_u0[nsys];
    T.e_wcol.assign(W + 1, 0);
    for (int w = 0; w <= W; ++w) T.e_wcol[w] = (long long)((__int128)Ctot * w / W);
    auto sys_of = [&](long long U) {   // system holding unit U (one with units)
        return (int)(std::upper_bound(T.sys_u0.begin(), T.sys_u0.end(), U) - T.sys_u0.begin()) - 1;
    };
    T.e_wrec.assign(W, 0);
    std::vector<int> r_first(nsys, -1);
    int rec = 0;
    for (int w = 0; w < W; ++w) {
        T.e_wrec[w] = rec;
        if (T.e_wcol[w] >= T.e_wcol[w + 1]) continue;
        const int sa = sys_of(T.e_wcol[w] / 64), sb = sys_of((T.e_wcol[w + 1] - 1) / 64);
        for (int s = sa; s <= sb; ++s) {
            if (T.sys_u0[s + 1] == T.sys_u0[s]) continue;
            if (r_first[s] < 0) r_first[s] = rec;
            ++rec;
        }
    }
    T.sys_r0.assign(nsys + 1, rec);
    for (int s = nsys - 1; s >= 0; --s) T.sys_r0[s] = r_first[s] >= 0 ? r_first[s] : T.sys_r0[s + 1];
    if (T.bchunk.empty()) T.bchunk.push_back(make_int4(0, 0, 0, 0));
    if (T.kchunk.empty()) T.kchunk.push_back(make_int4(0, 0, 0, 0));
    if (T.eitems.empty()) T.eitems.push_back(KickItem{0, 0, 0, 0, 0, 0});
}

// pairs (i, j), i < j, of the rows' bodies [i0, i0 + ni) with j < j_end
// (local indices; j_end >= i0)
double row_area(long long i0, long long ni, long long j_end)
{
    const long long m = j_end - i0;
    if (m <= ni) return 0.5 * (double)m * (double)(m - 1);
    return 0.5 * (double)ni * (double)(ni - 1) + (double)ni * (double)(m - ni);
}

// the smallest j_end whose row_area reaches `target`
long long row_end_for(long long i0, long long ni, double target)
{
    const double tri = 0.5 * (double)ni * (double)(ni - 1);
    long long j;
    if (target <= tri)
        j = i0 + (long long)std::ceil(0.5 * (1.0 + std::sqrt(1.0 + 8.0 * target)));
    else
        j = i0 + ni + (long long)std::ceil((target - tri) / (double)ni);
    while (j > i0 + 1 && row_area(i0, ni, j - 1) >= target) --j;
    while (row_area(i0, ni, j) < target) ++j;
    return j;
}

// Balanced rows (kSymRows): each system's upper triangle in rows of BI
// bodies, each row cut along j into items of about equal pair count, so
// that all items fit in one round of the `slots` resident workgroups and
// finish together.  The first item of a row holds its diagonal block.
// Item t of row r writes its i-side partials to slot t and its reactions
// to slot KX + r (KX = the system's largest row item count); krow holds the
// item count of every row.  Returns false when the items do not fit.
bool build_rows(qsym_ctx *c, const Shape &sh, int slots, std::vector<KickItem> &items,
                std::vector<int4> &sysK, std::vector<int> &krow, int krow_base)
{
    const long long BI = (long long)sh.block * sh.ipl;
    // row item counts for a target item area A (at least one item per row,
    // items at least 64 columns wide)
    auto counts = [&](double A, std::vector<std::vector<int>> *out) {
        long long tot = 0;
        for (int s = 0; s < c->nsys; ++s) {
            const long long n = nsys_bodies(c->off, s);
            if (out) (*out)[s].clear();
            // the partial-slot budget: KX i-side slots + one per row
            const long long rows = (n + BI - 1) / BI;
            const long long kcap = std::max<long long>(1, partial_slots(n, c->L.jchunk_min) - rows);
            for (long long i0 = 0; i0 < n; i0 += BI) {
                const long long ni = std::min(BI, n - i0);
                const double area = row_area(i0, ni, n);
                const long long kmax = std::min(kcap, std::max<long long>(1, (n - i0 - ni) / 64 + 1));
                const long long k = std::min<long long>(kmax, std::max<long long>(1, (long long)std::ceil(area / A)));
                tot += k;
                if (out) (*out)[s].push_back((int)k);
            }
        }
        return tot;
    };
    double P = 0.0;
    for (int s = 0; s < c->nsys; ++s) {
        const double n = (double)nsys_bodies(c->off, s);
        P += 0.5 * n * (n - 1.0);
    }
    double lo = std::max(P / std::max(slots, 1), 1.0), hi = std::max(P, 1.0);
    if (counts(lo, nullptr) > slots) {
        for (int it = 0; it < 100; ++it) {
            const double mid = 0.5 * (lo + hi);
            if (counts(mid, nullptr) > slots) lo = mid; else hi = mid;
        }
        lo = hi;
    }
    std::vector<std::vector<int>> K(c->nsys);
    counts(lo, &K);
    int kb = krow_base;
    for (int s = 0; s < c->nsys; ++s) {
        const long long n = nsys_bodies(c->off, s);
        const long long o = c->off[s];
        int KX = 0;
        for (int k : K[s]) KX = std::max(KX, k);
        sysK[s] = make_int4(KX, (int)BI, kb, 2);
        int r = 0;
        for (long long i0 = 0; i0 < n; i0 += BI, ++r) {
            const long long ni = std::min(BI, n - i0);
            const int k = K[s][r];
            krow.push_back(k);
            const double area = row_area(i0, ni, n);
            long long ja = i0;
            for (int t = 0; t < k; ++t) {
                long long jb = t + 1 == k ? n : row_end_for(i0, ni, area * (t + 1) / k);
                if (t == 0) jb = std::max(jb, i0 + ni);          // the whole diagonal block
                jb = std::min(std::max(jb, ja + 1), n - (k - 1 - t));
                items.push_back(KickItem{s, (int)(o + i0), (int)ni, (int)(o + ja), (int)(jb - ja), t,
                                         KX + r});
                ja = jb;
            }
        }
        kb += r;
    }
    return true;
}

// kick work items for a launch shape; systems largest first, each system's
// items j-chunk major (consecutive items share j data)
// pairs i < j of a symmetric-kick item: i in [i0, i0 + ni), j in [j0, j0 + nj)
long long item_pairs(const KickItem &it)
{
    const long long a = it.i0, b = (long long)it.i0 + it.ni, c0 = it.j0, e = (long long)it.j0 + it.nj;
    // i below the chunk meets all of it; i inside it the part above i
    long long p = std::max(0ll, std::min(b, c0) - a) * it.nj;
    const long long lo = std::max(a, c0), hi = std::min(b, e);
    if (hi > lo) p += (2 * e - lo - hi - 1) * (hi - lo) / 2;   // sum of e - 1 - i over [lo, hi)
    return p;
}

// Dispatch order of the symmetric kick's items when the shape asks for it
// (remap bit 1; else chunk by chunk): largest first (the
// diagonal items, with a half or less of a full item's pairs, and the short
// items of a ragged last chunk at the end), so the workgroups dispatched
// last are the short ones and the compute units finish together.  With
// the XCD-aware order (workgroup b runs item (b % 8) * per + b / 8) the
// sorted items are dealt round robin into the eight XCDs' runs, each run
// still largest first.  Results do not depend on the order: every item
// writes its own partial slots.
void order_items(std::vector<KickItem> &items, int remap)
{
    std::vector<std::pair<long long, int>> w(items.size());
    for (size_t k = 0; k < items.size(); ++k) w[k] = {-item_pairs(items[k]), (int)k};
    std::stable_sort(w.begin(), w.end(),
                     [](const std::pair<long long, int> &x, const std::pair<long long, int> &y) {
                         return x.first < y.first;
                     });
    std::vector<KickItem> out;
    out.reserve(items.size());
    if (!remap) {
        for (const auto &x : w) out.push_back(items[x.second]);
    } else {
        // run r holds the item indices [r per, (r + 1) per) below n, per =
        // grid / 8 (the grid's padding workgroups, indices n and up, have
        // no item)
        const int n = (int)items.size();
        const int per = std::max(8, (n + 7) / 8 * 8) / 8;
        std::vector<std::vector<int>> run(8);
        auto cap = [&](int r) { return std::max(0, std::min(per, n - r * per)); };
        int x = 0;
        for (const auto &v : w) {
            while ((int)run[x].size() >= cap(x)) x = (x + 1) % 8;
            run[x].push_back(v.second);
            x = (x + 1) % 8;
        }
        for (int r = 0; r < 8; ++r)
            for (int k : run[r]) out.push_back(items[k]);
    }
    items.swap(out);
}

int build_items(qsym_ctx *c, const Shape &sh, std::vector<KickItem> &items, std::vector<int4> &sysK,
                int slots, std::vector<int> &krow, int krow_base)
{
    const long long BI = (long long)sh.block * sh.ipl;
    const long long JC = sh.jchunk;
    items.clear();
    sysK.assign(c->nsys, make_int4(0, 0, 0, 0));
    krow.clear();
    if (sh.sym == kSymRows) {
        build_rows(c, sh, slots, items, sysK, krow, krow_base);
        return (int)items.size();
    }
    std::vector<int> order(c->nsys);
    for (int s = 0; s < c->nsys; ++s) order[s] = s;
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) {
        return nsys_bodies(c->off, a) > nsys_bodies(c->off, b);
    });
    for (int s : order) {
        const int n = nsys_bodies(c->off, s);
        const int S = (int)((n + JC - 1) / JC);
        const long long o = c->off[s];
        if (sh.sym == 0) {
            sysK[s] = make_int4(S, (int)JC, 0, 0);
            for (int ch = 0; ch < S; ++ch)
                for (long long ib = 0; ib < n; ib += BI) {
                    KickItem it{s, (int)(o + ib), (int)std::min<long long>(BI, n - ib),
                                (int)(o + ch * JC), (int)std::min<long long>(JC, n - ch * JC), ch, 0};
                    items.push_back(it);
                }
        } else {
            // chunk ch meets the i-bodies below its end, in ranges of RB
            const long long RB = BI * sh.sym;
            sysK[s] = make_int4(S, (int)JC, (int)RB, 0);
            for (int ch = 0; ch < S; ++ch) {
                const long long hi = std::min<long long>((ch + 1) * JC, n);
                const int R = (int)((hi + RB - 1) / RB);
                for (int r = 0; r < R; ++r) {
                    KickItem it{s, (int)(o + r * RB), (int)std::min<long long>(RB, hi - r * RB),
                                (int)(o + ch * JC), (int)std::min<long long>(JC, n - ch * JC), ch,
                                S + r};
                    items.push_back(it);
                }
            }
        }
    }
    if (sh.sym != 0 && (sh.remap & 2)) order_items(items, sh.remap & 1);
    return (int)items.size();
}

int kick_occupancy(qsym_ctx *c, int which, const Shape &sh);

int upload_shape(qsym_ctx *c, int which)
{
    std::vector<KickItem> items;
    std::vector<int4> sysK;
    std::vector<int> krow;
    const Shape &sh = c->shape[which];
    const int slots = sh.sym == kSymRows ? c->cus * kick_occupancy(c, which, sh) : 0;
    const int krow_base = which * (int)c->L.krow_cap;
    const int n = build_items(c, sh, items, sysK, slots, krow, krow_base);
    if ((long long)n > c->L.max_items)
        return fail(c, QSYM_EINVAL, "kick shape needs more work items than the workspace holds");
    if ((long long)krow.size() > c->L.krow_cap)
        return fail(c, QSYM_EINVAL, "kick shape has more rows than the workspace holds");
    for (int s = 0; s < c->nsys; ++s) {
        const long long ns = nsys_bodies(c->off, s);
        if (sysK[s].w == 2) {
            // balanced rows: KX i-side slots + one j-side slot per row
            const long long rows = (ns + sysK[s].y - 1) / sysK[s].y;
            if (sysK[s].x + rows > partial_slots(ns, c->L.jchunk_min))
                return fail(c, QSYM_EINVAL, "balanced rows need more partial slots than the workspace holds");
            continue;
        }
        const long long Smax = (ns + c->L.jchunk_min - 1) / c->L.jchunk_min;
        const long long slots = sysK[s].x + (sysK[s].z > 0 ? (ns + sysK[s].z - 1) / sysK[s].z : 0);
        if (sysK[s].x > Smax || slots > partial_slots(ns, c->L.jchunk_min))
            return fail(c, QSYM_EINVAL, "j-chunk smaller than the workspace allows");
    }
    if (!krow.empty())
        HIPCHK(c, hipMemcpyAsync(c->d.krow + krow_base, krow.data(), sizeof(int) * krow.size(),
                                 hipMemcpyHostToDevice, c->stream));
    c->nitems[which] = n;
    c->grid_kick[which] = std::max(8, (n + 7) / 8 * 8);
    if (n > 0)
        HIPCHK(c, hipMemcpyAsync(c->d.items + (size_t)which * c->L.max_items, items.data(),
                                 sizeof(KickItem) * n, hipMemcpyHostToDevice, c->stream));
    HIPCHK(c, hipMemcpyAsync(c->d.sys_K + (size_t)which * c->nsys, sysK.data(), sizeof(int4) * c->nsys,
                             hipMemcpyHostToDevice, c->stream));
    HIPCHK(c, hipStreamSynchronize(c->stream));
    for (auto &g : c->g) g.valid = false;
    return QSYM_OK;
}

// ---------------------------------------------------------------- launches
unsigned long long *rec_slot(qsym_ctx *c, int nwg, hipStream_t st);

template <int BS, int IPL>
hipError_t launch_kick_bs(qsym_ctx *c, int mode, int prec, hipStream_t st)
{
    const int w = mode ? 1 : 0;
    const int xcd = c->shape[w].remap & 1;
    KickArgs ka{c->d, c->d.items + (size_t)w * c->L.max_items, c->p.G, c->L.cap, c->nitems[w],
                xcd, c->p.hill_mode, c->p.aE, c->p.crude_safety, c->tau_crude, 1e-200, 1.875, 1.5};
    const dim3 g(xcd ? c->grid_kick[w] : std::max(c->nitems[w], 1)), b(BS);
    // workgroup records only for the symmetric kick (its recording variant)
    if (c->shape[w].sym) ka.rec = rec_slot(c, (int)g.x, st);
    if (c->shape[w].sym) {
        // one or two i per lane (the shape check admits no other)
        if constexpr (IPL <= 2) {
            auto launch = [&](auto unit, auto recv) {
                constexpr bool U = decltype(unit)::value, R = decltype(recv)::value;
                if (prec == 0) {
                    if (mode == 0) hipLaunchKernelGGL((k_kick_sym<BS, IPL, 0, 0, U, R>), g, b, 0, st, ka);
                    else if (mode == 1) hipLaunchKernelGGL((k_kick_sym<BS, IPL, 1, 0, U, R>), g, b, 0, st, ka);
                    else hipLaunchKernelGGL((k_kick_sym<BS, IPL, 2, 0, U, R>), g, b, 0, st, ka);
                } else {
                    if (mode == 0) hipLaunchKernelGGL((k_kick_sym<BS, IPL, 0, 1, U, R>), g, b, 0, st, ka);
                    else if (mode == 1) hipLaunchKernelGGL((k_kick_sym<BS, IPL, 1, 1, U, R>), g, b, 0, st, ka);
                    else hipLaunchKernelGGL((k_kick_sym<BS, IPL, 2, 1, U, R>), g, b, 0, st, ka);
                }
            };
            if (c->nsys == 1) {
                if (ka.rec) launch(std::true_type{}, std::true_type{});
                else launch(std::true_type{}, std::false_type{});
            } else {
                if (ka.rec) launch(std::false_type{}, std::true_type{});
                else launch(std::false_type{}, std::false_type{});
            }
            return hipGetLastError();
        }
        return hipErrorInvalidValue;
    }
    if (prec == 0) {
        if (mode == 0) hipLaunchKernelGGL((k_kick<BS, IPL, 0, 0>), g, b, 0, st, ka);
        else if (mode == 1) hipLaunchKernelGGL((k_kick<BS, IPL, 1, 0>), g, b, 0, st, ka);
        else hipLaunchKernelGGL((k_kick<BS, IPL, 2, 0>), g, b, 0, st, ka);
    } else {
        if (mode == 0) hipLaunchKernelGGL((k_kick<BS, IPL, 0, 1>), g, b, 0, st, ka);
        else if (mode == 1) hipLaunchKernelGGL((k_kick<BS, IPL, 1, 1>), g, b, 0, st, ka);
        else hipLaunchKernelGGL((k_kick<BS, IPL, 2, 1>), g, b, 0, st, ka);
    }
    return hipGetLastError();
}

// mode 0: plain kick; 1, 2: kick with the crude sweep (mutual, sum)
hipError_t launch_kick(qsym_ctx *c, int mode, hipStream_t st)
{
    const int w = mode ? 1 : 0;
    const int prec = c->p.precision;
    const int ipl = c->shape[w].ipl, bs = c->shape[w].block;
    if (c->nitems[w] == 0) return hipSuccess;
    if (bs == 256) {
        if (ipl == 1) return launch_kick_bs<256, 1>(c, mode, prec, st);
        if (ipl == 2) return launch_kick_bs<256, 2>(c, mode, prec, st);
        return launch_kick_bs<256, 4>(c, mode, prec, st);
    }
    if (ipl == 1) return launch_kick_bs<128, 1>(c, mode, prec, st);
    if (ipl == 2) return launch_kick_bs<128, 2>(c, mode, prec, st);
    return launch_kick_bs<128, 4>(c, mode, prec, st);
}

// resident workgroups per compute unit of the kick kernel a shape launches
template <int BS, int IPL, bool U>
int occ_bs(int mode, int prec)
{
    int occ = 0;
    hipError_t e = hipErrorInvalidValue;
    auto query = [&](auto kernel) { e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, kernel, BS, 0); };
    if (prec == 0) {
        if (mode == 0) query(k_kick_sym<BS, IPL, 0, 0, U>);
        else if (mode == 1) query(k_kick_sym<BS, IPL, 1, 0, U>);
        else query(k_kick_sym<BS, IPL, 2, 0, U>);
    } else {
        if (mode == 0) query(k_kick_sym<BS, IPL, 0, 1, U>);
        else if (mode == 1) query(k_kick_sym<BS, IPL, 1, 1, U>);
        else query(k_kick_sym<BS, IPL, 2, 1, U>);
    }
    return (e == hipSuccess && occ > 0) ? occ : 1;
}

int kick_occupancy(qsym_ctx *c, int which, const Shape &sh)
{
    const int mode = which ? 1 + c->p.hill_mode : 0;
    auto occ = [&](auto unit) {
        constexpr bool U = decltype(unit)::value;
        const int prec = c->p.precision;
        if (sh.block == 256) return sh.ipl == 1 ? occ_bs<256, 1, U>(mode, prec) : occ_bs<256, 2, U>(mode, prec);
        return sh.ipl == 1 ? occ_bs<128, 1, U>(mode, prec) : occ_bs<128, 2, U>(mode, prec);
    };
    return c->nsys == 1 ? occ(std::true_type{}) : occ(std::false_type{});
}

int nblocks_chunks(qsym_ctx *c) { return (int)c->T.bchunk.size(); }

constexpr int kRecLaunches = 64;

// Busy time of each compute unit in one recorded launch: the union of the
// [start, end] intervals of the workgroups it ran (workgroups resident
// together count once).  Adds the largest and the mean over the device's
// compute units (idle ones count as zero) to the phase's sums.
void busy_launch(qsym_ctx *c, int ph, const unsigned long long *r, int nwg)
{
    std::vector<std::array<unsigned long long, 3>> v;
    v.reserve(nwg);
    for (int k = 0; k < nwg; ++k)
        if (r[3 * k] != 0 && r[3 * k + 2] >= r[3 * k + 1]) v.push_back({r[3 * k], r[3 * k + 1], r[3 * k + 2]});
    if (v.empty()) return;
    std::sort(v.begin(), v.end());
    unsigned long long total = 0, most = 0;
    int units = 0;
    for (size_t a = 0; a < v.size();) {
        size_t b = a;
        unsigned long long busy = 0, lo = v[a][1], hi = v[a][2];
        for (; b < v.size() && v[b][0] == v[a][0]; ++b) {
            if (v[b][1] > hi) {
                busy += hi - lo;
                lo = v[b][1];
                hi = v[b][2];
            } else {
                hi = std::max(hi, v[b][2]);
            }
        }
        busy += hi - lo;
        total += busy;
        most = std::max(most, busy);
        ++units;
        a = b;
    }
    // ticks of the 100 MHz real-time clock: 0.01 us each
    c->busy_max_us[ph] += 0.01 * (double)most;
    c->busy_mean_us[ph] += 0.01 * (double)total / std::max(c->cus, units);
    c->busy_calls[ph] += 1;
    c->busy_units = std::max(c->busy_units, units);
}

// the busy figures of the pending workgroup records (waits for the stream)
void flush_records(qsym_ctx *c)
{
    if (c->rec_pend.empty()) return;
    const size_t words = 3 * (size_t)c->rec_wg;
    std::vector<unsigned long long> h(words * c->rec_pend.size());
    if (hipStreamSynchronize(c->stream) == hipSuccess &&
        hipMemcpy(h.data(), c->rec, sizeof(unsigned long long) * h.size(), hipMemcpyDeviceToHost) ==
            hipSuccess) {
        for (size_t k = 0; k < c->rec_pend.size(); ++k)
            busy_launch(c, c->rec_pend[k].first, h.data() + words * k, c->rec_pend[k].second);
    }
    c->rec_pend.clear();
}

// accumulate the timings of all pending event pairs (waits for them) and
// the busy figures of the pending workgroup records
void flush_profile(qsym_ctx *c)
{
    for (size_t k = 0; k < c->pend_phase.size(); ++k) {
        float ms = 0.f;
        (void)hipEventSynchronize(c->pool[2 * k + 1]);
        if (hipEventElapsedTime(&ms, c->pool[2 * k], c->pool[2 * k + 1]) == hipSuccess) {
            c->phase_us[c->pend_phase[k]] += 1000.0 * ms;
            c->phase_calls[c->pend_phase[k]] += 1;
        }
    }
    c->pend_phase.clear();
    c->pool_used = 0;
    flush_records(c);
}

// record slot for a launch of nwg workgroups in the current phase (cleared
// on st), or null when not profiling or no memory for the records.  Called
// inside the launch's Timer: only the records are flushed here, the Timer's
// own event pair stays pending.
unsigned long long *rec_slot(qsym_ctx *c, int nwg, hipStream_t st)
{
    if (c->profile < 2 || nwg <= 0) return nullptr;
    if ((int)c->rec_pend.size() == kRecLaunches || nwg > c->rec_wg) flush_records(c);
    if (nwg > c->rec_wg) {
        if (c->rec) (void)hipFree(c->rec);
        c->rec = nullptr;
        c->rec_wg = 0;
        const int w = std::max(nwg, 1024);
        if (hipMalloc((void **)&c->rec, sizeof(unsigned long long) * 3 * (size_t)w * kRecLaunches) !=
            hipSuccess) {
            c->rec = nullptr;
            return nullptr;
        }
        c->rec_wg = w;
    }
    unsigned long long *r = c->rec + 3 * (size_t)c->rec_wg * c->rec_pend.size();
    if (hipMemsetAsync(r, 0, sizeof(unsigned long long) * 3 * (size_t)nwg, st) != hipSuccess)
        return nullptr;
    c->rec_pend.push_back({c->cur_phase, nwg});
    return r;
}

hipEvent_t pool_event(qsym_ctx *c)
{
    if (c->pool_used == c->pool.size()) {
        hipEvent_t e = nullptr;
        if (hipEventCreate(&e) != hipSuccess) return nullptr;
        c->pool.push_back(e);
    }
    return c->pool[c->pool_used++];
}

struct Timer {
    qsym_ctx *c;
    int ph;
    hipEvent_t e1 = nullptr;
    Timer(qsym_ctx *cc, int p) : c(cc), ph(p)
    {
        if (!c->profile) return;
        if (c->pend_phase.size() >= 4096) flush_profile(c);
        hipEvent_t e0 = pool_event(c);
        e1 = pool_event(c);
        if (!e0 || !e1) { e1 = nullptr; return; }
        c->pend_phase.push_back(ph);
        c->cur_phase = ph;
        (void)hipEventRecord(e0, c->stream);
    }
    ~Timer()
    {
        if (e1) (void)hipEventRecord(e1, c->stream);
    }
};

// backup (first drift of a hybrid step) keeps the state at the step's
// start; restore (its last drift) puts it back when the step could not hold
// its encounter pairs
hipError_t run_drift(qsym_ctx *c, double dt, int prepass, double tau_crude, int reset,
                     hipStream_t st, int phase, int count_step = 0, int backup = 0,
                     int restore = 0, int fused = 0)
{
    Timer tm(c, phase);
    DriftArgs a{c->d, dt, c->p.G, tau_crude, c->p.aE, c->p.crude_safety, prepass, c->p.hill_mode,
                reset, count_step, prepass && c->p.sweep == 1, backup, restore, fused};
    hipLaunchKernelGGL(k_drift, dim3(nblocks_chunks(c)), dim3(kChunk), 0, st, a);
    return hipGetLastError();
}

hipError_t run_momentum(qsym_ctx *c, hipStream_t st)
{
    Timer tm(c, P_MOMENTUM);
    hipLaunchKernelGGL(k_momentum, dim3(nblocks_chunks(c)), dim3(kChunk), 0, st, c->d);
    return hipGetLastError();
}

// kick apply (+ snapshot, + Kepler, + momentum partials).  Launches with a
// Kepler pass use 64-body workgroups (the solve is latency bound, so every
// CU gets work); the momentum partials need the 256-body chunks.
hipError_t run_apply(qsym_ctx *c, double dt_kick, double dt_kep, int do_kick, int do_kep,
                     int snapshot, int momentum, hipStream_t st, int phase, int which)
{
    Timer tm(c, phase);
    // kChunkK bodies per workgroup (the momentum partials are per such chunk)
    ApplyArgs a{c->d, c->d.kchunk, c->d.sys_K + (size_t)which * c->nsys, dt_kick, dt_kep, c->p.G,
                do_kick, do_kep, snapshot, c->p.kepler_mode, momentum};
    // systems of many bodies (tens of partial-sum slots per body) share each
    // body's reduction over four threads; many small systems keep one
    // thread per body
    const dim3 gk((unsigned)c->T.kchunk.size());
    if (c->apply_parts == 4)
        hipLaunchKernelGGL((k_apply_kepler<kChunkK, 4>), gk, dim3(kChunkK * 4), 0, st, a);
    else
        hipLaunchKernelGGL((k_apply_kepler<kChunkK, 1>), gk, dim3(kChunkK), 0, st, a);
    return hipGetLastError();
}

hipError_t run_kick(qsym_ctx *c, int crude, double tau_crude, hipStream_t st, int phase)
{
    Timer tm(c, phase);
    c->tau_crude = std::fabs(tau_crude);
    return launch_kick(c, crude ? 1 + c->p.hill_mode : 0, st);
}

// grid crude sweep (qsym_params.sweep = 1): grid constants and bucket
// clear, binning, search; the candidates land where the fused sweep puts
// them.  Timed with the first kick by the caller.
hipError_t launch_sweep(qsym_ctx *c, double tau, hipStream_t st)
{
    c->tau_crude = std::fabs(tau);
    KickArgs ka{c->d, nullptr, c->p.G, c->L.cap, 0, 0, c->p.hill_mode, c->p.aE, c->p.crude_safety,
                c->tau_crude, 1e-200, 1.875, 1.5};
    long long nmax = 0;
    for (int s = 0; s < c->nsys; ++s) nmax = std::max<long long>(nmax, nsys_bodies(c->off, s));
    SweepArgs a;
    a.ka = ka;
    a.nsys = c->nsys;
    a.ntot = (int)c->ntot;
    a.nsmall = (int)((14 * c->ntot + kSweepThreads - 1) / kSweepThreads);
    a.tiles = (int)std::max<long long>(1, (nmax + kSweepLargeTile - 1) / kSweepLargeTile);
    hipLaunchKernelGGL(k_sweep_bin, dim3(nblocks_chunks(c)), dim3(kChunk), 0, st, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_sweep_search, dim3(a.nsmall + 256), dim3(kSweepThreads), 0, st, a);
    return hipGetLastError();
}

// the first kick with its crude sweep: fused into the kick's pair loop
// (kick shape 1), or on the grid ahead of a plain kick (kick shape 0)
hipError_t run_kick1(qsym_ctx *c, double tau, hipStream_t st)
{
    if (!c->p.sweep) return run_kick(c, 1, tau, st, P_KICK1);
    Timer tm(c, P_KICK1);
    hipError_t e = launch_sweep(c, tau, st);
    if (e != hipSuccess) return e;
    return launch_kick(c, 0, st);
}

// workgroups of k_fine: enough for the candidate list, and for the
// all-pairs tiles when the list overflows
int fine_grid(qsym_ctx *c)
{
    const long long g = std::min<long long>((c->L.cap + 255) / 256, 128);
    const long long ge = std::min<long long>((long long)c->T.eitems.size(), 1024);
    return (int)std::max<long long>(1, std::max(g, ge));
}

// one full hybrid step (Sec. 2.3) enqueued on st
// the first drift of a hybrid step (1: drift tau/2 + per-body encounter
// terms, reset per-step counters, copy of the state at the step's start);
// between two steps of one call the previous step's last drift is made in
// the same launch (fused), otherwise it is a launch of its own (last)
hipError_t enqueue_first_drift(qsym_ctx *c, double tau, hipStream_t st, int fused)
{
    const double half = tau / 2.0;
    return run_drift(c, half, 1, tau, 1, st, P_DRIFT, fused, 1, fused, fused);
}

hipError_t enqueue_last_drift(qsym_ctx *c, double tau, hipStream_t st)
{
    // 10: drift tau/2 (or, for a step that could not hold its encounter
    // pairs, the state at its start)
    return run_drift(c, tau / 2.0, 0, 0.0, 0, st, P_DRIFT2, 1, 0, 1);
}

// steps 2-9 of a hybrid step (Sec. 2.3), between its two drifts
hipError_t enqueue_step_body(qsym_ctx *c, double tau, hipStream_t st)
{
    hipError_t e;
    const double half = tau / 2.0;
    // 2: kick tau/2 with the crude sweep
    if ((e = run_kick1(c, tau, st)) != hipSuccess) return e;
    // 2-3: apply the kick, snapshot (q0, v0), Kepler tau -> (q1, v1)
    if ((e = run_apply(c, half, tau, 1, 1, 1, 0, st, P_APPLY1, c->p.sweep ? 0 : 1)) != hipSuccess)
        return e;
    // 4: fine sweep, sets, r_crit
    {
        Timer tm(c, P_FINE);
        FineArgs fa{c->d, tau, c->p.aE, c->p.crude_safety, std::fabs(tau), c->L.cap,
                    c->p.hill_mode, (int)c->T.eitems.size()};
        hipLaunchKernelGGL(k_fine, dim3(fine_grid(c)), dim3(256), 0, st, fa);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    {
        Timer tm(c, P_SETS);
        SetsArgs sa{c->d, c->p.aH, c->p.planet_mass};
        hipLaunchKernelGGL(k_sets, dim3(c->nsys), dim3(kSetsThreads), 0, st, sa);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    // 5-7: corrections and Hermite per set
    {
        Timer tm(c, P_HERMITE);
        // one workgroup per compute unit, all resident: the grid phase's
        // barriers need them together
        HermArgs ha{c->d, tau, c->p.G, c->p.epsH, c->p.eta, c->p.eta_s, c->p.max_substeps,
                    rec_slot(c, c->grid_blocks, st), c->d.gbar, c->d.hpart};
        hipLaunchKernelGGL(k_hermite, dim3(c->grid_blocks), dim3(kHermThreads), 0, st, ha);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    // 9: kick tau/2 (all pairs), applied with the momentum partials
    if ((e = run_kick(c, 0, 0.0, st, P_KICK2)) != hipSuccess) return e;
    return run_apply(c, half, 0.0, 1, 0, 0, 1, st, P_APPLY2, 0);
}

// body + the fused drift between this step and the next (the steps before a
// call's last), body + the last drift (its last step)
hipError_t enqueue_step_mid(qsym_ctx *c, double tau, hipStream_t st)
{
    hipError_t e = enqueue_step_body(c, tau, st);
    if (e != hipSuccess) return e;
    return enqueue_first_drift(c, tau, st, 1);
}

hipError_t enqueue_step_last(qsym_ctx *c, double tau, hipStream_t st)
{
    hipError_t e = enqueue_step_body(c, tau, st);
    if (e != hipSuccess) return e;
    return enqueue_last_drift(c, tau, st);
}

// Kick shape of both kicks until the autotuner or a tuned table replaces it.
//
// One system of 5000 bodies or more: the symmetric kick.  Its items should
// number some 1500 (about six a compute unit), so they grow with the system:
// 128, 256, then 512 i against enough j for that, up to 1536 j (longer items
// leave a ragged last round), largest first and XCD-aware; and i-ranges of
// as many blocks as the partial slots need.  Measured against
// the full-matrix shape, fused / plain kick in us: 4100 bodies 28.8 / 24.3
// against 29.5 / 23.7 (so the line is at 5000), 8200 53 / 47 against 76 / 64,
// 12,000 94 / 81 against 135 / 114, 25,000 281 / 252 against 528 / 458, 40,003
// 649 / 595 against 1293 / 1091, 90,000 3353 / 3014 against 6186 / 5502.
// Both kicks with their reductions on either side of the lines between the
// blocks, us of 128 / 256 / 512 i: 5200 bodies 87 / 92 / 180, 8200 119 / 132 /
// 180, 8500 148 / 134 / 182, 9999 175 / 165 / 185, 16,000 346 / 277 / 263, 18,000
// 463 / 340 / 349, 19,999 529 / 400 / 435, 20,500 537 / 448 / 444, 22,500 744 / 493
// / 453.  (The 256 i as 128 threads with two each: within 5% either way from
// 12,000 to 20,000, 277 / 281 and 340 / 358 at 16,000 and 18,000.)
// From 532,481 bodies on i-ranges of eight blocks need more partial slots than
// there are: the full matrix, as before the rule.
//
// Otherwise the full matrix, one i per lane, with j-chunks that give the
// grid 4096 workgroups where the size allows: small kicks are bound by the
// length of one workgroup's chain, which is shorter without the reactions,
// and the sums of a context of many systems keep their order.
Shape default_shape(qsym_ctx *c)
{
    Shape sh;
    const long long jmin = c->L.jchunk_min;
    const long long n = c->ntot;
    if (c->nsys == 1 && n >= 5000) {
        sh.block = n < 8400 ? 128 : 256;
        sh.ipl = n < 20000 ? 1 : 2;
        sh.remap = 3;
        const long long BI = (long long)sh.block * sh.ipl;
        const long long want = std::min<long long>(n * n / (3000 * BI), 1536);
        const long long jc = std::max((want + BI / 2) / BI * BI, (jmin + BI - 1) / BI * BI);
        sh.jchunk = std::max(jc, BI);
        const long long slots = partial_slots(n, jmin) - (n + sh.jchunk - 1) / sh.jchunk;
        sh.sym = 1;
        while (sh.sym < 8 && (n + BI * sh.sym - 1) / (BI * sh.sym) > slots) sh.sym *= 2;
        if ((n + BI * sh.sym - 1) / (BI * sh.sym) <= slots) return sh;
    }
    sh.block = 128;
    sh.ipl = 1;
    sh.remap = 0;
    sh.sym = 0;
    long long jc = 8192;
    while (jc > jmin) {
        long long items = 0;
        for (int s = 0; s < c->nsys; ++s) {
            const long long ns = nsys_bodies(c->off, s);
            items += ((ns + 127) / 128) * ((ns + jc - 1) / jc);
        }
        if (items >= 4096) break;
        jc /= 2;
    }
    sh.jchunk = std::max<long long>(jc, jmin);
    sh.jchunk = (sh.jchunk + 127) / 128 * 128;
    return sh;
}

void enter(qsym_ctx *c)
{
    (void)hipEventRecord(c->ev_in, c->ustream);
    (void)hipStreamWaitEvent(c->stream, c->ev_in, 0);
}

void leave(qsym_ctx *c)
{
    (void)hipEventRecord(c->ev_out, c->stream);
    (void)hipStreamWaitEvent(c->ustream, c->ev_out, 0);
}

int status_code(qsym_ctx *c, unsigned long long st)
{
    if (st & S_NONFINITE) return fail(c, QSYM_ENONFINITE, "non-finite value in the state");
    if (st & (S_CAND_OVF | S_ENC_OVF))
        return fail(c, QSYM_EOVERFLOW, (st & S_CAND_OVF)
                                           ? "crude-candidate capacity exceeded"
                                           : "a system had more encounter pairs than its segment "
                                             "holds (4 per body + 64); the state is that of the "
                                             "start of that step");
    if (st & (S_HERMITE | S_SET_BIG))
        return fail(c, QSYM_EHERMITE, "Hermite substep cap reached or set too large");
    if (st & S_KEPLER) return fail(c, QSYM_EKEPLER, "Kepler solver reached its iteration cap");
    return QSYM_OK;
}

int read_ctr(qsym_ctx *c, unsigned long long *h)
{
    HIPCHK(c, hipMemcpyAsync(h, c->d.ctr, sizeof(unsigned long long) * C_COUNT,
                             hipMemcpyDeviceToHost, c->stream));
    HIPCHK(c, hipStreamSynchronize(c->stream));
    return QSYM_OK;
}

int sync_status(qsym_ctx *c)
{
    unsigned long long h[C_COUNT];
    int rc = read_ctr(c, h);
    if (rc) return rc;
    return status_code(c, h[C_STATUS]);
}

// Whether one kernel may move a state from or to the caller's arrays of
// `bytes` each in place of a copy per coordinate: every array lies inside one
// allocation of this device's memory (a copy takes memory of any kind and
// refuses to run over an allocation's end), is aligned for its doubles and
// outside this workspace, and no two written arrays overlap.  The copies,
// which run one after another, give the same bits wherever both may run.
// set_state and get_state of 104 bodies: 88 -> 32 and 89 -> 33 us a call.
struct Span {
    const void *p;
    size_t bytes;
};

bool apart(const Span &a, const Span &b)
{
    const char *x = (const char *)a.p, *y = (const char *)b.p;
    return x + a.bytes <= y || y + b.bytes <= x;
}

bool one_kernel_moves(qsym_ctx *c, const Span *s, int count, bool written)
{
    const Span ws{c->base, c->L.total};
    for (int k = 0; k < count; ++k) {
        if (!s[k].p) continue;
        hipPointerAttribute_t at{};
        hipDeviceptr_t start = nullptr;
        size_t size = 0;
        if (hipPointerGetAttributes(&at, s[k].p) != hipSuccess ||
            hipMemGetAddressRange(&start, &size, (hipDeviceptr_t)s[k].p) != hipSuccess) {
            (void)hipGetLastError();
            return false;
        }
        const char *p = (const char *)s[k].p;
        if (at.type != hipMemoryTypeDevice || at.device != c->device || at.isManaged ||
            (uintptr_t)p % sizeof(double) || p < (const char *)start ||
            p + s[k].bytes > (const char *)start + size || !apart(s[k], ws))
            return false;
        for (int j = 0; written && j < k; ++j)
            if (s[j].p && !apart(s[j], s[k])) return false;
    }
    return true;
}

// Encounter-free step with the Keplerian and interaction operators swapped
// (Sec. 2, after the composition): E_Dft(tau/2) E_Kep(tau/2) E_Int(tau)
// E_Kep(tau/2) E_Dft(tau/2); one all-pairs kick per step.  The kick and the
// second Kepler half-step share one pass over the bodies.
// the swapped step E_Dft(tau/2) E_Kep(tau/2) E_Int(tau) E_Kep(tau/2)
// E_Dft(tau/2): its first drift (fused with the previous step's last
// between two steps of one call), its body, its last drift
hipError_t enqueue_swapped_first_drift(qsym_ctx *c, double tau, hipStream_t st, int fused)
{
    return run_drift(c, tau / 2.0, 0, 0.0, 1, st, P_DRIFT, fused, 0, 0, fused);
}

hipError_t enqueue_swapped_body(qsym_ctx *c, double tau, hipStream_t st)
{
    hipError_t e;
    const double half = tau / 2.0;
    if ((e = run_apply(c, 0.0, half, 0, 1, 0, 0, st, P_APPLY1, 0)) != hipSuccess) return e;
    if ((e = run_kick(c, 0, 0.0, st, P_KICK2)) != hipSuccess) return e;
    return run_apply(c, tau, half, 1, 1, 0, 1, st, P_APPLY2, 0);
}

hipError_t enqueue_swapped_mid(qsym_ctx *c, double tau, hipStream_t st)
{
    hipError_t e = enqueue_swapped_body(c, tau, st);
    if (e != hipSuccess) return e;
    return enqueue_swapped_first_drift(c, tau, st, 1);
}

hipError_t enqueue_swapped_last(qsym_ctx *c, double tau, hipStream_t st)
{
    hipError_t e = enqueue_swapped_body(c, tau, st);
    if (e != hipSuccess) return e;
    return run_drift(c, tau / 2.0, 0, 0.0, 0, st, P_DRIFT2, 1);
}

// Whether this context's systems belong in k_small_steps: their sizes say so,
// and the crude sweep is the fused one
bool small_context(const qsym_ctx *c)
{
    return c->L.small && !c->p.sweep && small_route(c->off.data(), c->nsys, c->cus);
}

// Whether the steps run there now: with full-matrix kicks (whose partial sums
// it reproduces) and no per-kernel timings asked for
bool small_steps(const qsym_ctx *c)
{
    return small_context(c) && !c->profile && !c->shape[0].sym && !c->shape[1].sym;
}

hipError_t run_small(qsym_ctx *c, double tau, int64_t nsteps, int kind)
{
    SmallArgs a{};
    a.d = c->d;
    a.w = (unsigned long long *)(c->base + c->L.off_small);
    a.st = a.w + SW_COUNT;
    a.h = HermArgs{c->d, tau, c->p.G, c->p.epsH, c->p.eta, c->p.eta_s, c->p.max_substeps};
    a.aE = c->p.aE;
    a.aH = c->p.aH;
    a.cs = c->p.crude_safety;
    a.planet_mass = c->p.planet_mass;
    a.r2seed = 1e-200;
    a.c158 = 1.875;
    a.c32 = 1.5;
    a.cap = c->L.cap;
    for (int w = 0; w < 2; ++w) a.jc[w] = (int)std::min<long long>(c->shape[w].jchunk, kSmallMax);
    a.hill_mode = c->p.hill_mode;
    a.kepler_mode = c->p.kepler_mode;
    a.nsys = c->nsys;
    for (int64_t k = 0; k < nsteps; k += kSmallSteps) {
        a.nsteps = (int)std::min<int64_t>(nsteps - k, kSmallSteps);
        a.first = k == 0;
        // with several systems: the second launch takes the steps again when
        // one of them overflowed its encounter segment, else it does nothing
        for (a.redo = 0; a.redo <= (c->nsys > 1 && kind == 0 ? 1 : 0); ++a.redo) {
            const dim3 g(c->nsys), b(kSmallThreads);
            if (kind == 0) {
                if (c->p.precision == 0) hipLaunchKernelGGL((k_small_steps<0, false>), g, b, 0, c->stream, a);
                else hipLaunchKernelGGL((k_small_steps<1, false>), g, b, 0, c->stream, a);
            } else {
                if (c->p.precision == 0) hipLaunchKernelGGL((k_small_steps<0, true>), g, b, 0, c->stream, a);
                else hipLaunchKernelGGL((k_small_steps<1, true>), g, b, 0, c->stream, a);
            }
            const hipError_t e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
    }
    return hipSuccess;
}

constexpr int kGraphSteps = 8;     // steps of one graph
constexpr int kGraphAfter = 64;    // steps of one tau before its graph is made
constexpr long long kGraphBodies = 8192;   // contexts of fewer bodies use graphs

// nsteps steps of one kind (0 hybrid, 1 swapped)
int run_steps(qsym_ctx *c, double tau, int64_t nsteps, int kind)
{
    if (!c || nsteps < 0 || !std::isfinite(tau)) return fail(c, QSYM_EINVAL, "step: bad argument");
    if (c->p.kepler_mode == 2 && !c->guess_loaded)
        return fail(c, QSYM_EINVAL, "kepler_mode 2 needs weights (qsym_set_guess)");
    if (nsteps == 0 || c->ntot == 0) return QSYM_OK;
    enter(c);
    if (small_steps(c)) {
        HIPCHK(c, run_small(c, tau, nsteps, kind));
        leave(c);
        return QSYM_OK;
    }
    // a call of n steps: the first drift, then n - 1 times the step body
    // with the fused drift between steps, then the last body and drift
    using Enq = hipError_t (*)(qsym_ctx *, double, hipStream_t);
    const Enq mid = kind == 0 ? enqueue_step_mid : enqueue_swapped_mid;
    const Enq last = kind == 0 ? enqueue_step_last : enqueue_swapped_last;
    auto first = [&]() {
        return kind == 0 ? enqueue_first_drift(c, tau, c->stream, 0)
                         : enqueue_swapped_first_drift(c, tau, c->stream, 0);
    };
    // Launched one by one, or, below kGraphBodies, in graphs of kGraphSteps
    // steps.  The device waits some 20 us between two graphs, more than the
    // host takes to launch a step's kernels, so a graph holds several steps;
    // and it costs 22 us a node to capture and instantiate, so it is made once
    // the steps already taken with this tau would have paid for it.
    // Intervals of 20 steps as graphs of one step, one by one, and as graphs
    // of eight, in us: 1024 bodies 1868, 1852, 1770; 4100: 2455, 2407, 2351;
    // 16,388: 7197, 7086, 7103; 8 steps of the 512-system batch 17,580,
    // 17,530, 17,970; first interval of a context, 1024 bodies: 2459, 2080.
    // A caller who captures the stream gets the launches: a capture cannot
    // begin inside another, and a graph launched there is not recorded.
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    HIPCHK(c, hipStreamIsCapturing(c->stream, &capture));
    const bool captured = capture != hipStreamCaptureStatusNone;
    auto &G = c->g[kind];
    if (!captured && G.tau != tau) {
        G.tau = tau;
        G.seen = 0;
        G.valid = false;
    }
    const int64_t mids = nsteps - 1;
    const bool graphs = !c->profile && !captured && c->ntot < kGraphBodies;
    if (graphs && !G.valid && G.seen >= kGraphAfter && mids >= kGraphSteps) {
        if (G.exec) { hipGraphExecDestroy(G.exec); G.exec = nullptr; }
        if (G.graph) { hipGraphDestroy(G.graph); G.graph = nullptr; }
        HIPCHK(c, hipStreamBeginCapture(c->stream, hipStreamCaptureModeThreadLocal));
        hipError_t e = hipSuccess;
        for (int k = 0; k < kGraphSteps && e == hipSuccess; ++k) e = mid(c, tau, c->stream);
        hipGraph_t g = nullptr;
        const hipError_t e2 = hipStreamEndCapture(c->stream, &g);
        if (e != hipSuccess || e2 != hipSuccess) {
            if (g) hipGraphDestroy(g);
            return fail(c, QSYM_EHIP, std::string("graph capture: ") +
                                          hipGetErrorString(e != hipSuccess ? e : e2));
        }
        G.graph = g;
        HIPCHK(c, hipGraphInstantiate(&G.exec, G.graph, nullptr, nullptr, 0));
        G.valid = true;
    }
    HIPCHK(c, first());
    int64_t k = 0;
    if (graphs && G.valid)
        for (; mids - k >= kGraphSteps; k += kGraphSteps) HIPCHK(c, hipGraphLaunch(G.exec, c->stream));
    for (; k < mids; ++k) HIPCHK(c, mid(c, tau, c->stream));
    HIPCHK(c, last(c, tau, c->stream));
    if (!captured) G.seen += nsteps;
    leave(c);
    return QSYM_OK;
}

}  // namespace

// ====================================================================== ABI
extern "C" {

int qsym_workspace_bytes(const qsym_params *p, int32_t nsys, const int64_t *offsets, int64_t *bytes)
{
    std::string msg;
    int rc = validate(p, nsys, offsets, msg);
    if (rc) return rc;
    if (!bytes) return QSYM_EINVAL;
    std::vector<long long> off(offsets, offsets + nsys + 1);
    *bytes = (int64_t)make_layout(*p, off).total;
    return QSYM_OK;
}

int qsym_create(const qsym_params *p, int32_t nsys, const int64_t *offsets, const double *m0,
                void *workspace, int64_t ws_bytes, void *stream, qsym_ctx **out)
{
    if (!out) return QSYM_EINVAL;
    *out = nullptr;
    std::string msg;
    int rc = validate(p, nsys, offsets, msg);
    if (rc) return rc;
    if (!m0 || !workspace) return QSYM_EINVAL;
    for (int s = 0; s < nsys; ++s)
        if (!(m0[s] > 0)) return QSYM_EINVAL;
    if (((uintptr_t)workspace) % 256) return QSYM_EINVAL;
    qsym_ctx *c = new qsym_ctx();
    c->p = *p;
    c->nsys = nsys;
    c->off.assign(offsets, offsets + nsys + 1);
    c->m0.assign(m0, m0 + nsys);
    c->ntot = c->off.back();
    c->L = make_layout(*p, c->off);
    if ((long long)ws_bytes < (long long)c->L.total) {
        delete c;
        return QSYM_ENOMEM;
    }
    c->base = (char *)workspace;
    c->d = bind(c->base, c->L);
    c->ustream = (hipStream_t)stream;
    auto bail = [&](int code, const char *what) {
        const hipError_t e = hipGetLastError();
        g_noctx_err = std::string("qsym_create: ") + what + ": " + hipGetErrorString(e);
        if (c->stream) (void)hipStreamDestroy(c->stream);
        if (c->result) (void)hipHostFree(c->result);
        delete c;
        return code;
    };
    if (hipStreamCreateWithFlags(&c->stream, hipStreamNonBlocking) != hipSuccess)
        return bail(QSYM_EHIP, "hipStreamCreateWithFlags");
    {
        int dev = 0, cus = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
            return bail(QSYM_EHIP, "hipDeviceGetAttribute");
        // the Hermite's grid phase needs every workgroup resident at once:
        // one per compute unit, and only if the kernel fits one per unit
        int occ = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, k_hermite, kHermThreads, 0) !=
                hipSuccess || occ < 1)
            return bail(QSYM_EHIP, "k_hermite does not fit a compute unit");
        c->grid_blocks = std::max(1, std::min(cus, kGridMax));
        c->cus = std::max(1, cus);
        c->device = dev;
    }
    if (hipHostMalloc((void **)&c->result, sizeof(unsigned long long) * (size_t)(1 + nsys)) != hipSuccess)
        return bail(QSYM_EHIP, "hipHostMalloc");
    if (hipEventCreateWithFlags(&c->ev_in, hipEventDisableTiming) != hipSuccess)
        return bail(QSYM_EHIP, "hipEventCreateWithFlags");
    if (hipEventCreateWithFlags(&c->ev_out, hipEventDisableTiming) != hipSuccess)
        return bail(QSYM_EHIP, "hipEventCreateWithFlags");
    build_tables(c);
    {
        long long nmax = 0;
        for (int k = 0; k < nsys; ++k) nmax = std::max<long long>(nmax, c->off[k + 1] - c->off[k]);
        c->apply_parts = nmax >= 8192 ? 4 : 1;
    }
    enter(c);
    hipStream_t st = c->stream;
    // zero the whole workspace once (outside any graph)
    if (hipMemsetAsync(c->base, 0, c->L.total, st) != hipSuccess) return bail(QSYM_EHIP, "hipMemsetAsync");
    const Tables &T = c->T;
    bool ok = true;
    ok &= hipMemcpyAsync(c->d.sys_off, T.sys_off.data(), sizeof(int) * T.sys_off.size(),
                         hipMemcpyHostToDevice, st) == hipSuccess;
    ok &= hipMemcpyAsync(c->d.sys_m0, c->m0.data(), sizeof(double) * nsys, hipMemcpyHostToDevice,
                         st) == hipSuccess;
    ok &= hipMemcpyAsync(c->d.sys_poff, T.sys_poff.data(), sizeof(long long) * nsys,
                         hipMemcpyHostToDevice, st) == hipSuccess;
    ok &= hipMemcpyAsync(c->d.sys_c0, T.sys_c0.data(), sizeof(int) * T.sys_c0.size(),
                         hipMemcpyHostToDevice, st) == hipSuccess;
    ok &= hipMemcpyAsync(c->d.sys_k0, T.sys_k0.data(), sizeof(int) * T.sys_k0.size(),
                         hipMemcpyHostToDevice, st) == hipSuccess;
    ok &= hipMemcpyAsync(c->d.sys_e0, T.sys_e0.data(), sizeof(int) * T.sys_e0.size(),
                         hipMemcpyHostToDevice, st) == hipSuccess;
    ok &= hipMemcpyAsync(c->d.sys_eoff, T.sys_eoff.data(), sizeof(int) * T.sys_eoff.size(),
                         hipMemcpyHostToDevice, st) == hipSuccess;
    ok &= hipMemcpyAsync(c->d.sys_goff, T.sys_goff.data(), sizeof(long long) * nsys,
                         hipMemcpyHostToDevice, st) == hipSuccess;
    ok &= hipMemcpyAsync(c->d.sys_u0, T.sys_u0.data(), sizeof(long long) * T.sys_u0.size(),
                         hipMemcpyHostToDevice, st) == hipSuccess;
    ok &= hipMemcpyAsync(c->d.e_wcol, T.e_wcol.data(), sizeof(long long) * T.e_wcol.size(),
                         hipMemcpyHostToDevice, st) == hipSuccess;
    ok &= hipMemcpyAsync(c->d.e_wrec, T.e_wrec.data(), sizeof(int) * T.e_wrec.size(),
                         hipMemcpyHostToDevice, st) == hipSuccess;
    ok &= hipMemcpyAsync(c->d.sys_r0, T.sys_r0.data(), sizeof(int) * T.sys_r0.size(),
                         hipMemcpyHostToDevice, st) == hipSuccess;
    ok &= hipMemcpyAsync(c->d.bchunk, T.bchunk.data(), sizeof(int4) * T.bchunk.size(),
                         hipMemcpyHostToDevice, st) == hipSuccess;
    ok &= hipMemcpyAsync(c->d.kchunk, T.kchunk.data(), sizeof(int4) * T.kchunk.size(),
                         hipMemcpyHostToDevice, st) == hipSuccess;
    ok &= hipMemcpyAsync(c->d.eitems, T.eitems.data(), sizeof(KickItem) * T.eitems.size(),
                         hipMemcpyHostToDevice, st) == hipSuccess;
    ok &= hipMemcpyAsync(c->d.body_sys, T.body_sys.data(), sizeof(int) * T.body_sys.size(),
                         hipMemcpyHostToDevice, st) == hipSuccess;
    ok &= hipStreamSynchronize(st) == hipSuccess;
    if (!ok) return bail(QSYM_EHIP, "table upload");
    c->shape[0] = c->shape[1] = default_shape(c);
    if (upload_shape(c, 0) != QSYM_OK || upload_shape(c, 1) != QSYM_OK) {
        g_noctx_err = c->err;
        return bail(QSYM_EINVAL, "kick shape upload");
    }
    leave(c);
    *out = c;
    return QSYM_OK;
}

void qsym_destroy(qsym_ctx *c)
{
    if (!c) return;
    if (c->stream) hipStreamSynchronize(c->stream);
    for (auto &g : c->g) {
        if (g.exec) hipGraphExecDestroy(g.exec);
        if (g.graph) hipGraphDestroy(g.graph);
    }
    for (hipEvent_t e : c->pool) (void)hipEventDestroy(e);
    if (c->rec) (void)hipFree(c->rec);
    if (c->ev_in) hipEventDestroy(c->ev_in);
    if (c->ev_out) hipEventDestroy(c->ev_out);
    if (c->stream) hipStreamDestroy(c->stream);
    if (c->result) hipHostFree(c->result);
    delete c;
}

int qsym_set_state(qsym_ctx *c, const double *m, const double *h, const double *q, const double *v,
                   int32_t where)
{
    if (!c || !m || !h || !q || !v || (where != QSYM_HOST && where != QSYM_DEVICE))
        return fail(c, QSYM_EINVAL, "set_state: bad argument");
    const long long n = c->ntot;
    const hipMemcpyKind kind = where == QSYM_HOST ? hipMemcpyHostToDevice : hipMemcpyDeviceToDevice;
    enter(c);
    hipStream_t st = c->stream;
    const size_t B = sizeof(double) * (size_t)n;
    const Span in[4] = {{m, B}, {h, B}, {q, 3 * B}, {v, 3 * B}};
    if (n > 0 && where == QSYM_DEVICE && one_kernel_moves(c, in, 4, false)) {
        {
            Timer tm(c, P_MOMENTUM);
            const LoadArgs a{c->d, m, h, q, v, n};
            hipLaunchKernelGGL(k_load_state, dim3(nblocks_chunks(c)), dim3(kChunk), 0, st, a);
            HIPCHK(c, hipGetLastError());
        }
        HIPCHK(c, hipStreamSynchronize(st));   // nothing is left for the caller's stream to wait for
        return QSYM_OK;
    }
    if (n > 0) {
        HIPCHK(c, hipMemcpyAsync(c->d.m, m, B, kind, st));
        HIPCHK(c, hipMemcpyAsync(c->d.h, h, B, kind, st));
        double *qd[3] = {c->d.x, c->d.y, c->d.z};
        double *vd[3] = {c->d.vx, c->d.vy, c->d.vz};
        for (int k = 0; k < 3; ++k) {
            HIPCHK(c, hipMemcpyAsync(qd[k], q + k * n, B, kind, st));
            HIPCHK(c, hipMemcpyAsync(vd[k], v + k * n, B, kind, st));
        }
    }
    HIPCHK(c, run_momentum(c, st));
    // a new state starts with a clear device status (the latched bits
    // described the state it replaces)
    HIPCHK(c, hipMemsetAsync(c->d.ctr + C_STATUS, 0, sizeof(unsigned long long), st));
    HIPCHK(c, hipStreamSynchronize(st));
    leave(c);
    return QSYM_OK;
}

int qsym_get_state(qsym_ctx *c, double *q, double *v, int32_t where)
{
    if (!c || (where != QSYM_HOST && where != QSYM_DEVICE)) return fail(c, QSYM_EINVAL, "get_state: bad argument");
    const long long n = c->ntot;
    const hipMemcpyKind kind = where == QSYM_HOST ? hipMemcpyDeviceToHost : hipMemcpyDeviceToDevice;
    enter(c);
    hipStream_t st = c->stream;
    const size_t B = sizeof(double) * (size_t)n;
    const Span out[2] = {{q, 3 * B}, {v, 3 * B}};
    if (n > 0 && where == QSYM_DEVICE && one_kernel_moves(c, out, 2, true)) {
        const StoreArgs a{c->d, q, v, n, c->result};
        hipLaunchKernelGGL(k_store_state, dim3((unsigned)((n + kChunk - 1) / kChunk)), dim3(kChunk), 0,
                           st, a);
        HIPCHK(c, hipGetLastError());
        HIPCHK(c, hipStreamSynchronize(st));
        return status_code(c, c->result[0]);
    }
    const double *qd[3] = {c->d.x, c->d.y, c->d.z};
    const double *vd[3] = {c->d.vx, c->d.vy, c->d.vz};
    for (int k = 0; k < 3 && n > 0; ++k) {
        if (q) HIPCHK(c, hipMemcpyAsync(q + k * n, qd[k], B, kind, st));
        if (v) HIPCHK(c, hipMemcpyAsync(v + k * n, vd[k], B, kind, st));
    }
    HIPCHK(c, hipStreamSynchronize(st));
    leave(c);
    return sync_status(c);
}

int qsym_step(qsym_ctx *c, double tau, int64_t nsteps) { return run_steps(c, tau, nsteps, 0); }

int qsym_step_swapped(qsym_ctx *c, double tau, int64_t nsteps)
{
    return run_steps(c, tau, nsteps, 1);
}

int qsym_set_guess(qsym_ctx *c, const float *weights, int32_t where)
{
    if (!c || !weights || (where != QSYM_HOST && where != QSYM_DEVICE))
        return fail(c, QSYM_EINVAL, "set_guess: bad argument");
    enter(c);
    HIPCHK(c, hipMemcpyAsync(c->d.guess, weights, sizeof(float) * kGuessWeights,
                             where == QSYM_HOST ? hipMemcpyHostToDevice : hipMemcpyDeviceToDevice,
                             c->stream));
    HIPCHK(c, hipStreamSynchronize(c->stream));
    leave(c);
    c->guess_loaded = true;
    return QSYM_OK;
}

int qsym_sync(qsym_ctx *c)
{
    if (!c) return QSYM_EINVAL;
    HIPCHK(c, hipStreamSynchronize(c->stream));
    return sync_status(c);
}

int qsym_energy(qsym_ctx *c, double *E)
{
    if (!c || !E) return fail(c, QSYM_EINVAL, "energy: bad argument");
    enter(c);
    hipStream_t st = c->stream;
    {
        Timer tm(c, P_ENERGY);
        EnergyArgs ea{c->d, c->p.G, c->nsys, c->result};
        hipLaunchKernelGGL(k_energy_pairs, dim3((unsigned)(c->L.e_waves / 4)), dim3(256), 0, st, ea);
        HIPCHK(c, hipGetLastError());
        hipLaunchKernelGGL(k_energy_final, dim3(c->nsys), dim3(256), 0, st, ea);
        HIPCHK(c, hipGetLastError());
    }
    HIPCHK(c, hipStreamSynchronize(st));
    std::memcpy(E, c->result + 1, sizeof(double) * (size_t)c->nsys);
    return status_code(c, c->result[0]);
}

int qsym_encounters(qsym_ctx *c, int32_t *pairs, int64_t cap, int64_t *n_pairs, int32_t *set_id)
{
    if (!c || !n_pairs || cap < 0 || (cap > 0 && !pairs)) return fail(c, QSYM_EINVAL, "encounters: bad argument");
    unsigned long long h[C_COUNT];
    int rc = read_ctr(c, h);
    if (rc) return rc;
    const long long ne = (long long)h[C_ENC];
    *n_pairs = ne;
    hipStream_t st = c->stream;
    if (cap > 0 && ne > 0) {
        // the device keeps per-system segments in append order; the
        // canonical (i < j, lexicographic) order is produced here
        std::vector<int> cnt(c->nsys);
        std::vector<int2> seg((size_t)c->L.ecap);
        HIPCHK(c, hipMemcpyAsync(cnt.data(), c->d.sys_ecnt, sizeof(int) * c->nsys, hipMemcpyDeviceToHost, st));
        HIPCHK(c, hipMemcpyAsync(seg.data(), c->d.enc, sizeof(int2) * c->L.ecap, hipMemcpyDeviceToHost, st));
        HIPCHK(c, hipStreamSynchronize(st));
        std::vector<int2> raw;
        for (int s = 0; s < c->nsys; ++s) {
            const int held = std::min(cnt[s], c->T.sys_eoff[s + 1] - c->T.sys_eoff[s]);
            for (int k = 0; k < held; ++k) raw.push_back(seg[(size_t)c->T.sys_eoff[s] + k]);
        }
        std::sort(raw.begin(), raw.end(), [](const int2 &a, const int2 &b) {
            return a.x != b.x ? a.x < b.x : a.y < b.y;
        });
        const long long k = std::min<long long>((long long)raw.size(), cap);
        for (long long q = 0; q < k; ++q) {
            pairs[2 * q] = raw[q].x;
            pairs[2 * q + 1] = raw[q].y;
        }
    }
    if (set_id) {
        for (long long i = 0; i < c->ntot; ++i) set_id[i] = -1;
        const long long ns = (long long)h[C_NSETS], nu = (long long)h[C_NU];
        if (ns > 0 && !(h[C_STATUS] & S_ENC_OVF)) {
            std::vector<int> start(ns), count(ns), mem(nu);
            HIPCHK(c, hipMemcpyAsync(start.data(), c->d.set_start, sizeof(int) * ns, hipMemcpyDeviceToHost, st));
            HIPCHK(c, hipMemcpyAsync(count.data(), c->d.set_count, sizeof(int) * ns, hipMemcpyDeviceToHost, st));
            HIPCHK(c, hipMemcpyAsync(mem.data(), c->d.set_mem, sizeof(int) * nu, hipMemcpyDeviceToHost, st));
            HIPCHK(c, hipStreamSynchronize(st));
            // sets are numbered by their smallest member (members ascend)
            std::vector<long long> order(ns);
            for (long long s = 0; s < ns; ++s) order[s] = s;
            std::sort(order.begin(), order.end(),
                      [&](long long a, long long b) { return mem[start[a]] < mem[start[b]]; });
            for (long long r = 0; r < ns; ++r) {
                const long long s = order[r];
                for (int b = start[s]; b < start[s] + count[s]; ++b) set_id[mem[b]] = (int32_t)r;
            }
        }
    }
    HIPCHK(c, hipStreamSynchronize(st));
    rc = status_code(c, h[C_STATUS]);
    if (rc) return rc;
    if (ne > cap) return fail(c, QSYM_ETRUNC, "encounter buffer shorter than the count");
    return QSYM_OK;
}

int qsym_set_rcrit(qsym_ctx *c, double *rcrit, int64_t cap, int64_t *n_sets)
{
    if (!c || !n_sets || cap < 0 || (cap > 0 && !rcrit)) return fail(c, QSYM_EINVAL, "set_rcrit: bad argument");
    unsigned long long h[C_COUNT];
    int rc = read_ctr(c, h);
    if (rc) return rc;
    rc = status_code(c, h[C_STATUS]);
    if (rc) return rc;
    const long long ns = (long long)h[C_NSETS], nu = (long long)h[C_NU];
    *n_sets = ns;
    if (ns > 0 && cap > 0) {
        hipStream_t st = c->stream;
        std::vector<int> start(ns), mem(nu);
        std::vector<double> rcv(ns);
        HIPCHK(c, hipMemcpyAsync(start.data(), c->d.set_start, sizeof(int) * ns, hipMemcpyDeviceToHost, st));
        HIPCHK(c, hipMemcpyAsync(mem.data(), c->d.set_mem, sizeof(int) * nu, hipMemcpyDeviceToHost, st));
        HIPCHK(c, hipMemcpyAsync(rcv.data(), c->d.set_rc, sizeof(double) * ns, hipMemcpyDeviceToHost, st));
        HIPCHK(c, hipStreamSynchronize(st));
        // sets numbered by their smallest member (members ascend), as in
        // qsym_encounters
        std::vector<long long> order(ns);
        for (long long s = 0; s < ns; ++s) order[s] = s;
        std::sort(order.begin(), order.end(),
                  [&](long long a, long long b) { return mem[start[a]] < mem[start[b]]; });
        const long long k = std::min<long long>(ns, cap);
        for (long long r = 0; r < k; ++r) rcrit[r] = rcv[order[r]];
    }
    if (ns > cap) return fail(c, QSYM_ETRUNC, "r_crit buffer shorter than the set count");
    return QSYM_OK;
}

int qsym_candidates(qsym_ctx *c, int32_t *pairs, int64_t cap, int64_t *n)
{
    if (!c || !n || cap < 0 || (cap > 0 && !pairs)) return fail(c, QSYM_EINVAL, "candidates: bad argument");
    unsigned long long h[C_COUNT];
    int rc = read_ctr(c, h);
    if (rc) return rc;
    const long long nc = (long long)h[C_CAND];
    *n = nc;
    const long long k = std::min<long long>(std::min<long long>(nc, c->L.cap), cap);
    if (k > 0) {
        HIPCHK(c, hipMemcpyAsync(pairs, c->d.cand, sizeof(int2) * k, hipMemcpyDeviceToHost, c->stream));
        HIPCHK(c, hipStreamSynchronize(c->stream));
    }
    if (nc > c->L.cap) return fail(c, QSYM_EOVERFLOW, "crude-candidate capacity exceeded");
    if (nc > cap) return fail(c, QSYM_ETRUNC, "candidate buffer shorter than the count");
    return QSYM_OK;
}

int qsym_stats(qsym_ctx *c, qsym_stats_t *out)
{
    if (!c || !out) return QSYM_EINVAL;
    unsigned long long h[C_COUNT];
    int rc = read_ctr(c, h);
    if (rc) return rc;
    flush_profile(c);
    std::memset(out, 0, sizeof(*out));
    out->steps = (int64_t)h[C_STEPS];
    out->n_candidates = (int64_t)h[C_CAND];
    out->n_encounters = (int64_t)h[C_ENC];
    out->n_sets = (int64_t)h[C_NSETS];
    out->max_set = (int64_t)h[C_MAXSET];
    out->substeps = (int64_t)h[C_SUB];
    out->total_encounters = (int64_t)h[C_TENC];
    out->total_substeps = (int64_t)h[C_TSUB];
    {
        // the striped Kepler statistics, added up here
        std::vector<unsigned long long> ks((size_t)kStatStripes * kStatStride);
        HIPCHK(c, hipMemcpyAsync(ks.data(), c->d.kstat, sizeof(unsigned long long) * ks.size(),
                                 hipMemcpyDeviceToHost, c->stream));
        HIPCHK(c, hipStreamSynchronize(c->stream));
        unsigned long long kit = 0, kmax = 0, hist[kHist] = {};
        for (int s = 0; s < kStatStripes; ++s) {
            const unsigned long long *k = ks.data() + (size_t)s * kStatStride;
            for (int b = 0; b < kHist; ++b) hist[b] += k[b];
            kit += k[kHist];
            kmax = std::max(kmax, k[kHist + 1]);
        }
        unsigned long long krs = 0;
        for (int s = 0; s < kStatStripes; ++s) krs += ks[(size_t)s * kStatStride + kHist + 2];
        out->kepler_restarts = (int64_t)krs;
        out->kepler_iters = (int64_t)kit;
        out->kepler_max = (int64_t)kmax;
        for (int b = 0; b < kHist; ++b) out->kepler_hist[b] = (int64_t)hist[b];
    }
    out->status = (int64_t)h[C_STATUS];
    out->whole_system = (int64_t)h[C_WHOLE];
    out->fallbacks = (int64_t)h[C_FALLBACK];
    out->overflows = (int64_t)h[C_OVERFLOW];
    out->global_sets = (int64_t)h[C_TBIGSYS];
    for (int k = 0; k < kPhases; ++k) {
        out->phase_us[k] = c->phase_us[k];
        out->phase_calls[k] = c->phase_calls[k];
        out->busy_max_us[k] = c->busy_max_us[k];
        out->busy_mean_us[k] = c->busy_mean_us[k];
        out->busy_calls[k] = c->busy_calls[k];
    }
    out->busy_units = c->busy_units;
    return QSYM_OK;
}

const char *qsym_last_error(const qsym_ctx *c) { return c ? c->err.c_str() : g_noctx_err.c_str(); }

int qsym_apply_drift(qsym_ctx *c, double dt)
{
    if (!c) return QSYM_EINVAL;
    enter(c);
    HIPCHK(c, run_drift(c, dt, 0, 0.0, 0, c->stream, P_DRIFT));
    leave(c);
    return QSYM_OK;
}

int qsym_apply_kick(qsym_ctx *c, double dt, double crude_tau)
{
    if (!c) return QSYM_EINVAL;
    enter(c);
    hipStream_t st = c->stream;
    const int crude = crude_tau != 0.0;
    if (crude) HIPCHK(c, run_drift(c, 0.0, 1, crude_tau, 1, st, P_DRIFT));
    if (crude)
        HIPCHK(c, run_kick1(c, crude_tau, st));
    else
        HIPCHK(c, run_kick(c, 0, 0.0, st, P_KICK2));
    HIPCHK(c, run_apply(c, dt, 0.0, 1, 0, 0, 1, st, P_APPLY2, crude && !c->p.sweep ? 1 : 0));
    leave(c);
    return QSYM_OK;
}

int qsym_apply_kepler(qsym_ctx *c, double dt)
{
    if (!c) return QSYM_EINVAL;
    if (c->p.kepler_mode == 2 && !c->guess_loaded)
        return fail(c, QSYM_EINVAL, "kepler_mode 2 needs weights (qsym_set_guess)");
    enter(c);
    HIPCHK(c, run_apply(c, 0.0, dt, 0, 1, 0, 1, c->stream, P_APPLY1, 0));
    leave(c);
    return QSYM_OK;
}

int qsym_fine_test(const qsym_params *p, double m0, double tau, int64_t n, const double *m,
                   const double *h, const double *A, const double *q0, const double *v0,
                   const double *q1, const double *v1, int64_t npairs, const int32_t *pairs,
                   int32_t *flags, double *lhs, double *rhs, void *stream)
{
    if (!p || npairs < 0 || n < 0 || !(m0 > 0)) return QSYM_EINVAL;
    if (npairs == 0) return QSYM_OK;
    if (!m || !h || !A || !q0 || !v0 || !q1 || !v1 || !pairs || !flags) return QSYM_EINVAL;
    hipStream_t st = (hipStream_t)stream;
    const unsigned grid = (unsigned)((npairs + 255) / 256);
    hipLaunchKernelGGL(k_fine_standalone, dim3(grid), dim3(256), 0, st, p->hill_mode, p->aE, m0, tau,
                       (long long)n, m, h, A, q0, v0, q1, v1, (long long)npairs, (const int *)pairs,
                       (int *)flags, lhs, rhs);
    if (hipGetLastError() != hipSuccess) return QSYM_EHIP;
    if (hipStreamSynchronize(st) != hipSuccess) return QSYM_EHIP;
    return QSYM_OK;
}

int qsym_set_kick_shape(qsym_ctx *c, int32_t which, int32_t ipl, int32_t block, int64_t jchunk,
                        int32_t remap, int32_t sym)
{
    if (!c) return QSYM_EINVAL;
    if ((which < -1 || which > 1) || (ipl != 1 && ipl != 2 && ipl != 4) ||
        (block != 128 && block != 256) || jchunk <= 0 || jchunk % block ||
        jchunk < c->L.jchunk_min || remap < 0 || remap > 3 || (remap > 1 && sym == 0) ||
        (sym != 0 && sym != 1 && sym != 2 && sym != 4 && sym != 8 && sym != kSymRows) ||
        (sym && (ipl > 2 || jchunk % ((long long)block * ipl))))
        return fail(c, QSYM_EINVAL, "kick shape out of range");
    for (int w = 0; w < 2; ++w) {
        if (which >= 0 && w != which) continue;
        const Shape old = c->shape[w];
        c->shape[w] = Shape{ipl, block, jchunk, remap, sym};
        const int rc = upload_shape(c, w);
        if (rc) {
            c->shape[w] = old;
            (void)upload_shape(c, w);
            return rc;
        }
    }
    return QSYM_OK;
}

int qsym_get_kick_shape(qsym_ctx *c, int32_t which, int32_t *ipl, int32_t *block, int64_t *jchunk,
                        int32_t *remap, int32_t *sym)
{
    if (!c || which < 0 || which > 1) return QSYM_EINVAL;
    const Shape &sh = c->shape[which];
    if (ipl) *ipl = sh.ipl;
    if (block) *block = sh.block;
    if (jchunk) *jchunk = sh.jchunk;
    if (remap) *remap = sh.remap;
    if (sym) *sym = sh.sym;
    return QSYM_OK;
}

int qsym_autotune(qsym_ctx *c, double tau, double *us)
{
    if (!c) return QSYM_EINVAL;
    if (c->ntot == 0) return QSYM_OK;
    enter(c);
    hipStream_t st = c->stream;
    // the crude sweep needs the per-body terms: compute them at the current
    // state without moving it (drift by 0)
    HIPCHK(c, run_drift(c, 0.0, 1, tau, 1, st, P_OTHER));
    c->tau_crude = std::fabs(tau);
    hipEvent_t e0, e1;
    HIPCHK(c, hipEventCreate(&e0));
    HIPCHK(c, hipEventCreate(&e1));
    const int ipls[3] = {1, 2, 4};
    const int blocks[2] = {128, 256};
    // a symmetric kick would take a small context out of k_small_steps for
    // the sake of one kernel (512 systems of 192 bodies: 131 us a step there,
    // 180 in the step's kernels)
    const bool full_only = small_context(c);
    int rc = QSYM_OK;
    for (int w = 0; w < 2; ++w) {
        const int mode = w ? 1 + c->p.hill_mode : 0;
        Shape best = c->shape[w];
        double best_us = 1e300;
        // full-matrix shapes, then symmetric ones (i-blocks per item 1, 2, 4)
        std::vector<Shape> cand;
        for (int bi = 0; bi < 2; ++bi)
            for (int ii = 0; ii < 3; ++ii)
                for (long long jc = c->L.jchunk_min; jc <= std::max<long long>(c->L.jchunk_min, 8192);
                     jc *= 2) {
                    const long long jcr = (jc + blocks[bi] - 1) / blocks[bi] * blocks[bi];
                    for (int rm = 0; rm < 2; ++rm) cand.push_back(Shape{ipls[ii], blocks[bi], jcr, rm, 0});
                    // symmetric kick: one or two i per lane
                    const long long BI = (long long)blocks[bi] * ipls[ii];
                    const long long jcs = (jc + BI - 1) / BI * BI;
                    if (ipls[ii] <= 2 && !full_only)
                        for (int sy = 1; sy <= 4; sy *= 2)
                            for (int rm = 0; rm < 4; ++rm)
                                cand.push_back(Shape{ipls[ii], blocks[bi], jcs, rm, sy});
                }
        // balanced rows (the j-chunk plays no part: the smallest allowed)
        for (int bi = 0; bi < 2 && !full_only; ++bi)
            for (int ii = 0; ii < 2; ++ii) {
                const long long BI = (long long)blocks[bi] * ipls[ii];
                const long long jcs = (c->L.jchunk_min + BI - 1) / BI * BI;
                cand.push_back(Shape{ipls[ii], blocks[bi], jcs, 0, kSymRows});
            }
        for (const Shape &sh : cand) {
            c->shape[w] = sh;
            if (upload_shape(c, w) != QSYM_OK) continue;
            // warm-up, then 3 timed launches of the kick and of the
            // reduction of its partial sums (an apply with dt = 0, which
            // leaves the state as it is): shapes with more partial slots
            // pay for them there
            (void)launch_kick(c, mode, st);
            (void)run_apply(c, 0.0, 0.0, 1, 0, 0, 0, st, P_OTHER, w);
            (void)hipEventRecord(e0, st);
            for (int r = 0; r < 3; ++r) {
                (void)launch_kick(c, mode, st);
                (void)run_apply(c, 0.0, 0.0, 1, 0, 0, 0, st, P_OTHER, w);
            }
            (void)hipEventRecord(e1, st);
            (void)hipEventSynchronize(e1);
            float ms = 0.f;
            (void)hipEventElapsedTime(&ms, e0, e1);
            const double t_us = 1000.0 * ms / 3.0;
            if (t_us < best_us) {
                best_us = t_us;
                best = c->shape[w];
            }
        }
        c->shape[w] = best;
        const int r = upload_shape(c, w);
        if (r) rc = r;
        if (us) us[w] = best_us;
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    // leave the counters of the next step clean
    HIPCHK(c, run_drift(c, 0.0, 1, tau, 1, st, P_OTHER));
    HIPCHK(c, hipStreamSynchronize(st));
    leave(c);
    return rc;
}

int qsym_profile(qsym_ctx *c, int32_t enable)
{
    if (!c) return QSYM_EINVAL;
    (void)hipStreamSynchronize(c->stream);
    flush_profile(c);
    c->profile = enable < 0 ? 0 : std::min(enable, 2);
    if (enable) {
        for (int k = 0; k < kPhases; ++k) {
            c->phase_us[k] = 0.0;
            c->phase_calls[k] = 0;
            c->busy_max_us[k] = c->busy_mean_us[k] = 0.0;
            c->busy_calls[k] = 0;
        }
        c->busy_units = 0;
    }
    return QSYM_OK;
}

}  // extern "C"
