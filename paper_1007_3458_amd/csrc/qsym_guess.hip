// qsym_guess.hip -- stand-alone Kepler solves and the training of the learned
// starting value of the Newton iteration (features, scalers, gradient of the
// loss by backpropagation, Adam) for MI355X / gfx950.
//
// The network and its features are defined in qsym_kepler.hpp.  Training
// samples are stored column-major in FP32: rows 0..3 of `feat` hold the
// features f0..f3 and row 4 the target y = ln(x / x_p) / T, each row `ld`
// floats apart.  The loss over n samples is (1/n) sum (o - (y - m_y)/s_y)^2.
#include "qsym.h"

#include <algorithm>
#include <cmath>
#include <mutex>
#include <string>

#include "qsym_kepler.hpp"

using namespace qsym;

namespace {

constexpr int kGPart = kGuessParams + 1;    // gradient sums + loss sum of one workgroup
constexpr int kGMaxParts = 4096;            // workgroups of one gradient launch
constexpr int kGMomBlocks = 1024;           // blocks of the moments reduction
constexpr int kGMaxEpochs = 4096;

struct State6 {
    const double *x, *y, *z, *vx, *vy, *vz;
};

__device__ __forceinline__ void body_terms(const State6 &s, long long i, double &r0, double &rv,
                                           double &vv)
{
    const double x = s.x[i], y = s.y[i], z = s.z[i], vx = s.vx[i], vy = s.vy[i], vz = s.vz[i];
    r0 = sqrt(x * x + y * y + z * z);
    vv = vx * vx + vy * vy + vz * vz;
    rv = x * vx + y * vy + z * vz;
}

// universal anomaly of each body for its own step (Appendix A solve);
// iters < 0 marks a solve that reached the cap from every start
__global__ __launch_bounds__(256) void k_kepler_solve(double mu, long long n, State6 s,
                                                      const double *__restrict__ dt, int mode,
                                                      const float *__restrict__ w,
                                                      double *__restrict__ xo, int *__restrict__ it)
{
    const long long i = blockIdx.x * 256LL + threadIdx.x;
    if (i >= n) return;
    const double h = dt[i];
    if (h == 0.0) {
        xo[i] = 0.0;
        if (it) it[i] = 0;
        return;
    }
    double r0, rv, vv;
    body_terms(s, i, r0, rv, vv);
    const double smu = sqrt(mu);
    const double alpha = 2.0 / r0 - vv / mu;
    int count = 0, restart;
    double x;
    const int ok = kepler_root(smu, r0, rv, alpha, h, mode, w, x, count, restart);
    xo[i] = x;
    if (it) it[i] = ok ? count : -count;
}

// learned start alone (0 for a zero step)
__global__ __launch_bounds__(256) void k_kepler_guess(double mu, long long n, State6 s,
                                                      const double *__restrict__ dt,
                                                      const float *__restrict__ w,
                                                      double *__restrict__ xo)
{
    const long long i = blockIdx.x * 256LL + threadIdx.x;
    if (i >= n) return;
    const double h = dt[i];
    if (h == 0.0) {
        xo[i] = 0.0;
        return;
    }
    double r0, rv, vv;
    body_terms(s, i, r0, rv, vv);
    const double smu = sqrt(mu);
    xo[i] = guess_start(w, smu, r0, rv, 2.0 / r0 - vv / mu, h);
}

// features (and targets when xr is given) of n solved bodies; *bad counts
// samples that cannot be used (zero step, non-finite feature or target)
__global__ __launch_bounds__(256) void k_guess_prepare(double mu, long long n, State6 s,
                                                       const double *__restrict__ dt,
                                                       const double *__restrict__ xr,
                                                       float *__restrict__ feat, long long ld,
                                                       unsigned long long *bad)
{
    const long long i = blockIdx.x * 256LL + threadIdx.x;
    if (i >= n) return;
    const double h = dt[i];
    double r0, rv, vv;
    body_terms(s, i, r0, rv, vv);
    const double smu = sqrt(mu);
    float f[4] = {NAN, NAN, NAN, NAN}, T = NAN;
    float y = 0.0f;
    bool ok = h != 0.0;
    if (ok) {
        guess_features(smu, r0, rv, 2.0 / r0 - vv / mu, h, f, T);
        if (xr) {
            const double Td = smu * fabs(h) / (r0 * sqrt(r0));
            y = (float)(log(xr[i] / (smu * h / r0)) / Td);
            ok = isfinite(y);
        }
        for (int c = 0; c < 4; ++c) ok = ok && isfinite(f[c]);
    }
    for (int c = 0; c < 4; ++c) feat[c * ld + i] = f[c];
    feat[4 * ld + i] = y;
    if (!ok) atomicAdd(bad, 1ULL);
}

// per-block FP64 sums of each of the 5 rows and of their squares
__global__ __launch_bounds__(256) void k_guess_moments(long long n, const float *__restrict__ feat,
                                                       long long ld, double *__restrict__ part)
{
    __shared__ double red[10][256];
    double a[10] = {};
    for (long long i = blockIdx.x * 256LL + threadIdx.x; i < n; i += 256LL * gridDim.x)
        for (int c = 0; c < 5; ++c) {
            const double v = feat[c * ld + i];
            a[c] += v;
            a[5 + c] += v * v;
        }
    for (int c = 0; c < 10; ++c) red[c][threadIdx.x] = a[c];
    __syncthreads();
    for (int st = 128; st > 0; st >>= 1) {
        if ((int)threadIdx.x < st)
            for (int c = 0; c < 10; ++c) red[c][threadIdx.x] += red[c][threadIdx.x + st];
        __syncthreads();
    }
    if (threadIdx.x < 10) part[blockIdx.x * 10 + threadIdx.x] = red[threadIdx.x][0];
}

// means and population deviations into the scaler slots of w (a deviation
// of 0 or a non-finite one becomes 1)
__global__ void k_guess_scalers(const double *__restrict__ part, int nb, long long n,
                                float *__restrict__ w)
{
    const int c = threadIdx.x;
    if (c >= 5) return;
    double s = 0.0, q = 0.0;
    for (int b = 0; b < nb; ++b) {
        s += part[b * 10 + c];
        q += part[b * 10 + 5 + c];
    }
    const double mean = s / (double)n;
    double var = q / (double)n - mean * mean;
    double sd = var > 0.0 ? sqrt(var) : 0.0;
    if (!(sd > 0.0) || !isfinite(sd)) sd = 1.0;
    float *sc = w + kGuessParams;
    if (c < 4) {
        sc[c] = (float)mean;
        sc[4 + c] = (float)sd;
    } else {
        sc[8] = (float)mean;
        sc[9] = (float)sd;
    }
}

// Loss gradient sums over n samples on the matrix cores: a workgroup of four
// waves takes tiles of 64 samples (strided over the grid), a wave 16 of them.
// All products are FP32 16x16x4 MFMA steps (A: row l % 16, k = l / 16 of lane
// l; B: column l % 16, k = l / 16; C: rows 4 (l / 16) + 0..3, column l % 16).
//
// Forward and back, a column is a sample and a row a unit: the four rows a
// lane holds of one result are the k = l / 16 terms of four steps of the next
// product, once the columns of its weights are taken in that order (k of
// step r: 4 (l / 16) + r), so layer follows layer without a move.  The
// gradient sums run over samples; for them the unit rows go through LDS once,
// transposed.  b1, b2, w3 and w1 take a product each whose B holds a column of
// ones, the errors or the inputs.
//
// A lane per sample, 1024 fma in a row per layer on 128 waves, was bound by
// that chain: 65 us at 8192 samples (of which the products need 0.7 us at the
// card's FP32 rate), this 8.0 us.  part[workgroup] receives sum e dO/dw (e
// = o - target; the factor 2/n is applied by the update) and sum e^2.
typedef float f32x4 __attribute__((ext_vector_type(4)));
constexpr int kGWaves = 4;
constexpr int kGStride = 36;   // floats per sample row of the transposed units (16-byte rows)

struct GradWave {
    float h1[16][kGStride], h2[16][kGStride], d1[16][kGStride], d2[16][kGStride];
    float in[16][8];   // standardised inputs, 1, e, 0, 0
};

__device__ __forceinline__ f32x4 mfma16(float a, float b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

__global__ __launch_bounds__(64 * kGWaves) void k_guess_grad(const float *__restrict__ w,
                                                             const float *__restrict__ feat,
                                                             long long ld, long long n,
                                                             float *__restrict__ part)
{
    __shared__ __align__(16) union {
        GradWave wave[kGWaves];
        float sum[kGWaves][kGPart];
    } L;
    const int t = threadIdx.x, l = t & 63, wv = t >> 6;
    const int u = l & 15, g = l >> 4;
    GradWave &S = L.wave[wv];
    const float *sc = w + kGuessParams;
    // weights in operand order: w1 rows, w2 rows and columns, biases and w3 in
    // the rows a lane holds
    float a1[2], a2[2][2][4], at[2][2][4];
    f32x4 b1[2], b2[2], w3[2];
#pragma unroll
    for (int m = 0; m < 2; ++m) {
        a1[m] = w[kGW1 + 4 * (16 * m + u) + g];
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                a2[m][k][r] = w[kGW2 + 32 * (16 * m + u) + 16 * k + 4 * g + r];
                at[m][k][r] = w[kGW2 + 32 * (16 * k + 4 * g + r) + 16 * m + u];
            }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            b1[m][r] = w[kGB1 + 16 * m + 4 * g + r];
            b2[m][r] = w[kGB2 + 16 * m + 4 * g + r];
            w3[m][r] = w[kGW3 + 16 * m + 4 * g + r];
        }
    }
    const float bias3 = w[kGB3];
    const float mean = sc[g], dev = sc[4 + g], ymean = sc[8], ydev = sc[9];
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    f32x4 gw2[2][2] = {{zero, zero}, {zero, zero}};   // [units of layer 2][of layer 1]
    f32x4 g1[2] = {zero, zero};                       // columns 0-3: w1, 4: b1
    f32x4 g2[2] = {zero, zero};                       // column 4: b2
    f32x4 g3[2] = {zero, zero};                       // column 5: w3
    float gb3 = 0.f, lsum = 0.f;
    for (long long tile = blockIdx.x; tile * 64 < n; tile += gridDim.x) {
        const long long s = tile * 64 + 16 * wv + u;
        const bool valid = s < n;
        const float in = valid ? (feat[g * ld + s] - mean) / dev : 0.f;
        const float yt = valid ? (feat[4 * ld + s] - ymean) / ydev : 0.f;
        f32x4 h1[2], h2[2], d1[2], d2[2];
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            h1[m] = mfma16(a1[m], in, b1[m]);
#pragma unroll
            for (int r = 0; r < 4; ++r) h1[m][r] = tanh_fast(h1[m][r]);
        }
        float o = 0.f;
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            f32x4 z = b2[m];
#pragma unroll
            for (int k = 0; k < 2; ++k)
#pragma unroll
                for (int r = 0; r < 4; ++r) z = mfma16(a2[m][k][r], h1[k][r], z);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                h2[m][r] = tanh_fast(z[r]);
                o = fmaf(w3[m][r], h2[m][r], o);
            }
        }
        o += __shfl_xor(o, 16, 64);
        o += __shfl_xor(o, 32, 64);
        const float e = valid ? o + bias3 - yt : 0.f;
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int r = 0; r < 4; ++r) d2[m][r] = e * w3[m][r] * (1.f - h2[m][r] * h2[m][r]);
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            f32x4 z = zero;
#pragma unroll
            for (int k = 0; k < 2; ++k)
#pragma unroll
                for (int r = 0; r < 4; ++r) z = mfma16(at[m][k][r], d2[k][r], z);
#pragma unroll
            for (int r = 0; r < 4; ++r) d1[m][r] = z[r] * (1.f - h1[m][r] * h1[m][r]);
        }
        // transposed through the wave's LDS (rows of a sample)
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            *reinterpret_cast<f32x4 *>(&S.h1[u][16 * m + 4 * g]) = h1[m];
            *reinterpret_cast<f32x4 *>(&S.h2[u][16 * m + 4 * g]) = h2[m];
            *reinterpret_cast<f32x4 *>(&S.d1[u][16 * m + 4 * g]) = d1[m];
            *reinterpret_cast<f32x4 *>(&S.d2[u][16 * m + 4 * g]) = d2[m];
        }
        S.in[u][g] = in;
        S.in[u][4 + g] = g == 0 ? 1.f : (g == 1 ? e : 0.f);
        __syncthreads();   // (every wave runs the same tiles)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int sm = 4 * q + g;   // the sample of this lane's k
            const float x = u < 5 ? S.in[sm][u] : 0.f;
            const float one = u == 4 ? 1.f : 0.f, err = u == 5 ? S.in[sm][5] : 0.f;
            const float hb[2] = {S.h1[sm][u], S.h1[sm][16 + u]};
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                const float dk = S.d2[sm][16 * m + u];
                gw2[m][0] = mfma16(dk, hb[0], gw2[m][0]);
                gw2[m][1] = mfma16(dk, hb[1], gw2[m][1]);
                g2[m] = mfma16(dk, one, g2[m]);
                g1[m] = mfma16(S.d1[sm][16 * m + u], x, g1[m]);
                g3[m] = mfma16(S.h2[sm][16 * m + u], err, g3[m]);
            }
        }
        gb3 += e;
        lsum = fmaf(e, e, lsum);
        __syncthreads();
    }
    // the waves' sums through LDS, added in wave order
    float *p = L.sum[wv];
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int row = 16 * m + 4 * g + r;
            p[kGW2 + 32 * row + u] = gw2[m][0][r];
            p[kGW2 + 32 * row + 16 + u] = gw2[m][1][r];
            if (u < 4) p[kGW1 + 4 * row + u] = g1[m][r];
            if (u == 4) {
                p[kGB1 + row] = g1[m][r];
                p[kGB2 + row] = g2[m][r];
            }
            if (u == 5) p[kGW3 + row] = g3[m][r];
        }
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) {
        gb3 += __shfl_xor(gb3, o, 64);
        lsum += __shfl_xor(lsum, o, 64);
    }
    if (l == 0) {
        p[kGB3] = gb3;
        p[kGuessParams] = lsum;
    }
    __syncthreads();
    for (int k = t; k < kGPart; k += 64 * kGWaves)
        part[(long long)blockIdx.x * kGPart + k] = (L.sum[0][k] + L.sum[1][k]) + (L.sum[2][k] + L.sum[3][k]);
}

// g_p = gscale * sum over nparts rows of gsrc (row stride `stride`), in a
// fixed order; optional gradient output, loss (column 1249, only when
// loss_acc is given: added to it, or stored) and Adam update (Kingma & Ba,
// Alg. 1, with c1 = 1 - b1^t, c2 = 1 - b2^t).  A workgroup takes 64 columns
// with 16 threads each, thread group q the rows q, q + 16, ..., eight in
// flight: a thread per column waited for 128 rows four at a time, 12 us
// against 4.0 us.
struct UpdateArgs {
    const float *gsrc;
    int nparts;
    long long stride;
    double gscale, lscale;
    float *gout;
    double *loss_acc;
    int loss_add;
    float *w, *m, *v;
    double lr, b1, b2, eps, c1, c2;
    int adam;
};

constexpr int kUCols = 64, kURows = 16;

__global__ __launch_bounds__(kUCols * kURows) void k_guess_update(UpdateArgs a)
{
    __shared__ double red[kURows][kUCols];
    const int c = threadIdx.x % kUCols, r = threadIdx.x / kUCols;
    const int p = blockIdx.x * kUCols + c;
    double s = 0.0;
    if (p <= kGuessParams && (p < kGuessParams || a.loss_acc)) {
        int q = r;
        for (; q + 7 * kURows < a.nparts; q += 8 * kURows) {
            float v[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = a.gsrc[(long long)(q + k * kURows) * a.stride + p];
#pragma unroll
            for (int k = 0; k < 8; ++k) s += (double)v[k];
        }
        for (; q < a.nparts; q += kURows) s += (double)a.gsrc[(long long)q * a.stride + p];
    }
    red[r][c] = s;
    __syncthreads();
    if (r != 0 || p > kGuessParams) return;
    for (int k = 1; k < kURows; ++k) s += red[k][c];
    if (p == kGuessParams) {
        if (a.loss_acc) *a.loss_acc = (a.loss_add ? *a.loss_acc : 0.0) + s * a.lscale;
        return;
    }
    const double g = s * a.gscale;
    if (a.gout) a.gout[p] = (float)g;
    if (a.adam) {
        const double mm = a.b1 * (double)a.m[p] + (1.0 - a.b1) * g;
        const double vv = a.b2 * (double)a.v[p] + (1.0 - a.b2) * g * g;
        a.m[p] = (float)mm;
        a.v[p] = (float)vv;
        const double mh = mm / a.c1, vh = vv / a.c2;
        a.w[p] = (float)((double)a.w[p] - a.lr * mh / (sqrt(vh) + a.eps));
    }
}

__global__ void k_zero_f64(double *p, int n)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < n) p[i] = 0.0;
}

State6 state6(const double *st, long long n)
{
    return State6{st, st + n, st + 2 * n, st + 3 * n, st + 4 * n, st + 5 * n};
}

unsigned grid_of(long long n, int bs) { return (unsigned)((n + bs - 1) / bs); }

}  // namespace

struct qsym_guess_trainer {
    hipStream_t stream = nullptr;
    long long max_batch = 0;
    int max_parts = 0;
    char *mem = nullptr;
    float *part = nullptr, *g = nullptr, *m = nullptr, *v = nullptr;
    double *loss = nullptr, *mom = nullptr, *curve = nullptr;
    unsigned long long *bad = nullptr;
    long long t = 0;
    std::string err;
};

namespace {

int tfail(qsym_guess_trainer *tr, int code, const std::string &msg)
{
    if (tr) tr->err = msg;
    return code;
}

#define TCHK(tr, call)                                                                        \
    do {                                                                                      \
        hipError_t e_ = (call);                                                               \
        if (e_ != hipSuccess)                                                                 \
            return tfail((tr), QSYM_EHIP, std::string(#call) + ": " + hipGetErrorString(e_)); \
    } while (0)

int launch_grad(qsym_guess_trainer *tr, const float *w, const float *feat, long long ld,
                long long n, int &nparts)
{
    nparts = (int)std::min<long long>((n + 63) / 64, tr->max_parts);
    hipLaunchKernelGGL(k_guess_grad, dim3(nparts), dim3(64 * kGWaves), 0, tr->stream, w, feat, ld, n,
                       tr->part);
    TCHK(tr, hipGetLastError());
    return QSYM_OK;
}

int launch_update(qsym_guess_trainer *tr, const UpdateArgs &a)
{
    hipLaunchKernelGGL(k_guess_update, dim3(grid_of(kGuessParams + 1, kUCols)), dim3(kUCols * kURows), 0,
                       tr->stream, a);
    TCHK(tr, hipGetLastError());
    return QSYM_OK;
}

bool bad_state_args(long long n, const void *st, const void *dt) { return n < 0 || (n > 0 && (!st || !dt)); }

}  // namespace

// ------------------------------------------------------------------------
// Scratch of the allocation-free loss gradient (qsym_guess_grad_static):
// the partial sums of up to kStaticParts workgroups (64 samples each)
// and the loss accumulator, in one file-scope device array.  Every device
// the library runs on holds its own copy until the process ends; host code
// reaches it only through the address hipGetSymbolAddress gives on that
// device (the array's name is a host-side stand-in).
// ------------------------------------------------------------------------
constexpr int kStaticParts = QSYM_GUESS_STATIC_MAX / 64;
constexpr size_t kStaticPartBytes = (size_t)kStaticParts * kGPart * sizeof(float);
constexpr size_t kStaticScratchBytes = kStaticPartBytes + 256;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

void qsym_noctx_error(const char *msg);

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices] = {};

// device address of this device's scratch, looked up once per device (with
// that device current) and kept
int static_scratch(void **out)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) {
        qsym_noctx_error("guess_grad_static: no current HIP device");
        return QSYM_EHIP;
    }
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) {
            qsym_noctx_error((std::string("guess_grad_static: hipGetSymbolAddress: ") +
                              hipGetErrorString(e)).c_str());
            return QSYM_EHIP;
        }
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return QSYM_OK;
}

}  // namespace

extern "C" {

int qsym_kepler_solve(double mu, int64_t n, const double *state, const double *dt, int32_t mode,
                      const float *weights, double *x_out, int32_t *iters, void *stream)
{
    if (!(mu > 0) || bad_state_args(n, state, dt) || mode < 0 || mode > 2 ||
        (mode == 2 && !weights) || (n > 0 && !x_out))
        return QSYM_EINVAL;
    if (n == 0) return QSYM_OK;
    hipLaunchKernelGGL(k_kepler_solve, dim3(grid_of(n, 256)), dim3(256), 0, (hipStream_t)stream, mu,
                       (long long)n, state6(state, n), dt, (int)mode, weights, x_out, (int *)iters);
    return hipGetLastError() == hipSuccess ? QSYM_OK : QSYM_EHIP;
}

int qsym_kepler_guess(double mu, int64_t n, const double *state, const double *dt,
                      const float *weights, double *x_out, void *stream)
{
    if (!(mu > 0) || bad_state_args(n, state, dt) || (n > 0 && (!weights || !x_out)))
        return QSYM_EINVAL;
    if (n == 0) return QSYM_OK;
    hipLaunchKernelGGL(k_kepler_guess, dim3(grid_of(n, 256)), dim3(256), 0, (hipStream_t)stream, mu,
                       (long long)n, state6(state, n), dt, weights, x_out);
    return hipGetLastError() == hipSuccess ? QSYM_OK : QSYM_EHIP;
}

int qsym_guess_trainer_create(int64_t max_batch, void *stream, qsym_guess_trainer **out)
{
    if (!out || max_batch < 1) return QSYM_EINVAL;
    *out = nullptr;
    auto *tr = new qsym_guess_trainer();
    tr->stream = (hipStream_t)stream;
    tr->max_batch = max_batch;
    tr->max_parts = (int)std::min<long long>((max_batch + 63) / 64, kGMaxParts);
    const size_t b_part = (size_t)tr->max_parts * kGPart * sizeof(float);
    const size_t b_vec = 1280 * sizeof(float);
    const size_t b_mom = (size_t)kGMomBlocks * 10 * sizeof(double);
    const size_t b_curve = kGMaxEpochs * sizeof(double);
    const size_t total = b_part + 3 * b_vec + 256 + b_mom + b_curve + 256;
    if (hipMalloc((void **)&tr->mem, total) != hipSuccess) {
        delete tr;
        return QSYM_ENOMEM;
    }
    char *p = tr->mem;
    tr->part = (float *)p; p += b_part;
    tr->g = (float *)p; p += b_vec;
    tr->m = (float *)p; p += b_vec;
    tr->v = (float *)p; p += b_vec;
    tr->loss = (double *)p; p += 256;
    tr->mom = (double *)p; p += b_mom;
    tr->curve = (double *)p; p += b_curve;
    tr->bad = (unsigned long long *)p;
    if (hipMemsetAsync(tr->mem, 0, total, tr->stream) != hipSuccess ||
        hipStreamSynchronize(tr->stream) != hipSuccess) {
        hipFree(tr->mem);
        delete tr;
        return QSYM_EHIP;
    }
    *out = tr;
    return QSYM_OK;
}

void qsym_guess_trainer_destroy(qsym_guess_trainer *tr)
{
    if (!tr) return;
    hipStreamSynchronize(tr->stream);
    hipFree(tr->mem);
    delete tr;
}

const char *qsym_guess_trainer_error(const qsym_guess_trainer *tr) { return tr ? tr->err.c_str() : ""; }

int qsym_guess_reset(qsym_guess_trainer *tr)
{
    if (!tr) return QSYM_EINVAL;
    TCHK(tr, hipMemsetAsync(tr->m, 0, 2 * 1280 * sizeof(float), tr->stream));
    tr->t = 0;
    return QSYM_OK;
}

int qsym_guess_prepare(qsym_guess_trainer *tr, double mu, int64_t n, const double *state,
                       const double *dt, const double *x_root, float *feat, int64_t ld)
{
    if (!tr) return QSYM_EINVAL;
    if (!(mu > 0) || bad_state_args(n, state, dt) || (n > 0 && !feat) || ld < n)
        return tfail(tr, QSYM_EINVAL, "guess_prepare: bad arguments (mu > 0, ld >= n)");
    if (n == 0) return QSYM_OK;
    TCHK(tr, hipMemsetAsync(tr->bad, 0, sizeof(unsigned long long), tr->stream));
    hipLaunchKernelGGL(k_guess_prepare, dim3(grid_of(n, 256)), dim3(256), 0, tr->stream, mu,
                       (long long)n, state6(state, n), dt, x_root, feat, (long long)ld, tr->bad);
    TCHK(tr, hipGetLastError());
    unsigned long long bad = 0;
    TCHK(tr, hipMemcpyAsync(&bad, tr->bad, sizeof bad, hipMemcpyDeviceToHost, tr->stream));
    TCHK(tr, hipStreamSynchronize(tr->stream));
    if (bad)
        return tfail(tr, QSYM_EINVAL,
                     std::to_string(bad) + " samples unusable (zero step or non-finite feature/target)");
    return QSYM_OK;
}

int qsym_guess_fit_scalers(qsym_guess_trainer *tr, const float *feat, int64_t ld, int64_t n,
                           float *weights)
{
    if (!tr) return QSYM_EINVAL;
    if (n < 1 || ld < n || !feat || !weights)
        return tfail(tr, QSYM_EINVAL, "guess_fit_scalers: need n >= 1, ld >= n");
    const int nb = (int)std::min<long long>((n + 255) / 256, kGMomBlocks);
    hipLaunchKernelGGL(k_guess_moments, dim3(nb), dim3(256), 0, tr->stream, (long long)n, feat,
                       (long long)ld, tr->mom);
    TCHK(tr, hipGetLastError());
    hipLaunchKernelGGL(k_guess_scalers, dim3(1), dim3(64), 0, tr->stream, tr->mom, nb,
                       (long long)n, weights);
    TCHK(tr, hipGetLastError());
    return QSYM_OK;
}

int qsym_guess_grad(qsym_guess_trainer *tr, const float *weights, const float *feat, int64_t ld,
                    int64_t n, float *grad, double *loss)
{
    if (!tr) return QSYM_EINVAL;
    if (n < 1 || n > tr->max_batch || ld < n || !weights || !feat || !grad)
        return tfail(tr, QSYM_EINVAL, "guess_grad: need 1 <= n <= max_batch, ld >= n");
    int nparts;
    if (int rc = launch_grad(tr, weights, feat, ld, n, nparts)) return rc;
    UpdateArgs a{};
    a.gsrc = tr->part;
    a.nparts = nparts;
    a.stride = kGPart;
    a.gscale = 2.0 / (double)n;
    a.lscale = 1.0 / (double)n;
    a.gout = grad;
    a.loss_acc = tr->loss;
    if (int rc = launch_update(tr, a)) return rc;
    if (loss) {
        TCHK(tr, hipMemcpyAsync(loss, tr->loss, sizeof(double), hipMemcpyDeviceToHost, tr->stream));
        TCHK(tr, hipStreamSynchronize(tr->stream));
    }
    return QSYM_OK;
}

int qsym_guess_grad_static(const float *weights, const float *feat, int64_t ld, int64_t n,
                           float *grad, double *loss, void *stream)
{
    if (n < 1 || n > QSYM_GUESS_STATIC_MAX || ld < n || !weights || !feat || !grad) {
        qsym_noctx_error("guess_grad_static: need 1 <= n <= QSYM_GUESS_STATIC_MAX (16384), "
                         "ld >= n and non-null weights, feat, grad");
        return QSYM_EINVAL;
    }
    void *base = nullptr;
    if (int rc = static_scratch(&base)) return rc;
    float *part = (float *)base;
    double *lacc = (double *)((char *)base + kStaticPartBytes);
    hipStream_t st = (hipStream_t)stream;
    // the same launches as qsym_guess_grad: one workgroup per 64 samples (every
    // partial row is written whole); the update stores the loss
    const int nparts = (int)((n + 63) / 64);
    hipLaunchKernelGGL(k_guess_grad, dim3(nparts), dim3(64 * kGWaves), 0, st, weights, feat,
                       (long long)ld, (long long)n, part);
    if (hipGetLastError() != hipSuccess) return QSYM_EHIP;
    UpdateArgs a{};
    a.gsrc = part;
    a.nparts = nparts;
    a.stride = kGPart;
    a.gscale = 2.0 / (double)n;
    a.lscale = 1.0 / (double)n;
    a.gout = grad;
    a.loss_acc = lacc;
    hipLaunchKernelGGL(k_guess_update, dim3(grid_of(kGuessParams + 1, kUCols)), dim3(kUCols * kURows),
                       0, st, a);
    if (hipGetLastError() != hipSuccess) return QSYM_EHIP;
    if (loss) {
        if (hipMemcpyAsync(loss, lacc, sizeof(double), hipMemcpyDeviceToHost, st) != hipSuccess ||
            hipStreamSynchronize(st) != hipSuccess)
            return QSYM_EHIP;
    }
    return QSYM_OK;
}

int qsym_guess_adam(qsym_guess_trainer *tr, float *weights, const float *grad, double lr,
                    double b1, double b2, double eps)
{
    if (!tr) return QSYM_EINVAL;
    if (!weights || !grad || !(lr >= 0) || !(b1 >= 0 && b1 < 1) || !(b2 >= 0 && b2 < 1) || !(eps >= 0))
        return tfail(tr, QSYM_EINVAL, "guess_adam: bad arguments");
    tr->t += 1;
    UpdateArgs a{};
    a.gsrc = grad;
    a.nparts = 1;
    a.stride = 0;
    a.gscale = 1.0;
    a.w = weights;
    a.m = tr->m;
    a.v = tr->v;
    a.lr = lr;
    a.b1 = b1;
    a.b2 = b2;
    a.eps = eps;
    a.c1 = 1.0 - std::pow(b1, (double)tr->t);
    a.c2 = 1.0 - std::pow(b2, (double)tr->t);
    a.adam = 1;
    return launch_update(tr, a);
}

int qsym_guess_train(qsym_guess_trainer *tr, float *weights, const float *feat, int64_t ld,
                     int64_t n, int64_t batch, int32_t epochs, double lr, double lr_final,
                     double *curve)
{
    if (!tr) return QSYM_EINVAL;
    if (!weights || !feat || n < 1 || ld < n || batch < 1 || batch > tr->max_batch || epochs < 1 ||
        epochs > kGMaxEpochs || !(lr > 0) || !(lr_final >= 0))
        return tfail(tr, QSYM_EINVAL,
                     "guess_train: need n >= 1, ld >= n, 1 <= batch <= max_batch, 1 <= epochs <= 4096, lr > 0");
    hipLaunchKernelGGL(k_zero_f64, dim3(grid_of(epochs, 256)), dim3(256), 0, tr->stream, tr->curve,
                       (int)epochs);
    TCHK(tr, hipGetLastError());
    const double b1 = 0.9, b2 = 0.999, eps = 1e-8;
    for (int e = 0; e < epochs; ++e) {
        // cosine decay from lr to lr_final over the epochs
        const double lre = lr_final + (lr - lr_final) * 0.5 * (1.0 + std::cos(kPi * e / epochs));
        for (long long b0 = 0; b0 < n; b0 += batch) {
            const long long nb = std::min<long long>(batch, n - b0);
            int nparts;
            if (int rc = launch_grad(tr, weights, feat + b0, ld, nb, nparts)) return rc;
            tr->t += 1;
            UpdateArgs a{};
            a.gsrc = tr->part;
            a.nparts = nparts;
            a.stride = kGPart;
            a.gscale = 2.0 / (double)nb;
            a.lscale = 1.0 / (double)n;
            a.loss_acc = tr->curve + e;
            a.loss_add = 1;
            a.w = weights;
            a.m = tr->m;
            a.v = tr->v;
            a.lr = lre;
            a.b1 = b1;
            a.b2 = b2;
            a.eps = eps;
            a.c1 = 1.0 - std::pow(b1, (double)tr->t);
            a.c2 = 1.0 - std::pow(b2, (double)tr->t);
            a.adam = 1;
            if (int rc = launch_update(tr, a)) return rc;
        }
    }
    if (curve)
        TCHK(tr, hipMemcpyAsync(curve, tr->curve, sizeof(double) * epochs, hipMemcpyDeviceToHost,
                                tr->stream));
    TCHK(tr, hipStreamSynchronize(tr->stream));
    return QSYM_OK;
}

}  // extern "C"
