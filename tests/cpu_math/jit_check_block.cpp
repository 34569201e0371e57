// Host check of the generated part of the block kernels (the adjoint, the adjoint
// at complex energies, the forward; AMI_JIT_KERNELS says which): one sample per
// block, a host thread per wave, driven through the kernels' steps on the LDS
// columns of lane 0 (column c at sm[64 c]) with a barrier for __syncthreads, so
// a test can compare values and gradients with the oracle.  The generated source
// is included through AMI_GENERATED without its two #include lines.
//
// stdin: "n_s n_f beta e_reg t mu", q (2 per external slot), the frequencies,
// then per sample its input (momenta, energies or complex energies) and, but for
// the forward, the cotangents.  stdout per sample: the values, and but for the
// forward the gradients by input, dL/dbeta, (real) dL/dmu, dL/dt, dL/dw.
#include <pthread.h>

#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <functional>
#include <thread>
#include <vector>

#include "../../paper_2311_17189_amd/csrc/device_common.hpp"

static pthread_barrier_t g_barrier;
static void block_barrier() { pthread_barrier_wait(&g_barrier); }
#define __syncthreads() block_barrier()

#include AMI_GENERATED

using namespace amijit;

constexpr int NXA = NX > 0 ? NX : 1, NIA = NI > 0 ? NI : 1, NGA = NG > 0 ? NG : 1;
constexpr bool kComplex = (AMI_JIT_KERNELS & 16384) != 0, kForward = (AMI_JIT_KERNELS & 32768) != 0;
constexpr int C = kComplex ? 2 : 1;                 // columns of a value

struct Sample {
    int n_f;
    double beta, e_reg, t, mu;
    const double *q;
    std::vector<double> w, in, cot;                 // n_f x NX complex, the input, n_f complex
    std::vector<double> sm, re, im, gw, grad;       // LDS; values, dL/dw and gradients
    double gbeta = 0.0;
};

static void frequency(const Sample &s, int f, double (&wr)[NXA], double (&wi)[NXA]) {
    for (int x = 0; x < NXA; ++x) {
        wr[x] = x < NX ? s.w[2 * (f * NX + x)] : 0.0;
        wi[x] = x < NX ? s.w[2 * (f * NX + x) + 1] : 0.0;
    }
}

static double total(const double *col, int first) {
    double v = 0.0;
    for (int w = 0; w < NW; ++w) v += col[64 * (first + w)];
    return v;
}

#if AMI_JIT_KERNELS & 32768
template <int WV>
static void wave(Sample &s) {
    double *col = s.sm.data(), E[NE], x[L];
    for (int i = 0; i < NE; ++i) E[i] = s.in[i];
    leaf_args(E, x);
    for (int l = WV; l < L; l += NW) {
        double f, fm;
        ami::leaf_pair(kBose[l], s.beta * (kBose[l] ? x[l] + s.e_reg : x[l]), f, fm);
        col[64 * (NE + l)] = f;
    }
    __syncthreads();
    blk_sums<WV>(col + 64 * NE, col + 64 * (NE + L));
    __syncthreads();
    for (int f = WV; f < s.n_f; f += NW) {
        double wr[NXA], wi[NXA], dr[D], di[D], xr[D], xi[D];
        frequency(s, f, wr, wi);
        den_args(E, wr, wi, dr, di);
        for (int k = 0; k < D; ++k) {
            const double inv = ami::rcp_nr(fma(dr[k], dr[k], di[k] * di[k]));
            xr[k] = dr[k] * inv;
            xi[k] = -di[k] * inv;
        }
        blk_row(col + 64 * (NE + L), xr, xi, s.re[f], s.im[f]);
    }
}
#else
template <int WV, bool ONE, typename Ft>
static void row(Sample &s, int f, Ft &ft, Ft &ftb, double (&gE)[C][NE]) {
    double *col = s.sm.data(), wr[NXA], wi[NXA], gwr[NXA] = {0.0}, gwi[NXA] = {0.0}, re = 0.0, im = 0.0;
    frequency(s, f, wr, wi);
    const double cr = s.cot[2 * f], ci = s.cot[2 * f + 1];
#if AMI_JIT_KERNELS & 16384
    blk_freq<WV, ONE>(col + 64 * kBE, wr, wi, col + 64 * kBT, ft[0], ft[1], cr, ci, ftb[0], ftb[1], re, im, gE[0], gE[1],
                      gwr, gwi);
#else
    blk_freq<WV, ONE>(col + 64 * kBE, wr, wi, col + 64 * kBT, ft[0], cr, ci, ftb[0], re, im, gE[0], gwr, gwi);
#endif
    if (f > 0) __syncthreads();
    col[64 * (kBA + WV)] = re;
    col[64 * (kBA + NW + WV)] = im;
    for (int x = 0; x < NX; ++x) {
        col[64 * (kBA + (2 + 2 * x) * NW + WV)] = gwr[x];
        col[64 * (kBA + (3 + 2 * x) * NW + WV)] = gwi[x];
    }
    __syncthreads();
    if (WV == f % NW) {
        s.re[f] = total(col, kBA);
        s.im[f] = total(col, kBA + NW);
        for (int x = 0; x < NX; ++x) {
            s.gw[2 * (f * NX + x)] = total(col, kBA + (2 + 2 * x) * NW);
            s.gw[2 * (f * NX + x) + 1] = -total(col, kBA + (3 + 2 * x) * NW);
        }
    }
}

template <int WV>
static void wave(Sample &s) {
    double *col = s.sm.data();
    double E[C][NE], x[C][L], gE[C][NE] = {}, ft[C][GW] = {}, ftb[C][GW] = {}, FB[C][L] = {}, gbeta = 0.0;
    for (int c = 0; c < C; ++c) {
        for (int i = 0; i < NE; ++i) {
            E[c][i] = s.in[C * i + c];
            if (i % NW == WV) col[64 * (kBE + c * NE + i)] = E[c][i];
        }
        leaf_args(E[c], x[c]);
    }
    for (int l = WV; l < L; l += NW) {
        double v[2 * C];                            // the leaf, its slope
        const double xr = kBose[l] ? x[0][l] + s.e_reg : x[0][l];
#if AMI_JIT_KERNELS & 16384
        blk_cleaf(kBose[l], s.beta * xr, s.beta * x[1][l], v[0], v[1], v[2], v[3]);
#else
        ami::leaf_and_slope(kBose[l], s.beta * xr, v[0], v[1]);
#endif
        for (int c = 0; c < C; ++c) {
            col[64 * (kBF + C * l + c)] = v[c];
            if (kBS >= 0) col[64 * (kBS + C * l + c)] = v[C + c];
        }
    }
    __syncthreads();
#if AMI_JIT_KERNELS & 16384
    blk_sums<WV>(col + 64 * kBF, col + 64 * kBT, ft[0], ft[1]);
#else
    blk_sums<WV>(col + 64 * kBF, col + 64 * kBT, ft[0]);
    if (kValueWave >= 0) __syncthreads();
#endif
    if (s.n_f == 1) {
        row<WV, true>(s, 0, ft, ftb, gE);
    } else {
        for (int f = 0; f < s.n_f; ++f) row<WV, false>(s, f, ft, ftb, gE);
#if AMI_JIT_KERNELS & 16384
        blk_keep<WV>(col + 64 * kBT, ftb[0], ftb[1]);
#else
        blk_keep<WV>(col + 64 * kBT, ftb[0]);
#endif
    }
#if AMI_JIT_KERNELS & 16384
    blk_leaf<WV>(col + 64 * kBF, col + 64 * kBT, ftb[0], ftb[1], FB[0], FB[1]);
    blk_rounds<WV>(FB[0], FB[1], s.beta, s.e_reg, col + 64 * kBE, col + 64 * kBU, col + 64 * kBS, gE[0], gE[1], gbeta);
#else
    blk_leaf<WV>(col + 64 * kBF, col + 64 * kBT, ftb[0], FB[0]);
    blk_rounds<WV>(FB[0], s.beta, s.e_reg, col + 64 * kBE, col + 64 * kBU, col + 64 * kBS, gE[0], gbeta);
#endif
    __syncthreads();
    for (int i = 0; i < NE; ++i)
        for (int c = 0; c < C; ++c) col[64 * (kBU + (C * i + c) * NW + WV)] = gE[c][i];
    col[64 * (kBU + C * NE * NW + WV)] = gbeta;
    __syncthreads();
    if (WV > 0) return;
    for (int i = 0; i < C * NE; ++i) s.grad[i] = total(col, kBU + i * NW);
    s.gbeta = total(col, kBU + C * NE * NW);
}
#endif

template <int WV>
static void start(std::vector<std::thread> &pool, Sample &s) {
    if constexpr (WV < NW) {
        pool.emplace_back(wave<WV>, std::ref(s));
        start<WV + 1>(pool, s);
    }
}

int main() {
    int n_s;
    Sample s;
    if (std::scanf("%d %d %lf %lf %lf %lf", &n_s, &s.n_f, &s.beta, &s.e_reg, &s.t, &s.mu) != 6) return 2;
    auto read = [](std::vector<double> &v, size_t n) {
        v.assign(n, 0.0);
        for (double &x : v)
            if (std::scanf("%lf", &x) != 1) std::exit(2);
    };
    std::vector<double> q, k;
    read(q, 2 * NX);
    read(s.w, 2 * static_cast<size_t>(s.n_f) * NX);
    pthread_barrier_init(&g_barrier, nullptr, NW);
    for (int n = 0; n < n_s; ++n) {
        double Kx[NGA] = {0.0}, Ky[NGA] = {0.0};
        if (AMI_JIT_HUB) {
            read(k, 2 * NI);
            double kx[NIA], ky[NIA];
            for (int l = 0; l < NI; ++l) {
                kx[l] = ami::reduce_2pi(k[2 * l]);
                ky[l] = ami::reduce_2pi(k[2 * l + 1]);
            }
            lines(kx, ky, q.data(), Kx, Ky);
            s.in.assign(NE, 0.0);
            for (int j = 0; j < NG; ++j) s.in[j] = fma(2.0 * s.t, ami::cos_red(Kx[j]) + ami::cos_red(Ky[j]), s.mu);
        } else {
            read(s.in, static_cast<size_t>(C) * NE);
        }
        if (!kForward) read(s.cot, 2 * static_cast<size_t>(s.n_f));
        s.sm.assign(64 * static_cast<size_t>(kBlockCols), std::nan(""));    // what was not written must not be read
        s.re.assign(s.n_f, 0.0);
        s.im.assign(s.n_f, 0.0);
        s.gw.assign(2 * static_cast<size_t>(s.n_f) * NX, 0.0);
        s.grad.assign(static_cast<size_t>(C) * NE, 0.0);
        std::vector<std::thread> pool;
        start<0>(pool, s);
        for (std::thread &th : pool) th.join();
        for (int f = 0; f < s.n_f; ++f) std::printf("%.17g %.17g ", s.re[f], s.im[f]);
#if AMI_JIT_KERNELS & 8192
        double gmu = 0.0, gt = 0.0;
        if (AMI_JIT_HUB) {
            double gx[NGA], gy[NGA], gkx[NIA] = {0.0}, gky[NIA] = {0.0};
            for (int j = 0; j < NG; ++j) {
                double sx, cx, sy, cy;
                ami::sincos_red(Kx[j], sx, cx);
                ami::sincos_red(Ky[j], sy, cy);
                gmu += s.grad[j];
                gt = fma(s.grad[j], 2.0 * (cx + cy), gt);
                gx[j] = -2.0 * s.t * s.grad[j] * sx;
                gy[j] = -2.0 * s.t * s.grad[j] * sy;
            }
            line_scatter(gx, gy, gkx, gky);
            for (int l = 0; l < NI; ++l) std::printf("%.17g %.17g ", gkx[l], gky[l]);
        } else {
            for (double g : s.grad) std::printf("%.17g ", g);
        }
        std::printf("%.17g %.17g %.17g ", s.gbeta, gmu, gt);
#elif AMI_JIT_KERNELS & 16384
        for (double g : s.grad) std::printf("%.17g ", g);
        std::printf("%.17g ", s.gbeta);
#endif
        if (!kForward)
            for (double g : s.gw) std::printf("%.17g ", g);
        std::printf("\n");
    }
    return 0;
}
