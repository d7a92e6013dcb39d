// Learned Davidson preconditioner: a two-layer perceptron applied to every
// element of the site tensor, its training pairs and its training.
//
// The paper leaves the local solver of Sec. 2.3 open; the library's solver
// is Davidson with the diagonal correction t = -r / (dh - theta dn).  The
// learned variant maps five features of each element,
//   f0 = |r_i| / rms(r), f1 = asinh(d_i), f2 = asinh(dn_i), f3 = asinh(-f0 / d_i'),
//   f4 = sign(r_i) t_i / rms(t)   (t = -r / d', the diagonal correction)
// (d = dh - theta dn, d' = d floored to |d'| >= floor) to
// t_i = sign(r_i) (w2 . relu(W1 f + b1) + b2): odd in r like a linear
// preconditioner, so the free sign of the Ritz vector does not matter.
// Davidson normalises t, so the scale is free.  Training targets are the
// solver's own exact corrections e_j = x*/(x_j . x*) - x_j (x_j the unit Ritz
// vector of iteration j, x* the converged one) divided by rms(e_j), times
// sign(r_i).
// Per-N-block scope: the root mean squares in f0 and f4 and in the targets
// are taken over the element's N-block of the site tensor (elements sharing
// both bond particle numbers), and the correction is scaled by the block's
// rms of the diagonal correction, so the model shapes the correction inside
// a block and the diagonal rule keeps the block's weight.
// Weights and recorded pairs are FP32 in memory; all arithmetic is FP64.
// Packed weights: W1 (H x 5, row-major) | b1 (H) | w2 (H) | b2.

#include <hip/hip_runtime.h>

#include <algorithm>

#include "kernels.h"
#include "mlp.h"

namespace spk {

namespace {

constexpr int kMlpThreads = 256;

__device__ inline double wsum(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// fixed-order sum over a work-group of blockDim.x (a multiple of 64) threads
__device__ inline double group_sum(double v, double* red) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    v = wsum(v);
    __syncthreads();
    if (lane == 0) red[wave] = v;
    __syncthreads();
    double r = 0.0;
    for (int w = 0; w < nw; ++w) r += red[w];
    return r;
}

__device__ inline double mlp_eval(const double* sw, int H, const double f[kMlpIn]) {
    const double* W1 = sw;
    const double* b1 = sw + H * kMlpIn;
    const double* w2 = b1 + H;
    double y = w2[H];  // b2
    for (int j = 0; j < H; ++j) {
        double z = b1[j];
#pragma unroll
        for (int c = 0; c < kMlpIn; ++c) z = fma(W1[j * kMlpIn + c], f[c], z);
        y = fma(w2[j], fmax(z, 0.0), y);
    }
    return y;
}

__device__ inline void load_weights(const float* __restrict__ w, int H, double* sw) {
    const int P = int(mlp_size(H));
    for (int p = threadIdx.x; p < P; p += blockDim.x) sw[p] = double(w[p]);
    __syncthreads();
}

__global__ __launch_bounds__(kMlpThreads) void k_sum_partials(const double* __restrict__ part, int nchunk, int stride,
                                                              int idx, double* __restrict__ out) {
    __shared__ double red[kMlpThreads / 64];
    double s = 0.0;
    for (int q = threadIdx.x; q < nchunk; q += kMlpThreads) s += part[(long long)q * stride + idx];
    s = group_sum(s, red);
    if (threadIdx.x == 0) *out = s;
}

// features of every element from the diagonal correction t = -r / d' (so
// r = -t d'), optionally recorded with sign(r_i) (feat, sgn), then optionally
// the model's correction in place of t
__global__ __launch_bounds__(kMlpThreads) void k_mlp_apply(const float* __restrict__ w, int H, double* __restrict__ t,
                                                           const double* __restrict__ dh,
                                                           const double* __restrict__ dn,
                                                           const double* __restrict__ theta,
                                                           const double* __restrict__ rr,
                                                           const double* __restrict__ tt, int n, double floor_,
                                                           float* __restrict__ feat, float* __restrict__ sgn,
                                                           const int* __restrict__ gid,
                                                           const double* __restrict__ grms) {
    extern __shared__ double sw[];
    if (w) load_weights(w, H, sw);
    const int i = blockIdx.x * kMlpThreads + threadIdx.x;
    if (i >= n) return;
    const double th = *theta;
    double rms, rmst;
    if (gid) {
        const int q = gid[i];
        rms = grms[2 * q];
        rmst = grms[2 * q + 1];
    } else {
        rms = sqrt(*rr / n);
        rmst = sqrt(*tt / n);
    }
    const double d = dh[i] - th * dn[i];
    const double dfl = fabs(d) < floor_ ? (d < 0.0 ? -floor_ : floor_) : d;
    const double r = -t[i] * dfl;
    const double sr = r > 0.0 ? 1.0 : (r < 0.0 ? -1.0 : 0.0);
    const double f0 = rms > 0.0 ? fabs(r) / rms : 0.0;
    double f[kMlpIn] = {f0, asinh(d), asinh(dn[i]), asinh(-f0 / dfl), rmst > 0.0 ? sr * t[i] / rmst : 0.0};
    if (feat) {
#pragma unroll
        for (int c = 0; c < kMlpIn; ++c) feat[(long long)i * kMlpIn + c] = float(f[c]);
        sgn[i] = float(sr);
    }
    if (w) t[i] = sr * mlp_eval(sw, H, f) * (gid ? rmst : 1.0);
}

// one work-group per group of element ranges: rms of r = -t d' and of t
__global__ __launch_bounds__(kMlpThreads) void k_mlp_group_rms(const double* __restrict__ t,
                                                               const double* __restrict__ dh,
                                                               const double* __restrict__ dn,
                                                               const double* __restrict__ theta, double floor_,
                                                               ElemGroups g, double* __restrict__ grms) {
    __shared__ double red[kMlpThreads / 64];
    const int q = blockIdx.x;
    const double th = *theta;
    double rr = 0.0, tt = 0.0;
    long long cnt = 0;
    for (int j = g.gptr[q]; j < g.gptr[q + 1]; ++j) {
        const long long o = g.roff[j];
        cnt += g.rlen[j];
        for (int e = threadIdx.x; e < g.rlen[j]; e += kMlpThreads) {
            const long long i = o + e;
            const double d = dh[i] - th * dn[i];
            const double dfl = fabs(d) < floor_ ? (d < 0.0 ? -floor_ : floor_) : d;
            const double r = -t[i] * dfl;
            rr = fma(r, r, rr);
            tt = fma(t[i], t[i], tt);
        }
    }
    rr = group_sum(rr, red);
    tt = group_sum(tt, red);
    if (threadIdx.x == 0) {
        grms[2 * q] = cnt > 0 ? sqrt(rr / double(cnt)) : 0.0;
        grms[2 * q + 1] = cnt > 0 ? sqrt(tt / double(cnt)) : 0.0;
    }
}

__global__ __launch_bounds__(1024) void k_sumsq(const double* __restrict__ v, int n, double* __restrict__ out) {
    __shared__ double red[16];
    double s = 0.0;
    for (int i = threadIdx.x; i < n; i += 1024) s = fma(v[i], v[i], s);
    s = group_sum(s, red);
    if (threadIdx.x == 0) *out = s;
}

// A tile of up to kTileRows rows (features in LDS as f(row, c) at
// row * kRow + c, rows past ns zero): the model's outputs without b2 in eight
// parts, one per wavefront.  Wavefront v takes hidden units [v H / 8, ..), a
// lane the rows lane + 64 i, so a weight read from LDS serves four rows (with
// one row per thread the reads, 16 values per clock and CU, take four times
// as long as the FMAs).
constexpr int kTileThreads = 512, kTileRows = 256, kTileWaves = kTileThreads / 64;
constexpr int kRow = 6, kUnit = 8;  // doubles per row (features, target) and per hidden unit (W1, b1, w2)

__device__ inline void load_units(const float* __restrict__ w, int H, double* su) {
    for (int p = threadIdx.x; p < H * (kMlpIn + 2); p += kTileThreads) {
        const int j = p < H * kMlpIn ? p / kMlpIn : (p - H * kMlpIn) % H;
        const int c = p < H * kMlpIn ? p % kMlpIn : kMlpIn + (p - H * kMlpIn) / H;
        su[j * kUnit + c] = double(w[p]);
    }
}

__device__ inline void tile_outputs(const double* __restrict__ su, int H, const double* __restrict__ sf, int ns,
                                    double (*__restrict__ part)[kTileRows]) {
    const int lane = threadIdx.x % 64, wave = threadIdx.x / 64, ng = (ns + 63) / 64;
    const int j0 = wave * H / kTileWaves, j1 = (wave + 1) * H / kTileWaves;
    double f[4][kMlpIn], y[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int c = 0; c < kMlpIn; ++c) f[i][c] = sf[(lane + 64 * i) * kRow + c];
    auto unit = [&](int j, int i) {
        const double* u = su + j * kUnit;
        double z = u[kMlpIn];
#pragma unroll
        for (int c = 0; c < kMlpIn; ++c) z = fma(u[c], f[i][c], z);
        y[i] = fma(u[kMlpIn + 1], fmax(z, 0.0), y[i]);
    };
    if (ng > 2) {
#pragma unroll 2
        for (int j = j0; j < j1; ++j)
#pragma unroll
            for (int i = 0; i < 4; ++i) unit(j, i);
    } else {
#pragma unroll 2
        for (int j = j0; j < j1; ++j)
#pragma unroll
            for (int i = 0; i < 2; ++i) unit(j, i);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) part[wave][lane + 64 * i] = y[i];
}

__global__ __launch_bounds__(kTileThreads) void k_mlp_forward(const float* __restrict__ w, int H,
                                                              const float* __restrict__ F, long long n, int rows,
                                                              float* __restrict__ y) {
    __shared__ double su[kMlpMaxHidden * kUnit], sf[kTileRows * kRow], part[kTileWaves][kTileRows];
    const long long q0 = (long long)blockIdx.x * rows;
    const int ns = int(min((long long)rows, n - q0));
    load_units(w, H, su);
    for (int e = threadIdx.x; e < kTileRows * kMlpIn; e += kTileThreads)
        sf[e / kMlpIn * kRow + e % kMlpIn] = e < ns * kMlpIn ? double(F[q0 * kMlpIn + e]) : 0.0;
    __syncthreads();
    tile_outputs(su, H, sf, ns, part);
    __syncthreads();
    const int r = threadIdx.x;
    if (r < ns) {
        double v = double(w[H * (kMlpIn + 2)]);
#pragma unroll
        for (int q = 0; q < kTileWaves; ++q) v += part[q][r];
        y[q0 + r] = float(v);
    }
}

// one work-group per recorded iteration j: Y_j = sign(r_j) e_j / rms(e_j),
// e_j = x*/(xh . x*) - xh, xh = x_j / |x_j|; Y_j holds sign(r_j) on entry
__global__ __launch_bounds__(1024) void k_mlp_targets(const double* __restrict__ X, long long ldx,
                                                      const double* __restrict__ xs, int n, float* __restrict__ Y) {
    __shared__ double red[16];
    const double* x = X + (long long)blockIdx.x * ldx;
    float* out = Y + (long long)blockIdx.x * n;
    double xx = 0.0, xy = 0.0;
    for (int i = threadIdx.x; i < n; i += 1024) {
        xx = fma(x[i], x[i], xx);
        xy = fma(x[i], xs[i], xy);
    }
    xx = group_sum(xx, red);
    xy = group_sum(xy, red);
    const double nx = sqrt(xx);
    const double c = xy / nx;  // xh . x*
    double ee = 0.0;
    for (int i = threadIdx.x; i < n; i += 1024) {
        const double e = xs[i] / c - x[i] / nx;
        ee = fma(e, e, ee);
    }
    ee = group_sum(ee, red);
    const double rms = sqrt(ee / n);
    const double inv = rms > 0.0 ? 1.0 / rms : 0.0;
    for (int i = threadIdx.x; i < n; i += 1024) out[i] = float(double(out[i]) * (xs[i] / c - x[i] / nx) * inv);
}

// grouped targets, first pass: one work-group per recorded iteration j,
// scal[2j] = |x_j|, scal[2j+1] = xh . x*
__global__ __launch_bounds__(1024) void k_mlp_target_dots(const double* __restrict__ X, long long ldx,
                                                          const double* __restrict__ xs, int n,
                                                          double* __restrict__ scal) {
    __shared__ double red[16];
    const double* x = X + (long long)blockIdx.x * ldx;
    double xx = 0.0, xy = 0.0;
    for (int i = threadIdx.x; i < n; i += 1024) {
        xx = fma(x[i], x[i], xx);
        xy = fma(x[i], xs[i], xy);
    }
    xx = group_sum(xx, red);
    xy = group_sum(xy, red);
    if (threadIdx.x == 0) {
        const double nx = sqrt(xx);
        scal[2 * blockIdx.x] = nx;
        scal[2 * blockIdx.x + 1] = xy / nx;
    }
}

// grouped targets, second pass: work-group (group q, iteration j) divides
// e_j on the group's ranges by its rms there; Y holds sign(r) on entry
__global__ __launch_bounds__(kMlpThreads) void k_mlp_targets_grouped(const double* __restrict__ X, long long ldx,
                                                                     const double* __restrict__ xs, int n,
                                                                     ElemGroups g, const double* __restrict__ scal,
                                                                     float* __restrict__ Y) {
    __shared__ double red[kMlpThreads / 64];
    const int q = blockIdx.x, j = blockIdx.y;
    const double* x = X + (long long)j * ldx;
    float* out = Y + (long long)j * n;
    const double nx = scal[2 * j], c = scal[2 * j + 1];
    double ee = 0.0;
    long long cnt = 0;
    for (int k = g.gptr[q]; k < g.gptr[q + 1]; ++k) {
        const long long o = g.roff[k];
        cnt += g.rlen[k];
        for (int e = threadIdx.x; e < g.rlen[k]; e += kMlpThreads) {
            const double v = xs[o + e] / c - x[o + e] / nx;
            ee = fma(v, v, ee);
        }
    }
    ee = group_sum(ee, red);
    const double rms = cnt > 0 ? sqrt(ee / double(cnt)) : 0.0;
    const double inv = rms > 0.0 ? 1.0 / rms : 0.0;
    for (int k = g.gptr[q]; k < g.gptr[q + 1]; ++k) {
        const long long o = g.roff[k];
        for (int e = threadIdx.x; e < g.rlen[k]; e += kMlpThreads) {
            const long long i = o + e;
            out[i] = float(double(out[i]) * (xs[i] / c - x[i] / nx) * inv);
        }
    }
}

// gradient partials of 0.5 * sum (y - Y)^2 over rows row0 + q * stride, q in
// this work-group's share of [0, count), a tile of kTileRows at a time: the
// outputs as above, then thread (column, split) owns hidden units column and
// column + ncol for every nsplit-th row, so that a row read from LDS serves
// two units; the splits' sums are added in order at the end.  FP64 FMAs bound
// it (7 us for 60001 rows of 256 units); four rows per work-group-wide
// reduction took 585 us, this form 26.
__global__ __launch_bounds__(kTileThreads) void k_mlp_grad(const float* __restrict__ w, int H,
                                                           const float* __restrict__ F, const float* __restrict__ Y,
                                                           long long row0, long long stride, long long count,
                                                           double* __restrict__ gpart) {
    constexpr int NG = kMlpIn + 2;  // gradients per unit: W1, b1, w2
    __shared__ double su[kMlpMaxHidden * kUnit], sf[kTileRows * kRow], red[kTileThreads / 64];
    __shared__ double sums[NG][2 * kTileThreads];
    double(*part)[kTileRows] = reinterpret_cast<double(*)[kTileRows]>(&sums[0][0]);
    static_assert(kTileWaves * kTileRows <= NG * 2 * kTileThreads, "outputs fit the sums' LDS");
    load_units(w, H, su);
    const double b2 = w[H * (kMlpIn + 2)];
    const int ncol = 64 * ((H + 127) / 128), nsplit = kTileThreads / ncol;
    const int col = threadIdx.x % ncol, split = threadIdx.x / ncol;
    __syncthreads();
    double W[2][NG], g[2][NG];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int c = 0; c < NG; ++c) {
            const int j = col + u * ncol;
            W[u][c] = j < H ? su[j * kUnit + c] : 0.0;
            g[u][c] = 0.0;
        }
    double gb2 = 0.0, loss = 0.0;
    const long long per = (count + gridDim.x - 1) / gridDim.x;
    const long long q0 = (long long)blockIdx.x * per, q1 = min(count, q0 + per);
    for (long long q = q0; q < q1; q += kTileRows) {
        const int ns = int(min((long long)kTileRows, q1 - q));
        for (int e = threadIdx.x; e < kTileRows * kRow; e += kTileThreads) {
            const int r = e / kRow, c = e % kRow;
            const long long row = row0 + (q + r) * stride;
            sf[e] = r < ns ? double(c < kMlpIn ? F[row * kMlpIn + c] : Y[row]) : 0.0;
        }
        __syncthreads();
        tile_outputs(su, H, sf, ns, part);
        __syncthreads();
        if (threadIdx.x < unsigned(ns)) {
            double y = b2;
#pragma unroll
            for (int v = 0; v < kTileWaves; ++v) y += part[v][threadIdx.x];
            const double dy = y - sf[threadIdx.x * kRow + kMlpIn];
            sf[threadIdx.x * kRow + kMlpIn] = dy;
            gb2 += dy;
            loss = fma(dy, dy, loss);
        }
        __syncthreads();
        for (int r = split; r < ns; r += nsplit) {
            double f[kRow];
#pragma unroll
            for (int c = 0; c < kRow; ++c) f[c] = sf[r * kRow + c];
            const double dy = f[kMlpIn];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                double z = W[u][kMlpIn];
#pragma unroll
                for (int c = 0; c < kMlpIn; ++c) z = fma(W[u][c], f[c], z);
                g[u][kMlpIn + 1] = fma(dy, fmax(z, 0.0), g[u][kMlpIn + 1]);
                if (z > 0.0) {
                    const double dz = dy * W[u][kMlpIn + 1];
                    g[u][kMlpIn] += dz;
#pragma unroll
                    for (int c = 0; c < kMlpIn; ++c) g[u][c] = fma(dz, f[c], g[u][c]);
                }
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int c = 0; c < NG; ++c) sums[c][u * kTileThreads + threadIdx.x] = g[u][c];
    gb2 = group_sum(gb2, red);
    loss = group_sum(loss, red);
    const long long P = mlp_size(H) + 1;
    double* out = gpart + (long long)blockIdx.x * P;
    for (int p = threadIdx.x; p < H * NG; p += kTileThreads) {
        const int j = p < H * kMlpIn ? p / kMlpIn : (p - H * kMlpIn) % H;
        const int c = p < H * kMlpIn ? p % kMlpIn : kMlpIn + (p - H * kMlpIn) / H;
        const double* v = &sums[c][j < ncol ? j : kTileThreads + j - ncol];
        double t = 0.0;
        for (int q = 0; q < nsplit; ++q) t += v[q * ncol];
        out[p] = t;
    }
    if (threadIdx.x == 0) {
        out[H * NG] = gb2;
        out[P - 1] = loss;
    }
}

// The same for up to kFewRows rows: a thread per hidden unit, and the rows'
// outputs summed by 16 lanes each.  The tiles above take 5 to 10 us however few
// their rows are (512 threads, six barriers and the splits' sums): with 256
// units 1 row 9.6 -> 4.0 us, 16 rows 10.4 -> 5.7; 20 rows in tiles 10.5.
constexpr int kFewRows = 16;
__global__ __launch_bounds__(kMlpThreads) void k_mlp_grad_few(const float* __restrict__ w, int H,
                                                              const float* __restrict__ F, const float* __restrict__ Y,
                                                              long long row0, long long stride, int count,
                                                              double* __restrict__ gpart) {
    static_assert(kMlpMaxHidden <= kMlpThreads && kFewRows * 16 <= kMlpThreads, "a thread per hidden unit, 16 per row");
    constexpr int NG = kMlpIn + 2, AT = 4;  // rows at once
    __shared__ double sf[kFewRows][kRow], hid[kFewRows][kMlpThreads + 2], err[kFewRows];
    const int j = threadIdx.x;
    double W[NG], g[NG], z[kFewRows];
#pragma unroll
    for (int c = 0; c < NG; ++c) {
        W[c] = j < H ? double(w[c < kMlpIn ? j * kMlpIn + c : H * c + j]) : 0.0;
        g[c] = 0.0;
    }
    const double b2 = w[H * NG];
    if (j < kFewRows * kRow) {
        const int r = j / kRow, c = j % kRow;
        const long long row = row0 + r * stride;
        sf[r][c] = r < count ? double(c < kMlpIn ? F[row * kMlpIn + c] : Y[row]) : 0.0;
    }
    __syncthreads();
#pragma unroll
    for (int r0 = 0; r0 < kFewRows; r0 += AT) {
        if (r0 >= count) break;
#pragma unroll
        for (int r = r0; r < r0 + AT; ++r) {
            z[r] = W[kMlpIn];
#pragma unroll
            for (int c = 0; c < kMlpIn; ++c) z[r] = fma(W[c], sf[r][c], z[r]);
            hid[r][j] = W[kMlpIn + 1] * fmax(z[r], 0.0);
        }
    }
    __syncthreads();
    if (j < 16 * count) {
        const int r = j / 16, q = j % 16;
        double p = 0.0;
        for (int i = 0; i < H; i += 64)
#pragma unroll
            for (int t = 0; t < 4; ++t) p += hid[r][i + 16 * t + q];
#pragma unroll
        for (int o = 8; o > 0; o >>= 1) p += __shfl_xor(p, o, 16);
        if (q == 0) err[r] = b2 + p - sf[r][kMlpIn];
    }
    __syncthreads();
    double gb2 = 0.0, loss = 0.0;
#pragma unroll
    for (int r0 = 0; r0 < kFewRows; r0 += AT) {
        if (r0 >= count) break;
#pragma unroll
        for (int r = r0; r < r0 + AT; ++r) {
            const double dy = r < count ? err[r] : 0.0;
            gb2 += dy;
            loss = fma(dy, dy, loss);
            g[kMlpIn + 1] = fma(dy, fmax(z[r], 0.0), g[kMlpIn + 1]);
            if (z[r] > 0.0) {
                const double dz = dy * W[kMlpIn + 1];
                g[kMlpIn] += dz;
#pragma unroll
                for (int c = 0; c < kMlpIn; ++c) g[c] = fma(dz, sf[r][c], g[c]);
            }
        }
    }
    if (j < H)
#pragma unroll
        for (int c = 0; c < NG; ++c) gpart[c < kMlpIn ? j * kMlpIn + c : H * c + j] = g[c];
    if (j == 0) {
        gpart[H * NG] = gb2;
        gpart[mlp_size(H)] = loss;
    }
}

// Adam step: gradient = scale * (sum of the partials, interleaved runs of
// work-groups added in order).  A work-group takes PAR neighbouring parameters:
// 16 of them where there are partials to sum, so that these are read as whole
// lines by many CUs (one work-group for all parameters took 109 us for 1793 of
// them, this 6); a single partial has nothing to spread, and fewer work-groups
// end sooner.
template <int PAR>
__global__ __launch_bounds__(kMlpThreads) void k_mlp_adam(float* __restrict__ w, double* __restrict__ m,
                                                          double* __restrict__ v, int H,
                                                          const double* __restrict__ gpart, int nparts,
                                                          double scale, double lr, int step,
                                                          double* __restrict__ loss_out) {
    constexpr int RUN = kMlpThreads / PAR;
    __shared__ double run[RUN][PAR];
    const long long P = mlp_size(H) + 1;
    const int i = threadIdx.x % PAR, r = threadIdx.x / PAR;
    const long long p = (long long)blockIdx.x * PAR + i;
    const double b1 = 0.9, b2 = 0.999, eps = 1e-8;
    double g = 0.0, mp = 0.0, vp = 0.0, wp = 0.0;
    if (r == 0 && p < P - 1) {  // read while the partials are
        mp = m[p];
        vp = v[p];
        wp = double(w[p]);
    }
    const double c1 = 1.0 - pow(b1, step), c2 = 1.0 - pow(b2, step);
    if (p < P)
#pragma unroll 8
        for (int b = r; b < nparts; b += RUN) g += gpart[b * P + p];
    if constexpr (RUN > 1) {
        run[r][i] = g;
        __syncthreads();
        g = 0.0;
#pragma unroll
        for (int q = 0; q < RUN; ++q) g += run[q][i];
    }
    if (r > 0 || p >= P) return;
    if (p == P - 1) {
        if (loss_out) *loss_out = 0.5 * g * scale;
        return;
    }
    g *= scale;
    const double mm = b1 * mp + (1.0 - b1) * g;
    const double vv = b2 * vp + (1.0 - b2) * g * g;
    m[p] = mm;
    v[p] = vv;
    w[p] = float(wp - lr * (mm / c1) / (sqrt(vv / c2) + eps));
}

inline int blocks_for(long long n) { return int((n + kMlpThreads - 1) / kMlpThreads); }

}  // namespace

void sum_partials(hipStream_t s, const double* part, int nchunk, int stride, int idx, double* out) {
    hipLaunchKernelGGL(k_sum_partials, dim3(1), dim3(kMlpThreads), 0, s, part, nchunk, stride, idx, out);
}

void mlp_apply(hipStream_t s, const float* w, int H, double* t, const double* dh, const double* dn,
               const double* theta, const double* rr, const double* tt, int n, double floor_, float* feat,
               float* sgn) {
    mlp_apply_grouped(s, w, H, t, dh, dn, theta, rr, tt, n, floor_, feat, sgn, nullptr, nullptr);
}

void mlp_apply_grouped(hipStream_t s, const float* w, int H, double* t, const double* dh, const double* dn,
                       const double* theta, const double* rr, const double* tt, int n, double floor_, float* feat,
                       float* sgn, const int* gid, const double* grms) {
    if (n <= 0) return;
    const size_t lds = w ? size_t(mlp_size(H)) * sizeof(double) : 0;
    hipLaunchKernelGGL(k_mlp_apply, dim3(blocks_for(n)), dim3(kMlpThreads), lds, s, w, H, t, dh, dn, theta, rr, tt,
                       n, floor_, feat, sgn, gid, grms);
}

void mlp_group_rms(hipStream_t s, const double* t, const double* dh, const double* dn, const double* theta,
                   double floor_, ElemGroups g, double* grms) {
    if (g.ng > 0)
        hipLaunchKernelGGL(k_mlp_group_rms, dim3(g.ng), dim3(kMlpThreads), 0, s, t, dh, dn, theta, floor_, g, grms);
}

void sumsq(hipStream_t s, const double* v, int n, double* out) {
    hipLaunchKernelGGL(k_sumsq, dim3(1), dim3(1024), 0, s, v, n, out);
}

void mlp_forward(hipStream_t s, const float* w, int H, const float* F, long long n, float* y) {
    if (n <= 0) return;
    // a work-group's time grows with its rows per lane, so as few as give no
    // more than one work-group per CU (256 units: 17000 rows 6.2 us, 8.3 in
    // tiles of 256, 33000 8.4 against 8.5, 60001 8.8 against 9.0)
    const int rows = 64 * int(std::min<long long>(kTileRows / 64, (n + 64 * 256 - 1) / (64 * 256)));
    hipLaunchKernelGGL(k_mlp_forward, dim3(int((n + rows - 1) / rows)), dim3(kTileThreads), 0, s, w, H, F, n, rows, y);
}

void mlp_targets(hipStream_t s, const double* X, long long ldx, int nrec, const double* xstar, int n, float* Y) {
    if (nrec > 0 && n > 0) hipLaunchKernelGGL(k_mlp_targets, dim3(nrec), dim3(1024), 0, s, X, ldx, xstar, n, Y);
}

void mlp_targets_grouped(hipStream_t s, const double* X, long long ldx, int nrec, const double* xstar, int n,
                         ElemGroups g, double* scal, float* Y) {
    if (nrec <= 0 || n <= 0 || g.ng <= 0) return;
    hipLaunchKernelGGL(k_mlp_target_dots, dim3(nrec), dim3(1024), 0, s, X, ldx, xstar, n, scal);
    hipLaunchKernelGGL(k_mlp_targets_grouped, dim3(g.ng, nrec), dim3(kMlpThreads), 0, s, X, ldx, xstar, n, g, scal,
                       Y);
}

void mlp_grad(hipStream_t s, const float* w, int H, const float* F, const float* Y, long long row0, long long stride,
              long long count, double* gpart, int nparts) {
    if (count <= kFewRows && nparts == 1)
        hipLaunchKernelGGL(k_mlp_grad_few, dim3(1), dim3(kMlpThreads), 0, s, w, H, F, Y, row0, stride, int(count), gpart);
    else
        hipLaunchKernelGGL(k_mlp_grad, dim3(nparts), dim3(kTileThreads), 0, s, w, H, F, Y, row0, stride, count, gpart);
}

void mlp_adam(hipStream_t s, float* w, double* m, double* v, int H, const double* gpart, int nparts, double scale,
              double lr, int step, double* loss_out) {
    const long long P = mlp_size(H) + 1;
    if (nparts == 1)
        hipLaunchKernelGGL(k_mlp_adam<kMlpThreads>, dim3(blocks_for(P)), dim3(kMlpThreads), 0, s, w, m, v, H, gpart, nparts,
                           scale, lr, step, loss_out);
    else
        hipLaunchKernelGGL(k_mlp_adam<16>, dim3(int((P + 15) / 16)), dim3(kMlpThreads), 0, s, w, m, v, H, gpart, nparts,
                           scale, lr, step, loss_out);
}

}  // namespace spk
