// Device kernels of the SP-MPS hot path for gfx950 (FP64).
//
// Every contraction of the one-site sweep -- environment updates (Fig.
// [spmpsOpt]) and the local products H_eff x, N_eff x (Eq. [geproblem]) --
// is a list of small dense products between particle-number blocks of the
// environments and (N, M) blocks of the site tensor.  The host runtime
// precomputes these lists once per site (the block structure is fixed); the
// kernels below execute them.  All reductions run in a fixed order (no
// floating-point atomics), so repeated calls give bitwise-identical results.
#include "kernels.h"

#include <type_traits>

namespace spk {

namespace {

constexpr int kThreads = 256;

__device__ inline double wave_sum64(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

__device__ inline double block_sum(double v, double* red) {
    // fixed-order tree reduction over the work-group (blockDim.x power of 2)
    red[threadIdx.x] = v;
    __syncthreads();
    for (int s = blockDim.x / 2; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
        __syncthreads();
    }
    double r = red[0];
    __syncthreads();
    return r;
}

__device__ inline double term_dot(const BufSet& bufs, const BTerm& tm, int r, int c) {
    const double* A = bufs.p[tm.a_buf] + tm.a_off + (long long)r * tm.a_rs;
    const double* B = bufs.p[tm.b_buf] + tm.b_off + (long long)c * tm.b_cs;
    double s = 0.0;
    for (int k = 0; k < tm.K; ++k) s = fma(A[(long long)k * tm.a_cs], B[(long long)k * tm.b_rs], s);
    return s;
}

__global__ __launch_bounds__(kThreads) void k_bgemm(const BTask* __restrict__ tasks,
                                                      const BTerm* __restrict__ terms, BufSet bufs,
                                                      const double* __restrict__ coef) {
    __shared__ double red[kThreads];
    const BTask tk = tasks[blockIdx.x];
    const int MN = tk.M * tk.N;
    if (MN <= 0) return;
    double* C = bufs.p[tk.c_buf] + tk.c_off;
    const int nt = tk.t1 - tk.t0;
    int S = 1;
    if (MN < kThreads && nt > 1) {
        S = kThreads / MN;
        if (S > nt) S = nt;
    }
    if (S == 1) {
        for (int o = threadIdx.x; o < MN; o += kThreads) {
            const int r = o / tk.N, c = o - r * tk.N;
            double acc = 0.0;
            for (int t = tk.t0; t < tk.t1; ++t) {
                const BTerm tm = terms[t];
                acc = fma(coef[tm.cidx], term_dot(bufs, tm, r, c), acc);
            }
            double* cp = C + (long long)r * tk.ldc + c;
            *cp = tk.accumulate ? *cp + acc : acc;
        }
    } else {
        // split the term list over S groups of MN threads, then add the S
        // partial sums in a fixed order
        const int o = threadIdx.x % MN;
        const int sp = threadIdx.x / MN;
        const int r = o / tk.N, c = o - r * tk.N;
        double acc = 0.0;
        if (sp < S) {
            for (int t = tk.t0 + sp; t < tk.t1; t += S) {
                const BTerm tm = terms[t];
                acc = fma(coef[tm.cidx], term_dot(bufs, tm, r, c), acc);
            }
        }
        red[threadIdx.x] = acc;
        __syncthreads();
        if ((int)threadIdx.x < MN) {
            double tot = 0.0;
            for (int q = 0; q < S; ++q) tot += red[q * MN + threadIdx.x];
            double* cp = C + (long long)r * tk.ldc + c;
            *cp = tk.accumulate ? *cp + tot : tot;
        }
    }
}

__global__ __launch_bounds__(kThreads) void k_combine(const CTask* __restrict__ tasks,
                                                        const CTerm* __restrict__ terms,
                                                        BufSet bufs, const double* __restrict__ coef) {
    // the task's terms (source pointer, coefficient) are staged in LDS by one
    // thread each, 64 at a time, so that the element loop issues independent
    // loads; every element still sums its terms in list order
    constexpr int kTermsAtOnce = 64, kPer = 4;
    __shared__ const double* sp[kTermsAtOnce];
    __shared__ double sc[kTermsAtOnce];
    const CTask tk = tasks[blockIdx.x];
    double* C = bufs.p[tk.c_buf] + tk.c_off;
    for (int eb = 0; eb < tk.n; eb += kPer * kThreads) {
        double acc[kPer];
#pragma unroll
        for (int u = 0; u < kPer; ++u) acc[u] = 0.0;
        for (int tb = tk.t0; tb < tk.t1; tb += kTermsAtOnce) {
            const int nt = min(kTermsAtOnce, tk.t1 - tb);
            __syncthreads();
            if ((int)threadIdx.x < nt) {
                const CTerm tm = terms[tb + threadIdx.x];
                sp[threadIdx.x] = bufs.p[tm.a_buf] + tm.a_off;
                sc[threadIdx.x] = coef[tm.cidx];
            }
            __syncthreads();
            for (int t = 0; t < nt; ++t) {
                const double* __restrict__ a = sp[t];
                const double c = sc[t];
#pragma unroll
                for (int u = 0; u < kPer; ++u) {
                    const int e = eb + threadIdx.x + u * kThreads;
                    if (e < tk.n) acc[u] = fma(c, a[e], acc[u]);
                }
            }
        }
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int e = eb + threadIdx.x + u * kThreads;
            if (e < tk.n) C[e] = acc[u];
        }
    }
}

// Diagonals of the environment blocks, compact: Ld/Rd(g, z, p).  blockIdx.y
// is g, blockIdx.z the side.  One strided 8-byte read per value; everything
// after it reads contiguous rows.
__global__ __launch_bounds__(kThreads) void k_diag_gather(DiagSide left, DiagSide right) {
    const DiagSide& S = blockIdx.z ? right : left;
    const int e = blockIdx.x * kThreads + threadIdx.x;
    if (e >= S.nz * S.D) return;
    const int z = e / S.D, p = e - z * S.D, g = blockIdx.y;
    const DiagSrc src = S.src[z * S.nnb + S.nb[p]];
    double v = 0.0;
    if (src.ld >= 0) v = S.env[g * S.esize + src.off + (long long)S.ro[p] * (src.ld + 1)];
    S.out[(long long)g * S.nz * S.D + e] = v;
}

// M(g, row, p) = sum over the row's terms of coef * Ld(g, z, p): one
// work-group per (row, g), the terms staged in LDS 64 at a time so that the
// loads of the sum are independent of each other.
__global__ __launch_bounds__(kThreads) void k_diag_mix(const DiagMix* __restrict__ mix,
                                                         const DiagMixTerm* __restrict__ terms,
                                                         const double* __restrict__ Ld, int nzl, int Dl,
                                                         const double* __restrict__ coef, int ncoef, int nmix,
                                                         double* __restrict__ M) {
    constexpr int kAtOnce = 64;
    __shared__ int sz[kAtOnce];
    __shared__ double sc[kAtOnce];
    const DiagMix m = mix[blockIdx.x];
    const int g = blockIdx.y;
    const double* __restrict__ src = Ld + (long long)g * nzl * Dl;
    double* __restrict__ out = M + ((long long)g * nmix + blockIdx.x) * Dl;
    for (int p0 = 0; p0 < Dl; p0 += blockDim.x) {
        const int p = p0 + threadIdx.x;
        double acc = 0.0;
        for (int tb = m.t0; tb < m.t1; tb += kAtOnce) {
            const int nt = min(kAtOnce, m.t1 - tb);
            __syncthreads();
            if ((int)threadIdx.x < nt) {
                const DiagMixTerm tm = terms[tb + threadIdx.x];
                sz[threadIdx.x] = tm.z * Dl;
                sc[threadIdx.x] = coef[(long long)g * ncoef + tm.cidx];
            }
            __syncthreads();
            if (p < Dl) {
#pragma unroll 8
                for (int t = 0; t < nt; ++t) acc = fma(sc[t], src[sz[t] + p], acc);
            }
        }
        if (p < Dl) out[p] = acc;
    }
}

// A tile of an outer-product sum out(r, c) = sum over units u0 .. u1 of
// lv(u, r) rv(u, c), staged through LDS 32 units at a time with the next
// chunk's loads issued before the products of the current one; a thread owns
// column tid % 32 and rows tid / 32 + 8 i.  value(u, x, l, r) gives the left
// value of row x and the right one of column x.
template <class F>
__device__ inline void diag_tile(const DiagBlk& b, int u0, int u1, double* __restrict__ out, F value) {
    constexpr int T = kDiagTile, U = 32, PER = U * T / kThreads;
    static_assert(PER == 4 && T == 32, "four staged values of either operand per thread");
    __shared__ double Ls[U][T], Rs[U][T];
    const int x = threadIdx.x % T, y = threadIdx.x / T;
    double lv[PER], rv[PER], acc[PER] = {0.0, 0.0, 0.0, 0.0};
    auto fetch = [&](int ub) {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int u = ub + y + 8 * i;
            lv[i] = rv[i] = 0.0;
            if (u < u1) value(u, x, lv[i], rv[i]);
        }
    };
    if (u0 < u1) fetch(u0);
    for (int ub = u0; ub < u1; ub += U) {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            Ls[y + 8 * i][x] = lv[i];
            Rs[y + 8 * i][x] = rv[i];
        }
        __syncthreads();
        if (ub + U < u1) fetch(ub + U);
        const int nu = min(U, u1 - ub);
        for (int u = 0; u < nu; ++u) {
            const double r = Rs[u][x];
#pragma unroll
            for (int i = 0; i < PER; ++i)
                if (8 * i < b.rows) acc[i] = fma(Ls[u][y + 8 * i], r, acc[i]);
        }
        __syncthreads();
    }
    if (x < b.cols) {
#pragma unroll
        for (int i = 0; i < PER; ++i)
            if (y + 8 * i < b.rows) out[b.x_off + (y + 8 * i) * b.ldc + x] = acc[i];
    }
}

// One tile of the diagonal of H_eff or N_eff from the gathered diagonals, its
// units u = (g, row).  Every environment value is read once per tile instead of
// once per element, and a right channel's terms are mixed once per bond state:
// the centre of the K = 12, D = 128, G = 11 ab-initio state has 8600 terms per
// sigma but 250 rows, and its three launches take the diagonal from 3.8 ms (one
// work-group summing every term of every element of a block) to under 0.1 ms.
// A part of 256 units is 8 staged chunks.
__global__ __launch_bounds__(kThreads) void k_diag(const DiagBlk* __restrict__ blks, const int* __restrict__ zlist,
                                                     const double* __restrict__ M, int nmix, int Dl,
                                                     const double* __restrict__ Rd, int nzr, int Dr, int G,
                                                     double* __restrict__ dh, double* __restrict__ dn,
                                                     double* __restrict__ part, long long ntot) {
    const DiagBlk b = blks[blockIdx.x];
    const int nsplit = b.is_n ? 1 : gridDim.y, j = blockIdx.y;
    if (j >= nsplit) return;
    const int UT = G * b.nrow;
    const int u0 = int((long long)UT * j / nsplit), u1 = int((long long)UT * (j + 1) / nsplit);
    double* __restrict__ out = b.is_n ? dn : (nsplit == 1 ? dh : part + (long long)j * ntot);
    diag_tile(b, u0, u1, out, [&](int u, int x, double& l, double& r) {
        const int g = u / b.nrow, q = u - g * b.nrow;
        if (x < b.rows) l = M[((long long)g * nmix + b.row0 + q) * Dl + b.p0 + x];
        if (x < b.cols) r = Rd[((long long)g * nzr + zlist[b.zl0 + q]) * Dr + b.q0 + x];
    });
}

// The same tile from the environments themselves, its units (g, term): one
// launch for both diagonals.  A chain of dependent reads bounds it (tile, term,
// coefficient and diagonals, 4 us in all for a few units); every tile reads the
// strided diagonals again, which many units or tiles make dearer than the
// gathered rows of three launches.
__global__ __launch_bounds__(kThreads) void k_diag_direct(const DiagBlk* __restrict__ blks, const DiagTerm* __restrict__ terms,
                                                            const double* __restrict__ lenv, long long lsize,
                                                            const double* __restrict__ renv, long long rsize,
                                                            const double* __restrict__ coef, int ncoef, int G,
                                                            double* __restrict__ dh, double* __restrict__ dn) {
    const DiagBlk b = blks[blockIdx.x];
    const int nt = b.t1 - b.t0;
    diag_tile(b, 0, G * nt, b.is_n ? dn : dh, [&](int u, int x, double& l, double& r) {
        const int g = u / nt;
        const DiagTerm t = terms[b.t0 + u - g * nt];
        if (x < b.rows) l = coef[(long long)g * ncoef + t.cidx] * lenv[g * lsize + t.l_off + (b.r0 + x) * (t.l_ld + 1LL)];
        if (x < b.cols) r = renv[g * rsize + t.r_off + (b.c0 + x) * (t.r_ld + 1LL)];
    });
}

__global__ __launch_bounds__(kThreads) void k_diag_sum(const double* __restrict__ part, int nsplit, long long ntot,
                                                         double* __restrict__ out) {
    const long long e = (long long)blockIdx.x * kThreads + threadIdx.x;
    if (e >= ntot) return;
    double acc = 0.0;
    for (int j = 0; j < nsplit; ++j) acc += part[(long long)j * ntot + e];
    out[e] = acc;
}

// Householder QR of one gathered sector matrix (rows >= cols), column-major
// in scratch; Q overwrites the pieces, R (cols x cols, row-major) goes to
// rout.  Signs are fixed so that diag(R) >= 0 (the unique QR of a full-rank
// matrix).
__global__ __launch_bounds__(kThreads) void k_qr(const QrTask* __restrict__ tasks,
                                                   const QrPiece* __restrict__ pieces,
                                                   double* __restrict__ site,
                                                   double* __restrict__ scratch,
                                                   double* __restrict__ rout) {
    __shared__ double red[kThreads];
    __shared__ double tau_s[256];
    __shared__ double diag_s[256];
    __shared__ double dots[256];
    const QrTask tk = tasks[blockIdx.x];
    const int rows = tk.rows, cols = tk.cols;
    double* S = scratch + tk.scratch_off;           // rows x cols, column-major
    double* Q = S + (long long)rows * cols;          // rows x cols, column-major
    // gather
    for (int p = tk.p0; p < tk.p1; ++p) {
        const QrPiece pc = pieces[p];
        const int nr = pc.transposed ? pc.pcol : pc.prow;
        const int nel = nr * cols;
        for (int e = threadIdx.x; e < nel; e += kThreads) {
            const int rr = e / cols, cc = e - rr * cols;
            const double v = pc.transposed ? site[pc.off + (long long)cc * pc.pcol + rr]
                                           : site[pc.off + (long long)rr * pc.pcol + cc];
            S[(long long)cc * rows + pc.row0 + rr] = v;
        }
    }
    __syncthreads();
    for (int j = 0; j < cols; ++j) {
        double ss = 0.0;
        for (int r = j + threadIdx.x; r < rows; r += kThreads) {
            const double v = S[(long long)j * rows + r];
            ss = fma(v, v, ss);
        }
        ss = block_sum(ss, red);
        if (threadIdx.x == 0) {
            const double x0 = S[(long long)j * rows + j];
            const double nrm = sqrt(ss);
            const double alpha = (x0 >= 0.0) ? -nrm : nrm;
            const double v0 = x0 - alpha;
            const double vv = ss - x0 * x0 + v0 * v0;
            tau_s[j] = (vv > 0.0) ? 2.0 / vv : 0.0;
            diag_s[j] = alpha;
            S[(long long)j * rows + j] = v0;
        }
        __syncthreads();
        const double tau = tau_s[j];
        for (int c = j + 1 + threadIdx.x; c < cols; c += kThreads) {
            double d = 0.0;
            for (int r = j; r < rows; ++r) d = fma(S[(long long)j * rows + r], S[(long long)c * rows + r], d);
            const double f = tau * d;
            for (int r = j; r < rows; ++r) S[(long long)c * rows + r] -= f * S[(long long)j * rows + r];
        }
        __syncthreads();
    }
    // R (row-major) with the sign fix
    double* R = rout + tk.r_off;
    for (int e = threadIdx.x; e < cols * cols; e += kThreads) {
        const int i = e / cols, c = e - i * cols;
        double v = 0.0;
        if (c == i) v = diag_s[i];
        else if (c > i) v = S[(long long)c * rows + i];
        if (diag_s[i] < 0.0) v = -v;
        R[e] = v;
    }
    // Q = H_0 ... H_{cols-1} [I; 0]
    for (int e = threadIdx.x; e < rows * cols; e += kThreads) {
        const int c = e / rows, r = e - c * rows;
        Q[e] = (r == c) ? 1.0 : 0.0;
    }
    __syncthreads();
    for (int j = cols - 1; j >= 0; --j) {
        const double tau = tau_s[j];
        for (int c = threadIdx.x; c < cols; c += kThreads) {
            double d = 0.0;
            for (int r = j; r < rows; ++r) d = fma(S[(long long)j * rows + r], Q[(long long)c * rows + r], d);
            dots[c] = tau * d;
        }
        __syncthreads();
        const int span = rows - j;
        for (int e = threadIdx.x; e < span * cols; e += kThreads) {
            const int c = e / span, r = j + (e - c * span);
            Q[(long long)c * rows + r] -= dots[c] * S[(long long)j * rows + r];
        }
        __syncthreads();
    }
    // scatter Q with the sign fix
    for (int p = tk.p0; p < tk.p1; ++p) {
        const QrPiece pc = pieces[p];
        const int nr = pc.transposed ? pc.pcol : pc.prow;
        const int nel = nr * cols;
        for (int e = threadIdx.x; e < nel; e += kThreads) {
            const int rr = e / cols, cc = e - rr * cols;
            double v = Q[(long long)cc * rows + pc.row0 + rr];
            if (diag_s[cc] < 0.0) v = -v;
            if (pc.transposed) site[pc.off + (long long)cc * pc.pcol + rr] = v;
            else site[pc.off + (long long)rr * pc.pcol + cc] = v;
        }
    }
}

// The same factorisation with both matrices in LDS: the norm of the pivot
// column is a wave reduction, and each trailing (or Q) column is updated by
// one wave (lanes over rows, dot product by cross-lane shuffles).
__global__ __launch_bounds__(kThreads) void k_qr_lds(const QrTask* __restrict__ tasks,
                                                       const QrPiece* __restrict__ pieces,
                                                       double* __restrict__ site, double* __restrict__ rout) {
    extern __shared__ double sh[];
    __shared__ double tau_s[256];
    __shared__ double diag_s[256];
    const QrTask tk = tasks[blockIdx.x];
    const int rows = tk.rows, cols = tk.cols;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    double* S = sh;                       // rows x cols, column-major
    double* Q = sh + (long long)rows * cols;
    for (int p = tk.p0; p < tk.p1; ++p) {
        const QrPiece pc = pieces[p];
        const int nr = pc.transposed ? pc.pcol : pc.prow;
        const int nel = nr * cols;
        for (int e = threadIdx.x; e < nel; e += kThreads) {
            const int rr = e / cols, cc = e - rr * cols;
            const double v = pc.transposed ? site[pc.off + (long long)cc * pc.pcol + rr]
                                           : site[pc.off + (long long)rr * pc.pcol + cc];
            S[cc * rows + pc.row0 + rr] = v;
        }
    }
    __syncthreads();
    for (int j = 0; j < cols; ++j) {
        const double* sj = S + j * rows;
        if (wave == 0) {
            double ss = 0.0;
            for (int r = j + lane; r < rows; r += 64) ss = fma(sj[r], sj[r], ss);
            ss = wave_sum64(ss);
            if (lane == 0) {
                const double x0 = sj[j];
                const double nrm = sqrt(ss);
                const double alpha = (x0 >= 0.0) ? -nrm : nrm;
                const double v0 = x0 - alpha;
                const double vv = ss - x0 * x0 + v0 * v0;
                tau_s[j] = (vv > 0.0) ? 2.0 / vv : 0.0;
                diag_s[j] = alpha;
                S[j * rows + j] = v0;
            }
        }
        __syncthreads();
        const double tau = tau_s[j];
        for (int c = j + 1 + wave; c < cols; c += kThreads / 64) {
            double* sc = S + c * rows;
            double d = 0.0;
            for (int r = j + lane; r < rows; r += 64) d = fma(sj[r], sc[r], d);
            const double f = tau * wave_sum64(d);
            for (int r = j + lane; r < rows; r += 64) sc[r] -= f * sj[r];
        }
        __syncthreads();
    }
    double* R = rout + tk.r_off;
    for (int e = threadIdx.x; e < cols * cols; e += kThreads) {
        const int i = e / cols, c = e - i * cols;
        double v = 0.0;
        if (c == i) v = diag_s[i];
        else if (c > i) v = S[c * rows + i];
        if (diag_s[i] < 0.0) v = -v;
        R[e] = v;
    }
    for (int e = threadIdx.x; e < rows * cols; e += kThreads) {
        const int c = e / rows, r = e - c * rows;
        Q[e] = (r == c) ? 1.0 : 0.0;
    }
    __syncthreads();
    for (int j = cols - 1; j >= 0; --j) {
        const double tau = tau_s[j];
        const double* sj = S + j * rows;
        for (int c = wave; c < cols; c += kThreads / 64) {
            double* qc = Q + c * rows;
            double d = 0.0;
            for (int r = j + lane; r < rows; r += 64) d = fma(sj[r], qc[r], d);
            const double f = tau * wave_sum64(d);
            for (int r = j + lane; r < rows; r += 64) qc[r] -= f * sj[r];
        }
        __syncthreads();
    }
    for (int p = tk.p0; p < tk.p1; ++p) {
        const QrPiece pc = pieces[p];
        const int nr = pc.transposed ? pc.pcol : pc.prow;
        const int nel = nr * cols;
        for (int e = threadIdx.x; e < nel; e += kThreads) {
            const int rr = e / cols, cc = e - rr * cols;
            double v = Q[cc * rows + pc.row0 + rr];
            if (diag_s[cc] < 0.0) v = -v;
            if (pc.transposed) site[pc.off + (long long)cc * pc.pcol + rr] = v;
            else site[pc.off + (long long)rr * pc.pcol + cc] = v;
        }
    }
}

// Sum over rows q + 16 i of a column in 16 lanes (acc[i % 4] adds them for
// ascending i / 4), the same bits in every lane: the order of wave_sum64 over
// rows dealt to 64 lanes, whichever row the lanes start at.
__device__ inline double column_sum(const double (&acc)[4]) {
    auto ror = [](double x, auto n) {
        constexpr int ctrl = 0x120 + decltype(n)::value;  // row_ror
        const long long b = __builtin_bit_cast(long long, x);
        const int lo = __builtin_amdgcn_mov_dpp(int(b), ctrl, 0xf, 0xf, false);
        const int hi = __builtin_amdgcn_mov_dpp(int(b >> 32), ctrl, 0xf, 0xf, false);
        return __builtin_bit_cast(double, (long long)((unsigned long long)(unsigned)lo | (unsigned long long)(unsigned)hi << 32));
    };
    double v = (acc[0] + acc[2]) + (acc[1] + acc[3]);
    v += ror(v, std::integral_constant<int, 8>{});
    v += ror(v, std::integral_constant<int, 4>{});
    v += ror(v, std::integral_constant<int, 2>{});
    v += ror(v, std::integral_constant<int, 1>{});
    return v;
}

// The same factorisation with a column per 16 lanes, its rows lane + 16 i
// in registers; only the Householder vectors are in LDS (zero above their
// diagonal and past the last row).  Latency bounds it: a chain of one LDS
// read, dot product, update, norm, square root and division per column, one
// barrier each -- the lanes of column j + 1 form their vector as soon as
// vector j is applied to it -- and no barrier at all in the Q pass.  Sums run
// in the order of k_qr_lds: the two give the same bits (near-dependent columns
// amplify any rounding).  With S
// and Q in LDS and a wavefront per column a gauge move at L = 32, D = 256 took
// 102 us on average, this 23; at D = 512 (S and Q in memory, a thread per
// column) 2.8 ms, this 71 us.
template <int RV>
__global__ __launch_bounds__(16 * kQrRegCols) void k_qr_reg(const QrTask* __restrict__ tasks,
                                                           const QrPiece* __restrict__ pieces,
                                                           double* __restrict__ site, double* __restrict__ rout) {
    extern __shared__ double sh[];  // Householder vectors, 16 nv values each
    __shared__ double tau_s[kQrRegCols], diag_s[kQrRegCols];
    const QrTask tk = tasks[blockIdx.x];
    const int rows = tk.rows, cols = tk.cols, nv = (rows + 15) / 16, ldv = 16 * nv;
    const int q = threadIdx.x % 16, c = threadIdx.x / 16;
    const int cw = __builtin_amdgcn_readfirstlane(c);  // first column of the wavefront
    double s[RV], v[RV];
#pragma unroll
    for (int i = 0; i < RV; ++i) s[i] = 0.0;
    if (c < cols)
        for (int p = tk.p0; p < tk.p1; ++p) {
            const QrPiece pc = pieces[p];
            const int nr = pc.transposed ? pc.pcol : pc.prow;
#pragma unroll
            for (int i = 0; i < RV; ++i) {
                const int rr = q + 16 * i - pc.row0;
                if (rr >= 0 && rr < nr)
                    s[i] = site[pc.off + (pc.transposed ? (long long)c * pc.pcol + rr : (long long)rr * pc.pcol + c)];
            }
        }
    // the Householder vector of column j = c from its rows >= j
    auto reflect = [&](int j) {
        double sq[4] = {}, top[4] = {};
#pragma unroll
        for (int i = 0; i < RV; ++i) {
            const int r = q + 16 * i;
            if (r >= j) sq[i % 4] = fma(s[i], s[i], sq[i % 4]);
            if (r == j) top[0] = s[i];
        }
        const double ss = column_sum(sq), x0 = column_sum(top);
        const double nrm = sqrt(ss);
        const double alpha = (x0 >= 0.0) ? -nrm : nrm;
        const double v0 = x0 - alpha;
        const double vv = ss - x0 * x0 + v0 * v0;
#pragma unroll
        for (int i = 0; i < RV; ++i) {
            const int r = q + 16 * i;
            if (i < nv) sh[j * ldv + r] = r > j ? s[i] : (r == j ? v0 : 0.0);
        }
        if (q == 0) {
            tau_s[j] = (vv > 0.0) ? 2.0 / vv : 0.0;
            diag_s[j] = alpha;
        }
    };
    // s -= tau (v_j . s) v_j
    auto apply = [&](int j) {
        const double tau = tau_s[j];
        double d[4] = {};
#pragma unroll
        for (int i = 0; i < RV; ++i) v[i] = i < nv ? sh[j * ldv + q + 16 * i] : 0.0;
#pragma unroll
        for (int i = 0; i < RV; ++i) d[i % 4] = fma(v[i], s[i], d[i % 4]);
        const double f = tau * column_sum(d);
#pragma unroll
        for (int i = 0; i < RV; ++i) s[i] = fma(-f, v[i], s[i]);
    };
    if (c == 0) reflect(0);
    __syncthreads();
    for (int j = 0; j + 1 < cols; ++j) {
        if (cw + 3 > j) {
            if (c > j && c < cols) apply(j);
            if (c == j + 1) reflect(j + 1);
        }
        __syncthreads();
    }
    if (c >= cols) return;
    double* R = rout + tk.r_off;
#pragma unroll
    for (int i = 0; i < RV; ++i) {
        const int r = q + 16 * i;
        if (r < cols) {
            const double dg = diag_s[r], x = r < c ? s[i] : (r == c ? dg : 0.0);
            R[r * cols + c] = dg < 0.0 ? -x : x;
        }
    }
    // column c of H_0 .. H_{cols-1} [I; 0]; vectors j > c leave it alone
#pragma unroll
    for (int i = 0; i < RV; ++i) s[i] = q + 16 * i == c ? 1.0 : 0.0;
    for (int j = min(cw + 3, cols - 1); j >= 0; --j) apply(j);
    const double sign = diag_s[c] < 0.0 ? -1.0 : 1.0;
    for (int p = tk.p0; p < tk.p1; ++p) {
        const QrPiece pc = pieces[p];
        const int nr = pc.transposed ? pc.pcol : pc.prow;
#pragma unroll
        for (int i = 0; i < RV; ++i) {
            const int rr = q + 16 * i - pc.row0;
            if (rr >= 0 && rr < nr)
                site[pc.off + (pc.transposed ? (long long)c * pc.pcol + rr : (long long)rr * pc.pcol + c)] = sign * s[i];
        }
    }
}

// ---- Davidson vector kernels --------------------------------------------

__global__ __launch_bounds__(kThreads) void k_fill(double* __restrict__ p, long long n, double value) {
    for (long long i = (long long)blockIdx.x * kThreads + threadIdx.x; i < n; i += (long long)gridDim.x * kThreads)
        p[i] = value;
}

__global__ __launch_bounds__(1024) void k_normalize(const double* __restrict__ in,
                                                     double* __restrict__ out, int n,
                                                     double* __restrict__ norm_out) {
    __shared__ double red[1024];
    double ss = 0.0;
    for (int e = threadIdx.x; e < n; e += 1024) ss = fma(in[e], in[e], ss);
    ss = block_sum(ss, red);
    const double nrm = sqrt(ss);
    const double inv = nrm > 0.0 ? 1.0 / nrm : 0.0;
    for (int e = threadIdx.x; e < n; e += 1024) out[e] = in[e] * inv;
    if (threadIdx.x == 0 && norm_out) *norm_out = nrm;
}

__global__ __launch_bounds__(kThreads) void k_multidot(const double* __restrict__ A, long long ld,
                                                         const double* __restrict__ u, int n,
                                                         double* __restrict__ out) {
    __shared__ double red[kThreads];
    const double* a = A + blockIdx.x * ld;
    double s = 0.0;
    for (int e = threadIdx.x; e < n; e += kThreads) s = fma(a[e], u[e], s);
    s = block_sum(s, red);
    if (threadIdx.x == 0) out[blockIdx.x] = s;
}

// out_i = sum_j Q[j][i] A_j for i < keep: eight outputs per pass, the A
// loads of a pass batched eight vectors at a time
__global__ __launch_bounds__(kThreads) void k_basis_rotate(const double* __restrict__ A,
                                                             long long ld, int m,
                                                             const double* __restrict__ Q, int keep,
                                                             double* __restrict__ out, int n) {
    const int e = blockIdx.x * kThreads + threadIdx.x;
    if (e >= n) return;
    for (int i0 = 0; i0 < keep; i0 += 8) {
        double acc[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) acc[u] = 0.0;
        for (int j0 = 0; j0 < m; j0 += 8) {
            double av[8];
#pragma unroll
            for (int v = 0; v < 8; ++v) av[v] = (j0 + v < m) ? A[(long long)(j0 + v) * ld + e] : 0.0;
#pragma unroll
            for (int v = 0; v < 8; ++v) {
                if (j0 + v >= m) break;
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    if (i0 + u < keep) acc[u] = fma(Q[(j0 + v) * keep + i0 + u], av[v], acc[u]);
            }
        }
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (i0 + u < keep) out[(long long)(i0 + u) * ld + e] = acc[u];
    }
}

__global__ __launch_bounds__(kThreads) void k_to_f32(const double* __restrict__ in, float* __restrict__ out,
                                                       long long n) {
    const long long e = (long long)blockIdx.x * kThreads + threadIdx.x;
    if (e < n) out[e] = float(in[e]);
}

// the sum of p[g stride + e] over g = 0..G-1 in order, U slots' loads issued
// together
template <int U>
__device__ inline double sum_slots(const double* __restrict__ p, long long stride, int G, long long e) {
    double s = 0.0;
    int g = 0;
    for (; g + U <= G; g += U) {
        double a[U];
#pragma unroll
        for (int u = 0; u < U; ++u) a[u] = p[(g + u) * stride + e];
#pragma unroll
        for (int u = 0; u < U; ++u) s += a[u];
    }
    for (; g < G; ++g) s += p[g * stride + e];
    return s;
}

// 64 elements per work-group (a wavefront's width: the vectors are short, so
// wider groups leave most of the chip idle); wavefront w adds its quarter of
// the slots, then the four sums are added in order.  blockIdx.y: the output.
__global__ __launch_bounds__(kThreads) void k_gsum2(const double* __restrict__ pa, const double* __restrict__ pb,
                                                      long long stride, int Ga, int Gb, int n,
                                                      double* __restrict__ outa, double* __restrict__ outb) {
    __shared__ double red[4][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int e = blockIdx.x * 64 + lane, G = blockIdx.y ? Gb : Ga;
    const int g0 = G * wave / 4, g1 = G * (wave + 1) / 4;
    const double* __restrict__ p = blockIdx.y ? pb : pa;
    red[wave][lane] = e < n ? sum_slots<8>(p + g0 * stride, stride, g1 - g0, e) : 0.0;
    __syncthreads();
    if (wave == 0 && e < n)
        (blockIdx.y ? outb : outa)[e] = (red[0][lane] + red[1][lane]) + (red[2][lane] + red[3][lane]);
}

// ---- grid-parallel Davidson passes ----------------------------------------
// A work-group owns kDavChunk consecutive elements.  The Ritz and CGS passes
// run 1024 threads per work-group: four groups of 256 threads split the
// subspace index, each thread loading all of its vectors in one batch, and
// their partial sums are added in LDS in a fixed order.

constexpr int kDavWide = 1024;
constexpr int kDavGroups = kDavWide / kDavChunk;  // 4
constexpr int kDavWaves = kDavWide / 64;          // 16
static_assert(kDavChunk == kThreads, "one element per thread of a group");
constexpr int kBatch = 8;

__device__ inline double wave_sum(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// out[j] = sum over q < nchunk of part[q * stride + j], for j < m.  Wave w
// of NW adds the chunks q = w mod NW (ascending), then the NW wave sums are
// added in wave order: a fixed order, so the result is deterministic.
template <int NW>
__device__ inline void reduce_partials(const double* __restrict__ part, int nchunk, int stride, int m,
                                       double (*wred)[64], double* out) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int j0 = 0; j0 < m; j0 += 64) {
        const int j = j0 + lane;
        double acc = 0.0;
        if (j < m) {
            int q = wave;
            for (; q + 3 * NW < nchunk; q += 4 * NW) {
                const double p0 = part[(long long)q * stride + j];
                const double p1 = part[(long long)(q + NW) * stride + j];
                const double p2 = part[(long long)(q + 2 * NW) * stride + j];
                const double p3 = part[(long long)(q + 3 * NW) * stride + j];
                acc += p0;
                acc += p1;
                acc += p2;
                acc += p3;
            }
            for (; q < nchunk; q += NW) acc += part[(long long)q * stride + j];
        }
        wred[wave][lane] = acc;
        __syncthreads();
        if (threadIdx.x < 64 && j < m) {
            double r = 0.0;
#pragma unroll
            for (int w = 0; w < NW; ++w) r += wred[w][lane];
            out[j] = r;
        }
        __syncthreads();
    }
}

// out[j] = sum over the chunk of src_j[e] w[e] for j < m, src_j = base + j ld,
// with w staged in LDS (ws, kDavChunk values).  Wave w of NW takes
// j = w mod NW, four vectors per pass (16 loads in flight per lane).
template <int NW>
__device__ inline void chunk_dots(const double* __restrict__ base, long long ld, int m, int e0, int n,
                                  const double* ws, double* __restrict__ out) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int nval = min(kDavChunk, n - e0);
    double wv[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) wv[q] = ws[lane + 64 * q];
    for (int j = wave; j < m; j += 4 * NW) {
        double acc[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            acc[u] = 0.0;
            const int jj = j + NW * u;
            if (jj < m) {
                const double* __restrict__ src = base + (long long)jj * ld + e0;
                double v[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) v[q] = (lane + 64 * q < nval) ? src[lane + 64 * q] : 0.0;
#pragma unroll
                for (int q = 0; q < 4; ++q) acc[u] = fma(v[q], wv[q], acc[u]);
            }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const double r = wave_sum(acc[u]);
            if (lane == 0 && j + NW * u < m) out[j + NW * u] = r;
        }
    }
}

// the subspace range [j0, j1) of thread group jg when m vectors are split
// over kDavGroups groups
__device__ inline void group_range(int m, int jg, int& j0, int& j1) {
    const int per = (m + kDavGroups - 1) / kDavGroups;
    j0 = min(m, jg * per);
    j1 = min(m, j0 + per);
}

__device__ inline void dav_ritz_body(const double* __restrict__ V, const double* __restrict__ HV,
                                                         const double* __restrict__ NV, long long ld, int m,
                                                         const double* __restrict__ aq,
                                                         const double* __restrict__ dh,
                                                         const double* __restrict__ dn, int n, double floor_,
                                                         double* __restrict__ x, double* __restrict__ t,
                                                         double* __restrict__ part_x, double* __restrict__ part_c, int chunk) {
    __shared__ double sa[kDavMaxVec + 1];
    __shared__ double red[3][kDavGroups][kDavChunk];
    __shared__ double ts[kDavChunk];
    __shared__ double wsum[4][3];
    for (int j = threadIdx.x; j <= m; j += kDavWide) sa[j] = aq[j];
    __syncthreads();
    const double theta = sa[m];
    const int el = threadIdx.x & (kDavChunk - 1), jg = threadIdx.x / kDavChunk;
    const int e0 = chunk * kDavChunk;
    const int e = e0 + el;
    {
        double xv = 0.0, hv = 0.0, nv = 0.0;
        if (e < n) {
            int j0, j1;
            group_range(m, jg, j0, j1);
            int j = j0;
            for (; j + kBatch <= j1; j += kBatch) {
                double v[kBatch], h[kBatch], q[kBatch];
#pragma unroll
                for (int u = 0; u < kBatch; ++u) {
                    const long long o = (long long)(j + u) * ld + e;
                    v[u] = V[o];
                    h[u] = HV[o];
                    q[u] = NV[o];
                }
#pragma unroll
                for (int u = 0; u < kBatch; ++u) {
                    xv = fma(sa[j + u], v[u], xv);
                    hv = fma(sa[j + u], h[u], hv);
                    nv = fma(sa[j + u], q[u], nv);
                }
            }
            for (; j < j1; ++j) {
                const long long o = (long long)j * ld + e;
                xv = fma(sa[j], V[o], xv);
                hv = fma(sa[j], HV[o], hv);
                nv = fma(sa[j], NV[o], nv);
            }
        }
        red[0][jg][el] = xv;
        red[1][jg][el] = hv;
        red[2][jg][el] = nv;
    }
    __syncthreads();
    if (jg == 0) {
        double tv = 0.0, xx = 0.0, uu = 0.0, xn = 0.0;
        if (e < n) {
            const double xv = (red[0][0][el] + red[0][1][el]) + (red[0][2][el] + red[0][3][el]);
            const double hv = (red[1][0][el] + red[1][1][el]) + (red[1][2][el] + red[1][3][el]);
            const double nv = (red[2][0][el] + red[2][1][el]) + (red[2][2][el] + red[2][3][el]);
            const double u = hv - theta * nv;
            double den = dh[e] - theta * dn[e];
            if (fabs(den) < floor_) den = (den < 0.0) ? -floor_ : floor_;
            tv = -u / den;
            x[e] = xv;
            t[e] = tv;
            xx = xv * xv;
            uu = u * u;
            xn = xv * nv;
        }
        ts[el] = tv;
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
        xx = wave_sum(xx);
        uu = wave_sum(uu);
        xn = wave_sum(xn);
        if (lane == 0) {
            wsum[wave][0] = xx;
            wsum[wave][1] = uu;
            wsum[wave][2] = xn;
        }
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        const int c = threadIdx.x;
        part_x[3 * chunk + c] = (wsum[0][c] + wsum[1][c]) + (wsum[2][c] + wsum[3][c]);
    }
    chunk_dots<kDavWaves>(V, ld, m, e0, n, ts, part_c + (long long)chunk * m);
}

__device__ inline void dav_cgs_body(const double* __restrict__ V, long long ld, int m,
                                                        int m_dot, const double* __restrict__ part_in, int nchunk,
                                                        double* __restrict__ t, int n,
                                                        double* __restrict__ part_out, int mode, int chunk) {
    __shared__ double c[kDavMaxVec];
    __shared__ double wred[kDavWaves][64];
    __shared__ double red[kDavGroups][kDavChunk];
    __shared__ double ts[kDavChunk];
    __shared__ double wsum[4];
    reduce_partials<kDavWaves>(part_in, nchunk, m, m, wred, c);
    const int el = threadIdx.x & (kDavChunk - 1), jg = threadIdx.x / kDavChunk;
    const int e0 = chunk * kDavChunk;
    const int e = e0 + el;
    {
        double s = 0.0;
        if (e < n) {
            int j0, j1;
            group_range(m, jg, j0, j1);
            int j = j0;
            for (; j + kBatch <= j1; j += kBatch) {
                double w[kBatch];
#pragma unroll
                for (int u = 0; u < kBatch; ++u) w[u] = V[(long long)(j + u) * ld + e];
#pragma unroll
                for (int u = 0; u < kBatch; ++u) s = fma(c[j + u], w[u], s);
            }
            for (; j < j1; ++j) s = fma(c[j], V[(long long)j * ld + e], s);
        }
        red[jg][el] = s;
    }
    __syncthreads();
    double v = 0.0;
    if (jg == 0) {
        if (e < n) {
            v = t[e] - ((red[0][el] + red[1][el]) + (red[2][el] + red[3][el]));
            t[e] = v;
        }
        ts[el] = v;
    }
    if (mode == 0) {
        __syncthreads();
        chunk_dots<kDavWaves>(V, ld, m_dot, e0, n, ts, part_out + (long long)chunk * m_dot);
    } else {
        // norm partial (the first four waves hold the chunk)
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
        double ss = wave_sum(v * v);
        if (jg == 0 && lane == 0) wsum[wave] = ss;
        __syncthreads();
        if (threadIdx.x == 0) part_out[chunk] = (wsum[0] + wsum[1]) + (wsum[2] + wsum[3]);
    }
}

__global__ __launch_bounds__(kThreads) void k_dav_normalize(const double* __restrict__ part, int nchunk,
                                                              const double* __restrict__ t,
                                                              double* __restrict__ vout, int n,
                                                              double* __restrict__ tnorm) {
    __shared__ double wred[4][64];
    __shared__ double tot[1];
    reduce_partials<4>(part, nchunk, 1, 1, wred, tot);
    const double nrm = sqrt(tot[0]);
    const double inv = nrm > 0.0 ? 1.0 / nrm : 0.0;
    const int e = blockIdx.x * kDavChunk + threadIdx.x;
    if (e < n) vout[e] = t[e] * inv;
    if (blockIdx.x == 0 && threadIdx.x == 0) *tnorm = nrm;
}

// Gram rows of the new vector m.  With t != nullptr the new vector is
// t / |t| (|t|^2 = the sum of the nchunk partials pn, written to *tnorm): the
// work-groups with blockIdx.y == 0 store it as V_m, and H_eff t, N_eff t are
// scaled by 1/|t| the same way (H_eff is linear).  With ypart != nullptr
// H_eff t and N_eff t are the sums over the G quadrature partials (ascending
// g) and stored, scaled, in HV_m, NV_m; else (t must then be nullptr) they
// are read from HV_m, NV_m as they are.
__device__ inline void dav_gram_body(double* __restrict__ V, double* __restrict__ HV,
                                                         double* __restrict__ NV, long long ld, int m, int n,
                                                         const double* __restrict__ t,
                                                         const double* __restrict__ pn, int npn,
                                                         double* __restrict__ tnorm,
                                                         const double* __restrict__ ypart,
                                                         const double* __restrict__ nypart, long long gstride, int G, int Gn,
                                                         double* __restrict__ part, int chunk, int grp) {
    __shared__ double vs[kDavChunk], hs[kDavChunk], ns[kDavChunk];
    __shared__ double wred[4][64];
    __shared__ double tot[1];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int nd = 4 * m + 2;
    const int e0 = chunk * kDavChunk;
    const int e = e0 + threadIdx.x;
    const int nval = min(kDavChunk, n - e0);
    double inv = 1.0;
    if (t) {
        reduce_partials<4>(pn, npn, 1, 1, wred, tot);
        const double nrm = sqrt(tot[0]);
        inv = nrm > 0.0 ? 1.0 / nrm : 0.0;
        if (chunk == 0 && grp == 0 && threadIdx.x == 0) *tnorm = nrm;
    }
    double vm = 0.0, hm = 0.0, nm = 0.0;
    if (e < n) {
        const long long o = (long long)m * ld + e;
        vm = t ? t[e] * inv : V[o];
        if (ypart) {
            hm = sum_slots<8>(ypart, gstride, G, e);
            nm = sum_slots<8>(nypart, gstride, Gn, e);
        } else {
            hm = HV[o];
            nm = NV[o];
        }
        hm *= inv;
        nm *= inv;
    }
    vs[threadIdx.x] = vm;
    hs[threadIdx.x] = hm;
    ns[threadIdx.x] = nm;
    __syncthreads();
    // every work-group has read what it needs of HV_m, NV_m (only its own
    // chunk, by its own threads) before the y == 0 groups overwrite them
    if (grp == 0 && e < n && ypart) {
        const long long o = (long long)m * ld + e;
        if (t) V[o] = vm;
        HV[o] = hm;
        NV[o] = nm;
    }
    double* out = part + (long long)chunk * nd;
    const int d0 = grp * kGramGroup;
    const int d1 = min(nd, d0 + kGramGroup);
    // d <= m: V_d.HV_m; then V_j.NV_m (j <= m); HV_j.V_m (j < m); NV_j.V_m (j < m).
    // V_m itself is taken from LDS (it may be being stored right now).
    for (int d = d0 + wave; d < d1; d += 16) {
        double acc[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            acc[u] = 0.0;
            const int dd = d + 4 * u;
            if (dd < d1) {
                int row;
                const double* __restrict__ base;
                const double* w;
                if (dd <= m) {
                    row = dd;
                    base = V;
                    w = hs;
                } else if (dd <= 2 * m + 1) {
                    row = dd - m - 1;
                    base = V;
                    w = ns;
                } else if (dd <= 3 * m + 1) {
                    row = dd - 2 * m - 2;
                    base = HV;
                    w = vs;
                } else {
                    row = dd - 3 * m - 2;
                    base = NV;
                    w = vs;
                }
                if (row == m) {  // V_m . (HV_m or NV_m), both in LDS
#pragma unroll
                    for (int q = 0; q < 4; ++q) acc[u] = fma(vs[lane + 64 * q], w[lane + 64 * q], acc[u]);
                } else {
                    const double* __restrict__ src = base + (long long)row * ld + e0;
                    double v[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) v[q] = (lane + 64 * q < nval) ? src[lane + 64 * q] : 0.0;
#pragma unroll
                    for (int q = 0; q < 4; ++q) acc[u] = fma(v[q], w[lane + 64 * q], acc[u]);
                }
            }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const double r = wave_sum(acc[u]);
            if (lane == 0 && d + 4 * u < d1) out[d + 4 * u] = r;
        }
    }
}

__global__ __launch_bounds__(kDavWide) void k_dav_ritz(const double* __restrict__ V, const double* __restrict__ HV,
                                                         const double* __restrict__ NV, long long ld, int m,
                                                         const double* __restrict__ aq,
                                                         const double* __restrict__ dh,
                                                         const double* __restrict__ dn, int n, double floor_,
                                                         double* __restrict__ x, double* __restrict__ t,
                                                         double* __restrict__ part_x, double* __restrict__ part_c) {
    dav_ritz_body(V, HV, NV, ld, m, aq, dh, dn, n, floor_, x, t, part_x, part_c, blockIdx.x);
}

__global__ __launch_bounds__(kDavWide) void k_dav_cgs(const double* __restrict__ V, long long ld, int m,
                                                        int m_dot, const double* __restrict__ part_in, int nchunk,
                                                        double* __restrict__ t, int n,
                                                        double* __restrict__ part_out, int mode) {
    dav_cgs_body(V, ld, m, m_dot, part_in, nchunk, t, n, part_out, mode, blockIdx.x);
}

__global__ __launch_bounds__(kThreads) void k_dav_gram(double* __restrict__ V, double* __restrict__ HV,
                                                         double* __restrict__ NV, long long ld, int m, int n,
                                                         const double* __restrict__ t,
                                                         const double* __restrict__ pn, int npn,
                                                         double* __restrict__ tnorm,
                                                         const double* __restrict__ ypart,
                                                         const double* __restrict__ nypart, long long gstride, int G, int Gn,
                                                         double* __restrict__ part) {
    dav_gram_body(V, HV, NV, ld, m, n, t, pn, npn, tnorm, ypart, nypart, gstride, G, Gn, part, blockIdx.x, blockIdx.y);
}

// batched passes: blockIdx.y (blockIdx.z for the Gram pass) is the instance;
// work-groups past an instance's chunk or dot count, or of an inactive
// instance, exit at once
__global__ __launch_bounds__(kDavWide) void k_bdav_ritz(const DavInst* __restrict__ insts) {
    const DavInst I = insts[blockIdx.y];
    if (!I.active || (int)blockIdx.x >= dav_chunks(I.n)) return;
    dav_ritz_body(I.V, I.HV, I.NV, I.ld, I.mr, I.aq, I.dh, I.dn, I.n, I.floor_, I.x, I.t, I.part_x, I.pc1, blockIdx.x);
}

__global__ __launch_bounds__(kDavWide) void k_bdav_cgs(const DavInst* __restrict__ insts, int mode) {
    const DavInst I = insts[blockIdx.y];
    if (!I.active || !I.ext || (int)blockIdx.x >= dav_chunks(I.n)) return;
    const int nch = dav_chunks(I.n);
    if (mode == 0) dav_cgs_body(I.V, I.ld, I.m, I.m, I.pc1, nch, I.t, I.n, I.pc2, 0, blockIdx.x);
    else if (mode == 1) dav_cgs_body(I.V, I.ld, I.m, 0, I.pc2, nch, I.t, I.n, I.pn, 1, blockIdx.x);
    else if (I.restart) dav_cgs_body(I.V, I.ld, 0, I.m, I.pc2, nch, I.t, I.n, I.pc1, 0, blockIdx.x);
}

__global__ __launch_bounds__(kThreads) void k_bdav_gram(const DavInst* __restrict__ insts) {
    const DavInst I = insts[blockIdx.z];
    const int nd = 4 * I.m + 2;
    if (!I.active || !I.ext || (int)blockIdx.x >= dav_chunks(I.n) || (int)blockIdx.y * kGramGroup >= nd) return;
    dav_gram_body(I.V, I.HV, I.NV, I.ld, I.m, I.n, I.from_t ? I.t : nullptr, I.pn, dav_chunks(I.n), I.tnorm,
                  I.ypart, I.nypart, I.gstride, I.G, I.Gn, I.pg, blockIdx.x, blockIdx.y);
}

inline int nblk(int n) { return (n + kThreads - 1) / kThreads; }

}  // namespace

void to_f32(hipStream_t s, const double* in, float* out, long long n) {
    if (n > 0)
        hipLaunchKernelGGL(k_to_f32, dim3((unsigned)((n + kThreads - 1) / kThreads)), dim3(kThreads), 0, s, in, out, n);
}
void gsum2(hipStream_t s, const double* pa, const double* pb, long long stride, int Ga, int Gb, int n, double* outa,
           double* outb) {
    hipLaunchKernelGGL(k_gsum2, dim3((n + 63) / 64, 2), dim3(kThreads), 0, s, pa, pb, stride, Ga, Gb, n, outa, outb);
}
void bgemm(hipStream_t s, const BTask* tasks, int ntasks, const BTerm* terms, BufSet bufs,
           const double* coef) {
    if (ntasks > 0) hipLaunchKernelGGL(k_bgemm, dim3(ntasks), dim3(kThreads), 0, s, tasks, terms, bufs, coef);
}
void combine(hipStream_t s, const CTask* tasks, int ntasks, const CTerm* terms, BufSet bufs,
             const double* coef) {
    if (ntasks > 0) hipLaunchKernelGGL(k_combine, dim3(ntasks), dim3(kThreads), 0, s, tasks, terms, bufs, coef);
}
void diag_gather(hipStream_t s, const DiagSide& left, const DiagSide& right, int G) {
    const int n = std::max(left.nz * left.D, right.nz * right.D);
    if (n > 0) hipLaunchKernelGGL(k_diag_gather, dim3(nblk(n), G, 2), dim3(kThreads), 0, s, left, right);
}
void diag_mix(hipStream_t s, const DiagMix* mix, int nmix, const DiagMixTerm* terms, const double* Ld, int nzl, int Dl,
              const double* coef, int ncoef, int G, double* M) {
    if (nmix > 0)
        hipLaunchKernelGGL(k_diag_mix, dim3(nmix, G), dim3(std::min(kThreads, (Dl + 63) / 64 * 64)), 0, s, mix, terms, Ld,
                           nzl, Dl, coef, ncoef, nmix, M);
}
void diag_blocks(hipStream_t s, const DiagBlk* blks, int nb, const int* zlist, const double* M, int nmix, int Dl,
                 const double* Rd, int nzr, int Dr, int G, double* dh, double* dn, int nsplit, double* part,
                 long long ntot) {
    if (nb <= 0) return;
    if (nsplit < 1 || (nsplit > 1 && !part)) nsplit = 1;
    hipLaunchKernelGGL(k_diag, dim3(nb, nsplit), dim3(kThreads), 0, s, blks, zlist, M, nmix, Dl, Rd, nzr, Dr, G, dh, dn,
                       part, ntot);
    if (nsplit > 1)
        hipLaunchKernelGGL(k_diag_sum, dim3((unsigned)((ntot + kThreads - 1) / kThreads)), dim3(kThreads), 0, s, part,
                           nsplit, ntot, dh);
}
void diag_direct(hipStream_t s, const DiagBlk* blks, int nb, const DiagTerm* terms, const double* lenv, long long lsize,
                 const double* renv, long long rsize, const double* coef, int ncoef, int G, double* dh, double* dn) {
    if (nb > 0)
        hipLaunchKernelGGL(k_diag_direct, dim3(nb), dim3(kThreads), 0, s, blks, terms, lenv, lsize, renv, rsize, coef, ncoef,
                           G, dh, dn);
}
void qr_sectors(hipStream_t s, const QrTask* tasks, int ntasks, const QrPiece* pieces, double* site,
                double* scratch, double* rout, const QrShape& shape) {
    if (ntasks <= 0) return;
    if (shape.cols <= kQrRegCols && shape.rows <= kQrRegRows) {
        const dim3 wg(64 * ((shape.cols + 3) / 4));
        const size_t lds = size_t(shape.area) * sizeof(double);
        if (shape.rows <= 64)
            hipLaunchKernelGGL(k_qr_reg<4>, dim3(ntasks), wg, lds, s, tasks, pieces, site, rout);
        else if (shape.rows <= 128)
            hipLaunchKernelGGL(k_qr_reg<8>, dim3(ntasks), wg, lds, s, tasks, pieces, site, rout);
        else
            hipLaunchKernelGGL(k_qr_reg<16>, dim3(ntasks), wg, lds, s, tasks, pieces, site, rout);
    } else if (shape.lds <= kQrLdsMax) {
        hipLaunchKernelGGL(k_qr_lds, dim3(ntasks), dim3(kThreads), size_t(shape.lds) * sizeof(double), s, tasks,
                           pieces, site, rout);
    } else {
        hipLaunchKernelGGL(k_qr, dim3(ntasks), dim3(kThreads), 0, s, tasks, pieces, site, scratch, rout);
    }
}
void fill(hipStream_t s, double* p, long long n, double value) {
    if (n <= 0) return;
    const long long nb = std::min<long long>((n + kThreads - 1) / kThreads, 4096);
    hipLaunchKernelGGL(k_fill, dim3(unsigned(nb)), dim3(kThreads), 0, s, p, n, value);
}
void normalize(hipStream_t s, const double* in, double* out, int n, double* norm_out) {
    hipLaunchKernelGGL(k_normalize, dim3(1), dim3(1024), 0, s, in, out, n, norm_out);
}
void multidot(hipStream_t s, const double* A, long long ld, int m, const double* u, int n, double* out) {
    if (m > 0) hipLaunchKernelGGL(k_multidot, dim3(m), dim3(kThreads), 0, s, A, ld, u, n, out);
}
void basis_rotate(hipStream_t s, const double* A, long long ld, int m, const double* Q, int keep,
                  double* out, int n) {
    hipLaunchKernelGGL(k_basis_rotate, dim3(nblk(n)), dim3(kThreads), 0, s, A, ld, m, Q, keep, out, n);
}
void dav_ritz(hipStream_t s, const double* V, const double* HV, const double* NV, long long ld, int m,
              const double* aq, const double* dh, const double* dn, int n, double floor_, double* x, double* t,
              double* part_x, double* part_c) {
    hipLaunchKernelGGL(k_dav_ritz, dim3(dav_chunks(n)), dim3(kDavWide), 0, s, V, HV, NV, ld, m, aq, dh, dn, n, floor_,
                       x, t, part_x, part_c);
}
void dav_cgs(hipStream_t s, const double* V, long long ld, int m_sub, int m_dot, const double* part_in,
             int nchunk, double* t, int n, double* part_out, int mode) {
    hipLaunchKernelGGL(k_dav_cgs, dim3(dav_chunks(n)), dim3(kDavWide), 0, s, V, ld, m_sub, m_dot, part_in, nchunk, t,
                       n, part_out, mode);
}
void dav_normalize(hipStream_t s, const double* part, int nchunk, const double* t, double* vout, int n,
                   double* tnorm) {
    hipLaunchKernelGGL(k_dav_normalize, dim3(dav_chunks(n)), dim3(kThreads), 0, s, part, nchunk, t, vout, n, tnorm);
}
void dav_gram(hipStream_t s, double* V, double* HV, double* NV, long long ld, int m, int n, const double* t,
              const double* pn, int npn, double* tnorm, const double* ypart, const double* nypart, long long gstride,
              int G, int Gn, double* part) {
    const int nd = 4 * m + 2;
    hipLaunchKernelGGL(k_dav_gram, dim3(dav_chunks(n), (nd + kGramGroup - 1) / kGramGroup), dim3(kThreads), 0, s, V, HV,
                       NV, ld, m, n, t, pn, npn, tnorm, ypart, nypart, gstride, G, Gn, part);
}

void bdav_ritz(hipStream_t s, const DavInst* insts, int ninst, int max_n) {
    if (ninst > 0) hipLaunchKernelGGL(k_bdav_ritz, dim3(dav_chunks(max_n), ninst), dim3(kDavWide), 0, s, insts);
}
void bdav_cgs(hipStream_t s, const DavInst* insts, int ninst, int max_n, int mode) {
    if (ninst > 0) hipLaunchKernelGGL(k_bdav_cgs, dim3(dav_chunks(max_n), ninst), dim3(kDavWide), 0, s, insts, mode);
}
void bdav_gram(hipStream_t s, const DavInst* insts, int ninst, int max_n, int max_m) {
    const int nd = 4 * max_m + 2;
    if (ninst > 0)
        hipLaunchKernelGGL(k_bdav_gram, dim3(dav_chunks(max_n), (nd + kGramGroup - 1) / kGramGroup, ninst),
                           dim3(kThreads), 0, s, insts);
}

}  // namespace spk
