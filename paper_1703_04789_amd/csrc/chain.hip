// Chained block products for gfx950: every contraction of the tiled path --
// H_eff x and N_eff x (Eq. [geproblem]) and the environment updates (Fig.
// [spmpsOpt]) -- is a sum of outputs
//     O(m x n) += P(m x kc) [ sum over segments coef A(kc x kj) B(kj x n) ]
// over steps (P, a range of kc, its segments).  The inner product I stays in
// registers: a matrix-core result holds, in lane l, rows that depend on l / 16
// and the column l % 16, which is exactly what the second operand of the next
// product takes, so I is never written to memory.
//   H_eff x (transposed): m = columns of the output block, n = its rows,
//     P = R(c') rows, A = the rotated site vector, B = L(c) or the left
//     environment with the MPO mixed in
//   left environment:  P = the bra tensor, A = L(c), B = the rotated ket tensor
//   right environment: P = the bra tensor, A = R(c'), B = the rotated ket tensor
// One work-group of four wavefronts per output tile; the steps of a tile are
// dealt to the wavefronts, whose sums are added through LDS in a fixed order.
// What bounds it: at narrow MPOs the latency of a wavefront's chain of loads
// (matrix cores 22 % busy at the L = 32, D = 256, G = 9 Hubbard centre); at
// wide ones the reads from the L2 (12.5 TB/s at the K = 12, D = 128, G = 11
// ab-initio centre, the matrix cores 41 % busy there, three fifths of that on
// padding).  The next chunk's loads are issued before the current chunk's
// products; deeper prefetch and tiles of 48 x 48 were slower (registers, so
// fewer wavefronts).  Calls of H_eff x and N_eff x, before (FP64 FMAs through
// LDS; block products with intermediates in memory) and now: Hubbard L = 32,
// D = 256 45 -> 24 us, L = 48, D = 512 145 -> 63, ab-initio K = 12, D = 128
// 497 -> 224; an environment update at L = 32, D = 256 (four launches of block
// products before) 75 -> 28 us.
#include "kernels.h"

#include <type_traits>

namespace spk {

namespace {

typedef double d4_t __attribute__((ext_vector_type(4)));
typedef float f4_t __attribute__((ext_vector_type(4)));
typedef short s4_t __attribute__((ext_vector_type(4)));
typedef double d2u_t __attribute__((ext_vector_type(2), aligned(8)));
typedef float f4u_t __attribute__((ext_vector_type(4), aligned(4)));

typedef __bf16 bf4_t __attribute__((ext_vector_type(4)));
// v ~ hi + lo, both bf16 rounded to nearest even, off by at most 2^-17 of v.
// The residue of an FP64 value is formed in FP64: what FP32 drops of v can
// decide how it rounds
template <class V>
__device__ inline void split_bf16(const V* v, s4_t& hi, s4_t& lo) {
    f4_t f, r;
#pragma unroll
    for (int t = 0; t < 4; ++t) f[t] = float(v[t]);
    const bf4_t h = __builtin_convertvector(f, bf4_t);
    const f4_t hf = __builtin_convertvector(h, f4_t);
#pragma unroll
    for (int t = 0; t < 4; ++t) r[t] = float(v[t] - V(hf[t]));
    const bf4_t l = __builtin_convertvector(r, bf4_t);
    hi = __builtin_bit_cast(s4_t, h);
    lo = __builtin_bit_cast(s4_t, l);
}

// the value at element i from a tile's first: a uniform base and a 32-bit
// byte offset per lane
template <class E>
__device__ inline E at(const E* __restrict__ p, unsigned i) {
    return *reinterpret_cast<const E*>(reinterpret_cast<const char*>(p) + unsigned(sizeof(E)) * i);
}
template <int N>
__device__ inline void read_run(const double* __restrict__ p, unsigned i, double (&v)[N]) {
#pragma unroll
    for (int t = 0; t < N; t += 2) {
        const d2u_t w = *reinterpret_cast<const d2u_t*>(reinterpret_cast<const char*>(p + t) + 8u * i);
        v[t] = w.x;
        v[t + 1] = w.y;
    }
}
template <int N>
__device__ inline void read_run(const float* __restrict__ p, unsigned i, float (&v)[N]) {
    static_assert(N == 4, "a run of four FP32 values");
    const f4u_t w = *reinterpret_cast<const f4u_t*>(reinterpret_cast<const char*>(p) + 4u * i);
    v[0] = w.x;
    v[1] = w.y;
    v[2] = w.z;
    v[3] = w.w;
}

// one chunk of an inner product in a lane: KL consecutive kj values of row
// (column) l % 16 of every block of A (B); the segment's coefficient, the kj
// values left in the segment, whether the chunk ends the step
template <class E, int NI, int NN, int KL>
struct Frag {
    E a[NI][KL], b[NN][KL];
    E cf;
    int nk;
    bool last;
};

// MODE kChainF64: FP64 on v_mfma_f64_16x16x4; kChainF32: FP32 operands on
// v_mfma_f32_16x16x4; kChainBF3: FP64 operands split into bf16 hi + lo, three
// v_mfma_f32_16x16x16_bf16 per step (lo lo dropped), FP32 accumulation.
// NM, NN: blocks of 16 of the output tile in m and n; NI: blocks of 16 kc
// values formed at once.
// Lane l holds kj = KL (l / 16) + t of a chunk in either operand (any
// assignment of k values to lanes and steps gives the same products as long as
// both operands share it).  Rows past an extent re-read its last one, kj and
// kc values past a range are read from what follows (the buffers end in
// read_pad values) and set to zero in both operands.
// Wavefronts per SIMD: as many as the registers of a tile leave without spills.
constexpr int chain_waves_per_simd(int lay, int nm) {
    return lay == kChainHeff ? (nm <= 4 ? 3 : 2) : (nm == 2 ? 5 : nm == 3 ? 4 : nm <= 6 ? 3 : 2);
}
template <int MODE, int LAY, int NM, int NI, int NN, int W, bool BATCH>
__global__ __launch_bounds__(64 * W, chain_waves_per_simd(LAY, NM)) void k_chain(const KInst* __restrict__ insts, KInst one) {
    typedef typename std::conditional<MODE == kChainF32, float, double>::type E;         // operands
    typedef typename std::conditional<MODE == kChainF64, d4_t, f4_t>::type A4;           // accumulators
    typedef typename std::conditional<MODE == kChainF64, double, float>::type AE;
    // sums over steps in the FP32 mode are FP64: a step's part is added to them
    typedef typename std::conditional<MODE == kChainBF3, float, double>::type SE;
    constexpr bool kFold = MODE == kChainF32;
    constexpr int KL = MODE == kChainF64 ? 2 : 4, KC = 4 * KL, NE = NM * NN * 4;
    typedef Frag<E, NI, NN, KL> F;
    // the sums of the wavefronts, and that of N_eff x
    __shared__ SE red[W + (LAY == kChainHeff ? 1 : 0)][W == 1 ? 1 : NE][64];
    const KInst& I = BATCH ? insts[blockIdx.y] : one;
    if (I.gate && *I.gate == 0) return;
    // work-group w runs on XCD w mod 8: contiguous runs of the g-major list of
    // tiles per XCD, so that its L2 holds the environments of a few g
    const int T = I.ntile * I.G, per = (T + 7) / 8, pos = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
    if (int(blockIdx.x >> 3) >= per || pos >= T) return;
    const int g = pos / I.ntile;
    const KTile* __restrict__ tp = I.tiles + (pos - g * I.ntile);
    const KTile& tk = *tp;
    const double* __restrict__ coef = I.coef + (long long)g * I.nc;
    const int lane = threadIdx.x % 64, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    const int li = lane % 16, lk = lane / 16;
    // row of A that lane li supplies: FP64 results hold row 4 v + l / 16 in
    // element v, so block row p carries kc = 4 (p mod 4) + p / 4 and a lane's
    // four values of I are consecutive kc, as P is read
    const int ai = MODE == kChainF64 ? 4 * (li % 4) + li / 4 : li;
    int pm[NM], bn[NN];
#pragma unroll
    for (int i = 0; i < NM; ++i) pm[i] = min(16 * i + li, tk.m - 1);
#pragma unroll
    for (int i = 0; i < NN; ++i) bn[i] = min(16 * i + li, tk.n - 1);
    const int nm = (tk.m + 15) / 16;
    A4 acc[NM][NN], in[NI][NN];
    d4_t sum64[kFold ? NM : 1][kFold ? NN : 1];
#pragma unroll
    for (int i = 0; i < NM; ++i)
#pragma unroll
        for (int j = 0; j < NN; ++j) {
            acc[i][j] = A4{0, 0, 0, 0};
            if constexpr (kFold) sum64[i][j] = d4_t{0, 0, 0, 0};
        }
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < NN; ++j) in[i][j] = A4{0, 0, 0, 0};

    // the chunks of this wavefront's steps as one sequence: every step holds
    // a segment and every segment a kj value (checked with the lists)
    const bool metric = LAY == kChainHeff && wave == W - 1 && tk.e1 > tk.e0;
    const int y0 = tk.s[wave], y1 = tk.s[wave + 1];
    int st = metric ? tk.e0 : y0, s1 = metric ? tk.e1 : y1;
    auto base = [&](int b) { return static_cast<const E*>(I.in[b].p) + g * I.in[b].gs; };
    const E* __restrict__ x0 = base(K_X);
    const E* __restrict__ x1 = base(K_XR);
    const E* __restrict__ e0 = base(LAY == kChainEnvR ? K_R : K_L);
    const E* __restrict__ e1 = base(K_LT);
    const E* __restrict__ pb = LAY == kChainHeff ? base(K_R) : x0;
    KStep fs{};
    KSeg sg{};
    int s = 0, kb = 0;
    if (st < s1) {
        fs = I.steps[st];
        s = fs.g0;
        sg = I.segs[s];
    }
    auto fetch = [&](F& f) {
        f.cf = E(sg.cf);
        f.nk = sg.nk - kb;
        const E* __restrict__ X = sg.alt_x ? x1 : x0;
        const E* __restrict__ V = sg.alt_e ? e1 : e0;
        const E* __restrict__ A = (LAY == kChainHeff ? X : V) + sg.a_off;
        const E* __restrict__ B = (LAY == kChainHeff ? V : X) + sg.b_off;
        if constexpr (LAY == kChainHeff) {  // A(kc, kj) at kj * lda + kc
            A += (long long)kb * sg.lda;
#pragma unroll
            for (int t = 0; t < KL; ++t) {
#pragma unroll
                for (int i = 0; i < NI; ++i) {
                    const int r = 16 * i + min(ai, fs.nkc - 1 - 16 * i);
                    f.a[i][t] = at(A, unsigned(KL * lk * sg.lda + r));
                }
                A += sg.lda;
            }
        } else {  // A(kc, kj) at kc * lda + kj
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                const int r = 16 * i + min(ai, fs.nkc - 1 - 16 * i);
                read_run(A + kb, unsigned(r * sg.lda + KL * lk), f.a[i]);
            }
        }
        if constexpr (LAY == kChainEnvL) {  // B(kj, n) at kj * ldb + n
            B += (long long)kb * sg.ldb;
#pragma unroll
            for (int t = 0; t < KL; ++t) {
#pragma unroll
                for (int j = 0; j < NN; ++j) f.b[j][t] = at(B, unsigned(KL * lk * sg.ldb + bn[j]));
                B += sg.ldb;
            }
        } else {  // B(kj, n) at n * ldb + kj
#pragma unroll
            for (int j = 0; j < NN; ++j) read_run(B + kb, unsigned(bn[j] * sg.ldb + KL * lk), f.b[j]);
        }
        kb += KC;
        f.last = false;
        if (kb >= sg.nk) {
            ++s;
            if (s >= fs.g1) {
                f.last = true;
                ++st;
                if (st < s1) {
                    fs = I.steps[st];
                    s = fs.g0;
                }
            }
            if (st < s1) sg = I.segs[s];
            kb = 0;
        }
    };
    KStep cs{};  // the step whose inner product is being formed
    int cst = st;
    if (cst < s1) cs = fs;
    auto products = [&](F& f) {
        if (f.nk < KC) {
#pragma unroll
            for (int t = 0; t < KL; ++t) {
                const bool on = KL * lk + t < f.nk;
#pragma unroll
                for (int i = 0; i < NI; ++i) f.a[i][t] = on ? f.a[i][t] : E(0);
#pragma unroll
                for (int j = 0; j < NN; ++j) f.b[j][t] = on ? f.b[j][t] : E(0);
            }
        }
#pragma unroll
        for (int j = 0; j < NN; ++j)
#pragma unroll
            for (int t = 0; t < KL; ++t) f.b[j][t] *= f.cf;
        const int ni = (cs.nkc + 15) / 16;
        if constexpr (MODE == kChainBF3) {
            s4_t bh[NN], bl[NN];
#pragma unroll
            for (int j = 0; j < NN; ++j) split_bf16(f.b[j], bh[j], bl[j]);
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                if (i >= ni) break;
                s4_t ah, al;
                split_bf16(f.a[i], ah, al);
#pragma unroll
                for (int j = 0; j < NN; ++j) {
                    in[i][j] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(al, bh[j], in[i][j], 0, 0, 0);
                    in[i][j] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(ah, bl[j], in[i][j], 0, 0, 0);
                    in[i][j] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(ah, bh[j], in[i][j], 0, 0, 0);
                }
            }
        } else {
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                if (i >= ni) break;
#pragma unroll
                for (int t = 0; t < KL; ++t)
#pragma unroll
                    for (int j = 0; j < NN; ++j) {
                        if constexpr (MODE == kChainF64)
                            in[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(f.a[i][t], f.b[j][t], in[i][j], 0, 0, 0);
                        else
                            in[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(f.a[i][t], f.b[j][t], in[i][j], 0, 0, 0);
                    }
            }
        }
        if (!f.last) return;
        // O += P I, 16 kc values at a time
        const E* __restrict__ P = pb + cs.p_off;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            if (i >= ni) break;
            const int k0 = 16 * i;
            E p[NM][4];
            if constexpr (LAY == kChainEnvL) {  // P(m, kc) at kc * ldp + m
                const E* __restrict__ q = P + (long long)k0 * cs.ldp;
#pragma unroll
                for (int v = 0; v < 4; ++v) {
#pragma unroll
                    for (int a = 0; a < NM; ++a) p[a][v] = at(q, unsigned(4 * lk * cs.ldp + pm[a]));
                    q += cs.ldp;
                }
            } else {  // P(m, kc) at m * ldp + kc
#pragma unroll
                for (int a = 0; a < NM; ++a) read_run(P + k0, unsigned(pm[a] * cs.ldp + 4 * lk), p[a]);
            }
            if (k0 + 16 > cs.nkc) {
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const bool on = k0 + 4 * lk + v < cs.nkc;
#pragma unroll
                    for (int a = 0; a < NM; ++a) p[a][v] = on ? p[a][v] : E(0);
#pragma unroll
                    for (int j = 0; j < NN; ++j) in[i][j][v] = on ? in[i][j][v] : AE(0);
                }
            }
            if constexpr (MODE == kChainBF3) {
                s4_t ih[NN], il[NN];
#pragma unroll
                for (int j = 0; j < NN; ++j) {
                    float v[4] = {in[i][j][0], in[i][j][1], in[i][j][2], in[i][j][3]};
                    split_bf16(v, ih[j], il[j]);
                }
#pragma unroll
                for (int a = 0; a < NM; ++a) {
                    if (a >= nm) break;
                    s4_t ph, pl;
                    split_bf16(p[a], ph, pl);
#pragma unroll
                    for (int j = 0; j < NN; ++j) {
                        acc[a][j] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(pl, ih[j], acc[a][j], 0, 0, 0);
                        acc[a][j] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(ph, il[j], acc[a][j], 0, 0, 0);
                        acc[a][j] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(ph, ih[j], acc[a][j], 0, 0, 0);
                    }
                }
            } else {
#pragma unroll
                for (int a = 0; a < NM; ++a) {
                    if (a >= nm) break;
#pragma unroll
                    for (int v = 0; v < 4; ++v)
#pragma unroll
                        for (int j = 0; j < NN; ++j) {
                            if constexpr (MODE == kChainF64)
                                acc[a][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(p[a][v], in[i][j][v], acc[a][j], 0, 0, 0);
                            else
                                acc[a][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(p[a][v], in[i][j][v], acc[a][j], 0, 0, 0);
                        }
                }
            }
#pragma unroll
            for (int j = 0; j < NN; ++j) in[i][j] = A4{0, 0, 0, 0};
        }
        if constexpr (kFold) {
#pragma unroll
            for (int a = 0; a < NM; ++a)
#pragma unroll
                for (int j = 0; j < NN; ++j) {
                    sum64[a][j] += __builtin_convertvector(acc[a][j], d4_t);
                    acc[a][j] = A4{0, 0, 0, 0};
                }
        }
        ++cst;
        if (cst < s1) cs = I.steps[cst];
    };
    auto total = [&](int a, int j, int v) {
        if constexpr (kFold) return sum64[a][j][v];
        else return acc[a][j][v];
    };
    for (int pass = metric ? 0 : 1; pass < 2; ++pass) {
        if (pass == 1 && metric) {  // N_eff x is done: its sum to LDS, then this wavefront's own steps
#pragma unroll
            for (int a = 0; a < NM; ++a)
#pragma unroll
                for (int j = 0; j < NN; ++j) {
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        if constexpr (LAY == kChainHeff) red[W][(a * NN + j) * 4 + v][lane] = total(a, j, v);
                    acc[a][j] = A4{0, 0, 0, 0};
                    if constexpr (kFold) sum64[a][j] = d4_t{0, 0, 0, 0};
                }
            st = cst = y0;
            s1 = y1;
            if (st < s1) {
                cs = fs = I.steps[st];
                s = fs.g0;
                sg = I.segs[s];
                kb = 0;
            }
        }
        if (st >= s1) continue;
        // the loads of the next chunk are issued whether there is one or not
        // (past the end the last segment's first chunk again): behind a branch
        // the wait for the current chunk would have to take them in as well
        F f0, f1;
        fetch(f0);
        for (;;) {
            const bool m1 = st < s1;
            fetch(f1);
            products(f0);
            if (!m1) break;
            const bool m0 = st < s1;
            fetch(f0);
            products(f1);
            if (!m0) break;
        }
    }
    const double scale = tk.cidx < 0 ? 1.0 : coef[tk.cidx];
    double* __restrict__ out = I.out[0] + g * I.ogs + tk.o_off;
    if constexpr (W == 1) {
#pragma unroll
        for (int a = 0; a < NM; ++a)
#pragma unroll
            for (int j = 0; j < NN; ++j)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int m = 16 * a + (MODE == kChainF64 ? 4 * v + lk : 4 * lk + v), n = 16 * j + li;
                    if (m < tk.m && n < tk.n) out[(long long)m * tk.ldo + n] = scale * double(total(a, j, v));
                }
        return;
    } else {
        // the wavefronts' sums in wavefront order
#pragma unroll
        for (int a = 0; a < NM; ++a)
#pragma unroll
            for (int j = 0; j < NN; ++j)
#pragma unroll
                for (int v = 0; v < 4; ++v) red[wave][(a * NN + j) * 4 + v][lane] = total(a, j, v);
        __syncthreads();
        double* __restrict__ out2 = I.out[1] + g * I.ogs;
        const bool both = LAY == kChainHeff && tk.e1 > tk.e0;
        for (int e = wave; e < nm * NN * 4; e += W) {
            const int v = e % 4, j = (e / 4) % NN, a = e / (4 * NN);
            const int m = 16 * a + (MODE == kChainF64 ? 4 * v + lk : 4 * lk + v), n = 16 * j + li;
            if (m >= tk.m || n >= tk.n) continue;
            double sum = red[0][e][lane];
#pragma unroll
            for (int w = 1; w < W; ++w) sum += double(red[w][e][lane]);
            if constexpr (LAY == kChainHeff) {
                const int q = I.map[tk.map_off + (long long)n * tk.ldo + m];
                if (q >= 0) {
                    out[q] = scale * sum;
                    if (both) out2[q] = scale * double(red[W][e][lane]);
                }
            } else {
                out[(long long)m * tk.ldo + n] = scale * sum;
            }
        }
    }
}

// dense particle-number blocks of the site vector (blockIdx.y = 0) and, for
// g = blockIdx.y - 1, the blocks of the two singly occupied states rotated by
// r(beta_g) (Eq. [expSy]; it leaves the other two states alone)
template <class E, bool BATCH>
__global__ __launch_bounds__(256) void k_xprep(const KPrep* __restrict__ insts, KPrep one) {
    const KPrep& I = BATCH ? insts[blockIdx.z] : one;
    if (I.gate && *I.gate == 0) return;
    const long long e = blockIdx.x * 256LL + threadIdx.x;
    if (blockIdx.y == 0) {
        if (e >= I.nd) return;
        const int q = I.map[e];
        static_cast<E*>(I.xd)[e] = q >= 0 ? E(I.x[q]) : E(0);
        return;
    }
    const int g = int(blockIdx.y) - 1;
    if (g >= I.G || e >= I.nr) return;
    const int qa = I.rmap[2 * e], qb = I.rmap[2 * e + 1];
    const double a = qa >= 0 ? I.x[qa] : 0.0, b = qb >= 0 ? I.x[qb] : 0.0;
    const double* __restrict__ r = I.coef + (long long)g * I.nc + I.crot;  // r(s, u) at 4 s + u
    E* __restrict__ out = static_cast<E*>(I.xr) + g * 2 * I.nr;
    out[e] = E(r[4 * 1 + 1] * a + r[4 * 1 + 2] * b);
    out[I.nr + e] = E(r[4 * 2 + 1] * a + r[4 * 2 + 2] * b);
}

template <int MODE, int LAY, int W>
void launch_shape(hipStream_t s, int shape, dim3 grid, const KInst* insts, const KInst& one) {
#define SPK_CHAIN(NM, NN)                                                                                          \
    if (LAY == kChainHeff && insts)                                                                                \
        hipLaunchKernelGGL((k_chain<MODE, LAY, NM, 2, NN, W, LAY == kChainHeff>), grid, dim3(64 * W), 0, s, insts, one); \
    else                                                                                                           \
        hipLaunchKernelGGL((k_chain<MODE, LAY, NM, 2, NN, W, false>), grid, dim3(64 * W), 0, s, insts, one)
    switch (shape) {
        case 0: SPK_CHAIN(2, 1); return;
        case 1: SPK_CHAIN(3, 1); return;
        case 2: SPK_CHAIN(4, 1); return;
        case 3: SPK_CHAIN(6, 1); return;
        case 4: SPK_CHAIN(8, 1); return;
        default: break;
    }
    if constexpr (LAY == kChainHeff) {  // environments use the narrow shapes
        switch (shape) {
            case 5: SPK_CHAIN(2, 2); break;
            case 6: SPK_CHAIN(3, 2); break;
            default: SPK_CHAIN(4, 2); break;
        }
    }
#undef SPK_CHAIN
}

// The pre-mixed environment of one side, blockIdx.y = g.  Wide MPOs sum tens
// of blocks into one and use every block in hundreds of sums, so the sources
// are staged in LDS, and since a sum's sources are set by its channel and
// operator type, whole groups of blocks share them: one LDS read serves up to
// kMixGroup sums (the LDS gives 16 values per clock and CU, the FMAs take 64).
// K = 12, D = 128, site 7, G = 11: 261 us, of which writing the 700 MB of
// mixed blocks takes about 160; a work-group per 64 elements of one block with
// terms read from memory 870, one block at a time from LDS 650.
template <class E>
__global__ __launch_bounds__(kMixThreads) void k_premix(MixLists m, const E* __restrict__ in, long long igs,
                                                        E* __restrict__ out, long long ogs) {
    __shared__ E src[kMixTile][64];
    constexpr int NW = kMixThreads / 64;
    const MixWork* __restrict__ w = m.work + blockIdx.x;
    const int lane = threadIdx.x % 64, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    const bool on = w->e0 + lane < w->n;
    in += blockIdx.y * igs + w->e0 + lane;
    out += blockIdx.y * ogs + w->e0 + lane;
    for (int t = w->tile0; t < w->tile1; ++t) {
        const MixTileRec* __restrict__ tl = m.tiles + t;
        const int s0 = tl->s0, ns = tl->s1 - s0;
#pragma unroll 4
        for (int q = wave; q < ns; q += NW) src[q][lane] = on ? in[m.src[s0 + q]] : E(0);
        __syncthreads();
        for (int i = tl->i0 + wave; i < tl->i1; i += NW) {
            const MixGroup* __restrict__ it = m.groups + i;
            const int t1 = it->t1, n = it->n;
            double acc[kMixGroup];
#pragma unroll
            for (int b = 0; b < kMixGroup; ++b) acc[b] = it->first || b >= n || !on ? 0.0 : double(out[it->o[b]]);
#pragma unroll 4
            for (int q = it->t0; q < t1; ++q) {
                const double v = double(src[m.at[q]][lane]);
                const double* __restrict__ c = m.cf + kMixGroup * (long long)q;
#pragma unroll
                for (int b = 0; b < kMixGroup; ++b) acc[b] = fma(c[b], v, acc[b]);
            }
            if (on)
#pragma unroll
                for (int b = 0; b < kMixGroup; ++b)
                    if (b < n) out[it->o[b]] = E(acc[b]);
        }
        __syncthreads();
    }
}

}  // namespace

const KShape kChainShapes[kNumChainShapes] = {{2, 2, 1}, {3, 2, 1}, {4, 2, 1}, {6, 2, 1}, {8, 2, 1},
                                               {2, 2, 2}, {3, 2, 2}, {4, 2, 2}};

void chain(hipStream_t s, int mode, int lay, int shape, int waves, int max_tiles, int ninst, const KInst* insts,
           const KInst& one) {
    if (max_tiles <= 0 || ninst <= 0) return;
    const dim3 grid((max_tiles + 7) / 8 * 8, ninst);
    if (lay == kChainHeff) {
        if (mode == kChainF64) launch_shape<kChainF64, kChainHeff, kChainWaves>(s, shape, grid, insts, one);
        else if (mode == kChainF32) launch_shape<kChainF32, kChainHeff, kChainWaves>(s, shape, grid, insts, one);
        else launch_shape<kChainBF3, kChainHeff, kChainWaves>(s, shape, grid, insts, one);
    } else if (lay == kChainEnvL) {
        if (waves == 1) launch_shape<kChainF64, kChainEnvL, 1>(s, shape, grid, insts, one);
        else launch_shape<kChainF64, kChainEnvL, kChainWaves>(s, shape, grid, insts, one);
    } else {
        if (waves == 1) launch_shape<kChainF64, kChainEnvR, 1>(s, shape, grid, insts, one);
        else launch_shape<kChainF64, kChainEnvR, kChainWaves>(s, shape, grid, insts, one);
    }
}

void xprep(hipStream_t s, bool f32, long long max_n, int max_G, int ninst, const KPrep* insts, const KPrep& one) {
    if (max_n <= 0 || ninst <= 0) return;
    const dim3 grid(unsigned((max_n + 255) / 256), max_G + 1, ninst);
    if (f32 && insts) hipLaunchKernelGGL((k_xprep<float, true>), grid, dim3(256), 0, s, insts, one);
    else if (f32) hipLaunchKernelGGL((k_xprep<float, false>), grid, dim3(256), 0, s, insts, one);
    else if (insts) hipLaunchKernelGGL((k_xprep<double, true>), grid, dim3(256), 0, s, insts, one);
    else hipLaunchKernelGGL((k_xprep<double, false>), grid, dim3(256), 0, s, insts, one);
}

void premix(hipStream_t s, bool f32, const MixLists& m, const void* in, long long igs, void* out, long long ogs, int G) {
    if (m.nwork <= 0) return;
    const dim3 grid(m.nwork, G), wg(kMixThreads);
    if (f32)
        hipLaunchKernelGGL(k_premix<float>, grid, wg, 0, s, m, static_cast<const float*>(in), igs, static_cast<float*>(out), ogs);
    else
        hipLaunchKernelGGL(k_premix<double>, grid, wg, 0, s, m, static_cast<const double*>(in), igs, static_cast<double*>(out), ogs);
}

}  // namespace spk
