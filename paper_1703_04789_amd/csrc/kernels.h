// Device kernels of the SP-MPS hot path (gfx950) and their launch wrappers.
#pragma once
#include <hip/hip_runtime.h>
#include <cstdint>

namespace spk {

constexpr int kMaxBufs = 10;

// One output block C (M x N, row stride ldc) = sum over terms of
// coef[cidx] * A(M x K) B(K x N); accumulate != 0 adds to C.  A term with
// strides (a_rs, a_cs) reads A(r, k) = bufs[a_buf][a_off + r*a_rs + k*a_cs].
struct BTask {
    long long c_off;
    int c_buf, M, N, ldc;
    int t0, t1, accumulate, pad;
};
struct BTerm {
    long long a_off, b_off;
    int a_buf, b_buf;
    int a_rs, a_cs, b_rs, b_cs;
    int K, cidx;
};
// C[e] = sum_terms coef[cidx] * A[a_off + e], e < n.
struct CTask {
    long long c_off;
    int c_buf, n, t0, t1;
};
struct CTerm {
    long long a_off;
    int a_buf, cidx;
};
struct BufSet {
    double* p[kMaxBufs];
};

// Diagonal of H_eff / N_eff (the spin-diagonal part of the rotated MPO acts on
// the diagonals of the environments alone).  Narrow MPOs sum every term in
// one launch (DiagTerm); wide ones take three:
//   gather  Ld(g, z, p), Rd(g, z, p): the diagonals of the environment
//           blocks of the particle-conserving channels z, state p of the bond
//   mix     M(g, row, p) = sum over terms of coef * Ld(g, z, p)
//   blocks  out(r, c) = sum over g and the block's units of
//           M(g, row, r) Rd(g, z, c): one work-group per tile of at most
//           kDiagTile x kDiagTile elements of an (N, M) block
struct DiagSrc {
    long long off;  // environment block (within one g); ld < 0: no block, zeros
    int ld, pad;
};
// one side of the gather: element (z, p) is env[src[z * nnb + nb[p]].off +
// ro[p] * (ld + 1)], nb/ro the particle-number block of state p and its place
struct DiagSide {
    const DiagSrc* src;
    const int* nb;
    const int* ro;
    const double* env;
    long long esize;  // environment values per g
    double* out;      // nz * D values per g
    int nz, D, nnb, pad;
};
struct DiagMix {
    int t0, t1;  // terms of one row of M
};
struct DiagMixTerm {
    int z, cidx;
};
struct DiagBlk {
    int x_off, ldc;        // element (r, c) of the tile at x_off + r * ldc + c
    int rows, cols;
    int row0, nrow;        // units: M rows row0 .. row0 + nrow
    int p0, q0;            // first state of the tile on the left, right bond
    int zl0;               // Rd channel of unit u: zlist[zl0 + u]
    int is_n;              // 1: N_eff
    int t0, t1;            // one launch: the terms of the tile's (N, M) block
    int r0, c0;            // and the tile's first row and column in it
};
// coef[cidx] L(r, r) R(c, c): the diagonals of an (N, M) block's rows and
// columns, elements ld + 1 apart
struct DiagTerm {
    long long l_off, r_off;
    int l_ld, r_ld, cidx, pad;
};

// QR of one gathered sector matrix: pieces are row-major blocks of a packed
// site tensor; transposed pieces contribute their columns as rows.
struct QrTask {
    long long scratch_off;  // rows*cols doubles of scratch (column-major)
    long long r_off;        // cols*cols output (row-major)
    int rows, cols, p0, p1;
};
struct QrPiece {
    long long off;  // block offset in the site tensor
    int prow, pcol;  // stored block dims (row-major, ld = pcol)
    int transposed, row0;  // row offset in the gathered matrix
};

// outa[e] = sum over Ga slots of pa[slot * stride + e], outb likewise over Gb,
// in a fixed order
void gsum2(hipStream_t s, const double* pa, const double* pb, long long stride, int Ga, int Gb, int n, double* outa,
           double* outb);

// Chained block products (chain.hip): the lists of one launch, the same for
// every quadrature point; a buffer's values of point g start at g * gs.
constexpr int kChainF64 = 0, kChainF32 = 1, kChainBF3 = 2;     // arithmetic
constexpr int kChainHeff = 0, kChainEnvL = 1, kChainEnvR = 2;  // operand layouts
constexpr int kChainWaves = 4;  // wavefronts of a tile, at most
// operand buffers: the environments left and right of the site, the dense
// site tensor, its rotated singly occupied blocks, the pre-mixed environment
enum KBufId { K_L = 0, K_R = 1, K_X = 2, K_XR = 3, K_LT = 4, K_NBUF = 5 };
struct KBuf {
    const void* p;
    long long gs;
};
// Offsets of a tile, a step and a segment are those of their first element
// (first row, column, kc and kj value), 64 bits wide and the same for every
// lane; a lane adds the rows and values of its tile alone, 32 bits of bytes.
// one product of the inner sum: cf A(kc, kj) B(kj, n) over nk values of kj.
// Each operand is one of two buffers: the site tensor's is K_X or (alt_x)
// K_XR, the environment's K_L (right updates: K_R) or (alt_e) K_LT
struct KSeg {
    long long a_off, b_off;
    double cf;
    int lda, ldb, nk, alt_x, alt_e, pad;
};
// nkc values of kc of P (H_eff x: of K_R, environments: of K_X) and the
// segments [g0, g1) of the inner sum
struct KStep {
    long long p_off;
    int ldp, nkc, g0, g1;
};
// output tile of m x n elements, the steps [s[w], s[w + 1]) of wavefront w,
// the sum times coef[cidx] (cidx < 0: 1).  Environments: element (m, n) at
// o_off + m * ldo + n; H_eff x: at o_off + map[map_off + n * ldo + m] where
// that is >= 0, and the steps [e0, e1) of N_eff x (second output, no o_off),
// taken by the last wavefront before its own
struct KTile {
    long long o_off, map_off;
    int m, n, ldo, cidx, s[5], e0, e1, pad;
};
// first elements in blocks at off with rows ld apart: of P from row m0, value
// kc0, of A from kc0, kj0, of B from kj0, column n0, and of an output tile
inline long long chain_p(int lay, long long off, int ld, long long m0, long long kc0) {
    return off + (lay == kChainEnvL ? kc0 * ld + m0 : m0 * ld + kc0);
}
inline long long chain_a(int lay, long long off, int ld, long long kc0, long long kj0) {
    return off + (lay == kChainHeff ? kj0 * ld + kc0 : kc0 * ld + kj0);
}
inline long long chain_b(int lay, long long off, int ld, long long kj0, long long n0) {
    return off + (lay == kChainEnvL ? kj0 * ld + n0 : n0 * ld + kj0);
}
struct KInst {
    const KTile* tiles;
    const KStep* steps;
    const KSeg* segs;
    const int* map;
    const double* coef;
    KBuf in[K_NBUF];  // FP64, or FP32 in the FP32 mode
    double* out[2];
    long long ogs;    // output values per g
    const int* gate;  // when set, the instance's work-groups return at once while *gate == 0
    int ntile, nc, G, pad;
};
// dense and rotated site vectors of one instance: xd (nd values, x[map] or 0)
// and per g xr (2 nr values: states 1, then 2, from x[rmap[2 e]], x[rmap[2 e + 1]])
struct KPrep {
    const double* x;
    const int* map;
    const int* rmap;
    const double* coef;
    void* xd;
    void* xr;
    const int* gate;
    long long nd, nr;
    int nc, crot, G, pad;
};
// blocks of 16 of a tile in m, of kc values formed at once, in n
struct KShape {
    int nm, ni, nn;
};
constexpr int kNumChainShapes = 8, kNarrowShapes = 5;  // the first kNarrowShapes have nn = 1
extern const KShape kChainShapes[kNumChainShapes];
// a lane stays within kLaneRows rows of its tile's or chunk's first element,
// and within that many values of the last of them: rows ld apart have to be
// few enough for 32 bits of bytes, whatever the block's size
constexpr int kLaneRows = 128;
inline bool chain_lanes_fit(int ld) { return 8 * (kLaneRows * (long long)ld + kLaneRows) < (1LL << 32); }
// values that may be read past the end of an operand buffer of blocks at most
// ld wide
inline long long read_pad(int ld) { return 16LL * ld + 64; }
// Pre-mixed environments: blocks that are sums of environment blocks of one
// shape (bra and ket particle number).  A work item sums 64 consecutive
// elements of every such block; its sources are staged in LDS kMixTile at a
// time, and up to kMixGroup blocks of the same sources are summed together.
constexpr int kMixTile = 160, kMixThreads = 1024, kMixGroup = 8;
struct MixWork {
    int tile0, tile1, e0, n;  // tiles of the shape, elements [e0, min(e0 + 64, n))
};
struct MixTileRec {
    int s0, s1, i0, i1;  // sources, groups
};
struct MixGroup {
    long long o[kMixGroup];
    int t0, t1, n, first;  // terms, blocks; first: the first tile of these blocks (they start from zero)
};
struct MixLists {
    const MixWork* work;
    const MixTileRec* tiles;
    const long long* src;  // environment block of every source
    const MixGroup* groups;
    const double* cf;  // term t of a group: kMixGroup coefficients
    const int* at;     // and the source within the tile
    int nwork, pad;
};
void premix(hipStream_t s, bool f32, const MixLists& m, const void* in, long long igs, void* out, long long ogs, int G);
// waves: wavefronts per tile (1 or kChainWaves; H_eff x: kChainWaves);
// max_tiles: the largest tile count times G of the instances; insts = null:
// the one instance `one`
void chain(hipStream_t s, int mode, int lay, int shape, int waves, int max_tiles, int ninst, const KInst* insts, const KInst& one);
void xprep(hipStream_t s, bool f32, long long max_n, int max_G, int ninst, const KPrep* insts, const KPrep& one);

// out = float(in), n elements
void to_f32(hipStream_t s, const double* in, float* out, long long n);

void bgemm(hipStream_t s, const BTask* tasks, int ntasks, const BTerm* terms, BufSet bufs,
           const double* coef);
void combine(hipStream_t s, const CTask* tasks, int ntasks, const CTerm* terms, BufSet bufs,
             const double* coef);
// the three launches of the diagonals.  mix row r reads terms mix[r]; M is
// mstride values per g.  nsplit > 1: the units of every H_eff tile are cut
// into nsplit parts summed in a fixed order through part (nsplit x ntot
// doubles, ntot = the site size); nsplit = 1 sums straight into dh
constexpr int kDiagTile = 32;
constexpr int kDiagSplitMax = 8;
// One launch up to so many terms of an (N, M) block, times G: its cost grows
// with them (4 us, and 0.12 for each), that of three launches starts at 9.5.
// 5: 4.3 us against 9.7 (L = 8, D = 64, G = 5); 27: 7.0 against 11.4 (L = 32,
// D = 256, G = 9); 75: 17.9 against 18.3 (the same, G = 25); 114: 32.6 against
// 26.8 (D = 400, G = 38), 15.5 against 17.8 at the second site of it
constexpr int kDiagDirectMax = 80;
void diag_direct(hipStream_t s, const DiagBlk* blks, int nblk, const DiagTerm* terms, const double* lenv, long long lsize,
                 const double* renv, long long rsize, const double* coef, int ncoef, int G, double* dh, double* dn);
void diag_gather(hipStream_t s, const DiagSide& left, const DiagSide& right, int G);
void diag_mix(hipStream_t s, const DiagMix* mix, int nmix, const DiagMixTerm* terms, const double* Ld, int nzl, int Dl,
              const double* coef, int ncoef, int G, double* M);
void diag_blocks(hipStream_t s, const DiagBlk* blks, int nblk, const int* zlist, const double* M, int nmix, int Dl,
                 const double* Rd, int nzr, int Dr, int G, double* dh, double* dn, int nsplit, double* part,
                 long long ntot);
// Per-sector positive-diagonal QR.  A list whose sectors fit kQrRegRows x
// kQrRegCols (every configuration up to D = 512) keeps its columns in
// registers; one whose two rows x cols matrices fit kQrLdsMax doubles runs in
// LDS; others use the scratch buffer in global memory.
constexpr int kQrLdsMax = 12288, kQrRegCols = 64, kQrRegRows = 256;
// the largest rows, cols, rows (rounded up to 16) * cols and 2 rows cols of a
// list's tasks
struct QrShape {
    int rows = 0, cols = 0, area = 0, lds = 0;
    void add(int r, int c) {
        auto up = [](int& a, long long b) { a = int(b > a ? (b < INT32_MAX ? b : INT32_MAX) : a); };
        up(rows, r);
        up(cols, c);
        up(area, (r + 15) / 16 * 16LL * c);
        up(lds, 2LL * r * c);
    }
};
void qr_sectors(hipStream_t s, const QrTask* tasks, int ntasks, const QrPiece* pieces, double* site,
                double* scratch, double* rout, const QrShape& shape);

// Davidson vector kernels (n = vector length, ld = stride between vectors)
void normalize(hipStream_t s, const double* in, double* out, int n, double* norm_out);
// p[0..n) = value
void fill(hipStream_t s, double* p, long long n, double value);
void multidot(hipStream_t s, const double* A, long long ld, int m, const double* u, int n,
              double* out);
void basis_rotate(hipStream_t s, const double* A, long long ld, int m, const double* Q, int keep,
                  double* out, int n);
// Grid-parallel Davidson passes.  Each work-group owns kDavChunk consecutive
// elements and writes per-chunk partial sums; consumers add the partials of
// all chunks in ascending chunk order (deterministic).  m <= kDavMaxVec.
constexpr int kDavChunk = 256;
constexpr int kGramGroup = 16;  // dots per work-group of the Gram pass
constexpr int kDavMaxVec = 256;
__host__ __device__ inline int dav_chunks(int n) { return (n + kDavChunk - 1) / kDavChunk; }
// aq = (a_0 .. a_{m-1}, theta) (device or mapped host memory); x = V a,
// u = HV a - theta NV a, t = -u / floor(dh - theta dn); part_x[3 per chunk] =
// (x.x, u.u, x.(NV a)); part_c[m per chunk] = V_j . t
void dav_ritz(hipStream_t s, const double* V, const double* HV, const double* NV, long long ld, int m,
              const double* aq, const double* dh, const double* dn, int n, double floor_, double* x, double* t,
              double* part_x, double* part_c);
// c = sum of part_in over chunks; t -= V c; then part_out = V_j . t (mode 0)
// or part_out = t.t per chunk (mode 1)
void dav_cgs(hipStream_t s, const double* V, long long ld, int m_sub, int m_dot, const double* part_in,
             int nchunk, double* t, int n, double* part_out, int mode);
// vout = t / sqrt(sum part), tnorm = sqrt(sum part)
void dav_normalize(hipStream_t s, const double* part, int nchunk, const double* t, double* vout, int n,
                   double* tnorm);
// Gram rows of the new vector m, per chunk: V_j.HV_m (j<=m), V_j.NV_m (j<=m),
// HV_j.V_m (j<m), NV_j.V_m (j<m).  With t != nullptr, V_m = t / |t| where
// |t|^2 = the sum of the npn partials pn (|t| -> *tnorm) and H_eff t, N_eff t
// are scaled by 1/|t| (t needs ypart); with ypart != nullptr they are the
// sums over the partials (G slots of H_eff, Gn of N_eff, stride gstride) and
// V_m (if t), HV_m and NV_m are stored, else they are read from HV_m, NV_m.
void dav_gram(hipStream_t s, double* V, double* HV, double* NV, long long ld, int m, int n, const double* t,
              const double* pn, int npn, double* tnorm, const double* ypart, const double* nypart, long long gstride,
              int G, int Gn, double* part);

// One instance of the batched Davidson passes (many SP-MPS states advanced
// together): the arguments of the single-instance passes above, with the
// partial-sum buffers pc1 (Ritz -> first CGS), pc2 (first -> second CGS)
// and pn (second CGS -> Gram).  The Gram pass forms V_m from t when
// from_t != 0 (then ypart must be set).
struct DavInst {
    double* V;
    double* HV;
    double* NV;
    long long ld;
    const double* aq;  // (a_0 .. a_{m-1}, theta), mapped host memory
    const double* dh;
    const double* dn;
    double floor_;
    double* x;
    double* t;
    double* part_x;  // 3 per chunk (mapped host memory)
    double* pc1;
    double* pc2;
    double* pn;
    double* pg;     // Gram rows, 4m+2 per chunk (mapped host memory)
    double* tnorm;  // (mapped host memory)
    const double* ypart;
    const double* nypart;
    long long gstride;
    int G, Gn, m, n, active, from_t, mr;  // mr: subspace size of the Ritz pass
    int ext;  // the search space grows this iteration (CGS, H_eff and Gram passes run)
    // device-resident iteration (davdev.hip): the state the host-driven
    // solver keeps on the host, here in this record on the device
    int it, max_iter, max_sub, keep, nk, restart, last, converged, matvecs, err, S, nch;
    double tol, drop, theta, rnorm, pnorm;
    double* Ht;      // S x S projected H_eff (device)
    double* Nt;      // S x S projected N_eff (device)
    double* Qk;      // restart rotation, m x nk (device)
    double* aqd;     // where the subspace solve writes (a, theta); aq reads it
    double* status;  // 8 doubles per instance for the host (mapped memory)
};
void bdav_ritz(hipStream_t s, const DavInst* insts, int ninst, int max_n);
// mode 0, 1: the two CGS passes; mode 2: after a restart, the dots of the
// correction with the rotated basis (instances without a restart skip it)
void bdav_cgs(hipStream_t s, const DavInst* insts, int ninst, int max_n, int mode);
void bdav_gram(hipStream_t s, const DavInst* insts, int ninst, int max_n, int max_m);

// Device-resident Davidson iteration (davdev.hip).  Subspace sizes up to
// kDevSubMax - 1 vectors and restarts keeping up to kDevKeepMax.
constexpr int kDevSubMax = 48;
constexpr int kDevKeepMax = 16;
// LDS bytes of the subspace solve for m vectors
__host__ __device__ inline int dev_solve_lds(int m) { return (7 * m * m + 8 * m + 512) * 8; }
// after the first product and Gram pass of a local solve: Ht[0], Nt[0] from
// the Gram partials, m = 1, iteration counters reset
void bdav_start(hipStream_t s, DavInst* insts, int ninst);
// one subspace solve per active instance (one work-group each): lowest pair
// of the projected pencil by canonical orthogonalisation, the restart
// rotation when the space is full, the fields the passes of the iteration read
void bdav_solve(hipStream_t s, DavInst* insts, int ninst, int max_m);
// restart: V, HV, NV rotated in place by Qk (instances without a restart skip)
void bdav_rotate(hipStream_t s, const DavInst* insts, int ninst, int max_n);
// end of an iteration: residual norm, convergence, the new Gram row, status
void bdav_update(hipStream_t s, DavInst* insts, int ninst);
// one instance's subspace solve on host data (tests): H, N m x m row-major;
// need_all != 0 also forms the restart rotation of `keep` vectors into Qk
// (m x keep) and the rotated H, N (keep x keep, into H and N); returns the
// rank kept (0: the metric vanishes)
int dev_small_solve(int m, double* H, double* N, double drop, int need_all, int keep, double* theta, double* a,
                    double* Qk);

// Learned Davidson preconditioner (mlp.hip): two-layer perceptron on five
// features per element; packed weights W1 (H x 5) | b1 (H) | w2 (H) | b2
constexpr int kMlpIn = 5;
constexpr int kMlpMaxHidden = 256;
__host__ __device__ inline long long mlp_size(int H) { return (long long)H * (kMlpIn + 2) + 1; }
// *out = sum over chunks of part[q * stride + idx] (fixed order)
void sum_partials(hipStream_t s, const double* part, int nchunk, int stride, int idx, double* out);
// features of every element from t = -r / d' (rr = |r|^2, tt = |t|^2,
// theta device scalars); feat (n x 5 FP32) and sgn (n, sign(r_i)) if feat is not null;
// t replaced by the model's correction if w is not null
void mlp_apply(hipStream_t s, const float* w, int H, double* t, const double* dh, const double* dn,
               const double* theta, const double* rr, const double* tt, int n, double floor_, float* feat,
               float* sgn);
// *out = v . v (one work-group, fixed order)
void sumsq(hipStream_t s, const double* v, int n, double* out);
void mlp_forward(hipStream_t s, const float* w, int H, const float* F, long long n, float* y);
// targets of nrec recorded iterations (Ritz vectors ldx apart) against the
// unit vector xstar, n per iteration; Y holds sign(r) on entry
void mlp_targets(hipStream_t s, const double* X, long long ldx, int nrec, const double* xstar, int n, float* Y);
// per-work-group gradient partials (mlp_size(H) + 1 doubles each, the last
// the summed squared error) over rows row0 + q * stride, q < count
void mlp_grad(hipStream_t s, const float* w, int H, const float* F, const float* Y, long long row0, long long stride,
              long long count, double* gpart, int nparts);
void mlp_adam(hipStream_t s, float* w, double* m, double* v, int H, const double* gpart, int nparts, double scale,
              double lr, int step, double* loss_out);

}  // namespace spk
