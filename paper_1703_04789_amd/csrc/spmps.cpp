// Host runtime and C ABI of the SP-MPS hot path (one MI355X, FP64).
//
// Holds the block structure of an (N, 2M)-symmetric MPS, the quadrature of
// the spin projector (Eqs. [PSMM], [pmpo]), the rotated MPO W[k] r(beta_g)
// (Eq. [expSy]), the environments of every quadrature point, and for every
// site the precomputed task lists that the device kernels execute:
//
//   left  pass:  T_g = L_g[k-1] x            (env blocks (N_bra, N_ket) times
//                                             (N, M) blocks of the site)
//                V_g = sum W~_g T_g           (W~_g = W[k] r_g, the rotation
//                                             acting on the ket index)
//   y   = P_NM sum_g coef_g V_g R_g[k+1]^T    (H_eff x)
//   ny  = P_NM sum_g coef_g r_g T_g R^I_g^T   (N_eff x, identity channels)
//   L_g[k] = A^T V_g                          (left environment update)
//   right pass mirrors it for R_g[k].
//
// These are the plain path's passes; the tiled path runs each line's products
// as one chained launch (y and ny together) that keeps T and V in registers.
//
// The environments are blocked by particle number only: the rotation
// exp(-i beta S_y) mixes M, so every (N_bra, N_ket) block is dense in M
// (the subduction described in Sec. 2.3).  Site tensors and H_eff vectors
// keep the (N, M) blocks.
#include "spmps.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <array>
#include <atomic>
#include <condition_variable>
#include <chrono>
#include <climits>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <exception>
#include <functional>
#include <map>
#include <numeric>
#include <memory>
#include <mutex>
#include <set>
#include <stdexcept>
#include <string>
#include <thread>
#include <vector>

#include "host_linalg.h"
#include "kernels.h"
#include "mlp.h"

namespace {

thread_local std::string g_last_error;

struct SpError : std::runtime_error {
    int code;
    SpError(int c, const std::string& m) : std::runtime_error(m), code(c) {}
};

#define SP_REQUIRE(cond, msg)                                  \
    do {                                                       \
        if (!(cond)) throw SpError(SP_EINVAL, std::string(msg)); \
    } while (0)

inline void hip_check(hipError_t e, const char* what) {
    if (e != hipSuccess) {
        if (e == hipErrorOutOfMemory) throw SpError(SP_ENOMEM, std::string(what) + ": out of device memory");
        throw SpError(SP_EHIP, std::string(what) + ": " + hipGetErrorString(e));
    }
}
#define HIPCK(x) hip_check((x), #x)

constexpr int kSigmaN[4] = {0, 1, 1, 2};
constexpr int kSigma2M[4] = {0, -1, 1, 0};

template <class T>
struct DArr {  // owned device array
    T* p = nullptr;
    size_t n = 0;
    DArr() = default;
    DArr(const DArr&) = delete;
    DArr& operator=(const DArr&) = delete;
    DArr(DArr&& o) noexcept : p(o.p), n(o.n) {
        o.p = nullptr;
        o.n = 0;
    }
    DArr& operator=(DArr&& o) noexcept {
        if (this != &o) {
            release();
            p = o.p;
            n = o.n;
            o.p = nullptr;
            o.n = 0;
        }
        return *this;
    }
    ~DArr() { release(); }
    void release() {
        if (p) (void)hipFree(p);
        p = nullptr;
        n = 0;
    }
    void alloc(size_t count) {
        release();
        n = count;
        if (count) HIPCK(hipMalloc(&p, count * sizeof(T)));
    }
    void upload(const std::vector<T>& v, hipStream_t s) {
        alloc(v.size());
        if (!v.empty()) HIPCK(hipMemcpyAsync(p, v.data(), v.size() * sizeof(T), hipMemcpyHostToDevice, s));
    }
};

template <class T>
struct DRef {  // view of device memory owned elsewhere
    T* p = nullptr;
};

// Many small host arrays as one device block and one copy: the lists of a
// state's sites are about forty arrays each, and an allocation, a copy and a
// free apiece cost 9 us (10.7 of the 31 ms of an expectation value at L = 32).
struct Upload {
    std::vector<char> host;
    std::vector<std::pair<void**, size_t>> views;
    template <class T>
    void add(DRef<T>& d, const std::vector<T>& v) {
        d.p = nullptr;
        if (v.empty()) return;
        const size_t off = (host.size() + 255) / 256 * 256;
        host.resize(off + v.size() * sizeof(T));
        std::memcpy(host.data() + off, v.data(), v.size() * sizeof(T));
        views.push_back({reinterpret_cast<void**>(&d.p), off});
    }
    void finish(DArr<char>& mem, hipStream_t s) {
        mem.alloc(host.size());
        if (host.empty()) return;
        HIPCK(hipMemcpyAsync(mem.p, host.data(), host.size(), hipMemcpyHostToDevice, s));
        for (const auto& v : views) *v.first = mem.p + v.second;
        HIPCK(hipStreamSynchronize(s));
    }
};

struct Sector {
    int n, m2, dim, off, nb, ro;
};
struct NBlock {
    int n, dim, off, s0, s1;
};
struct Bond {
    std::vector<Sector> sec;
    std::vector<NBlock> nb;
    int D = 0;
    std::map<std::pair<int, int>, int> sidx;
    std::map<int, int> nidx;
    int sector(int n, int m2) const {
        auto it = sidx.find({n, m2});
        return it == sidx.end() ? -1 : it->second;
    }
    int nblock(int n) const {
        auto it = nidx.find(n);
        return it == nidx.end() ? -1 : it->second;
    }
};
struct XBlk {
    int sa, s, sb, rows, cols;
    long long off;
};
struct SiteInfo {
    std::vector<XBlk> blk;
    long long size = 0, goff = 0;
    std::map<std::pair<int, int>, int> by_sa_s;  // (left sector, sigma) -> block
    int find(int sa, int s) const {
        auto it = by_sa_s.find({sa, s});
        return it == by_sa_s.end() ? -1 : it->second;
    }
};
// N-blocks of one site tensor (elements sharing both bond particle numbers)
// as groups of contiguous block ranges, and the group of every element; the
// host vectors stay alive as the sources of the uploads
struct NBlocks {
    int ng = 0;
    std::vector<int> gptr_h, rlen_h, gid_h;
    std::vector<long long> roff_h;
    DArr<int> gptr, rlen, gid;
    DArr<long long> roff;
    spk::ElemGroups groups() const { return spk::ElemGroups{ng, gptr.p, roff.p, rlen.p}; }
};
struct EnvBlk {
    int c, i, j, rows, cols;
    long long off;
};
struct EnvLayout {
    int nc = 0, nnb = 0;
    std::vector<EnvBlk> blk;
    std::vector<int> idx;  // c * nnb + i -> block
    long long size = 0;    // per quadrature point
    int find(int c, int i) const { return idx[size_t(c) * nnb + i]; }
};

// task list of one launch (host copy + device copy)
struct BList {
    std::vector<spk::BTask> tasks;
    std::vector<spk::BTerm> terms;
    DRef<spk::BTask> dtasks;
    DRef<spk::BTerm> dterms;
    double flops = 0.0;
    void add_task(int c_buf, long long c_off, int M, int N, int ldc, int accumulate = 0) {
        spk::BTask t{};
        t.c_off = c_off;
        t.c_buf = c_buf;
        t.M = M;
        t.N = N;
        t.ldc = ldc;
        t.t0 = t.t1 = int(terms.size());
        t.accumulate = accumulate;
        tasks.push_back(t);
    }
    void add_term(int a_buf, long long a_off, int a_rs, int a_cs, int b_buf, long long b_off, int b_rs,
                  int b_cs, int K, int cidx) {
        spk::BTerm m{};
        m.a_off = a_off;
        m.b_off = b_off;
        m.a_buf = a_buf;
        m.b_buf = b_buf;
        m.a_rs = a_rs;
        m.a_cs = a_cs;
        m.b_rs = b_rs;
        m.b_cs = b_cs;
        m.K = K;
        m.cidx = cidx;
        terms.push_back(m);
        tasks.back().t1 = int(terms.size());
        flops += 2.0 * tasks.back().M * tasks.back().N * K;
    }
    void upload(Upload& u) {
        u.add(dtasks, tasks);
        u.add(dterms, terms);
    }
    void launch(hipStream_t s, const spk::BufSet& b, const double* coef) const {
        spk::bgemm(s, dtasks.p, int(tasks.size()), dterms.p, b, coef);
    }
};
struct CList {
    std::vector<spk::CTask> tasks;
    std::vector<spk::CTerm> terms;
    DRef<spk::CTask> dtasks;
    DRef<spk::CTerm> dterms;
    double flops = 0.0;
    void add_task(int c_buf, long long c_off, int n) {
        spk::CTask t{};
        t.c_off = c_off;
        t.c_buf = c_buf;
        t.n = n;
        t.t0 = t.t1 = int(terms.size());
        tasks.push_back(t);
    }
    void add_term(int a_buf, long long a_off, int cidx) {
        spk::CTerm m{};
        m.a_off = a_off;
        m.a_buf = a_buf;
        m.cidx = cidx;
        terms.push_back(m);
        tasks.back().t1 = int(terms.size());
        flops += 2.0 * tasks.back().n;
    }
    void upload(Upload& u) {
        u.add(dtasks, tasks);
        u.add(dterms, terms);
    }
    void launch(hipStream_t s, const spk::BufSet& b, const double* coef) const {
        spk::combine(s, dtasks.p, int(tasks.size()), dterms.p, b, coef);
    }
};

// lists of a chained product (the same for every quadrature point)
struct ChainList {
    int lay = spk::kChainHeff, shape = 0, waves = spk::kChainWaves;
    std::vector<spk::KTile> tiles;
    std::vector<spk::KStep> steps;
    std::vector<spk::KSeg> segs;
    DRef<spk::KTile> dtiles;
    DRef<spk::KStep> dsteps;
    DRef<spk::KSeg> dsegs;
    // the steps of the tile being built: of the sum, and of N_eff x
    std::vector<spk::KStep> own, metric;
    int tile_m0 = 0, tile_n0 = 0, step_kc0 = 0;
    // the tile from row m0 and column n0 of its block
    void begin_tile(int m0, int n0) {
        tile_m0 = m0;
        tile_n0 = n0;
    }
    void begin_step(long long p_off, int ldp, int kc0, int kc1, bool of_metric = false) {
        step_kc0 = kc0;
        (of_metric ? metric : own)
            .push_back(spk::KStep{spk::chain_p(lay, p_off, ldp, tile_m0, kc0), ldp, kc1 - kc0, int(segs.size()), int(segs.size())});
    }
    // alt_x: the rotated site tensor, alt_e: the mixed environment
    void add_seg(long long a_off, int lda, long long b_off, int ldb, int k0, int k1, double cf, bool alt_x, bool alt_e,
                 bool of_metric = false) {
        segs.push_back(spk::KSeg{spk::chain_a(lay, a_off, lda, step_kc0, k0), spk::chain_b(lay, b_off, ldb, k0, tile_n0), cf,
                                 lda, ldb, k1 - k0, alt_x, alt_e, 0});
        (of_metric ? metric : own).back().g1 = int(segs.size());
    }
    // matrix-core steps of a step (blocks of 16 kc values times the 8-deep
    // chunks of its segments, then the outer product), plus its latency
    int weight(const spk::KStep& p, int nm) const {
        const int ni = (p.nkc + 15) / 16;
        int w = 12 + 4 * ni * nm;
        for (int g = p.g0; g < p.g1; ++g) w += 2 * ni * ((segs[g].nk + 7) / 8);
        return w;
    }
    // closes the tile: steps without segments are dropped, the others dealt to
    // the wavefronts, the heaviest first to the least loaded
    void end_tile(spk::KTile t) {
        auto has = [](const spk::KStep& p) { return p.g1 > p.g0; };
        const int nm = (t.m + 15) / 16;
        t.e0 = int(steps.size());
        int load[spk::kChainWaves] = {};
        for (const spk::KStep& p : metric)
            if (has(p)) {
                steps.push_back(p);
                load[waves - 1] += weight(p, nm);
            }
        t.e1 = int(steps.size());
        std::vector<std::pair<int, int>> order;
        for (int i = 0; i < int(own.size()); ++i)
            if (has(own[i])) order.push_back({-weight(own[i], nm), i});
        std::sort(order.begin(), order.end());
        std::vector<int> of[spk::kChainWaves];
        for (const auto& o : order) {
            const int w = int(std::min_element(load, load + waves) - load);
            load[w] -= o.first;
            of[w].push_back(o.second);
        }
        t.s[0] = int(steps.size());
        for (int w = 0; w < spk::kChainWaves; ++w) {
            std::sort(of[w].begin(), of[w].end());
            for (int i : of[w]) steps.push_back(own[i]);
            t.s[w + 1] = int(steps.size());
        }
        own.clear();
        metric.clear();
        tiles.push_back(t);
    }
    void upload(Upload& u) {
        u.add(dtiles, tiles);
        u.add(dsteps, steps);
        u.add(dsegs, segs);
    }
};
// one side's environment with the unrotated MPO mixed in
struct MixList {
    std::vector<spk::MixWork> work;
    std::vector<spk::MixTileRec> tiles;
    std::vector<long long> src;
    std::vector<spk::MixGroup> groups;
    std::vector<double> cf;
    std::vector<int> at;
    DRef<spk::MixWork> dwork;
    DRef<spk::MixTileRec> dtiles;
    DRef<long long> dsrc;
    DRef<spk::MixGroup> dgroups;
    DRef<double> dcf;
    DRef<int> dat;
    long long size = 0;  // values per quadrature point
    double flops = 0.0;  // per quadrature point
    // blocks to be mixed by shape (bra block, ket block): offset, then the
    // terms (environment block, coefficient)
    struct Block {
        long long off;
        std::vector<std::pair<int, double>> terms;
    };
    std::map<std::pair<int, int>, std::vector<Block>> shapes;
    long long add(int i, int j, int n, std::vector<std::pair<int, double>> t) {
        flops += 2.0 * n * t.size();
        std::sort(t.begin(), t.end());
        shapes[{i, j}].push_back({size, std::move(t)});
        size += n;
        return size - n;
    }
    bool empty() const { return shapes.empty(); }
    void finish(const EnvLayout& env) {
        std::vector<int> weight;
        for (const auto& sh : shapes) {
            std::set<int> used;
            for (const Block& b : sh.second)
                for (const auto& t : b.terms) used.insert(t.first);
            const std::vector<int> blk(used.begin(), used.end());
            // blocks of the same sources
            std::map<std::vector<int>, std::vector<const Block*>> alike;
            for (const Block& b : sh.second) {
                std::vector<int> from;
                for (const auto& t : b.terms) from.push_back(t.first);
                alike[from].push_back(&b);
            }
            const int tile0 = int(tiles.size());
            for (size_t s0 = 0; s0 < blk.size(); s0 += spk::kMixTile) {
                const size_t s1 = std::min(blk.size(), s0 + spk::kMixTile);
                spk::MixTileRec tr{int(src.size()), 0, int(groups.size()), 0};
                for (size_t q = s0; q < s1; ++q) src.push_back(env.blk[blk[q]].off);
                tr.s1 = int(src.size());
                for (const auto& al : alike) {
                    const std::vector<int>& from = al.first;
                    const size_t q0 = std::lower_bound(from.begin(), from.end(), blk[s0]) - from.begin(),
                                 q1 = std::upper_bound(from.begin(), from.end(), blk[s1 - 1]) - from.begin();
                    if (q0 == q1) continue;
                    for (size_t b0 = 0; b0 < al.second.size(); b0 += spk::kMixGroup) {
                        spk::MixGroup gr{};
                        gr.n = int(std::min<size_t>(spk::kMixGroup, al.second.size() - b0));
                        gr.first = q0 == 0;
                        gr.t0 = int(at.size());
                        for (int b = 0; b < gr.n; ++b) gr.o[b] = al.second[b0 + b]->off;
                        for (size_t q = q0; q < q1; ++q) {
                            at.push_back(int(std::lower_bound(blk.begin(), blk.end(), from[q]) - blk.begin() - s0));
                            for (int b = 0; b < spk::kMixGroup; ++b)
                                cf.push_back(b < gr.n ? al.second[b0 + b]->terms[q].second : 0.0);
                        }
                        gr.t1 = int(at.size());
                        groups.push_back(gr);
                    }
                }
                tr.i1 = int(groups.size());
                // the longest sums first
                std::stable_sort(groups.begin() + tr.i0, groups.end(), [](const spk::MixGroup& a, const spk::MixGroup& b) {
                    return a.t1 - a.t0 > b.t1 - b.t0;
                });
                tiles.push_back(tr);
            }
            const EnvBlk& e = env.blk[blk[0]];
            const int n = e.rows * e.cols;
            for (int e0 = 0; e0 < n; e0 += 64) work.push_back(spk::MixWork{tile0, int(tiles.size()), e0, n});
            weight.resize(work.size(), terms_of(work.back()));
        }
        // the shapes with the most terms first
        std::vector<int> ord(work.size());
        std::iota(ord.begin(), ord.end(), 0);
        std::stable_sort(ord.begin(), ord.end(), [&](int a, int b) { return weight[a] > weight[b]; });
        std::vector<spk::MixWork> by(work.size());
        for (size_t i = 0; i < ord.size(); ++i) by[i] = work[ord[i]];
        work.swap(by);
    }
    int terms_of(const spk::MixWork& w) const {
        int n = 0;
        for (int i = tiles[w.tile0].i0; i < tiles[w.tile1 - 1].i1; ++i) n += groups[i].t1 - groups[i].t0;
        return n;
    }
    void upload(Upload& u) {
        u.add(dwork, work);
        u.add(dtiles, tiles);
        u.add(dsrc, src);
        u.add(dgroups, groups);
        u.add(dcf, cf);
        u.add(dat, at);
    }
    spk::MixLists lists() const {
        return spk::MixLists{dwork.p, dtiles.p, dsrc.p, dgroups.p, dcf.p, dat.p, int(work.size()), 0};
    }
};

// buffer slots of a launch; B_BRA is the site tensor on the bra side of the
// plain-path environment updates (the same as B_X except for the mixed
// environments of an orthogonality constraint)
enum Buf { B_ENVL = 0, B_ENVR = 1, B_X = 2, B_T = 3, B_V = 4, B_Y = 5, B_NY = 6, B_OUT = 7, B_BRA = 8 };

struct SitePlan {
    // coefficient table [G][nc]
    int nW = 0, nc = 0;
    std::vector<std::array<int, 4>> went;  // (a, b, s, u) of the rotated MPO pattern
    std::vector<double> coef_h;
    DRef<double> coef;
    int c_wt(int e) const { return e; }
    int c_cwt(int e) const { return nW + e; }
    int c_g() const { return 2 * nW; }
    int c_gr(int s, int u) const { return 2 * nW + 1 + 4 * s + u; }
    int c_one() const { return 2 * nW + 17; }
    // unrotated MPO entries W[a, b, s, s'] (block-product path) and the
    // rotation r_g(s, u) itself
    int nWr = 0;
    int c_wr(int e) const { return 2 * nW + 18 + e; }
    int c_r(int s, int u) const { return 2 * nW + 18 + nWr + 4 * s + u; }
    // scratch of the plain path's passes per quadrature point
    long long Tsize = 0, Vsize = 0, Zsize = 0, Ztsize = 0;
    BList p1, yout, envl_out, p1r, envr_out;
    CList mixl, mixr;
    double heff_flops = 0.0;
    // diagonal
    int dg_nzl = 0, dg_nzr = 0, dg_split = 1;  // particle-conserving channels of both bonds, parts of a tile
    std::vector<spk::DiagSrc> dg_src;           // left, then right (nz * nnb each)
    std::vector<int> dg_idx;                    // left nb, ro, right nb, ro, then the channel lists of the tiles
    std::vector<spk::DiagMix> dg_mix;
    std::vector<spk::DiagMixTerm> dg_term;
    std::vector<spk::DiagBlk> dg_blk;
    bool dg_direct = false;                     // one launch over dg_dterm, without the lists above
    std::vector<spk::DiagTerm> dg_dterm;
    DRef<spk::DiagSrc> ddg_src;
    DRef<int> ddg_idx;
    DRef<spk::DiagMix> ddg_mix;
    DRef<spk::DiagMixTerm> ddg_term;
    DRef<spk::DiagBlk> ddg_blk;
    DRef<spk::DiagTerm> ddg_dterm;
    // gauge moves
    std::vector<spk::QrTask> qr_tasks, lq_tasks;
    std::vector<spk::QrPiece> qr_pieces, lq_pieces;
    DRef<spk::QrTask> dqr_tasks, dlq_tasks;
    DRef<spk::QrPiece> dqr_pieces, dlq_pieces;
    long long qr_scratch = 0, lq_scratch = 0, qr_rsize = 0, lq_rsize = 0;
    spk::QrShape qr_shape, lq_shape;
    std::vector<long long> qr_roff;  // per right sector of bond k
    std::vector<long long> lq_roff;  // per left sector of bond k-1
    BList absorb_right;  // R of site k into site k+1
    BList absorb_left;   // L of site k into site k-1
    // tiled path: dense particle-number layout of the site
    long long Xd_size = 0;
    std::vector<int> xmap_h;  // dense element -> packed index or -1
    DRef<int> xmap;
    // chained products: the environment updates, the pre-mixed environments
    // they (and H_eff x at wide MPOs) use, the packed indices of the rotated
    // site vector's two states
    std::vector<std::array<int, 4>> wr_ent;  // unrotated MPO entries (a, b, s, s')
    ChainList c_heff, c_envl, c_envr;
    int y_split = 1;                         // channel chunks of H_eff x (partials of y: y_split * G)
    MixList mix_l, mix_r;                    // empty: the products read the environment itself
    std::vector<int> rmap_h;
    DRef<int> rmap;
    // fused plan of H_eff x, which sets its arithmetic in the reduced
    // precisions: rows per task and LDS (doubles); 0: the site's MPO is too
    // wide for one
    int h_rows = 0;
    int h_lds = 0;
};

}  // namespace

struct sp_handle {
    hipStream_t stream = nullptr;
    int device = 0;
    int L = 0, N = 0, twoS = 0, twoM = 0, G = 0;
    bool inexact = false;
    std::vector<double> qx, qw, qc, qs, qcoef;
    std::vector<int> w;                    // MPO bond dimensions
    std::vector<std::vector<int>> dn;      // per bond, per channel: particle change
    std::vector<std::vector<double>> W;    // per site (index k-1)
    std::vector<Bond> bonds;
    std::vector<SiteInfo> sites;           // index k-1
    std::vector<EnvLayout> env;            // per bond
    // Environments per bond, G * size each.  An interior bond keeps one
    // buffer for both sides: a sweep builds L[k] only after its last use of
    // R[k] and the other way round, so at most one of the two is valid at a
    // time (Lvalid/Rvalid); the boundary bonds 0 and L keep both.
    DArr<char> plan_mem;  // the lists of every site
    std::vector<DArr<double>> envmem;
    std::vector<DArr<float>> envmem32;     // FP32 copies (reduced precisions)
    std::vector<DRef<double>> envL, envR;
    std::vector<DRef<float>> envL32, envR32;
    std::vector<int> tab_nsec, tab_n, tab_2m, tab_dim;  // the block table as given
    int precision = SP_FP64;
    std::vector<char> Lvalid, Rvalid;
    DArr<double> mps;
    long long mps_size = 0, max_site = 0;
    std::vector<SitePlan> plan;            // index k-1
    int path = SP_PATH_TILED;
    DArr<double> T, V, qr_scratch, qr_r, tmp_site, Xd, Xr, ypart, nypart;
    // pre-mixed environment of one site (tiled path): the left one is valid
    // for site lt_site while the generation of L[lt_site - 1] is lt_gen
    DArr<double> LT;
    long long LT_cap = 0;
    DArr<double> diag_part;  // partial sums of the split diagonal (kDiagSplitMax x max_site)
    std::vector<long long> Lgen;
    int lt_site = -1;   // -1: none (the scratch holds a right environment, or nothing)
    long long lt_gen = -1;
    bool lt_f32 = false;
    // the caller's capture that recorded it (0: it was launched), and whether
    // calls were ever recorded: their replays, which the handle does not see,
    // write the scratch and the environments
    unsigned long long lt_capture = 0;
    bool recorded = false;
    bool mixes = false;  // some site's MPO is mixed into an environment
    long long Xr_cap = 0;
    long long Xd_cap = 0;
    int y_split_max = 1;  // partial slots of y per quadrature point
    long long T_cap = 0, V_cap = 0, qr_scratch_cap = 0, qr_r_cap = 0;
    int center = 1;
    // Davidson workspace
    int dav_sub = 0;
    long long ld = 0;
    DArr<double> dV, dHV, dNV, dRot, dx, dt, ddh, ddn, dpart, dsmall, dy, dny;
    DArr<double> dHt, dNt;  // projected H_eff, N_eff of the device-resident solve ((dav_sub+1)^2)
    double* pin = nullptr;  // pinned host staging (device -> host)
    double* pin_dev = nullptr;  // the same memory as kernels address it
    size_t pin_n = 0;
    double* pin_up = nullptr;  // pinned host staging (host -> device)
    double* pin_up_dev = nullptr;
    size_t pin_up_n = 0;
    // orthogonality constraints (excited states): one identity-MPO handle per
    // lower state whose environments are mixed (bra: this state, ket: the
    // lower state), the orthonormalised constraint vectors of the current
    // site (cld apart) and their projection partials
    std::vector<std::unique_ptr<sp_handle>> cons;
    DArr<double> conB, conPart;
    long long cld = 0;
    int con_active = 0;
    double* con_pin = nullptr;  // mapped: norm partials read by the host
    double* con_pin_dev = nullptr;
    // learned preconditioner: the model used for corrections and the one
    // collecting training pairs (either may be null), Ritz vectors of the
    // current solve for the targets, device scalars
    sp_mlp* mlp_use = nullptr;
    sp_mlp* mlp_rec = nullptr;
    DArr<double> xrec, mlp_scal, mlp_grms, mlp_tscal;
    std::vector<NBlocks> nblocks;  // per site (index k-1), built on first use
    ~sp_handle() {
        if (pin) (void)hipHostFree(pin);
        if (pin_up) (void)hipHostFree(pin_up);
        if (con_pin) (void)hipHostFree(con_pin);
    }
};

// reduced-precision local solves (SP_FP32 or SP_BF16X3): FP32 products at
// sites with a fused plan, FP64 Rayleigh quotient per site step, looser canonical orthogonalisation
inline bool reduced(const sp_handle* h) { return h->precision != SP_FP64; }
// canonical orthogonalisation of the projected metric: eigenvalues below
// drop x the largest are discarded; the threshold sits above the relative
// noise of the products (FP64 ~1e-15, FP32 ~1e-7, split BF16 ~5e-6) by two
// orders, one order for split BF16 (1e-3 there slowed the descent of the
// sweeps by discarding directions of small spin-S weight)
inline double metric_drop(const sp_handle* h) {
    return h->precision == SP_FP64 ? 1e-10 : (h->precision == SP_FP32 ? 1e-5 : 1e-4);
}

// a learned Davidson preconditioner and its training pairs (one device)
struct sp_mlp {
    int hidden = 0, device = 0;
    DArr<float> w;       // packed weights
    DArr<double> m, v;   // Adam moments
    int step = 0;
    long long cap = 0, rows = 0;
    DArr<float> F, Y;    // recorded pairs: cap x 5 features, cap targets
    DArr<double> gpart, scal;
    int nparts = 0;
    int scope = SP_MLP_VECTOR;  // rms over the site vector or per N-block
};

namespace {

// ---------------------------------------------------------------------------
// setup

void build_bonds(sp_handle* h, const sp_block_table* bt) {
    const int L = h->L;
    h->bonds.assign(L + 1, Bond{});
    long long pos = 0;
    for (int k = 0; k <= L; ++k) {
        Bond& b = h->bonds[k];
        const int ns = bt->nsec[k];
        SP_REQUIRE(ns >= 1, "every bond needs at least one sector");
        int off = 0;
        for (int i = 0; i < ns; ++i, ++pos) {
            Sector s{bt->sec_n[pos], bt->sec_2m[pos], bt->sec_dim[pos], off, -1, 0};
            SP_REQUIRE(s.dim >= 1, "sector dimensions must be positive");
            if (i > 0) {
                const Sector& p = b.sec.back();
                SP_REQUIRE(p.n < s.n || (p.n == s.n && p.m2 < s.m2), "sectors must be sorted by (N, 2M)");
            }
            off += s.dim;
            b.sec.push_back(s);
        }
        b.D = off;
        for (int i = 0; i < ns; ++i) {
            Sector& s = b.sec[i];
            if (b.nb.empty() || b.nb.back().n != s.n) b.nb.push_back(NBlock{s.n, 0, s.off, i, i});
            NBlock& nb = b.nb.back();
            s.nb = int(b.nb.size()) - 1;
            s.ro = nb.dim;
            nb.dim += s.dim;
            nb.s1 = i + 1;
            b.sidx[{s.n, s.m2}] = i;
        }
        for (int i = 0; i < int(b.nb.size()); ++i) b.nidx[b.nb[i].n] = i;
    }
    SP_REQUIRE(h->bonds[0].sec.size() == 1 && h->bonds[0].sec[0].n == 0 && h->bonds[0].sec[0].m2 == 0 &&
                   h->bonds[0].sec[0].dim == 1,
               "bond 0 must be the single sector (0, 0) of dimension 1");
    SP_REQUIRE(h->bonds[L].sec.size() == 1 && h->bonds[L].sec[0].n == h->N &&
                   h->bonds[L].sec[0].m2 == h->twoM && h->bonds[L].sec[0].dim == 1,
               "bond L must be the single sector (N, 2M) of dimension 1");
    // reachability: a sector cannot hold more states than its neighbours reach
    for (int k = 1; k < L; ++k) {
        for (const Sector& s : h->bonds[k].sec) {
            int left = 0, right = 0;
            for (int q = 0; q < 4; ++q) {
                int a = h->bonds[k - 1].sector(s.n - kSigmaN[q], s.m2 - kSigma2M[q]);
                if (a >= 0) left += h->bonds[k - 1].sec[a].dim;
                int c = h->bonds[k + 1].sector(s.n + kSigmaN[q], s.m2 + kSigma2M[q]);
                if (c >= 0) right += h->bonds[k + 1].sec[c].dim;
            }
            SP_REQUIRE(s.dim <= left && s.dim <= right,
                       "block table: a sector is wider than its support in a neighbouring bond");
        }
    }
    // site blocks in canonical order
    h->sites.assign(L, SiteInfo{});
    long long goff = 0;
    for (int k = 1; k <= L; ++k) {
        SiteInfo& si = h->sites[k - 1];
        si.goff = goff;
        const Bond& bl = h->bonds[k - 1];
        const Bond& br = h->bonds[k];
        long long off = 0;
        for (int a = 0; a < int(bl.sec.size()); ++a) {
            for (int q = 0; q < 4; ++q) {
                const int b = br.sector(bl.sec[a].n + kSigmaN[q], bl.sec[a].m2 + kSigma2M[q]);
                if (b < 0) continue;
                XBlk x{a, q, b, bl.sec[a].dim, br.sec[b].dim, off};
                si.by_sa_s[{a, q}] = int(si.blk.size());
                si.blk.push_back(x);
                off += (long long)x.rows * x.cols;
            }
        }
        si.size = off;
        SP_REQUIRE(off > 0, "a site has no allowed block");
        goff += off;
        h->max_site = std::max(h->max_site, off);
    }
    h->mps_size = goff;
}

void build_mpo(sp_handle* h, const sp_mpo* Wm) {
    const int L = h->L;
    h->w.assign(Wm->w, Wm->w + L + 1);
    SP_REQUIRE(h->w[0] == 1 && h->w[L] == 1, "MPO: w[0] and w[L] must be 1");
    for (int k = 0; k <= L; ++k) SP_REQUIRE(h->w[k] >= 1 && h->w[k] <= 4096, "MPO: bad bond dimension");
    h->W.assign(L, {});
    long long pos = 0;
    for (int k = 1; k <= L; ++k) {
        const long long n = (long long)h->w[k - 1] * h->w[k] * 16;
        h->W[k - 1].assign(Wm->data + pos, Wm->data + pos + n);
        pos += n;
    }
    // particle change of every channel, propagated from bond 0
    h->dn.assign(L + 1, {});
    h->dn[0] = {0};
    for (int k = 1; k <= L; ++k) {
        const int wl = h->w[k - 1], wr = h->w[k];
        std::vector<int> d(wr, INT32_MIN);
        const auto& Wk = h->W[k - 1];
        for (int a = 0; a < wl; ++a)
            for (int b = 0; b < wr; ++b)
                for (int s = 0; s < 4; ++s)
                    for (int t = 0; t < 4; ++t) {
                        const double v = Wk[((size_t(a) * wr + b) * 4 + s) * 4 + t];
                        if (v == 0.0) continue;
                        const int val = h->dn[k - 1][a] + kSigmaN[s] - kSigmaN[t];
                        if (d[b] == INT32_MIN) d[b] = val;
                        SP_REQUIRE(d[b] == val, "MPO: an operator entry changes the particle number inconsistently");
                    }
        for (int b = 0; b < wr; ++b)
            if (d[b] == INT32_MIN) d[b] = 0;  // channel never reached: unused
        h->dn[k] = d;
    }
    SP_REQUIRE(h->dn[L][0] == 0, "MPO: the full operator must conserve the particle number");
    // identity channels: column 0 (k < L) and the last row (k > 1)
    auto op = [&](int k, int a, int b, int s, int t) {
        return h->W[k - 1][((size_t(a) * h->w[k] + b) * 4 + s) * 4 + t];
    };
    for (int k = 1; k <= L; ++k) {
        const int wl = h->w[k - 1], wr = h->w[k];
        if (k < L)
            for (int a = 0; a < wl; ++a)
                for (int s = 0; s < 4; ++s)
                    for (int t = 0; t < 4; ++t)
                        SP_REQUIRE(op(k, a, 0, s, t) == ((a == 0 && s == t) ? 1.0 : 0.0),
                                   "MPO: channel 0 must be the left identity string");
        if (k > 1)
            for (int b = 0; b < wr; ++b)
                for (int s = 0; s < 4; ++s)
                    for (int t = 0; t < 4; ++t)
                        SP_REQUIRE(op(k, wl - 1, b, s, t) == ((b == wr - 1 && s == t) ? 1.0 : 0.0),
                                   "MPO: the last channel must be the right identity string");
    }
}

void build_env_layouts(sp_handle* h) {
    const int L = h->L;
    h->env.assign(L + 1, EnvLayout{});
    for (int k = 0; k <= L; ++k) {
        EnvLayout& e = h->env[k];
        const Bond& b = h->bonds[k];
        e.nc = h->w[k];
        e.nnb = int(b.nb.size());
        e.idx.assign(size_t(e.nc) * e.nnb, -1);
        long long off = 0;
        for (int c = 0; c < e.nc; ++c)
            for (int i = 0; i < e.nnb; ++i) {
                const int j = b.nblock(b.nb[i].n - h->dn[k][c]);
                if (j < 0) continue;
                e.idx[size_t(c) * e.nnb + i] = int(e.blk.size());
                e.blk.push_back(EnvBlk{c, i, j, b.nb[i].dim, b.nb[j].dim, off});
                off += (long long)b.nb[i].dim * b.nb[j].dim;
            }
        e.size = off;
    }
    SP_REQUIRE(h->env[0].size == 1 && h->env[L].size == 1, "boundary environments must be 1x1");
    h->Lvalid.assign(L + 1, 0);
    h->Rvalid.assign(L + 1, 0);
    h->Lgen.assign(L + 1, 0);
}

// values the block products may read past the end of an operand buffer
long long read_pad(const sp_handle* h) {
    int ld = 1;
    for (const Bond& b : h->bonds)
        for (const NBlock& nb : b.nb) ld = std::max(ld, nb.dim);
    return spk::read_pad(ld);
}

// Interior bonds 1..L-1 hold one buffer shared by L[k] and R[k]; bonds 0
// and L hold two (the boundary ones and the full contractions).
template <class T>
void alloc_env_set(const sp_handle* h, std::vector<DArr<T>>& mem, std::vector<DRef<T>>& l,
                   std::vector<DRef<T>>& r) {
    const int L = h->L;
    mem.clear();
    mem.resize(L + 3);
    l.assign(L + 1, {});
    r.assign(L + 1, {});
    for (int k = 0; k <= L; ++k) {
        mem[k].alloc(size_t(h->G) * h->env[k].size + read_pad(h));
        l[k].p = r[k].p = mem[k].p;
    }
    mem[L + 1].alloc(size_t(h->G) * h->env[0].size + read_pad(h));
    mem[L + 2].alloc(size_t(h->G) * h->env[L].size + read_pad(h));
    r[0].p = mem[L + 1].p;
    r[L].p = mem[L + 2].p;
}

// an interior bond's two environments share storage
inline bool env_shared(const sp_handle* h, int k) { return k > 0 && k < h->L; }

void alloc_envs(sp_handle* h) {
    const int L = h->L;
    alloc_env_set(h, h->envmem, h->envL, h->envR);
    // boundary environments: one 1x1 block equal to 1 for every g
    std::vector<double> ones(h->G, 1.0);
    HIPCK(hipMemcpyAsync(h->envL[0].p, ones.data(), h->G * sizeof(double), hipMemcpyHostToDevice, h->stream));
    HIPCK(hipMemcpyAsync(h->envR[L].p, ones.data(), h->G * sizeof(double), hipMemcpyHostToDevice, h->stream));
    if (reduced(h)) {
        alloc_env_set(h, h->envmem32, h->envL32, h->envR32);
        spk::to_f32(h->stream, h->envL[0].p, h->envL32[0].p, h->G);
        spk::to_f32(h->stream, h->envR[L].p, h->envR32[L].p, h->G);
    }
    HIPCK(hipStreamSynchronize(h->stream));
    h->Lvalid[0] = 1;
    h->Rvalid[L] = 1;
    ++h->Lgen[0];
}

// rotated MPO W[k] r(beta_g): pattern and values
bool rot_nonzero(int t, int u) { return (t == u) || ((t == 1 || t == 2) && (u == 1 || u == 2)); }
double rot_value(int t, int u, double c, double s) {
    if (t == 0 || t == 3) return t == u ? 1.0 : 0.0;
    if (u == 0 || u == 3) return 0.0;
    if (t == u) return c;
    return (t == 1) ? s : -s;  // r[1][2] = s, r[2][1] = -s  (Eq. [expSy])
}

void build_plan(sp_handle* h, int k) {
    SitePlan& P = h->plan[k - 1];
    const int G = h->G;
    // the tiled path runs the chained lists and only counts the passes below:
    // one quadrature point stands for all
    const bool plain = h->path == SP_PATH_PLAIN;
    const int Gl = plain ? G : 1;
    const Bond& bl = h->bonds[k - 1];
    const Bond& br = h->bonds[k];
    const SiteInfo& si = h->sites[k - 1];
    const EnvLayout& el = h->env[k - 1];  // L env at bond k-1 (also output of the right pass)
    const EnvLayout& er = h->env[k];      // R env at bond k (also output of the left pass)
    const int wl = h->w[k - 1], wr = h->w[k];
    const auto& Wk = h->W[k - 1];
    // ---- rotated MPO pattern and coefficient table
    for (int a = 0; a < wl; ++a)
        for (int b = 0; b < wr; ++b) {
            const double* op = &Wk[(size_t(a) * wr + b) * 16];
            bool any = false;
            for (int e = 0; e < 16; ++e) any = any || op[e] != 0.0;
            if (!any) continue;
            for (int s = 0; s < 4; ++s)
                for (int u = 0; u < 4; ++u) {
                    bool nz = false;
                    for (int t = 0; t < 4; ++t)
                        if (op[s * 4 + t] != 0.0 && rot_nonzero(t, u)) nz = true;
                    if (nz) P.went.push_back({a, b, s, u});
                }
        }
    P.nW = int(P.went.size());
    // the rotated-MPO entries by (sigma, right channel) as (left channel,
    // sigma', entry), by (sigma, left channel) as (right channel, sigma',
    // entry), and the diagonal ones (sigma' = sigma) by sigma as (left
    // channel, right channel, entry), each in ascending order (the order of
    // the entry list)
    std::vector<std::vector<std::array<int, 3>>> byL(size_t(4) * wr), byR(size_t(4) * wl), byD(4);
    for (int e = 0; e < P.nW; ++e) {
        const auto& q = P.went[e];
        byL[size_t(q[2]) * wr + q[1]].push_back({q[0], q[3], e});
        byR[size_t(q[2]) * wl + q[0]].push_back({q[1], q[3], e});
        if (q[2] == q[3]) byD[q[2]].push_back({q[0], q[1], e});
    }
    // the unrotated entries W[a, b, s, s'] of the blocks in the pattern: the
    // chained products rotate the site vector instead (Eq. [expSy] acts on s'
    // only)
    std::vector<double> wr_val;
    {
        std::set<std::pair<int, int>> blocks;
        for (const auto& q : P.went) blocks.insert({q[0], q[1]});
        for (const auto& ab : blocks) {
            const double* op = &Wk[(size_t(ab.first) * wr + ab.second) * 16];
            for (int s2 = 0; s2 < 4; ++s2)
                for (int v = 0; v < 4; ++v)
                    if (op[s2 * 4 + v] != 0.0) {
                        wr_val.push_back(op[s2 * 4 + v]);
                        P.wr_ent.push_back({ab.first, ab.second, s2, v});
                    }
        }
    }
    P.nWr = int(wr_val.size());
    P.nc = 2 * P.nW + 18 + P.nWr + 16;
    P.coef_h.assign(size_t(G) * P.nc, 0.0);
    for (int g = 0; g < G; ++g) {
        double* cf = &P.coef_h[size_t(g) * P.nc];
        for (int e = 0; e < P.nW; ++e) {
            const auto& q = P.went[e];
            double v = 0.0;
            for (int t = 0; t < 4; ++t)
                v += Wk[((size_t(q[0]) * wr + q[1]) * 4 + q[2]) * 4 + t] * rot_value(t, q[3], h->qc[g], h->qs[g]);
            cf[P.c_wt(e)] = v;
            cf[P.c_cwt(e)] = h->qcoef[g] * v;
        }
        cf[P.c_g()] = h->qcoef[g];
        for (int s = 0; s < 4; ++s)
            for (int u = 0; u < 4; ++u) cf[P.c_gr(s, u)] = h->qcoef[g] * rot_value(s, u, h->qc[g], h->qs[g]);
        cf[P.c_one()] = 1.0;
        for (int e = 0; e < P.nWr; ++e) cf[P.c_wr(e)] = wr_val[e];
        for (int s = 0; s < 4; ++s)
            for (int u = 0; u < 4; ++u) cf[P.c_r(s, u)] = rot_value(s, u, h->qc[g], h->qs[g]);
    }
    const long long Lsz = el.size, Rsz = er.size;

    // ---- left pass, phase 1: T(eb, sigma') = L(eb) X(j, sigma', jb)
    std::vector<long long> Toff(el.blk.size() * 4, -1);
    std::vector<int> Tcols(el.blk.size() * 4, 0);
    long long toff = 0;
    for (size_t e = 0; e < el.blk.size(); ++e)
        for (int q = 0; q < 4; ++q) {
            const EnvBlk& eb = el.blk[e];
            const int jb = br.nblock(bl.nb[eb.j].n + kSigmaN[q]);
            if (jb < 0) continue;
            Toff[e * 4 + q] = toff;
            Tcols[e * 4 + q] = br.nb[jb].dim;
            toff += (long long)eb.rows * br.nb[jb].dim;
        }
    P.Tsize = toff;
    for (int g = 0; g < Gl; ++g) {
        for (size_t e = 0; e < el.blk.size(); ++e)
            for (int q = 0; q < 4; ++q) {
                if (Toff[e * 4 + q] < 0) continue;
                const EnvBlk& eb = el.blk[e];
                const int jb = br.nblock(bl.nb[eb.j].n + kSigmaN[q]);
                const NBlock& NB = br.nb[jb];
                for (int sb = NB.s0; sb < NB.s1; ++sb) {
                    const Sector& SB = br.sec[sb];
                    const long long coff = g * P.Tsize + Toff[e * 4 + q] + SB.ro;
                    P.p1.add_task(B_T, coff, eb.rows, SB.dim, NB.dim);
                    const int sa = bl.sector(SB.n - kSigmaN[q], SB.m2 - kSigma2M[q]);
                    if (sa < 0) continue;
                    const int xb = si.find(sa, q);
                    if (xb < 0) continue;
                    const XBlk& X = si.blk[xb];
                    P.p1.add_term(B_ENVL, g * Lsz + eb.off + bl.sec[sa].ro, eb.cols, 1, B_X, X.off, X.cols, 1,
                                  X.rows, g * P.nc + P.c_one());
                }
            }
    }
    // ---- left pass, mixing: V(sigma, c', i) = sum W~[c, c', sigma, sigma'] T(eb(c, i), sigma')
    std::map<std::array<int, 3>, long long> Voff;  // (sigma, c', i) -> offset
    std::map<std::array<int, 3>, int> Vcols;
    long long voff = 0;
    struct VTerm { int sig, cp, i; long long toffv; int widx, e, q; };
    std::vector<VTerm> vterms;
    for (int sig = 0; sig < 4; ++sig)
        for (int cp = 0; cp < wr; ++cp)
            for (int i = 0; i < int(bl.nb.size()); ++i) {
                const int nbk = br.nblock(bl.nb[i].n + kSigmaN[sig]);
                if (nbk < 0) continue;
                const int nbp = br.nblock(br.nb[nbk].n - h->dn[k][cp]);
                if (nbp < 0) continue;
                bool any = false;
                for (const auto& ent : byL[size_t(sig) * wr + cp]) {
                    const int c = ent[0], q = ent[1];
                    const int e = el.find(c, i);
                    if (e < 0 || Toff[size_t(e) * 4 + q] < 0) continue;
                    const int jb = br.nblock(bl.nb[el.blk[e].j].n + kSigmaN[q]);
                    SP_REQUIRE(jb == nbp, "internal: inconsistent particle numbers in the MPO mixing");
                    vterms.push_back({sig, cp, i, Toff[size_t(e) * 4 + q], ent[2], e, q});
                    any = true;
                }
                if (!any) continue;
                Voff[{sig, cp, i}] = voff;
                Vcols[{sig, cp, i}] = br.nb[nbp].dim;
                voff += (long long)bl.nb[i].dim * br.nb[nbp].dim;
            }
    P.Vsize = voff;
    for (int g = 0; g < Gl; ++g) {
        size_t t = 0;
        while (t < vterms.size()) {
            const VTerm& v0 = vterms[t];
            const long long vo = Voff[{v0.sig, v0.cp, v0.i}];
            const int n = bl.nb[v0.i].dim * Vcols[{v0.sig, v0.cp, v0.i}];
            P.mixl.add_task(B_V, g * P.Vsize + vo, n);
            while (t < vterms.size() && vterms[t].sig == v0.sig && vterms[t].cp == v0.cp && vterms[t].i == v0.i) {
                P.mixl.add_term(B_T, g * P.Tsize + vterms[t].toffv, g * P.nc + P.c_wt(vterms[t].widx));
                ++t;
            }
        }
    }
    // ---- y = sum_g coef_g V R^T  and  ny = sum_g coef_g r T0 R_last^T, per (N, M) block
    const int lastR = wr - 1;
    for (const XBlk& X : si.blk) {
        const Sector& SA = bl.sec[X.sa];
        const Sector& SB = br.sec[X.sb];
        P.yout.add_task(B_Y, X.off, X.rows, X.cols, X.cols);
        for (int g = 0; g < Gl; ++g)
            for (int cp = 0; cp < wr; ++cp) {
                auto it = Voff.find({X.s, cp, SA.nb});
                if (it == Voff.end()) continue;
                const int re = er.find(cp, SB.nb);
                if (re < 0) continue;
                const EnvBlk& RB = er.blk[re];
                const int K = Vcols[{X.s, cp, SA.nb}];
                SP_REQUIRE(K == RB.cols, "internal: V and R blocks disagree");
                P.yout.add_term(B_V, g * P.Vsize + it->second + (long long)SA.ro * K, K, 1, B_ENVR,
                                g * Rsz + RB.off + (long long)SB.ro * RB.cols, 1, RB.cols, K, g * P.nc + P.c_g());
            }
    }
    for (const XBlk& X : si.blk) {
        const Sector& SA = bl.sec[X.sa];
        const Sector& SB = br.sec[X.sb];
        P.yout.add_task(B_NY, X.off, X.rows, X.cols, X.cols);
        const int e0 = el.find(0, SA.nb);
        const int re = er.find(lastR, SB.nb);
        if (e0 < 0 || re < 0) continue;
        SP_REQUIRE(el.blk[e0].j == SA.nb && er.blk[re].j == SB.nb, "internal: identity channels must conserve N");
        for (int g = 0; g < Gl; ++g)
            for (int q = 0; q < 4; ++q) {
                if (!rot_nonzero(X.s, q)) continue;
                const long long to = Toff[size_t(e0) * 4 + q];
                if (to < 0) continue;
                const int K = Tcols[size_t(e0) * 4 + q];
                const EnvBlk& RB = er.blk[re];
                SP_REQUIRE(K == RB.cols, "internal: T and R identity blocks disagree");
                P.yout.add_term(B_T, g * P.Tsize + to + (long long)SA.ro * K, K, 1, B_ENVR,
                                g * Rsz + RB.off + (long long)SB.ro * RB.cols, 1, RB.cols, K,
                                g * P.nc + P.c_gr(X.s, q));
            }
    }
    // ---- left environment update: L[k](c', b, b') rows of sector s_b = sum_sigma A^T V
    for (int g = 0; g < Gl; ++g)
        for (const EnvBlk& OB : er.blk) {
            const NBlock& NB = br.nb[OB.i];
            for (int sb = NB.s0; sb < NB.s1; ++sb) {
                const Sector& SB = br.sec[sb];
                P.envl_out.add_task(B_OUT, g * Rsz + OB.off + (long long)SB.ro * OB.cols, SB.dim, OB.cols, OB.cols);
                for (int q = 0; q < 4; ++q) {
                    const int sa = bl.sector(SB.n - kSigmaN[q], SB.m2 - kSigma2M[q]);
                    if (sa < 0) continue;
                    const int xb = si.find(sa, q);
                    if (xb < 0) continue;
                    const XBlk& X = si.blk[xb];
                    auto it = Voff.find({q, OB.c, bl.sec[sa].nb});
                    if (it == Voff.end()) continue;
                    SP_REQUIRE((Vcols[{q, OB.c, bl.sec[sa].nb}] == OB.cols), "internal: V and L blocks disagree");
                    P.envl_out.add_term(B_BRA, X.off, 1, X.cols, B_V,
                                        g * P.Vsize + it->second + (long long)bl.sec[sa].ro * OB.cols, OB.cols, 1,
                                        X.rows, g * P.nc + P.c_one());
                }
            }
        }
    // ---- right pass, phase 1: Z(rb, sigma') rows of sector s_a' = X R(rb)^T
    std::vector<long long> Zoff(er.blk.size() * 4, -1);
    long long zoff = 0;
    for (size_t e = 0; e < er.blk.size(); ++e)
        for (int q = 0; q < 4; ++q) {
            const EnvBlk& rb = er.blk[e];
            const int i = bl.nblock(br.nb[rb.j].n - kSigmaN[q]);
            if (i < 0) continue;
            Zoff[e * 4 + q] = zoff;
            zoff += (long long)bl.nb[i].dim * rb.rows;
        }
    P.Zsize = zoff;
    for (int g = 0; g < Gl; ++g)
        for (size_t e = 0; e < er.blk.size(); ++e)
            for (int q = 0; q < 4; ++q) {
                if (Zoff[e * 4 + q] < 0) continue;
                const EnvBlk& rb = er.blk[e];
                const int i = bl.nblock(br.nb[rb.j].n - kSigmaN[q]);
                const NBlock& NA = bl.nb[i];
                for (int sa = NA.s0; sa < NA.s1; ++sa) {
                    const Sector& SA = bl.sec[sa];
                    P.p1r.add_task(B_T, g * P.Zsize + Zoff[e * 4 + q] + (long long)SA.ro * rb.rows, SA.dim, rb.rows,
                                   rb.rows);
                    const int xb = si.find(sa, q);
                    if (xb < 0) continue;
                    const XBlk& X = si.blk[xb];
                    const Sector& SB = br.sec[X.sb];
                    P.p1r.add_term(B_X, X.off, X.cols, 1, B_ENVR, g * Rsz + rb.off + SB.ro, 1, rb.cols, X.cols,
                                   g * P.nc + P.c_one());
                }
            }
    // ---- right pass, mixing: Zt(sigma, c, i') = sum W~[c, c', sigma, sigma'] Z(rb(c', b), sigma')
    std::map<std::array<int, 3>, long long> Ztoff;
    std::map<std::array<int, 3>, int> Ztcols;
    long long ztoff = 0;
    std::vector<VTerm> zterms;
    for (int sig = 0; sig < 4; ++sig)
        for (int c = 0; c < wl; ++c)
            for (int ip = 0; ip < int(bl.nb.size()); ++ip) {
                const int ia = bl.nblock(bl.nb[ip].n + h->dn[k - 1][c]);
                if (ia < 0) continue;
                const int nbb = br.nblock(bl.nb[ia].n + kSigmaN[sig]);
                if (nbb < 0) continue;
                bool any = false;
                for (const auto& ent : byR[size_t(sig) * wl + c]) {
                    const int cp = ent[0], q = ent[1];
                    const int e = er.find(cp, nbb);
                    if (e < 0 || Zoff[size_t(e) * 4 + q] < 0) continue;
                    const int irow = bl.nblock(br.nb[er.blk[e].j].n - kSigmaN[q]);
                    SP_REQUIRE(irow == ip, "internal: inconsistent particle numbers in the right mixing");
                    zterms.push_back({sig, c, ip, Zoff[size_t(e) * 4 + q], ent[2]});
                    any = true;
                }
                if (!any) continue;
                Ztoff[{sig, c, ip}] = ztoff;
                Ztcols[{sig, c, ip}] = br.nb[nbb].dim;
                ztoff += (long long)bl.nb[ip].dim * br.nb[nbb].dim;
            }
    P.Ztsize = ztoff;
    for (int g = 0; g < Gl; ++g) {
        size_t t = 0;
        while (t < zterms.size()) {
            const VTerm& v0 = zterms[t];
            const long long zo = Ztoff[{v0.sig, v0.cp, v0.i}];
            const int n = bl.nb[v0.i].dim * Ztcols[{v0.sig, v0.cp, v0.i}];
            P.mixr.add_task(B_V, g * P.Ztsize + zo, n);
            while (t < zterms.size() && zterms[t].sig == v0.sig && zterms[t].cp == v0.cp && zterms[t].i == v0.i) {
                P.mixr.add_term(B_T, g * P.Zsize + zterms[t].toffv, g * P.nc + P.c_wt(zterms[t].widx));
                ++t;
            }
        }
    }
    // ---- right environment update: R(c, a, a') rows of sector s_a = sum_sigma A Zt^T
    for (int g = 0; g < Gl; ++g)
        for (const EnvBlk& OB : el.blk) {
            const NBlock& NA = bl.nb[OB.i];
            for (int sa = NA.s0; sa < NA.s1; ++sa) {
                const Sector& SA = bl.sec[sa];
                P.envr_out.add_task(B_OUT, g * Lsz + OB.off + (long long)SA.ro * OB.cols, SA.dim, OB.cols, OB.cols);
                for (int q = 0; q < 4; ++q) {
                    const int xb = si.find(sa, q);
                    if (xb < 0) continue;
                    const XBlk& X = si.blk[xb];
                    const Sector& SB = br.sec[X.sb];
                    auto it = Ztoff.find({q, OB.c, OB.j});
                    if (it == Ztoff.end()) continue;
                    const int nbcols = Ztcols[{q, OB.c, OB.j}];
                    P.envr_out.add_term(B_BRA, X.off, X.cols, 1, B_V, g * P.Ztsize + it->second + SB.ro, 1, nbcols,
                                        X.cols, g * P.nc + P.c_one());
                }
            }
        }
    // ---- diagonal of H_eff and N_eff: tiles of the site's blocks
    // the particle-conserving blocks of an MPO entry at an (N, M) block
    auto diag_blocks = [&](int c, int cp, const XBlk& X, int& e, int& re) {
        const int i = bl.sec[X.sa].nb, j = br.sec[X.sb].nb;
        e = el.find(c, i);
        re = er.find(cp, j);
        return e >= 0 && el.blk[e].j == i && re >= 0 && er.blk[re].j == j;
    };
    P.dg_direct = true;
    for (size_t q = 0; q < si.blk.size() && P.dg_direct; ++q) {
        int units = 0, e, re;
        for (const auto& ent : byD[si.blk[q].s])
            if (diag_blocks(ent[0], ent[1], si.blk[q], e, re) && (units += G) > spk::kDiagDirectMax) break;
        P.dg_direct = units <= spk::kDiagDirectMax;
    }
    std::array<int, 4> row0{}, nrow{}, zl0{}, row_n{};
    int zn = 0;
    // with many terms: the particle-conserving channels z of both bonds, and
    // per sigma one mixed row per right channel with terms
    if (!P.dg_direct) {
        std::vector<int> zl(wl, -1), zr(wr, -1);
        auto side = [&](const Bond& bd, const EnvLayout& e, std::vector<int>& z, int& nz) {
            for (int c = 0; c < e.nc; ++c) {
                bool any = false;
                for (int i = 0; i < e.nnb && !any; ++i) any = e.find(c, i) >= 0 && e.blk[e.find(c, i)].j == i;
                if (!any) continue;
                z[c] = nz++;
                for (int i = 0; i < e.nnb; ++i) {
                    const int q = e.find(c, i);
                    P.dg_src.push_back(q >= 0 && e.blk[q].j == i ? spk::DiagSrc{e.blk[q].off, e.blk[q].cols, 0}
                                                                 : spk::DiagSrc{0, -1, 0});
                }
            }
            for (int i = 0; i < int(bd.nb.size()); ++i)
                P.dg_idx.insert(P.dg_idx.end(), bd.nb[i].dim, i);
            for (const NBlock& nb : bd.nb)
                for (int p = 0; p < nb.dim; ++p) P.dg_idx.push_back(p);
        };
        side(bl, el, zl, P.dg_nzl);
        side(br, er, zr, P.dg_nzr);
        SP_REQUIRE(zl[0] >= 0 && zr[lastR] >= 0, "internal: identity channels must conserve N");
        int most = 1;
        for (int sig = 0; sig < 4; ++sig) {
            std::vector<std::vector<spk::DiagMixTerm>> of(wr);
            for (const auto& ent : byD[sig])
                if (zl[ent[0]] >= 0 && zr[ent[1]] >= 0) of[ent[1]].push_back({zl[ent[0]], P.c_cwt(ent[2])});
            row0[sig] = int(P.dg_mix.size());
            zl0[sig] = int(P.dg_idx.size());
            for (int cp = 0; cp < wr; ++cp) {
                if (of[cp].empty()) continue;
                const int t0 = int(P.dg_term.size());
                P.dg_term.insert(P.dg_term.end(), of[cp].begin(), of[cp].end());
                P.dg_mix.push_back(spk::DiagMix{t0, int(P.dg_term.size())});
                P.dg_idx.push_back(zr[cp]);
            }
            nrow[sig] = int(P.dg_mix.size()) - row0[sig];
            most = std::max(most, G * nrow[sig]);
        }
        zn = int(P.dg_idx.size());  // N_eff: the two identity strings
        P.dg_idx.push_back(zr[lastR]);
        for (int sig = 0; sig < 4; ++sig) {
            row_n[sig] = int(P.dg_mix.size());
            P.dg_term.push_back({zl[0], P.c_gr(sig, sig)});
            P.dg_mix.push_back(spk::DiagMix{int(P.dg_term.size()) - 1, int(P.dg_term.size())});
        }
        // parts of a tile: about 256 units (8 staged chunks) each, so that
        // the hundreds of rows of a wide MPO run as parallel work-groups
        P.dg_split = std::min(std::max(most / 256, 1), spk::kDiagSplitMax);
    }
    for (const XBlk& X : si.blk) {
        const Sector& SA = bl.sec[X.sa];
        const Sector& SB = br.sec[X.sb];
        const int t0 = int(P.dg_dterm.size());
        int t1 = t0;  // H_eff: terms t0 .. t1, N_eff: the one after them
        if (P.dg_direct) {
            auto term = [&](int c, int cp, int cidx) {
                int e, re;
                if (!diag_blocks(c, cp, X, e, re)) return;
                const EnvBlk &l = el.blk[e], &r = er.blk[re];
                P.dg_dterm.push_back(spk::DiagTerm{l.off + SA.ro * (l.cols + 1LL), r.off + SB.ro * (r.cols + 1LL), l.cols, r.cols, cidx, 0});
            };
            for (const auto& ent : byD[X.s]) term(ent[0], ent[1], P.c_cwt(ent[2]));
            t1 = int(P.dg_dterm.size());
            term(0, lastR, P.c_gr(X.s, X.s));
        }
        SP_REQUIRE(X.off + (long long)X.rows * X.cols < INT32_MAX, "site too large for 32-bit offsets");
        for (int r = 0; r < X.rows; r += spk::kDiagTile)
            for (int c = 0; c < X.cols; c += spk::kDiagTile)
                for (int n = 0; n < 2; ++n) {
                    spk::DiagBlk d{};
                    d.x_off = int(X.off) + r * X.cols + c;
                    d.ldc = X.cols;
                    d.rows = std::min(spk::kDiagTile, X.rows - r);
                    d.cols = std::min(spk::kDiagTile, X.cols - c);
                    d.row0 = n ? row_n[X.s] : row0[X.s];
                    d.nrow = n ? 1 : nrow[X.s];
                    d.p0 = SA.off + r;
                    d.q0 = SB.off + c;
                    d.zl0 = n ? zn : zl0[X.s];
                    d.is_n = n;
                    d.t0 = n ? t1 : t0;
                    d.t1 = n ? int(P.dg_dterm.size()) : t1;
                    d.r0 = r;
                    d.c0 = c;
                    P.dg_blk.push_back(d);
                }
    }
    // ---- QR per right sector (left-orthonormalise) and LQ per left sector
    P.qr_roff.assign(br.sec.size(), -1);
    long long sc = 0, ro = 0;
    for (int sb = 0; sb < int(br.sec.size()); ++sb) {
        spk::QrTask t{};
        t.p0 = int(P.qr_pieces.size());
        int rows = 0;
        for (const XBlk& X : si.blk)
            if (X.sb == sb) {
                P.qr_pieces.push_back(spk::QrPiece{X.off, X.rows, X.cols, 0, rows});
                rows += X.rows;
            }
        t.p1 = int(P.qr_pieces.size());
        t.rows = rows;
        t.cols = br.sec[sb].dim;
        SP_REQUIRE(t.cols <= 256, "a sector wider than 256 states is not supported");
        if (rows == 0) continue;
        SP_REQUIRE(rows >= t.cols, "block table: a sector is wider than its left support");
        t.scratch_off = sc;
        t.r_off = ro;
        P.qr_roff[sb] = ro;
        sc += 2LL * rows * t.cols;
        ro += (long long)t.cols * t.cols;
        P.qr_shape.add(t.rows, t.cols);
        P.qr_tasks.push_back(t);
    }
    P.qr_scratch = sc;
    P.qr_rsize = ro;
    P.lq_roff.assign(bl.sec.size(), -1);
    sc = 0;
    ro = 0;
    for (int sa = 0; sa < int(bl.sec.size()); ++sa) {
        spk::QrTask t{};
        t.p0 = int(P.lq_pieces.size());
        int rows = 0;
        for (const XBlk& X : si.blk)
            if (X.sa == sa) {
                P.lq_pieces.push_back(spk::QrPiece{X.off, X.rows, X.cols, 1, rows});
                rows += X.cols;
            }
        t.p1 = int(P.lq_pieces.size());
        t.rows = rows;
        t.cols = bl.sec[sa].dim;
        SP_REQUIRE(t.cols <= 256, "a sector wider than 256 states is not supported");
        if (rows == 0) continue;
        SP_REQUIRE(rows >= t.cols, "block table: a sector is wider than its right support");
        t.scratch_off = sc;
        t.r_off = ro;
        P.lq_roff[sa] = ro;
        sc += 2LL * rows * t.cols;
        ro += (long long)t.cols * t.cols;
        P.lq_shape.add(t.rows, t.cols);
        P.lq_tasks.push_back(t);
    }
    P.lq_scratch = sc;
    P.lq_rsize = ro;
    // absorb R of this site into site k+1: A[k+1](sb, ., .) <- R_sb A[k+1](sb, ., .)
    if (k < h->L) {
        const SiteInfo& sn = h->sites[k];
        for (const XBlk& X : sn.blk) {
            P.absorb_right.add_task(B_OUT, X.off, X.rows, X.cols, X.cols);
            const long long r = P.qr_roff[X.sa];
            SP_REQUIRE(r >= 0, "internal: missing R factor");
            P.absorb_right.add_term(B_V, r, X.rows, 1, B_X, X.off, X.cols, 1, X.rows, P.c_one());
        }
    }
    // absorb L of this site into site k-1: A[k-1](., ., sa) <- A[k-1](., ., sa) L_sa, L = R'^T
    if (k > 1) {
        const SiteInfo& sp = h->sites[k - 2];
        for (const XBlk& X : sp.blk) {
            P.absorb_left.add_task(B_OUT, X.off, X.rows, X.cols, X.cols);
            const long long r = P.lq_roff[X.sb];
            SP_REQUIRE(r >= 0, "internal: missing L factor");
            P.absorb_left.add_term(B_X, X.off, X.cols, 1, B_V, r, 1, X.cols, X.cols, P.c_one());
        }
    }
    // algorithmic flops of one H_eff x: per g the left product, the mixing and
    // the right product for y, and the right product of ny
    P.heff_flops = (P.p1.flops + P.mixl.flops + P.yout.flops) * (plain ? 1 : G);
    if (!plain) {
        P.p1 = P.p1r = P.yout = P.envl_out = P.envr_out = BList{};
        P.mixl = P.mixr = CList{};
        P.Tsize = P.Vsize = P.Zsize = P.Ztsize = 0;
    }

    // ================= tiled path =================
    // dense particle-number blocks Xd(j, sigma, jb) of the site (zero outside
    // the (N, M) blocks) and the map from dense elements to packed indices
    std::vector<long long> Xdoff(bl.nb.size() * 4, -1);
    long long xd = 0;
    for (int j = 0; j < int(bl.nb.size()); ++j)
        for (int q = 0; q < 4; ++q) {
            const int jb = br.nblock(bl.nb[j].n + kSigmaN[q]);
            if (jb < 0) continue;
            Xdoff[size_t(j) * 4 + q] = xd;
            xd += (long long)bl.nb[j].dim * br.nb[jb].dim;
        }
    P.Xd_size = xd;
    P.xmap_h.assign(size_t(std::max(1LL, xd)), -1);
    for (const XBlk& X : si.blk) {
        const Sector& SA = bl.sec[X.sa];
        const Sector& SB = br.sec[X.sb];
        const int ldb = br.nb[SB.nb].dim;
        const long long base = Xdoff[size_t(SA.nb) * 4 + X.s];
        for (int r = 0; r < X.rows; ++r)
            for (int c = 0; c < X.cols; ++c)
                P.xmap_h[base + (long long)(SA.ro + r) * ldb + SB.ro + c] = int(X.off + (long long)r * X.cols + c);
    }
}

// partial slots of sp_heff_apply_noalloc, doubles per output (y, ny): 16 MiB each
constexpr long long kNoAllocSlots = 1LL << 21;

// H_eff x of a wide MPO: work-groups aimed at, and the fewest channels of one
// (centre products in us, ab initio).  4096 work-groups: K = 14, D = 181 662 ->
// 793, K = 12, D = 128 194 -> 217, but K = 14, D = 64 76 -> 71; 16384: the first
// two 4 % slower.  4 channels: K = 8, D = 48 31 -> 34, K = 10, D = 24 21 -> 26;
// 16: K = 6, D = 16 13.5 -> 15.8, outer sites 10-20 % slower, K = 10, D = 24
// 21 -> 20
constexpr long long kChainGroups = 8192;
constexpr int kChainMinChannels = 8;

// chained-product lists of site k (tiled path)
void build_chain(sp_handle* h, int k) {
    SitePlan& P = h->plan[k - 1];
    const Bond& bl = h->bonds[k - 1];
    const Bond& br = h->bonds[k];
    const SiteInfo& si = h->sites[k - 1];
    const EnvLayout& el = h->env[k - 1];
    const EnvLayout& er = h->env[k];
    const int wl = h->w[k - 1], wr = h->w[k], nl = int(bl.nb.size());
    // dense particle-number blocks X(j, sigma) (the layout of xmap) and, for
    // the singly occupied states, the rotated ones
    std::vector<long long> xd(size_t(nl) * 4, -1), xr(size_t(nl) * 4, -1);
    long long nd = 0, nr = 0;
    auto right_nb = [&](int j, int q) { return br.nblock(bl.nb[j].n + kSigmaN[q]); };
    for (int j = 0; j < nl; ++j)
        for (int q = 0; q < 4; ++q)
            if (right_nb(j, q) >= 0) {
                xd[size_t(j) * 4 + q] = nd;
                nd += (long long)bl.nb[j].dim * br.nb[right_nb(j, q)].dim;
            }
    SP_REQUIRE(nd == P.Xd_size, "internal: dense site layout");
    for (int j = 0; j < nl; ++j)
        if (right_nb(j, 1) >= 0) {
            const long long n = (long long)bl.nb[j].dim * br.nb[right_nb(j, 1)].dim;
            for (long long e = 0; e < n; ++e) {
                P.rmap_h.push_back(P.xmap_h[xd[size_t(j) * 4 + 1] + e]);
                P.rmap_h.push_back(P.xmap_h[xd[size_t(j) * 4 + 2] + e]);
            }
            xr[size_t(j) * 4 + 1] = nr;
            nr += n;
        }
    for (int j = 0; j < nl; ++j)
        if (xr[size_t(j) * 4 + 1] >= 0) xr[size_t(j) * 4 + 2] = nr + xr[size_t(j) * 4 + 1];
    auto rotates = [](int q) { return q == 1 || q == 2; };
    auto xoff = [&](int j, int q) { return (q == 1 || q == 2 ? xr : xd)[size_t(j) * 4 + q]; };
    // the rows of N-block j that columns [c0, c1) of N-block jb reach through
    // the rotated state q (every state the rotation mixes into q), and the
    // columns that rows reach, as one range
    auto rows_of = [&](int jb, int q, int c0, int c1, bool rotated, int& k0, int& k1) {
        k0 = INT32_MAX;
        k1 = -1;
        const NBlock& NB = br.nb[jb];
        for (int sb = NB.s0; sb < NB.s1; ++sb) {
            const Sector& SB = br.sec[sb];
            if (SB.ro + SB.dim <= c0 || SB.ro >= c1) continue;
            for (int u = 0; u < 4; ++u) {
                if (rotated ? !rot_nonzero(q, u) : u != q) continue;
                const int sa = bl.sector(SB.n - kSigmaN[u], SB.m2 - kSigma2M[u]);
                if (sa < 0) continue;
                k0 = std::min(k0, bl.sec[sa].ro);
                k1 = std::max(k1, bl.sec[sa].ro + bl.sec[sa].dim);
            }
        }
        return k1 > k0;
    };
    auto cols_of = [&](int j, int q, int r0, int r1, bool rotated, int& k0, int& k1) {
        k0 = INT32_MAX;
        k1 = -1;
        const NBlock& NA = bl.nb[j];
        for (int sa = NA.s0; sa < NA.s1; ++sa) {
            const Sector& SA = bl.sec[sa];
            if (SA.ro + SA.dim <= r0 || SA.ro >= r1) continue;
            for (int u = 0; u < 4; ++u) {
                if (rotated ? !rot_nonzero(q, u) : u != q) continue;
                const int sb = br.sector(SA.n + kSigmaN[u], SA.m2 + kSigma2M[u]);
                if (sb < 0) continue;
                k0 = std::min(k0, br.sec[sb].ro);
                k1 = std::max(k1, br.sec[sb].ro + br.sec[sb].dim);
            }
        }
        return k1 > k0;
    };
    // entries by (sigma, right channel) as (left channel, sigma', entry) and
    // by (sigma, left channel) as (right channel, sigma', entry); where many
    // channels meet in one (wide MPOs) the environment is mixed first: once
    // for all the groups (sigma, channel, sigma') that sum the same blocks with
    // the same coefficients up to a common sign (an operator that acts as the
    // identity or the parity gives one group per local state), and groups of
    // one term read the environment block itself (K = 12 centre: 231 mixed
    // blocks instead of 1414).  The line is at 1.5 entries per group: at 1 the
    // Hubbard chain would mix (L = 32, D = 256 environment update 28 -> 67 us);
    // at 3, K = 8, D = 100 updates next to the centre go from 25 to 43 us and the
    // K = 6, D = 16 product from 13.5 to 22, while outer sites of small states,
    // where a mixing launch is half the call, would gain (18 -> 10 us)
    std::vector<std::vector<std::array<int, 3>>> byR(size_t(4) * wr), byL(size_t(4) * wl);
    std::set<std::array<int, 3>> gl, gr;
    for (int e = 0; e < int(P.wr_ent.size()); ++e) {
        const auto& q = P.wr_ent[e];
        byR[size_t(q[2]) * wr + q[1]].push_back({q[0], q[3], e});
        byL[size_t(q[2]) * wl + q[0]].push_back({q[1], q[3], e});
        gl.insert({q[2], q[1], q[3]});
        gr.insert({q[2], q[0], q[3]});
    }
    const bool mixed_l = 2 * P.wr_ent.size() > 3 * gl.size(), mixed_r = 2 * P.wr_ent.size() > 3 * gr.size();
    // V(sigma, c', i) = sum of (block, coefficient, ket block j, sigma') terms
    // of the left environment, Zt(sigma, c, b) likewise of the right one
    struct Src {
        bool mixed;
        int cols, j, q;
        double cf;
        long long off;
    };
    std::map<std::array<int, 3>, std::vector<Src>> vsrc, zsrc;
    const double* wval = P.coef_h.data() + P.c_wr(0);
    for (int side = 0; side < 2; ++side) {
        const auto& by = side ? byL : byR;
        const EnvLayout& e = side ? er : el;
        MixList& mix = side ? P.mix_r : P.mix_l;
        auto& src = side ? zsrc : vsrc;
        const int nch = side ? wl : wr, nb = int((side ? br : bl).nb.size());
        std::map<std::vector<std::pair<int, double>>, std::pair<long long, double>> same;  // terms -> mixed block, its sign
        for (int sig = 0; sig < 4; ++sig)
            for (int c = 0; c < nch; ++c)
                for (int i = 0; i < nb; ++i) {
                    std::map<std::pair<int, int>, std::vector<std::pair<int, int>>> groups;  // (j, q) -> (block, entry)
                    for (const auto& ent : by[size_t(sig) * nch + c]) {
                        const int b = e.find(ent[0], i), q = ent[1];
                        if (b < 0) continue;
                        const int j = e.blk[b].j;
                        if (side == 0 ? right_nb(j, q) < 0 : bl.nblock(br.nb[j].n - kSigmaN[q]) < 0) continue;
                        groups[{j, q}].push_back({b, ent[2]});
                    }
                    for (const auto& g : groups) {
                        const EnvBlk& b0 = e.blk[g.second[0].first];
                        if (!(side ? mixed_r : mixed_l) || g.second.size() == 1) {
                            for (const auto& t : g.second)
                                src[{sig, c, i}].push_back(Src{false, b0.cols, g.first.first, g.first.second, wval[t.second],
                                                               e.blk[t.first].off});
                            continue;
                        }
                        const double sgn = wval[g.second[0].second] < 0.0 ? -1.0 : 1.0;
                        std::vector<std::pair<int, double>> key;
                        for (const auto& t : g.second) key.push_back({t.first, sgn * wval[t.second]});
                        auto it = same.find(key);
                        if (it == same.end()) {
                            std::vector<std::pair<int, double>> terms;
                            for (const auto& t : g.second) terms.push_back({t.first, wval[t.second]});
                            it = same.emplace(key, std::make_pair(mix.add(b0.i, b0.j, b0.rows * b0.cols, terms), sgn)).first;
                        }
                        src[{sig, c, i}].push_back(Src{true, b0.cols, g.first.first, g.first.second,
                                                       it->second.second == sgn ? 1.0 : -1.0, it->second.first});
                    }
                }
    }
    P.mix_l.finish(el);
    P.mix_r.finish(er);
    auto shape_for = [](int m, bool wide) {  // the smallest tile that takes m, or the largest
        int sh = wide ? spk::kNarrowShapes : 0;
        const int end = wide ? spk::kNumChainShapes : spk::kNarrowShapes;
        while (sh + 1 < end && 16 * spk::kChainShapes[sh].nm < m) ++sh;
        return sh;
    };
    // Two blocks in n halve the reads of A and P per product.  The BF16 matrix
    // cores wait for reads and splits, and gain (K = 14, D = 181, site 6: 541 us
    // against 645 with one; K = 12, D = 128 200 against 203); FP64 needs its
    // registers for wavefronts in flight (K = 12, D = 128, site 7: 361 us against
    // 297 with one; at the wider blocks of K = 16, D = 256 1837 against 2056)
    const bool wide_h = mixed_l && h->precision == SP_BF16X3;
    // Environment updates: an output block is a sum over few steps with a
    // narrow MPO, split over four wavefronts (L = 32, D = 256: 28 us against
    // 70 with one); a wide MPO has thousands of blocks of many steps each, and
    // a wavefront per tile saves the LDS sums (K = 12, D = 128, site 6: 221 us
    // against 260 with four for the left update, 380 with either for the right;
    // small wide states have too few tiles for it: K = 6, D = 16 16 us against 13)
    if (mixed_l || mixed_r) P.c_envl.waves = P.c_envr.waves = 1;
    int dl = 1, dr = 1;
    for (const NBlock& nb : bl.nb) dl = std::max(dl, nb.dim);
    for (const NBlock& nb : br.nb) dr = std::max(dr, nb.dim);
    // H_eff x, transposed: y(a, sigma, b) = sum_c' sum_k R(c')(b, k) V(sigma, c', i)(a, k)
    // in tiles of 16 rows a by the columns b that those rows reach; N_eff x
    // from the identity strings, V = L(0) X and R of the last channel
    {
        ChainList& C = P.c_heff;
        C.lay = spk::kChainHeff;
        const int lastR = wr - 1, TN = 16 * spk::kChainShapes[shape_for(1, wide_h)].nn;
        struct Tile {
            int i, q, b, n0, n1, m0, m1;
        };
        std::vector<Tile> rows, tiles;
        int widest = 1;
        for (int i = 0; i < nl; ++i)
            for (int q = 0; q < 4; ++q) {
                const int b = right_nb(i, q);
                if (b < 0) continue;
                for (int n0 = 0; n0 < bl.nb[i].dim; n0 += TN) {
                    const int n1 = std::min(bl.nb[i].dim, n0 + TN);
                    int c0, c1;
                    if (!cols_of(i, q, n0, n1, false, c0, c1)) continue;
                    rows.push_back({i, q, b, n0, n1, c0, c1});
                    widest = std::max(widest, c1 - c0);
                }
            }
        C.shape = shape_for(widest, wide_h);
        const int TM = 16 * spk::kChainShapes[C.shape].nm, TI = 16 * spk::kChainShapes[C.shape].ni;
        for (const Tile& t : rows)
            for (int m0 = t.m0; m0 < t.m1; m0 += TM) tiles.push_back({t.i, t.q, t.b, t.n0, t.n1, m0, std::min(t.m1, m0 + TM)});
        // the widest first: the launch ends with the short ones
        std::stable_sort(tiles.begin(), tiles.end(), [&](const Tile& x, const Tile& y) { return br.nb[x.b].dim > br.nb[y.b].dim; });
        // channels of a tile in chunks, each its own work-group and partial
        // slot, where the tiles alone leave the chip short of work-groups
        int most = 1;
        for (const Tile& t : tiles) {
            int n = 0;
            for (int cp = 0; cp < wr; ++cp) n += vsrc.count({t.q, cp, t.i}) && er.find(cp, t.b) >= 0;
            most = std::max(most, n);
        }
        long long want = std::max<long long>(1, kChainGroups / std::max<long long>(1, (long long)tiles.size() * h->G));
        // a site with a fused plan keeps to the fixed slots wherever one slot
        // per g does
        const long long per = std::max<long long>(1, h->G * si.size);
        if (P.h_rows > 0 && per <= kNoAllocSlots) want = std::min(want, kNoAllocSlots / per);
        const int chunk = int(std::max<long long>(kChainMinChannels, (most + want - 1) / want));
        P.y_split = std::max(1, (most + chunk - 1) / chunk);
        for (const Tile& t : tiles) {
            const long long mo = xd[size_t(t.i) * 4 + t.q];
            const int nn = br.nb[t.b].dim;
            int n = 0, slot = 0;
            auto end = [&]() {
                C.end_tile(spk::KTile{(long long)slot * h->G * si.size, mo + (long long)t.n0 * nn + t.m0, t.m1 - t.m0, t.n1 - t.n0,
                                      nn, P.c_g(), {}, 0, 0, 0});
                ++slot;
            };
            const int e0 = el.find(0, t.i), rl = er.find(lastR, t.b);
            SP_REQUIRE(e0 >= 0 && rl >= 0 && el.blk[e0].j == t.i && er.blk[rl].j == t.b, "internal: identity channels must conserve N");
            C.begin_tile(t.m0, t.n0);
            for (int c0 = 0; c0 < nn; c0 += TI) {  // N_eff x, with the first chunk
                const int c1 = std::min(nn, c0 + TI);
                int k0, k1;
                C.begin_step(er.blk[rl].off, nn, c0, c1, true);
                if (rows_of(t.b, t.q, c0, c1, true, k0, k1))
                    C.add_seg(xoff(t.i, t.q), nn, el.blk[e0].off, el.blk[e0].cols, k0, k1, 1.0, rotates(t.q), false, true);
            }
            for (int cp = 0; cp < wr; ++cp) {
                auto it = vsrc.find({t.q, cp, t.i});
                const int re = er.find(cp, t.b);
                if (it == vsrc.end() || re < 0) continue;
                if (n > 0 && n % chunk == 0) end();
                ++n;
                const EnvBlk& RB = er.blk[re];
                for (int c0 = 0; c0 < RB.cols; c0 += TI) {
                    const int c1 = std::min(RB.cols, c0 + TI);
                    C.begin_step(RB.off, RB.cols, c0, c1);
                    for (const Src& v : it->second) {
                        int k0, k1;
                        SP_REQUIRE(right_nb(v.j, v.q) == RB.j, "internal: H_eff particle numbers");
                        if (rows_of(RB.j, v.q, c0, c1, true, k0, k1))
                            C.add_seg(xoff(v.j, v.q), RB.cols, v.off, v.cols, k0, k1, v.cf, rotates(v.q), v.mixed);
                    }
                }
            }
            while (slot < P.y_split) end();  // slots without channels: zeros
        }
    }
    // left environment L[k](c', b, b') = sum_sigma X(a, sigma, b)^T V(sigma, c', a)(a, b')
    P.c_envl.lay = spk::kChainEnvL;
    P.c_envl.shape = shape_for(dr, false);
    P.c_envr.lay = spk::kChainEnvR;
    P.c_envr.shape = shape_for(dl, false);
    for (int side = 0; side < 2; ++side) {
        ChainList& C = side ? P.c_envr : P.c_envl;
        const spk::KShape sh = spk::kChainShapes[C.shape];
        const int TM = 16 * sh.nm, TI = 16 * sh.ni, TN = 16 * sh.nn;
        for (const EnvBlk& OB : (side ? el : er).blk)
            for (int m0 = 0; m0 < OB.rows; m0 += TM)
                for (int n0 = 0; n0 < OB.cols; n0 += TN) {
                    const int m1 = std::min(OB.rows, m0 + TM), n1 = std::min(OB.cols, n0 + TN);
                    C.begin_tile(m0, n0);
                    for (int q = 0; q < 4; ++q) {
                        int b0, b1;
                        if (side == 0) {  // X(a, q)^T: b = OB.i, a on the left bond
                            const int a = bl.nblock(br.nb[OB.i].n - kSigmaN[q]);
                            if (a < 0) continue;
                            auto it = vsrc.find({q, OB.c, a});
                            if (it == vsrc.end() || !rows_of(OB.i, q, m0, m1, false, b0, b1)) continue;
                            for (int c0 = b0; c0 < b1; c0 += TI) {
                                C.begin_step(xd[size_t(a) * 4 + q], OB.rows, c0, std::min(b1, c0 + TI));
                                for (const Src& v : it->second) {
                                    int k0, k1;
                                    SP_REQUIRE(right_nb(v.j, v.q) == OB.j, "internal: left environment particle numbers");
                                    if (rows_of(OB.j, v.q, n0, n1, true, k0, k1))
                                        C.add_seg(v.off, v.cols, xoff(v.j, v.q), OB.cols, k0, k1, v.cf, rotates(v.q), v.mixed);
                                }
                            }
                        } else {  // X(a, q): a = OB.i, b on the right bond
                            const int b = right_nb(OB.i, q);
                            if (b < 0) continue;
                            auto it = zsrc.find({q, OB.c, b});
                            if (it == zsrc.end() || !cols_of(OB.i, q, m0, m1, false, b0, b1)) continue;
                            for (int c0 = b0; c0 < b1; c0 += TI) {
                                C.begin_step(xd[size_t(OB.i) * 4 + q], br.nb[b].dim, c0, std::min(b1, c0 + TI));
                                for (const Src& v : it->second) {
                                    int k0, k1;
                                    SP_REQUIRE(right_nb(OB.j, v.q) == v.j, "internal: right environment particle numbers");
                                    if (cols_of(OB.j, v.q, n0, n1, true, k0, k1))
                                        C.add_seg(v.off, v.cols, xoff(OB.j, v.q), br.nb[v.j].dim, k0, k1, v.cf, rotates(v.q), v.mixed);
                                }
                            }
                        }
                    }
                    C.end_tile(spk::KTile{OB.off + (long long)m0 * OB.cols + n0, 0, m1 - m0, n1 - n0, OB.cols, -1, {}, 0, 0, 0});
                }
    }
}

// LDS budget of a fused plan of H_eff x (doubles): the default, and the
// largest the autotuner tries (the 160 KB of a CU less static arrays)
constexpr int kHeffLdsBudget = 9216;
constexpr int kHeffLdsMax = 18432;
constexpr int kHeffMaxRows = 8;

// The fused plan of site k for an LDS budget: rows per task RC such that RC
// rows of every left-environment block, of every product L(c) x[sigma'] and
// of the right channels of one sigma fit.  Every site runs the same chained
// lists; the plan decides in which arithmetic they run in the reduced
// precisions: FP32 (RC >= 1), or as block products (RC = 0: the MPO is too
// wide, or the caller chose so).  Returns false where no row fits.
bool build_fused(sp_handle* h, int k, int lds_budget = kHeffLdsBudget) {
    SitePlan& P = h->plan[k - 1];
    const Bond& bl = h->bonds[k - 1];
    const Bond& br = h->bonds[k];
    const EnvLayout& el = h->env[k - 1];
    const EnvLayout& er = h->env[k];
    const int wl = h->w[k - 1], wr = h->w[k];
    std::vector<std::vector<std::array<int, 2>>> by(size_t(4) * wr);  // (left channel, sigma') by (sigma, right channel)
    for (const auto& q : P.went) by[size_t(q[2]) * wr + q[1]].push_back({q[0], q[3]});
    auto right_nb = [&](int j, int q) { return br.nblock(bl.nb[j].n + kSigmaN[q]); };
    int need1 = 1;
    for (int i = 0; i < int(bl.nb.size()); ++i) {
        int lsum = 0, tsum = 0, vmax = 0;
        for (int c = 0; c < wl; ++c) {
            const int e = el.find(c, i);
            if (e < 0) continue;
            lsum += el.blk[e].cols;
            for (int q = 0; q < 4; ++q)
                if (right_nb(el.blk[e].j, q) >= 0) tsum += br.nb[right_nb(el.blk[e].j, q)].dim;
        }
        for (int sig = 0; sig < 4; ++sig) {
            const int nbb = right_nb(i, sig);
            if (nbb < 0) continue;
            int v = 0;
            for (int cp = 0; cp < wr; ++cp) {
                const int re = er.find(cp, nbb);
                if (re < 0) continue;
                for (const auto& ent : by[size_t(sig) * wr + cp]) {
                    const int e = el.find(ent[0], i);
                    if (e < 0 || right_nb(el.blk[e].j, ent[1]) < 0) continue;
                    v += er.blk[re].cols;
                    break;
                }
            }
            const int e0 = el.find(0, i), re = er.find(wr - 1, nbb);
            if (re >= 0 && e0 >= 0) v += er.blk[re].cols;  // N_eff
            vmax = std::max(vmax, v);
        }
        need1 = std::max(need1, lsum + tsum + vmax);
    }
    const int RC = std::min(kHeffMaxRows, lds_budget / need1);
    P.h_rows = std::max(0, RC);
    P.h_lds = P.h_rows * need1;
    return RC >= 1;
}

// f(1) .. f(L) on up to eight threads (sites only write their own plan); the
// error of the lowest site, if any
template <class F>
void for_sites(int L, F f) {
    std::vector<std::exception_ptr> err(L);
    std::atomic<int> next{0};
    auto work = [&]() {
        for (int k = next++; k < L; k = next++) try {
                f(k + 1);
            } catch (...) {
                err[k] = std::current_exception();
            }
    };
    const int nt = std::min({8, L / 2, int(std::thread::hardware_concurrency())});
    std::vector<std::thread> threads;
    try {
        threads.reserve(std::max(nt, 1));
        for (int t = 1; t < nt; ++t) threads.emplace_back(work);
    } catch (...) {  // no more threads: those there, and this one, do the work
    }
    work();
    for (auto& t : threads) t.join();
    for (const auto& e : err)
        if (e) std::rethrow_exception(e);
}

void upload_plan(sp_handle* h, int k, Upload& u) {
    SitePlan& P = h->plan[k - 1];
    u.add(P.coef, P.coef_h);
    P.p1.upload(u);
    P.mixl.upload(u);
    P.yout.upload(u);
    P.envl_out.upload(u);
    P.p1r.upload(u);
    P.mixr.upload(u);
    P.envr_out.upload(u);
    u.add(P.ddg_src, P.dg_src);
    u.add(P.ddg_idx, P.dg_idx);
    u.add(P.ddg_mix, P.dg_mix);
    u.add(P.ddg_term, P.dg_term);
    u.add(P.ddg_blk, P.dg_blk);
    u.add(P.ddg_dterm, P.dg_dterm);
    u.add(P.dqr_tasks, P.qr_tasks);
    u.add(P.dlq_tasks, P.lq_tasks);
    u.add(P.dqr_pieces, P.qr_pieces);
    u.add(P.dlq_pieces, P.lq_pieces);
    P.absorb_right.upload(u);
    P.absorb_left.upload(u);
    u.add(P.xmap, P.xmap_h);
    P.c_heff.upload(u);
    P.c_envl.upload(u);
    P.c_envr.upload(u);
    P.mix_l.upload(u);
    P.mix_r.upload(u);
    u.add(P.rmap, P.rmap_h);
}

// ---------------------------------------------------------------------------
// bounds validation of every task list against the buffers it will touch
// (host side, at init): a descriptor error becomes SP_EINVAL, never a device
// memory fault

using Sizes = std::array<long long, spk::kMaxBufs>;

void check_span(long long off, long long last, long long size, const char* what) {
    if (off < 0 || last < off || last >= size) throw SpError(SP_EINVAL, std::string("internal bounds check: ") + what);
}

void validate(const BList& b, const Sizes& sz, long long ncoef, const char* what) {
    for (const spk::BTask& t : b.tasks) {
        if (t.M <= 0 || t.N <= 0) continue;
        check_span(t.c_off, t.c_off + (long long)(t.M - 1) * t.ldc + (t.N - 1), sz[t.c_buf], what);
        for (int i = t.t0; i < t.t1; ++i) {
            const spk::BTerm& m = b.terms[i];
            if (m.K <= 0) throw SpError(SP_EINVAL, std::string("internal: empty term in ") + what);
            check_span(m.a_off, m.a_off + (long long)(t.M - 1) * m.a_rs + (long long)(m.K - 1) * m.a_cs,
                       sz[m.a_buf], what);
            check_span(m.b_off, m.b_off + (long long)(m.K - 1) * m.b_rs + (long long)(t.N - 1) * m.b_cs,
                       sz[m.b_buf], what);
            check_span(m.cidx, m.cidx, ncoef, what);
        }
    }
}

void validate(const CList& b, const Sizes& sz, long long ncoef, const char* what) {
    for (const spk::CTask& t : b.tasks) {
        check_span(t.c_off, t.c_off + t.n - 1, sz[t.c_buf], what);
        for (int i = t.t0; i < t.t1; ++i) {
            check_span(b.terms[i].a_off, b.terms[i].a_off + t.n - 1, sz[b.terms[i].a_buf], what);
            check_span(b.terms[i].cidx, b.terms[i].cidx, ncoef, what);
        }
    }
}

// bounds of a chained product: in[] the values per quadrature point of every
// operand buffer, nout of the output, npart the outputs a tile may scatter to
void validate(const ChainList& C, const std::array<long long, spk::K_NBUF>& in, long long nout, long long map_size,
              long long npart, long long ncoef, const char* what) {
    if (C.shape < 0 || C.shape >= spk::kNumChainShapes) throw SpError(SP_EINVAL, std::string("internal shape: ") + what);
    const spk::KShape sh = spk::kChainShapes[C.shape];
    for (const spk::KTile& t : C.tiles) {
        if (t.m < 1 || t.n < 1 || t.m > 16 * sh.nm || t.n > 16 * sh.nn || t.e0 < 0 || t.e1 < t.e0 ||
            (C.lay != spk::kChainHeff && t.e1 > t.e0) || t.s[0] < t.e1 || !std::is_sorted(t.s, t.s + 5) ||
            t.s[4] > int(C.steps.size()) || t.s[C.waves] != t.s[4])
            throw SpError(SP_EINVAL, std::string("internal tile: ") + what);
        if (t.cidx >= 0) check_span(t.cidx, t.cidx, ncoef, what);
        if (C.lay == spk::kChainHeff) {
            check_span(t.map_off, t.map_off + (t.n - 1LL) * t.ldo + t.m - 1, map_size, what);
            check_span(t.o_off, t.o_off + npart - 1, nout, what);
        } else {
            check_span(t.o_off, t.o_off + (t.m - 1LL) * t.ldo + t.n - 1, nout, what);
        }
        for (int q = t.e0; q < t.s[4]; ++q) {
            if (q >= t.e1 && q < t.s[0]) continue;
            const spk::KStep& p = C.steps[q];
            if (p.nkc < 1 || p.nkc > 16 * sh.ni || p.g0 < 0 || p.g1 <= p.g0 || p.g1 > int(C.segs.size()))
                throw SpError(SP_EINVAL, std::string("internal step: ") + what);
            const bool pt = C.lay == spk::kChainEnvL;
            // the last element from the first, rows ld apart
            auto span = [&](long long off, long long rows, int ld, int run, long long size) {
                if (!spk::chain_lanes_fit(ld)) throw SpError(SP_EINVAL, std::string("block too wide: ") + what);
                check_span(off, off + (rows - 1) * ld + run - 1, size, what);
            };
            span(p.p_off, pt ? p.nkc : t.m, p.ldp, pt ? t.m : p.nkc, in[C.lay == spk::kChainHeff ? spk::K_R : spk::K_X]);
            for (int i = p.g0; i < p.g1; ++i) {
                const spk::KSeg& g = C.segs[i];
                if (g.nk < 1) throw SpError(SP_EINVAL, std::string("internal segment: ") + what);
                const bool at = C.lay == spk::kChainHeff, bt = C.lay == spk::kChainEnvL;
                const long long nx = in[g.alt_x ? spk::K_XR : spk::K_X];
                const long long ne = in[g.alt_e ? spk::K_LT : (C.lay == spk::kChainEnvR ? spk::K_R : spk::K_L)];
                span(g.a_off, at ? g.nk : p.nkc, g.lda, at ? p.nkc : g.nk, at ? nx : ne);
                span(g.b_off, bt ? g.nk : t.n, g.ldb, bt ? t.n : g.nk, at ? ne : nx);
            }
        }
    }
}

void validate(const MixList& m, long long nin, long long nout, const char* what) {
    for (const spk::MixWork& w : m.work) {
        if (w.tile0 < 0 || w.tile1 <= w.tile0 || w.tile1 > int(m.tiles.size()) || w.e0 < 0 || w.e0 >= w.n)
            throw SpError(SP_EINVAL, std::string("internal work: ") + what);
        if (w.e0 > 0) continue;  // the first chunk of a shape stands for all
        for (int t = w.tile0; t < w.tile1; ++t) {
            const spk::MixTileRec& r = m.tiles[t];
            if (r.s0 < 0 || r.s1 < r.s0 || r.s1 - r.s0 > spk::kMixTile || r.s1 > int(m.src.size()) || r.i0 < 0 || r.i1 < r.i0 ||
                r.i1 > int(m.groups.size()))
                throw SpError(SP_EINVAL, std::string("internal tile: ") + what);
            for (int q = r.s0; q < r.s1; ++q) check_span(m.src[q], m.src[q] + w.n - 1, nin, what);
            for (int i = r.i0; i < r.i1; ++i) {
                const spk::MixGroup& it = m.groups[i];
                if (it.n < 1 || it.n > spk::kMixGroup || it.t0 < 0 || it.t1 <= it.t0 || it.t1 > int(m.at.size()) ||
                    m.cf.size() != m.at.size() * spk::kMixGroup)
                    throw SpError(SP_EINVAL, std::string("internal terms: ") + what);
                for (int b = 0; b < it.n; ++b) check_span(it.o[b], it.o[b] + w.n - 1, nout, what);
                for (int q = it.t0; q < it.t1; ++q) check_span(m.at[q], m.at[q], r.s1 - r.s0, what);
            }
        }
    }
}

// bounds of the lists of the diagonals of site k
void validate_diag(const sp_handle* h, int k) {
    const SitePlan& P = h->plan[k - 1];
    const Bond& bl = h->bonds[k - 1];
    const Bond& br = h->bonds[k];
    const int nidx = int(P.dg_idx.size()), nmix = int(P.dg_mix.size());
    const size_t nl = size_t(P.dg_nzl) * bl.nb.size(), nr = size_t(P.dg_nzr) * br.nb.size();
    const bool direct = P.dg_direct;
    if (P.dg_src.size() != nl + nr || (!direct && nidx < 2 * (bl.D + br.D))) throw SpError(SP_EINVAL, "internal: diagonal sources");
    for (size_t q = 0; q < nl + nr; ++q) {
        const spk::DiagSrc& d = P.dg_src[q];
        if (d.ld < 0) continue;
        const NBlock& nb = q < nl ? bl.nb[q % bl.nb.size()] : br.nb[(q - nl) % br.nb.size()];
        check_span(d.off, d.off + (long long)(nb.dim - 1) * (d.ld + 1), h->env[q < nl ? k - 1 : k].size, "diagonal source");
    }
    for (const spk::DiagMix& m : P.dg_mix)
        if (m.t0 < 0 || m.t1 <= m.t0 || m.t1 > int(P.dg_term.size())) throw SpError(SP_EINVAL, "internal: diagonal row");
    for (const spk::DiagMixTerm& t : P.dg_term) {
        check_span(t.z, t.z, P.dg_nzl, "diagonal term");
        check_span(t.cidx, t.cidx, P.nc, "diagonal coefficient");
    }
    for (const spk::DiagBlk& d : P.dg_blk) {
        if (d.rows < 1 || d.cols < 1 || d.rows > spk::kDiagTile || d.cols > spk::kDiagTile || d.nrow < 0)
            throw SpError(SP_EINVAL, "internal: diagonal tile");
        check_span(d.x_off, d.x_off + (long long)(d.rows - 1) * d.ldc + d.cols - 1, h->sites[k - 1].size, "diagonal block");
        if (direct) {
            if (d.t0 < 0 || d.t1 < d.t0 || d.t1 > int(P.dg_dterm.size()) || d.r0 < 0 || d.c0 < 0)
                throw SpError(SP_EINVAL, "internal: diagonal terms");
            for (int i = d.t0; i < d.t1; ++i) {
                const spk::DiagTerm& t = P.dg_dterm[i];
                check_span(t.l_off, t.l_off + (d.r0 + d.rows - 1) * (t.l_ld + 1LL), h->env[k - 1].size, "diagonal rows");
                check_span(t.r_off, t.r_off + (d.c0 + d.cols - 1) * (t.r_ld + 1LL), h->env[k].size, "diagonal columns");
                check_span(t.cidx, t.cidx, P.nc, "diagonal coefficient");
            }
            continue;
        }
        check_span(d.p0, d.p0 + d.rows - 1, bl.D, "diagonal rows");
        check_span(d.q0, d.q0 + d.cols - 1, br.D, "diagonal columns");
        if (d.nrow == 0) continue;
        check_span(d.row0, d.row0 + d.nrow - 1, nmix, "diagonal units");
        check_span(d.zl0, d.zl0 + d.nrow - 1, nidx, "diagonal channels");
        for (int u = 0; u < d.nrow; ++u) check_span(P.dg_idx[d.zl0 + u], P.dg_idx[d.zl0 + u], P.dg_nzr, "diagonal channel");
    }
    const long long G = h->G;
    if (G * ((long long)P.dg_nzl * bl.D + (long long)P.dg_nzr * br.D) > h->T_cap || G * nmix * bl.D > h->V_cap)
        throw SpError(SP_EINVAL, "internal: diagonal scratch too small");
}

void validate_plans(sp_handle* h) {
    const long long G = h->G;
    for (int k = 1; k <= h->L; ++k) {
        const SitePlan& P = h->plan[k - 1];
        const long long nco = G * P.nc;
        const long long xs = h->sites[k - 1].size;
        const long long Lb = G * h->env[k - 1].size, Rb = G * h->env[k].size;
        const long long Tb = h->T_cap, Vb = h->V_cap;
        Sizes z{};
        z.fill(0);
        z[B_ENVL] = Lb;
        z[B_ENVR] = Rb;
        z[B_X] = xs;
        z[B_T] = Tb;
        z[B_V] = Vb;
        z[B_Y] = xs;
        z[B_NY] = xs;
        z[B_BRA] = xs;
        if (G * P.Tsize > Tb || G * P.Vsize > Vb || G * P.Zsize > Tb || G * P.Ztsize > Vb)
            throw SpError(SP_EINVAL, "internal: scratch too small");
        validate(P.p1, z, nco, "left product");
        validate(P.mixl, z, nco, "left mixing");
        validate(P.yout, z, nco, "H_eff output");
        validate(P.p1r, z, nco, "right product");
        validate(P.mixr, z, nco, "right mixing");
        z[B_OUT] = Rb;
        validate(P.envl_out, z, nco, "left environment");
        z[B_OUT] = Lb;
        validate(P.envr_out, z, nco, "right environment");
        {
            for (int e : P.xmap_h)
                if (e >= xs) throw SpError(SP_EINVAL, "internal: packed map out of range");
            const long long ms = (long long)P.xmap_h.size();
            if (h->path == SP_PATH_TILED) {
                const long long Lg = h->env[k - 1].size, Rg = h->env[k].size;
                if (G * std::max(P.mix_l.size, P.mix_r.size) > h->LT_cap || G * (long long)P.rmap_h.size() > h->Xr_cap)
                    throw SpError(SP_EINVAL, "internal: scratch of the chained products too small");
                for (int e : P.rmap_h)
                    if (e >= xs) throw SpError(SP_EINVAL, "internal: packed map out of range");
                validate(P.mix_l, Lg, P.mix_l.size, "pre-mixed left environment");
                validate(P.mix_r, Rg, P.mix_r.size, "pre-mixed right environment");
                const long long nxr = (long long)P.rmap_h.size();
                validate(P.c_heff, {Lg, Rg, P.Xd_size, nxr, P.mix_l.size}, P.y_split * G * xs, ms, xs, P.nc, "H_eff x");
                validate(P.c_envl, {Lg, 0, P.Xd_size, nxr, P.mix_l.size}, Rg, 0, 0, P.nc, "left environment update");
                validate(P.c_envr, {0, Rg, P.Xd_size, nxr, P.mix_r.size}, Lg, 0, 0, P.nc, "right environment update");
            }
            if (P.Xd_size > h->Xd_cap) throw SpError(SP_EINVAL, "internal: dense site scratch too small");
        }
        if (k < h->L) {
            Sizes a{};
            a.fill(0);
            a[B_V] = h->qr_r_cap;
            a[B_X] = h->sites[k].size;
            a[B_OUT] = std::min<long long>(h->sites[k].size, h->max_site);
            validate(P.absorb_right, a, P.nc, "absorb right");
        }
        if (k > 1) {
            Sizes a{};
            a.fill(0);
            a[B_V] = h->qr_r_cap;
            a[B_X] = h->sites[k - 2].size;
            a[B_OUT] = std::min<long long>(h->sites[k - 2].size, h->max_site);
            validate(P.absorb_left, a, P.nc, "absorb left");
        }
        for (int pass = 0; pass < 2; ++pass) {
            const auto& tasks = pass ? P.lq_tasks : P.qr_tasks;
            const auto& pieces = pass ? P.lq_pieces : P.qr_pieces;
            for (const spk::QrTask& t : tasks) {
                if (t.cols > 256 || t.rows < t.cols) throw SpError(SP_EINVAL, "internal: bad QR task");
                check_span(t.scratch_off, t.scratch_off + 2LL * t.rows * t.cols - 1, h->qr_scratch_cap, "QR scratch");
                check_span(t.r_off, t.r_off + (long long)t.cols * t.cols - 1, h->qr_r_cap, "QR factor");
                int rows = 0;
                for (int i = t.p0; i < t.p1; ++i) {
                    const spk::QrPiece& pc = pieces[i];
                    check_span(pc.off, pc.off + (long long)pc.prow * pc.pcol - 1, xs, "QR piece");
                    if ((pc.transposed ? pc.prow : pc.pcol) != t.cols || pc.row0 != rows)
                        throw SpError(SP_EINVAL, "internal: QR piece shape");
                    rows += pc.transposed ? pc.pcol : pc.prow;
                }
                if (rows != t.rows) throw SpError(SP_EINVAL, "internal: QR rows");
            }
        }
        validate_diag(h, k);
    }
}

// ---------------------------------------------------------------------------
// operations

double* site_ptr(sp_handle* h, int k) { return h->mps.p + h->sites[k - 1].goff; }

// the N-blocks of site k's tensor: its (left sector, sigma) blocks grouped by
// the left bond's particle number and that of sigma (hence also the right
// bond's), whatever their M
const NBlocks& site_nblocks(sp_handle* h, int k) {
    if (h->nblocks.size() != size_t(h->L)) h->nblocks.resize(h->L);
    NBlocks& nb = h->nblocks[k - 1];
    if (nb.ng > 0) return nb;
    const SiteInfo& si = h->sites[k - 1];
    const Bond& bl = h->bonds[k - 1];
    std::map<std::pair<int, int>, int> key;
    std::vector<int> grp(si.blk.size());
    for (size_t b = 0; b < si.blk.size(); ++b) {
        const XBlk& x = si.blk[b];
        grp[b] = key.emplace(std::make_pair(bl.sec[x.sa].n, kSigmaN[x.s]), int(key.size())).first->second;
    }
    const int ng = int(key.size());
    nb.gptr_h.assign(ng + 1, 0);
    for (int g : grp) ++nb.gptr_h[g + 1];
    for (int g = 0; g < ng; ++g) nb.gptr_h[g + 1] += nb.gptr_h[g];
    nb.roff_h.assign(si.blk.size(), 0);
    nb.rlen_h.assign(si.blk.size(), 0);
    nb.gid_h.assign(size_t(si.size), 0);
    std::vector<int> fill(nb.gptr_h.begin(), nb.gptr_h.end() - 1);
    for (size_t b = 0; b < si.blk.size(); ++b) {  // site order inside a group
        const XBlk& x = si.blk[b];
        const long long len = (long long)x.rows * x.cols;
        const int j = fill[grp[b]]++;
        nb.roff_h[j] = x.off;
        nb.rlen_h[j] = int(len);
        std::fill(nb.gid_h.begin() + x.off, nb.gid_h.begin() + x.off + len, grp[b]);
    }
    nb.gptr.upload(nb.gptr_h, h->stream);
    nb.roff.upload(nb.roff_h, h->stream);
    nb.rlen.upload(nb.rlen_h, h->stream);
    nb.gid.upload(nb.gid_h, h->stream);
    nb.ng = ng;
    return nb;
}

spk::BufSet bufset(sp_handle* h, int k, const double* x, double* y, double* ny, double* out) {
    spk::BufSet b{};
    b.p[B_ENVL] = h->envL[k - 1].p;
    b.p[B_ENVR] = h->envR[k].p;
    b.p[B_X] = const_cast<double*>(x);
    b.p[B_T] = h->T.p;
    b.p[B_V] = h->V.p;
    b.p[B_Y] = y;
    b.p[B_NY] = ny;
    b.p[B_OUT] = out;
    b.p[B_BRA] = const_cast<double*>(x);
    return b;
}

void check_site(const sp_handle* h, int k) { SP_REQUIRE(k >= 1 && k <= h->L, "site out of range"); }

// operands of a chained product at site k (x prepared by site_vectors)
spk::KInst chain_inst(sp_handle* h, int k, const ChainList& C, const MixList& mix) {
    const SitePlan& P = h->plan[k - 1];
    spk::KInst I{};
    I.tiles = C.dtiles.p;
    I.steps = C.dsteps.p;
    I.segs = C.dsegs.p;
    I.map = P.xmap.p;
    I.coef = P.coef.p;
    I.in[spk::K_L] = {h->envL[k - 1].p, h->env[k - 1].size};
    I.in[spk::K_R] = {h->envR[k].p, h->env[k].size};
    I.in[spk::K_X] = {h->Xd.p, 0};
    I.in[spk::K_XR] = {h->Xr.p, (long long)P.rmap_h.size()};
    I.in[spk::K_LT] = {h->LT.p, mix.size};
    I.ntile = int(C.tiles.size());
    I.nc = P.nc;
    I.G = h->G;
    return I;
}

// dense and rotated copies of the packed site vector x
spk::KPrep prep_inst(sp_handle* h, int k, const double* x) {
    const SitePlan& P = h->plan[k - 1];
    spk::KPrep I{};
    I.x = x;
    I.map = P.xmap.p;
    I.rmap = P.rmap.p;
    I.coef = P.coef.p;
    I.xd = h->Xd.p;
    I.xr = h->Xr.p;
    I.nd = P.Xd_size;
    I.nr = (long long)P.rmap_h.size() / 2;
    I.nc = P.nc;
    I.crot = P.c_r(0, 0);
    I.G = h->G;
    return I;
}
void site_vectors(sp_handle* h, int k, const double* x, bool f32 = false) {
    const spk::KPrep I = prep_inst(h, k, x);
    spk::xprep(h->stream, f32, std::max(I.nd, I.nr), h->G, 1, nullptr, I);
}

// arithmetic of H_eff x at site k: fused plans follow the precision of the
// local solves, block products are FP64 or split BF16
int heff_mode(const sp_handle* h, int k, bool force_fp64) {
    if (force_fp64 || !reduced(h)) return spk::kChainF64;
    if (h->plan[k - 1].h_rows > 0) return spk::kChainF32;
    return h->precision == SP_BF16X3 ? spk::kChainBF3 : spk::kChainF64;
}

// partial slots of y that H_eff x leaves (of ny: G), in units of the site size
int heff_parts(const sp_handle* h, int k) {
    return h->path == SP_PATH_TILED ? h->G * h->plan[k - 1].y_split : h->G;
}

// the capture that the handle's stream is under, 0 if none
unsigned long long capture_of(sp_handle* h) {
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    unsigned long long id = 0;
    if (hipStreamGetCaptureInfo(h->stream, &st, &id) != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    if (st == hipStreamCaptureStatusNone) return 0;
    h->recorded = true;
    return id;
}
// start of a public call that mixes environments: after a replay the scratch
// may hold another site's, or the environment it was mixed from may be new
void forget_mix(sp_handle* h) {
    if (h->recorded && capture_of(h) == 0) h->lt_site = -1;
}

// the left environment with the MPO mixed in, once per local problem: it
// depends on L[k-1] only.  A capture records its own, so that every replay
// mixes the environment of the moment
void premix_left(sp_handle* h, int k, int mode) {
    const SitePlan& P = h->plan[k - 1];
    const MixList& m = P.mix_l;
    const bool f32 = mode == spk::kChainF32;
    if (m.empty()) return;
    const unsigned long long capture = capture_of(h);
    if (h->lt_site == k && h->lt_gen == h->Lgen[k - 1] && h->lt_f32 == f32 && h->lt_capture == capture) return;
    const void* env = f32 ? (const void*)h->envL32[k - 1].p : (const void*)h->envL[k - 1].p;
    spk::premix(h->stream, f32, m.lists(), env, h->env[k - 1].size, h->LT.p, m.size, h->G);
    h->lt_site = k;
    h->lt_gen = h->Lgen[k - 1];
    h->lt_f32 = f32;
    h->lt_capture = capture;
}

// H_eff x as a chained product into the partial slots yp, nyp
spk::KInst heff_inst(sp_handle* h, int k, int mode, double* yp, double* nyp) {
    const SitePlan& P = h->plan[k - 1];
    spk::KInst I = chain_inst(h, k, P.c_heff, P.mix_l);
    if (mode == spk::kChainF32) {
        I.in[spk::K_L].p = h->envL32[k - 1].p;
        I.in[spk::K_R].p = h->envR32[k].p;
    }
    I.out[0] = yp;
    I.out[1] = nyp;
    I.ogs = h->sites[k - 1].size;
    return I;
}

void need_envs(const sp_handle* h, int k) {
    if (!h->Lvalid[k - 1] || !h->Rvalid[k])
        throw SpError(SP_ESTATE, "H_eff needs L[site-1] and R[site+1]; build them with sp_env_update");
}

// H_eff x of several states as one launch per arithmetic and tile shape: the
// instances in launch order and the launches over them
struct HeffBatch {
    struct Launch {
        int mode, shape, first, count, max_tiles, max_G;
        long long max_n;
    };
    std::vector<spk::KInst> insts;
    std::vector<spk::KPrep> preps;
    std::vector<Launch> launches;
    std::vector<std::tuple<int, int, spk::KInst, spk::KPrep>> items;  // (mode, shape, ..)
    // adds x at site k of h (mixing its left environment if it is due); gate:
    // see KInst
    void add(sp_handle* h, int k, const double* x, const int* gate) {
        const int mode = heff_mode(h, k, false);
        need_envs(h, k);
        premix_left(h, k, mode);
        spk::KInst I = heff_inst(h, k, mode, h->ypart.p, h->nypart.p);
        spk::KPrep q = prep_inst(h, k, x);
        I.gate = q.gate = gate;
        items.push_back({mode, h->plan[k - 1].c_heff.shape, I, q});
    }
    void finish() {
        std::stable_sort(items.begin(), items.end(), [](const auto& a, const auto& b) {
            return std::tie(std::get<0>(a), std::get<1>(a)) < std::tie(std::get<0>(b), std::get<1>(b));
        });
        for (const auto& it : items) {
            const spk::KInst& I = std::get<2>(it);
            const spk::KPrep& q = std::get<3>(it);
            if (launches.empty() || launches.back().mode != std::get<0>(it) || launches.back().shape != std::get<1>(it))
                launches.push_back({std::get<0>(it), std::get<1>(it), int(insts.size()), 0, 0, 0, 0});
            Launch& l = launches.back();
            ++l.count;
            l.max_tiles = std::max(l.max_tiles, I.ntile * I.G);
            l.max_n = std::max(l.max_n, std::max(q.nd, q.nr));
            l.max_G = std::max(l.max_G, I.G);
            insts.push_back(I);
            preps.push_back(q);
        }
    }
    size_t bytes() const { return insts.size() * (sizeof(spk::KInst) + sizeof(spk::KPrep)); }
    // the records as one block: the instances, then the site vectors
    void pack(void* dst) const {
        std::memcpy(dst, insts.data(), insts.size() * sizeof(spk::KInst));
        std::memcpy(static_cast<char*>(dst) + insts.size() * sizeof(spk::KInst), preps.data(), preps.size() * sizeof(spk::KPrep));
    }
    void launch(hipStream_t s, const void* dev) const {
        const spk::KInst* di = static_cast<const spk::KInst*>(dev);
        const spk::KPrep* dp = reinterpret_cast<const spk::KPrep*>(di + insts.size());
        for (const Launch& l : launches) {
            spk::xprep(s, l.mode == spk::kChainF32, l.max_n, l.max_G, l.count, dp + l.first, preps[l.first]);
            spk::chain(s, l.mode, spk::kChainHeff, l.shape, spk::kChainWaves, l.max_tiles, l.count, di + l.first, insts[l.first]);
        }
    }
};

// H_eff x at site k into the partial slots, whatever the environments hold
void heff_partials(sp_handle* h, int k, const double* x, int mode, double* yp, double* nyp) {
    const SitePlan& P = h->plan[k - 1];
    premix_left(h, k, mode);
    site_vectors(h, k, x, mode == spk::kChainF32);
    const spk::KInst I = heff_inst(h, k, mode, yp, nyp);
    spk::chain(h->stream, mode, spk::kChainHeff, P.c_heff.shape, spk::kChainWaves, I.ntile * I.G, 1, nullptr, I);
}

// With defer_gsum on the tiled path only the per-quadrature-point partials
// (h->ypart, h->nypart) are produced and the function returns true: the
// caller adds them (the Davidson Gram pass does).
// yp, nyp: where the partials go (null = the handle's own slots)
bool heff_apply(sp_handle* h, int k, const double* x, double* y, double* ny, bool defer_gsum = false,
                bool force_fp64 = false, double* yp = nullptr, double* nyp = nullptr) {
    need_envs(h, k);
    SitePlan& P = h->plan[k - 1];
    hipStream_t s = h->stream;
    if (h->path == SP_PATH_PLAIN) {
        const spk::BufSet b = bufset(h, k, x, y, ny, nullptr);
        P.p1.launch(s, b, P.coef.p);
        P.mixl.launch(s, b, P.coef.p);
        P.yout.launch(s, b, P.coef.p);
        return false;
    }
    const int n = int(h->sites[k - 1].size);
    if (!yp) yp = h->ypart.p;
    if (!nyp) nyp = h->nypart.p;
    heff_partials(h, k, x, heff_mode(h, k, force_fp64), yp, nyp);
    if (defer_gsum) return true;
    spk::gsum2(s, yp, nyp, n, heff_parts(h, k), h->G, n, y, ny);
    return false;
}

// one environment update as a chained product: out, of the given values per g
void env_chain(sp_handle* h, int k, const ChainList& C, const MixList& mix, const double* env, long long esize, double* out,
               long long osize) {
    const SitePlan& P = h->plan[k - 1];
    if (h->mixes) (void)capture_of(h);  // a recorded update writes an environment when it is replayed
    site_vectors(h, k, site_ptr(h, k));
    if (&mix == &P.mix_l) {
        premix_left(h, k, spk::kChainF64);  // there already if H_eff was applied at this site
    } else if (!mix.empty()) {
        spk::premix(h->stream, false, mix.lists(), env, esize, h->LT.p, mix.size, h->G);
        h->lt_site = -1;
    }
    spk::KInst I = chain_inst(h, k, C, mix);
    I.out[0] = out;
    I.ogs = osize;
    spk::chain(h->stream, spk::kChainF64, C.lay, C.shape, C.waves, I.ntile * I.G, 1, nullptr, I);
}

void env_left(sp_handle* h, int k) {
    if (!h->Lvalid[k - 1]) throw SpError(SP_ESTATE, "left environment of the previous bond is not built");
    SitePlan& P = h->plan[k - 1];
    hipStream_t s = h->stream;
    if (h->path == SP_PATH_PLAIN) {
        const spk::BufSet b = bufset(h, k, site_ptr(h, k), nullptr, nullptr, h->envL[k].p);
        P.p1.launch(s, b, P.coef.p);
        P.mixl.launch(s, b, P.coef.p);
        P.envl_out.launch(s, b, P.coef.p);
    } else {
        env_chain(h, k, P.c_envl, P.mix_l, h->envL[k - 1].p, h->env[k - 1].size, h->envL[k].p, h->env[k].size);
    }
    if (reduced(h))
        spk::to_f32(s, h->envL[k].p, h->envL32[k].p, (long long)h->G * h->env[k].size);
    h->Lvalid[k] = 1;
    ++h->Lgen[k];
    if (env_shared(h, k)) h->Rvalid[k] = 0;
    for (int q = k + 1; q <= h->L; ++q) h->Lvalid[q] = 0;
}

void env_right(sp_handle* h, int k) {
    if (!h->Rvalid[k]) throw SpError(SP_ESTATE, "right environment of the next bond is not built");
    SitePlan& P = h->plan[k - 1];
    hipStream_t s = h->stream;
    if (h->path == SP_PATH_PLAIN) {
        const spk::BufSet b = bufset(h, k, site_ptr(h, k), nullptr, nullptr, h->envR[k - 1].p);
        P.p1r.launch(s, b, P.coef.p);
        P.mixr.launch(s, b, P.coef.p);
        P.envr_out.launch(s, b, P.coef.p);
    } else {
        env_chain(h, k, P.c_envr, P.mix_r, h->envR[k].p, h->env[k].size, h->envR[k - 1].p, h->env[k - 1].size);
    }
    if (reduced(h))
        spk::to_f32(s, h->envR[k - 1].p, h->envR32[k - 1].p, (long long)h->G * h->env[k - 1].size);
    h->Rvalid[k - 1] = 1;
    if (env_shared(h, k - 1)) h->Lvalid[k - 1] = 0;
    for (int q = 0; q < k - 1; ++q) h->Rvalid[q] = 0;
}

void diag(sp_handle* h, int k, double* dh, double* dn) {
    if (!h->Lvalid[k - 1] || !h->Rvalid[k]) throw SpError(SP_ESTATE, "environments for the diagonal are not built");
    SitePlan& P = h->plan[k - 1];
    if (P.dg_direct) {
        spk::diag_direct(h->stream, P.ddg_blk.p, int(P.dg_blk.size()), P.ddg_dterm.p, h->envL[k - 1].p, h->env[k - 1].size,
                         h->envR[k].p, h->env[k].size, P.coef.p, P.nc, h->G, dh, dn);
        return;
    }
    const Bond& bl = h->bonds[k - 1];
    const Bond& br = h->bonds[k];
    const int* idx = P.ddg_idx.p;
    const int nnbl = int(bl.nb.size()), nnbr = int(br.nb.size()), nmix = int(P.dg_mix.size());
    double* Ld = h->T.p;  // on the plain path scratch of the block products, idle here
    double* Rd = h->T.p + (long long)h->G * P.dg_nzl * bl.D;
    const spk::DiagSide left{P.ddg_src.p, idx, idx + bl.D, h->envL[k - 1].p, h->env[k - 1].size, Ld, P.dg_nzl, bl.D, nnbl, 0};
    const spk::DiagSide right{P.ddg_src.p + (size_t)P.dg_nzl * nnbl, idx + 2 * bl.D, idx + 2 * bl.D + br.D, h->envR[k].p,
                              h->env[k].size, Rd, P.dg_nzr, br.D, nnbr, 0};
    spk::diag_gather(h->stream, left, right, h->G);
    spk::diag_mix(h->stream, P.ddg_mix.p, nmix, P.ddg_term.p, Ld, P.dg_nzl, bl.D, P.coef.p, P.nc, h->G, h->V.p);
    spk::diag_blocks(h->stream, P.ddg_blk.p, int(P.dg_blk.size()), idx, h->V.p, nmix, bl.D, Rd, P.dg_nzr, br.D, h->G, dh,
                     dn, P.dg_split, h->diag_part.p, h->sites[k - 1].size);
}

// positive-diagonal QR per right sector of site k, R pushed into site k+1
void move_right(sp_handle* h, int k) {
    SitePlan& P = h->plan[k - 1];
    spk::qr_sectors(h->stream, P.dqr_tasks.p, int(P.qr_tasks.size()), P.dqr_pieces.p, site_ptr(h, k),
                    h->qr_scratch.p, h->qr_r.p, P.qr_shape);
    if (k < h->L) {
        spk::BufSet b{};
        b.p[B_V] = h->qr_r.p;
        b.p[B_X] = site_ptr(h, k + 1);
        b.p[B_OUT] = h->tmp_site.p;
        P.absorb_right.launch(h->stream, b, P.coef.p);
        HIPCK(hipMemcpyAsync(site_ptr(h, k + 1), h->tmp_site.p, h->sites[k].size * sizeof(double),
                             hipMemcpyDeviceToDevice, h->stream));
    }
}

// positive-diagonal LQ per left sector of site k, L pushed into site k-1
void move_left(sp_handle* h, int k) {
    SitePlan& P = h->plan[k - 1];
    spk::qr_sectors(h->stream, P.dlq_tasks.p, int(P.lq_tasks.size()), P.dlq_pieces.p, site_ptr(h, k),
                    h->qr_scratch.p, h->qr_r.p, P.lq_shape);
    if (k > 1) {
        spk::BufSet b{};
        b.p[B_V] = h->qr_r.p;
        b.p[B_X] = site_ptr(h, k - 1);
        b.p[B_OUT] = h->tmp_site.p;
        P.absorb_left.launch(h->stream, b, P.coef.p);
        HIPCK(hipMemcpyAsync(site_ptr(h, k - 1), h->tmp_site.p, h->sites[k - 2].size * sizeof(double),
                             hipMemcpyDeviceToDevice, h->stream));
    }
}

void invalidate_for_site(sp_handle* h, int k) {
    for (int q = k; q <= h->L; ++q) h->Lvalid[q] = 0;
    for (int q = 0; q <= k - 1; ++q) h->Rvalid[q] = 0;
}

// ---------------------------------------------------------------------------
// Davidson for the singular pencil H_eff x = theta N_eff x (Eq. [geproblem])

// Pinned, mapped and coherent host memory: the Davidson kernels read the
// subspace coefficients from it and write their per-chunk partial sums into
// it directly, so an iteration needs no copy in either direction.
// ---------------------------------------------------------------------------
// Orthogonality constraints (Sec. 2.3, Eq. [orthoB]).  A constraint handle
// holds a lower state Psi_0 with the identity MPO on the plain path; its
// environments are rebuilt with this state on the bra side, so that its
// N_eff applied to Psi_0's site tensor k gives B[k] = d<Psi|P|Psi_0>/dA[k]
// in this state's packed layout.

constexpr int kMaxConstraints = 8;

void env_left_mixed(sp_handle* a, int k, const double* bra) {
    SitePlan& P = a->plan[k - 1];
    spk::BufSet b = bufset(a, k, site_ptr(a, k), nullptr, nullptr, a->envL[k].p);
    b.p[B_BRA] = const_cast<double*>(bra);
    P.p1.launch(a->stream, b, P.coef.p);
    P.mixl.launch(a->stream, b, P.coef.p);
    P.envl_out.launch(a->stream, b, P.coef.p);
    a->Lvalid[k] = 1;
    ++a->Lgen[k];
    if (env_shared(a, k)) a->Rvalid[k] = 0;
}

void env_right_mixed(sp_handle* a, int k, const double* bra) {
    SitePlan& P = a->plan[k - 1];
    spk::BufSet b = bufset(a, k, site_ptr(a, k), nullptr, nullptr, a->envR[k - 1].p);
    b.p[B_BRA] = const_cast<double*>(bra);
    P.p1r.launch(a->stream, b, P.coef.p);
    P.mixr.launch(a->stream, b, P.coef.p);
    P.envr_out.launch(a->stream, b, P.coef.p);
    a->Rvalid[k - 1] = 1;
    if (env_shared(a, k - 1)) a->Lvalid[k - 1] = 0;
}

// B[k] of constraint handle a into out (ny: scratch of the site's size)
void constraint_vector(sp_handle* a, int k, double* out, double* ny) {
    SitePlan& P = a->plan[k - 1];
    const spk::BufSet b = bufset(a, k, site_ptr(a, k), out, ny, nullptr);
    P.p1.launch(a->stream, b, P.coef.p);
    P.mixl.launch(a->stream, b, P.coef.p);
    P.yout.launch(a->stream, b, P.coef.p);
}

// u -= C (C^T u) for the con_active orthonormal constraint vectors, twice
// (classical Gram-Schmidt with one reorthogonalisation)
void project_out(sp_handle* h, double* u, int n) {
    const int m = h->con_active;
    if (m == 0) return;
    hipStream_t s = h->stream;
    const int nch = spk::dav_chunks(n);
    double* P1 = h->conPart.p;
    double* P2 = P1 + (size_t)nch * m;
    spk::dav_cgs(s, h->conB.p, h->cld, 0, m, P1, nch, u, n, P1, 0);  // dots only
    spk::dav_cgs(s, h->conB.p, h->cld, m, m, P1, nch, u, n, P2, 0);  // subtract, dots again
    spk::dav_cgs(s, h->conB.p, h->cld, m, 0, P2, nch, u, n, P1, 0);  // subtract
}

// the orthonormal constraint vectors at site k: B[k] of every constraint in
// order, each orthogonalised against the ones kept before it and dropped
// when its remainder is below 1e-10 of its own norm
void prepare_constraints(sp_handle* h, int k) {
    h->con_active = 0;
    if (h->cons.empty()) return;
    hipStream_t s = h->stream;
    const int n = int(h->sites[k - 1].size);
    const int nch = spk::dav_chunks(n);
    double* p0 = h->con_pin_dev;  // raw norm partials
    double* p1 = p0 + nch;        // norm partials after the projection
    for (auto& a : h->cons) {
        double* row = h->conB.p + (size_t)h->con_active * h->cld;
        constraint_vector(a.get(), k, row, h->tmp_site.p);
        spk::dav_cgs(s, h->conB.p, h->cld, 0, 0, p0, nch, row, n, p0, 1);  // |B|^2 partials
        project_out(h, row, n);
        spk::dav_cgs(s, h->conB.p, h->cld, 0, 0, p1, nch, row, n, p1, 1);
        HIPCK(hipStreamSynchronize(s));
        double n0 = 0.0, n1 = 0.0;
        for (int q = 0; q < nch; ++q) {
            n0 += h->con_pin[q];
            n1 += h->con_pin[nch + q];
        }
        if (!(n0 > 0.0) || !(n1 > 1e-20 * n0)) continue;  // dependent on the kept vectors
        spk::dav_normalize(s, p1, nch, row, row, n, p0 + 2 * nch);
        h->con_active++;
    }
}

void ensure_pinned(sp_handle* h, size_t n, size_t n_up) {
    const unsigned flags = hipHostMallocMapped | hipHostMallocCoherent;
    if (h->pin_n < n) {
        if (h->pin) HIPCK(hipHostFree(h->pin));
        h->pin = nullptr;
        h->pin_dev = nullptr;
        HIPCK(hipHostMalloc(&h->pin, n * sizeof(double), flags));
        HIPCK(hipHostGetDevicePointer((void**)&h->pin_dev, h->pin, 0));
        h->pin_n = n;
    }
    if (h->pin_up_n < n_up) {
        if (h->pin_up) HIPCK(hipHostFree(h->pin_up));
        h->pin_up = nullptr;
        h->pin_up_dev = nullptr;
        HIPCK(hipHostMalloc(&h->pin_up, n_up * sizeof(double), flags));
        HIPCK(hipHostGetDevicePointer((void**)&h->pin_up_dev, h->pin_up, 0));
        h->pin_up_n = n_up;
    }
}

// device small area of the Davidson solve (offsets in doubles)
struct DavLayout {
    long long a, theta, q, pc1, pc2, pn, out, tn, px, pg, total;
    DavLayout(int max_sub, int nch) {
        a = 0;
        theta = max_sub + 2;
        q = max_sub + 4;
        pc1 = q + (long long)max_sub * max_sub;
        pc2 = pc1 + (long long)nch * max_sub;
        pn = pc2 + (long long)nch * max_sub;
        out = pn + nch;
        tn = out;
        px = out + 1;
        pg = px + 3LL * nch;
        total = pg + (long long)nch * (4 * max_sub + 2) + 8;
    }
};

void ensure_davidson(sp_handle* h, int max_sub) {
    if (h->dav_sub >= max_sub && h->ld > 0) return;
    SP_REQUIRE(max_sub + 1 <= spk::kDavMaxVec, "max_sub too large");
    h->ld = (h->max_site + 63) / 64 * 64;
    const size_t vec = size_t(max_sub + 1) * h->ld;
    h->dV.alloc(vec);
    h->dHV.alloc(vec);
    h->dNV.alloc(vec);
    h->dRot.alloc(size_t(max_sub + 1) * h->ld);
    h->dx.alloc(h->ld);
    h->dt.alloc(h->ld);
    h->ddh.alloc(h->ld);
    h->ddn.alloc(h->ld);
    const int nch = spk::dav_chunks(int(h->ld));
    const DavLayout lay(max_sub, nch);
    h->dsmall.alloc(lay.total);
    h->dHt.alloc(size_t(max_sub + 1) * (max_sub + 1));
    h->dNt.alloc(size_t(max_sub + 1) * (max_sub + 1));
    h->dav_sub = max_sub;
    ensure_pinned(h, lay.total - lay.out + 8, lay.pc1 + 8);
}

// tot[i] = the sum over chunks q < nch of part[q * stride + i], i < stride,
// each in ascending q, read from the chunk-major partials in one contiguous
// pass (the same sums as chunk by chunk per i, without the strided reads)
void chunk_totals(const double* part, int nch, int stride, double* tot) {
    for (int i = 0; i < stride; ++i) tot[i] = 0.0;
    for (int q = 0; q < nch; ++q) {
        const double* row = part + (size_t)q * stride;
        for (int i = 0; i < stride; ++i) tot[i] += row[i];
    }
}

struct DavOut {
    double theta = 0, rnorm = 0, pnorm = 0;
    int iters = 0, matvecs = 0;
    bool converged = false;
};

// lowest eigenpair of the pencil restricted to range(Nt) (canonical
// orthogonalisation); returns false if the projected metric vanishes.  gp
// (may be null) keeps the reduction of the pencil between the calls of one
// solve, which grows it by one row and column per call until a restart
bool small_solve(int m, const std::vector<double>& Ht, const std::vector<double>& Nt, int stride, double drop,
                 bool need_all, double& theta, std::vector<double>& a, std::vector<double>& Xc, int& rk,
                 sph::GrowingPencil* gp) {
    std::vector<double> Hs(size_t(m) * m), Ns(size_t(m) * m);
    for (int i = 0; i < m; ++i)
        for (int j = 0; j < m; ++j) {
            Hs[size_t(i) * m + j] = 0.5 * (Ht[size_t(i) * stride + j] + Ht[size_t(j) * stride + i]);
            Ns[size_t(i) * m + j] = 0.5 * (Nt[size_t(i) * stride + j] + Nt[size_t(j) * stride + i]);
        }
    a.assign(m, 0.0);
    if (gp && need_all) gp->reset();
    if (gp && !need_all) {
        const int r = gp->lowest(m, Hs.data(), Ns.data(), drop, &theta, a.data());
        if (r == -1) throw SpError(SP_ENAN, "subspace eigensolver failed");
        if (r == m) {
            if (!std::isfinite(theta)) throw SpError(SP_ENAN, "non-finite Ritz value");
            rk = m;
            return true;
        }
        a.assign(m, 0.0);
    }
    if (need_all) Xc.assign(size_t(m) * m, 0.0);
    const int r = sph::gen_lowest(m, Hs.data(), Ns.data(), drop, &theta, a.data(), need_all ? Xc.data() : nullptr, &rk);
    if (r < 0) throw SpError(SP_ENAN, "subspace eigensolver failed");
    if (r == 0) return false;
    if (!std::isfinite(theta)) throw SpError(SP_ENAN, "non-finite Ritz value");
    if (need_all) Xc.resize(size_t(m) * rk);
    return true;
}

// FP64 Rayleigh quotient at site k for the device vector x (any norm):
// theta = x.H_eff x / x.N_eff x, pnorm = x.N_eff x / x.x; uses dHV[0], dNV[0]
void rayleigh64(sp_handle* h, int k, const double* x, double& theta, double& pnorm, double& xx_out) {
    const int n = int(h->sites[k - 1].size);
    heff_apply(h, k, x, h->dHV.p, h->dNV.p, false, true);
    double* sm = h->dsmall.p;
    spk::multidot(h->stream, h->dHV.p, 0, 1, x, n, sm);
    spk::multidot(h->stream, h->dNV.p, 0, 1, x, n, sm + 1);
    spk::multidot(h->stream, x, 0, 1, x, n, sm + 2);
    HIPCK(hipMemcpyAsync(h->pin, sm, 3 * sizeof(double), hipMemcpyDeviceToHost, h->stream));
    HIPCK(hipStreamSynchronize(h->stream));
    const double xy = h->pin[0], xny = h->pin[1], xx = h->pin[2];
    xx_out = xx;
    theta = xy / xny;
    pnorm = xx > 0.0 ? xny / xx : 0.0;
}

DavOut davidson(sp_handle* h, int k, const sp_sweep_opts& o) {
    const int n = int(h->sites[k - 1].size);
    const int max_sub = std::max(2, o.max_sub);
    const int keep = std::max(1, std::min(o.keep, max_sub - 1));
    const int max_iter = std::max(1, o.max_iter);
    ensure_davidson(h, max_sub);
    hipStream_t s = h->stream;
    const long long ld = h->ld;
    double* V = h->dV.p;
    double* HV = h->dHV.p;
    double* NV = h->dNV.p;
    const int nch = spk::dav_chunks(n);
    const DavLayout lay(h->dav_sub, spk::dav_chunks(int(ld)));
    double* sm = h->dsmall.p;
    double* up = h->pin_up;
    double* dn = h->pin;
    double* dn_dev = h->pin_dev;  // device view of dn: partial sums land here
    // new vector mm: on the tiled path H_eff is applied to the unnormalised
    // correction t (or V_0 for mm = 0) and the Gram pass normalises V_mm,
    // HV_mm and NV_mm; the plain path normalises first
    auto extend = [&](int mm, bool from_t) {
        double* vm = V + size_t(mm) * ld;
        double* tn = dn_dev + (lay.tn - lay.out);
        if (h->path == SP_PATH_PLAIN) {
            if (from_t) spk::dav_normalize(s, sm + lay.pn, nch, h->dt.p, vm, n, tn);
            heff_apply(h, k, vm, HV + size_t(mm) * ld, NV + size_t(mm) * ld);
            spk::dav_gram(s, V, HV, NV, ld, mm, n, nullptr, nullptr, 0, nullptr, nullptr, nullptr, n, h->G, h->G,
                          dn_dev + (lay.pg - lay.out));
        } else {
            heff_apply(h, k, from_t ? h->dt.p : vm, nullptr, nullptr, true);
            spk::dav_gram(s, V, HV, NV, ld, mm, n, from_t ? h->dt.p : nullptr, sm + lay.pn, nch, tn, h->ypart.p,
                          h->nypart.p, n, heff_parts(h, k), h->G, dn_dev + (lay.pg - lay.out));
        }
        // constrained pencil (Q H Q, Q N Q): the Gram rows above are the same
        // for the projected products, since every V_j is orthogonal to C
        project_out(h, HV + size_t(mm) * ld, n);
        project_out(h, NV + size_t(mm) * ld, n);
    };
    // canonical orthogonalisation threshold: with FP32 products the null
    // space of the projected metric is only resolved to about 1e-7 of its
    // largest eigenvalue, so directions below 1e-5 are dropped there
    const double drop = metric_drop(h), floor_ = 1e-8;
    DavOut out;
    // fixed-order sums of per-chunk partials (host side)
    auto chunk_total = [&](const double* part, int stride, int idx) {
        double acc = 0.0;
        for (int q = 0; q < nch; ++q) acc += part[(size_t)q * stride + idx];
        return acc;
    };

    // learned preconditioner: corrections from the model while the residual
    // keeps reaching new minima and halves at least every four iterations
    // (abandoned for the rest of the solve otherwise); training pairs
    // recorded for every iteration of a converged solve
    sp_mlp* use = h->mlp_use;
    sp_mlp* rec = h->mlp_rec;
    bool use_model = use != nullptr;
    double best_r = INFINITY;
    std::vector<double> rhist;
    int stall = 0, nrec = 0, rec_last_it = 0;
    const long long rec_base = rec ? rec->rows : 0;
    if (rec && h->xrec.n < size_t(max_iter) * ld) h->xrec.alloc(size_t(max_iter) * ld);
    if ((use || rec) && h->mlp_scal.n < 4) h->mlp_scal.alloc(4);
    SP_REQUIRE(!use || !rec || use->scope == rec->scope, "the model in use and the recording one differ in scope");
    const NBlocks* nbk = ((use && use->scope == SP_MLP_NBLOCK) || (rec && rec->scope == SP_MLP_NBLOCK))
                             ? &site_nblocks(h, k)
                             : nullptr;
    if (nbk && h->mlp_grms.n < size_t(2 * nbk->ng)) h->mlp_grms.alloc(2 * nbk->ng);
    if (nbk && rec && h->mlp_tscal.n < size_t(2 * max_iter)) h->mlp_tscal.alloc(2 * max_iter);
    diag(h, k, h->ddh.p, h->ddn.p);
    spk::normalize(s, site_ptr(h, k), V, n, nullptr);
    if (h->con_active) {  // start in the complement of the constraints
        project_out(h, V, n);
        spk::normalize(s, V, V, n, nullptr);
    }
    extend(0, false);
    out.matvecs = 1;
    HIPCK(hipStreamSynchronize(s));
    const int S = max_sub + 1;
    std::vector<double> Ht(size_t(S) * S, 0.0), Nt(size_t(S) * S, 0.0);
    Ht[0] = chunk_total(dn + (lay.pg - lay.out), 2, 0);
    Nt[0] = chunk_total(dn + (lay.pg - lay.out), 2, 1);
    int m = 1;
    std::vector<double> a, Xc, gt;
    sph::GrowingPencil gp;
    for (int it = 1; it <= max_iter; ++it) {
        out.iters = it;
        double theta;
        int rk = 0;
        const bool last = (it == max_iter);
        const bool restart = !last && m >= max_sub;
        if (!small_solve(m, Ht, Nt, S, drop, restart, theta, a, Xc, rk, &gp))
            throw SpError(SP_ENORM, "projected norm vanishes in the search space");
        out.theta = theta;
        int nk = 0;
        std::vector<double> Qk;
        if (restart) {
            // the lowest Ritz vectors, Euclidean-orthonormalised (modified
            // Gram-Schmidt on their coefficient vectors)
            nk = std::min(keep, rk);
            Qk.assign(size_t(m) * nk, 0.0);
            for (int c = 0; c < nk; ++c) {
                std::vector<double> v(m);
                for (int i = 0; i < m; ++i) v[i] = Xc[i * rk + c];
                for (int p = 0; p < c; ++p) {
                    double d = 0.0;
                    for (int i = 0; i < m; ++i) d += Qk[i * nk + p] * v[i];
                    for (int i = 0; i < m; ++i) v[i] -= d * Qk[i * nk + p];
                }
                double nr = 0.0;
                for (int i = 0; i < m; ++i) nr += v[i] * v[i];
                nr = std::sqrt(nr);
                for (int i = 0; i < m; ++i) Qk[i * nk + c] = v[i] / nr;
            }
        }
        // a and theta are read by the Ritz kernel straight from mapped host
        // memory; the restart rotation is copied to the device
        for (int i = 0; i < m; ++i) up[lay.a + i] = a[i];
        up[lay.a + m] = theta;
        if (restart) {
            std::copy(Qk.begin(), Qk.end(), up + lay.q);
            HIPCK(hipMemcpyAsync(sm + lay.q, up + lay.q, Qk.size() * sizeof(double), hipMemcpyHostToDevice, s));
        }
        spk::dav_ritz(s, V, HV, NV, ld, m, h->pin_up_dev + lay.a, h->ddh.p, h->ddn.p, n, floor_, h->dx.p, h->dt.p,
                      dn_dev + (lay.px - lay.out), sm + lay.pc1);
        if (!last) {
            const bool record_now = rec && rec_base + (long long)(nrec + 1) * n <= rec->cap;
            if (use_model || record_now) {
                if (nbk) {
                    spk::mlp_group_rms(s, h->dt.p, h->ddh.p, h->ddn.p, h->pin_up_dev + lay.a + m, floor_,
                                       nbk->groups(), h->mlp_grms.p);
                } else {
                    spk::sum_partials(s, dn_dev + (lay.px - lay.out), nch, 3, 1, h->mlp_scal.p);
                    spk::sumsq(s, h->dt.p, n, h->mlp_scal.p + 1);
                }
                spk::mlp_apply_grouped(
                    s, use_model ? use->w.p : nullptr, use ? use->hidden : 0, h->dt.p, h->ddh.p, h->ddn.p,
                    h->pin_up_dev + lay.a + m, h->mlp_scal.p, h->mlp_scal.p + 1, n, floor_,
                    record_now ? rec->F.p + (rec_base + (long long)nrec * n) * spk::kMlpIn : nullptr,
                    record_now ? rec->Y.p + rec_base + (long long)nrec * n : nullptr, nbk ? nbk->gid.p : nullptr,
                    nbk ? h->mlp_grms.p : nullptr);
                if (record_now) {
                    HIPCK(hipMemcpyAsync(h->xrec.p + size_t(nrec) * ld, h->dx.p, size_t(n) * sizeof(double),
                                         hipMemcpyDeviceToDevice, s));
                    ++nrec;
                    rec_last_it = it;
                }
                // the dots of the new correction with the search space
                if (use_model) spk::dav_cgs(s, V, ld, 0, m, sm + lay.pc1, nch, h->dt.p, n, sm + lay.pc1, 0);
            }
            // the correction stays in the complement of the constraints (its
            // dots with V are unchanged, V being orthogonal to them)
            project_out(h, h->dt.p, n);
            if (restart) {
                for (double* B : {V, HV, NV}) {
                    spk::basis_rotate(s, B, ld, m, sm + lay.q, nk, h->dRot.p, n);
                    HIPCK(hipMemcpyAsync(B, h->dRot.p, size_t(nk) * ld * sizeof(double), hipMemcpyDeviceToDevice, s));
                }
                auto rot = [&](std::vector<double>& M) {
                    std::vector<double> tmp(size_t(m) * nk, 0.0), res(size_t(S) * S, 0.0);
                    for (int i = 0; i < m; ++i)
                        for (int c = 0; c < nk; ++c) {
                            double v = 0.0;
                            for (int j = 0; j < m; ++j) v += M[i * S + j] * Qk[j * nk + c];
                            tmp[i * nk + c] = v;
                        }
                    for (int r = 0; r < nk; ++r)
                        for (int c = 0; c < nk; ++c) {
                            double v = 0.0;
                            for (int i = 0; i < m; ++i) v += Qk[i * nk + r] * tmp[i * nk + c];
                            res[r * S + c] = v;
                        }
                    M.swap(res);
                };
                rot(Ht);
                rot(Nt);
                m = nk;
                // the first projections must be taken against the new basis
                spk::dav_cgs(s, V, ld, 0, m, sm + lay.pc2, nch, h->dt.p, n, sm + lay.pc1, 0);
            }
            // CGS2 of the correction against the search space, then normalise
            spk::dav_cgs(s, V, ld, m, m, sm + lay.pc1, nch, h->dt.p, n, sm + lay.pc2, 0);
            spk::dav_cgs(s, V, ld, m, 0, sm + lay.pc2, nch, h->dt.p, n, sm + lay.pn, 1);
            extend(m, true);
            out.matvecs++;
        }
        HIPCK(hipStreamSynchronize(s));
        double xt[3];
        chunk_totals(dn + (lay.px - lay.out), nch, 3, xt);
        const double xx = xt[0], uu = xt[1], xn = xt[2];
        if (!std::isfinite(xx) || !std::isfinite(uu) || !(xx > 0.0)) throw SpError(SP_ENAN, "non-finite Ritz vector");
        out.rnorm = std::sqrt(uu / xx);
        out.pnorm = xn / xx;
        if (out.rnorm <= o.tol) {
            out.converged = true;
            break;
        }
        if (use_model) {
            if (out.rnorm < best_r) {
                best_r = out.rnorm;
                stall = 0;
            } else {
                ++stall;
            }
            rhist.push_back(out.rnorm);
            const size_t nh = rhist.size();
            const bool slow = nh >= 5 && out.rnorm > 0.5 * rhist[nh - 5];
            if (stall >= 3 || slow) use_model = false;
        }
        if (last) break;
        const double tn = dn[lay.tn - lay.out];
        if (!(tn >= 1e-14)) break;
        // extend the projected matrices with the new vector m
        const int nd = 4 * m + 2;
        gt.resize(nd);
        chunk_totals(dn + (lay.pg - lay.out), nch, nd, gt.data());
        for (int j = 0; j <= m; ++j) {
            const double hv_new = gt[j];          // V_j . HV_m
            const double nv_new = gt[m + 1 + j];  // V_j . NV_m
            const double hv_old = (j < m) ? gt[2 * m + 2 + j] : hv_new;  // V_m . HV_j
            const double nv_old = (j < m) ? gt[3 * m + 2 + j] : nv_new;
            Ht[j * S + m] = hv_new;
            Ht[m * S + j] = hv_old;
            Nt[j * S + m] = nv_new;
            Nt[m * S + j] = nv_old;
        }
        ++m;
    }
    // normalise x and write it into the site
    spk::normalize(s, h->dx.p, site_ptr(h, k), n, nullptr);
    if (rec && out.converged && nrec > 0) {
        // iterations before the converged one: targets against the final x
        const int keep = nrec - (rec_last_it == out.iters ? 1 : 0);
        if (nbk)
            spk::mlp_targets_grouped(s, h->xrec.p, ld, keep, site_ptr(h, k), n, nbk->groups(), h->mlp_tscal.p,
                                     rec->Y.p + rec_base);
        else
            spk::mlp_targets(s, h->xrec.p, ld, keep, site_ptr(h, k), n, rec->Y.p + rec_base);
        rec->rows = rec_base + (long long)keep * n;
    }
    if (reduced(h)) {
        // the reported energy and norm: one FP64 product with the FP64
        // environments (the vector itself comes from the FP32 solve)
        double th, pn, xx;
        rayleigh64(h, k, site_ptr(h, k), th, pn, xx);
        if (!std::isfinite(th)) throw SpError(SP_ENAN, "non-finite Rayleigh quotient");
        out.theta = th;
        out.pnorm = pn;
    }
    return out;
}

// ---------------------------------------------------------------------------
// Batched sweeps: many SP-MPS states advanced together, one site step of
// each per round.  Within a round the Davidson iterations of all states run
// in lockstep: their subspace solves on a host thread pool, then one Ritz,
// two CGS and one Gram launch for all of them and one fused H_eff launch
// per row count (every state's quadrature points in the same launch).

class Pool {
  public:
    explicit Pool(int n) {
        for (int i = 0; i < n; ++i) th_.emplace_back([this] { loop(); });
    }
    ~Pool() {
        {
            std::lock_guard<std::mutex> l(mu_);
            stop_ = true;
        }
        cv_.notify_all();
        for (auto& t : th_) t.join();
    }
    // fn(i) for i < n on the pool and the calling thread
    void run(int n, const std::function<void(int)>& fn) {
        if (th_.empty() || n <= 1) {
            for (int i = 0; i < n; ++i) fn(i);
            return;
        }
        {
            std::lock_guard<std::mutex> l(mu_);
            job_ = &fn;
            njobs_ = n;
            next_ = 0;
            ++gen_;
        }
        cv_.notify_all();
        for (int i = next_.fetch_add(1); i < n; i = next_.fetch_add(1)) fn(i);
        std::unique_lock<std::mutex> l(mu_);
        done_.wait(l, [&] { return busy_ == 0; });
        job_ = nullptr;
    }

  private:
    void loop() {
        long seen = 0;
        for (;;) {
            const std::function<void(int)>* fn;
            int nj;
            {
                std::unique_lock<std::mutex> l(mu_);
                cv_.wait(l, [&] { return stop_ || gen_ != seen; });
                if (stop_) return;
                seen = gen_;
                fn = job_;
                nj = njobs_;
                if (!fn) continue;
                ++busy_;
            }
            for (int i = next_.fetch_add(1); i < nj; i = next_.fetch_add(1)) (*fn)(i);
            {
                std::lock_guard<std::mutex> l(mu_);
                if (--busy_ == 0) done_.notify_all();
            }
        }
    }
    std::vector<std::thread> th_;
    std::mutex mu_;
    std::condition_variable cv_, done_;
    const std::function<void(int)>* job_ = nullptr;
    int njobs_ = 0, busy_ = 0;
    std::atomic<int> next_{0};
    long gen_ = 0;
    bool stop_ = false;
};

struct BatchState {
    sph::GrowingPencil gp;  // reduction of the growing subspace pencil
    sp_handle* h = nullptr;
    std::vector<std::pair<int, int>> order;  // (site, dir) of every step
    size_t step = 0;
    int sweep_len = 1;
    // Davidson state of the current step
    int k = 0, n = 0, nch = 0, m = 0, it = 0, rk = 0, nk = 0;
    bool last = false, restart = false;
    double theta = 0;
    std::vector<double> Ht, Nt, a, Xc, Qk;
    DavOut out;
    std::chrono::steady_clock::time_point t0;
    std::string err;
    int err_code = 0;
};

struct BatchBufs {
    DArr<char> insts;
    DArr<spk::DavInst> dav;
    double* pin = nullptr;  // staging of the per-round uploads
    size_t pin_n = 0;
    ~BatchBufs() {
        if (pin) (void)hipHostFree(pin);
    }
    double* staging(size_t bytes) {
        const size_t n = (bytes + 7) / 8;
        if (pin_n < n) {
            if (pin) HIPCK(hipHostFree(pin));
            pin = nullptr;
            HIPCK(hipHostMalloc(&pin, n * 8, hipHostMallocDefault));
            pin_n = n;
        }
        return pin;
    }
};

// one fused H_eff application for every state in `idx` (tiled path), with
// x = V_0 where from_v0[i] else t; outputs stay as per-g partials in each
// handle.  The staging buffer is rewritten by the next call only after the
// caller has synchronised the stream (once per round).
void batch_heff_mixed(std::vector<BatchState>& B, const std::vector<int>& idx, const std::vector<int>& from_v0,
                      BatchBufs& bb, hipStream_t s) {
    if (idx.empty()) return;
    HeffBatch hb;
    for (int i : idx) hb.add(B[i].h, B[i].k, from_v0[i] ? B[i].h->dV.p : B[i].h->dt.p, nullptr);
    hb.finish();
    void* stage = bb.staging(hb.bytes());
    hb.pack(stage);
    if (bb.insts.n < hb.bytes()) bb.insts.alloc(hb.bytes());
    HIPCK(hipMemcpyAsync(bb.insts.p, stage, hb.bytes(), hipMemcpyHostToDevice, s));
    hb.launch(s, bb.insts.p);
}

void batch_dav_upload(std::vector<spk::DavInst>& D, BatchBufs& bb, hipStream_t s) {
    if (bb.dav.n < D.size()) bb.dav.alloc(D.size());
    HIPCK(hipMemcpyAsync(bb.dav.p, D.data(), D.size() * sizeof(spk::DavInst), hipMemcpyHostToDevice, s));
}

spk::DavInst dav_inst(BatchState& st) {
    sp_handle* h = st.h;
    const long long ld = h->ld;
    const DavLayout lay(h->dav_sub, spk::dav_chunks(int(ld)));
    double* sm = h->dsmall.p;
    double* dn_dev = h->pin_dev;
    spk::DavInst I{};
    I.V = h->dV.p;
    I.HV = h->dHV.p;
    I.NV = h->dNV.p;
    I.ld = ld;
    I.aq = h->pin_up_dev + lay.a;
    I.dh = h->ddh.p;
    I.dn = h->ddn.p;
    I.floor_ = 1e-8;
    I.x = h->dx.p;
    I.t = h->dt.p;
    I.part_x = dn_dev + (lay.px - lay.out);
    I.pc1 = sm + lay.pc1;
    I.pc2 = sm + lay.pc2;
    I.pn = sm + lay.pn;
    I.pg = dn_dev + (lay.pg - lay.out);
    I.tnorm = dn_dev + (lay.tn - lay.out);
    I.ypart = h->ypart.p;
    I.nypart = h->nypart.p;
    I.gstride = st.n;
    I.G = heff_parts(h, st.k);
    I.Gn = h->G;
    I.m = st.m;
    I.mr = st.m;
    I.n = st.n;
    I.active = 1;
    I.ext = 1;
    I.from_t = 1;
    return I;
}

// A finished site step: into the caller's report (while it has room) and,
// when asked, one line on stderr.
void record_step(sp_sweep_report* r, int verbose, int state, const sp_step_report& st) {
    if (r && r->steps && r->n_steps < r->capacity) r->steps[r->n_steps++] = st;
    if (verbose)
        std::fprintf(stderr, "[sp_sweep] state %d sweep %d site %d dir %+d: theta %.12f, %d matvecs%s, %.1f ms\n",
                     state, st.sweep, st.site, st.dir, st.theta, st.matvecs, st.converged ? "" : " (not converged)",
                     st.usec * 1e-3);
}

// One Davidson iteration of every running state per round (states are not
// aligned on site steps: a state that finishes its local solve moves its
// gauge, updates its environments and starts its next step at once).
int sweep_batch(std::vector<BatchState>& B, const sp_sweep_opts& o, std::vector<sp_sweep_report*>& reps) {
    hipStream_t s = B[0].h->stream;
    const int max_sub = std::max(2, o.max_sub);
    const int keep = std::max(1, std::min(o.keep, max_sub - 1));
    const int max_iter = std::max(1, o.max_iter);
    const int S = max_sub + 1;
    BatchBufs bb;
    const int nthreads =
        std::max(0, std::min<int>(int(B.size()), std::min(16u, std::thread::hardware_concurrency())) - 1);
    Pool pool(nthreads);
    int status = SP_OK;
    for (auto& st : B) ensure_davidson(st.h, max_sub);
    auto chunk_total = [](const double* part, int nch, int stride, int idx) {
        double acc = 0.0;
        for (int q = 0; q < nch; ++q) acc += part[(size_t)q * stride + idx];
        return acc;
    };
    // phase: 0 = start a step, 1 = Davidson iterations, 2 = done
    std::vector<int> phase(B.size());
    for (size_t i = 0; i < B.size(); ++i) phase[i] = B[i].order.empty() ? 2 : 0;
    for (;;) {
        std::vector<int> starting, iterating;
        for (size_t i = 0; i < B.size(); ++i) {
            if (phase[i] == 0) starting.push_back(int(i));
            else if (phase[i] == 1) iterating.push_back(int(i));
        }
        if (starting.empty() && iterating.empty()) break;
        // step start: diagonal and V_0
        for (int i : starting) {
            BatchState& st = B[i];
            sp_handle* h = st.h;
            st.k = st.order[st.step].first;
            st.n = int(h->sites[st.k - 1].size);
            st.nch = spk::dav_chunks(st.n);
            st.m = 0;
            st.it = 0;
            st.out = DavOut{};
            st.t0 = std::chrono::steady_clock::now();
            st.Ht.assign(size_t(S) * S, 0.0);
            st.Nt.assign(size_t(S) * S, 0.0);
            diag(h, st.k, h->ddh.p, h->ddn.p);
            spk::normalize(s, site_ptr(h, st.k), h->dV.p, st.n, nullptr);
        }
        // subspace solves of the iterating states
        pool.run(int(iterating.size()), [&](int q) {
            BatchState& st = B[iterating[q]];
            try {
                st.it += 1;
                st.out.iters = st.it;
                st.last = (st.it == max_iter);
                st.restart = !st.last && st.m >= max_sub;
                const double drop = metric_drop(st.h);
                if (!small_solve(st.m, st.Ht, st.Nt, S, drop, st.restart, st.theta, st.a, st.Xc, st.rk, &st.gp))
                    throw SpError(SP_ENORM, "projected norm vanishes in the search space");
                st.out.theta = st.theta;
                st.nk = 0;
                if (st.restart) {
                    const int m = st.m;
                    st.nk = std::min(keep, st.rk);
                    st.Qk.assign(size_t(m) * st.nk, 0.0);
                    for (int c = 0; c < st.nk; ++c) {
                        std::vector<double> v(m);
                        for (int r = 0; r < m; ++r) v[r] = st.Xc[r * st.rk + c];
                        for (int p = 0; p < c; ++p) {
                            double d = 0.0;
                            for (int r = 0; r < m; ++r) d += st.Qk[r * st.nk + p] * v[r];
                            for (int r = 0; r < m; ++r) v[r] -= d * st.Qk[r * st.nk + p];
                        }
                        double nr = 0.0;
                        for (int r = 0; r < m; ++r) nr += v[r] * v[r];
                        nr = std::sqrt(nr);
                        for (int r = 0; r < m; ++r) st.Qk[r * st.nk + c] = v[r] / nr;
                    }
                }
                sp_handle* h = st.h;
                const DavLayout lay(h->dav_sub, spk::dav_chunks(int(h->ld)));
                for (int r = 0; r < st.m; ++r) h->pin_up[lay.a + r] = st.a[r];
                h->pin_up[lay.a + st.m] = st.theta;
                if (st.restart) std::copy(st.Qk.begin(), st.Qk.end(), h->pin_up + lay.q);
            } catch (const SpError& e) {
                st.err = e.what();
                st.err_code = e.code;
            }
        });
        for (int i : iterating)
            if (B[i].err_code) throw SpError(B[i].err_code, B[i].err);
        std::vector<spk::DavInst> D;
        int max_n = 0, max_m = 0;
        if (!iterating.empty()) {
            for (int i : iterating) {
                D.push_back(dav_inst(B[i]));
                max_n = std::max(max_n, B[i].n);
            }
            batch_dav_upload(D, bb, s);
            spk::bdav_ritz(s, bb.dav.p, int(D.size()), max_n);
        }
        std::vector<int> ext;
        for (int i : iterating) {
            BatchState& st = B[i];
            if (st.last) continue;
            ext.push_back(i);
            st.out.matvecs++;
            if (!st.restart) continue;
            sp_handle* h = st.h;
            const long long ld = h->ld;
            const DavLayout lay(h->dav_sub, spk::dav_chunks(int(ld)));
            double* sm = h->dsmall.p;
            HIPCK(hipMemcpyAsync(sm + lay.q, h->pin_up + lay.q, st.Qk.size() * sizeof(double), hipMemcpyHostToDevice,
                                 s));
            for (double* Bv : {h->dV.p, h->dHV.p, h->dNV.p}) {
                spk::basis_rotate(s, Bv, ld, st.m, sm + lay.q, st.nk, h->dRot.p, st.n);
                HIPCK(hipMemcpyAsync(Bv, h->dRot.p, size_t(st.nk) * ld * sizeof(double), hipMemcpyDeviceToDevice, s));
            }
            const int m = st.m, nk = st.nk;
            auto rot = [&](std::vector<double>& M) {
                std::vector<double> tmp(size_t(m) * nk, 0.0), res(size_t(S) * S, 0.0);
                for (int r = 0; r < m; ++r)
                    for (int c = 0; c < nk; ++c) {
                        double v = 0.0;
                        for (int j = 0; j < m; ++j) v += M[r * S + j] * st.Qk[j * nk + c];
                        tmp[r * nk + c] = v;
                    }
                for (int r = 0; r < nk; ++r)
                    for (int c = 0; c < nk; ++c) {
                        double v = 0.0;
                        for (int j = 0; j < m; ++j) v += st.Qk[j * nk + r] * tmp[j * nk + c];
                        res[r * S + c] = v;
                    }
                M.swap(res);
            };
            rot(st.Ht);
            rot(st.Nt);
            st.m = nk;
            spk::dav_cgs(s, h->dV.p, ld, 0, st.m, sm + lay.pc2, st.nch, h->dt.p, st.n, sm + lay.pc1, 0);
        }
        // CGS2 of the extending states
        D.clear();
        max_n = 0;
        for (int i : ext) {
            D.push_back(dav_inst(B[i]));
            max_n = std::max(max_n, B[i].n);
        }
        if (!D.empty()) {
            batch_dav_upload(D, bb, s);
            spk::bdav_cgs(s, bb.dav.p, int(D.size()), max_n, 0);
            spk::bdav_cgs(s, bb.dav.p, int(D.size()), max_n, 1);
        }
        // one fused product for the new vectors (x = t) and the starting
        // vectors (x = V_0), then their Gram rows
        std::vector<int> prod = ext;
        prod.insert(prod.end(), starting.begin(), starting.end());
        if (!prod.empty()) {
            std::vector<int> from_v0(B.size(), 0);
            for (int i : starting) from_v0[i] = 1;
            batch_heff_mixed(B, prod, from_v0, bb, s);
            D.clear();
            max_n = 0;
            max_m = 0;
            for (int i : prod) {
                spk::DavInst I = dav_inst(B[i]);
                I.from_t = from_v0[i] ? 0 : 1;
                D.push_back(I);
                max_n = std::max(max_n, B[i].n);
                max_m = std::max(max_m, B[i].m);
            }
            batch_dav_upload(D, bb, s);
            spk::bdav_gram(s, bb.dav.p, int(D.size()), max_n, max_m);
        }
        HIPCK(hipStreamSynchronize(s));
        // results
        for (int i : starting) {
            BatchState& st = B[i];
            sp_handle* h = st.h;
            const DavLayout lay(h->dav_sub, spk::dav_chunks(int(h->ld)));
            const double* pg = h->pin + (lay.pg - lay.out);
            st.Ht[0] = chunk_total(pg, st.nch, 2, 0);
            st.Nt[0] = chunk_total(pg, st.nch, 2, 1);
            st.m = 1;
            st.out.matvecs = 1;
            phase[i] = 1;
        }
        std::vector<int> finished;
        for (int i : iterating) {
            BatchState& st = B[i];
            sp_handle* h = st.h;
            const DavLayout lay(h->dav_sub, spk::dav_chunks(int(h->ld)));
            const double* dn = h->pin;
            double xt[3];
            chunk_totals(dn + (lay.px - lay.out), st.nch, 3, xt);
            const double xx = xt[0], uu = xt[1], xn = xt[2];
            if (!std::isfinite(xx) || !std::isfinite(uu) || !(xx > 0.0)) throw SpError(SP_ENAN, "non-finite Ritz vector");
            st.out.rnorm = std::sqrt(uu / xx);
            st.out.pnorm = xn / xx;
            if (st.out.rnorm <= o.tol) {
                st.out.converged = true;
                finished.push_back(i);
                continue;
            }
            if (st.last) {
                finished.push_back(i);
                continue;
            }
            const double tn = dn[lay.tn - lay.out];
            if (!(tn >= 1e-14)) {
                finished.push_back(i);
                continue;
            }
            const int m = st.m, nd = 4 * m + 2;
            std::vector<double> gt(nd);
            chunk_totals(dn + (lay.pg - lay.out), st.nch, nd, gt.data());
            for (int j = 0; j <= m; ++j) {
                const double hv_new = gt[j];
                const double nv_new = gt[m + 1 + j];
                const double hv_old = (j < m) ? gt[2 * m + 2 + j] : hv_new;
                const double nv_old = (j < m) ? gt[3 * m + 2 + j] : nv_new;
                st.Ht[j * S + m] = hv_new;
                st.Nt[j * S + m] = nv_new;
                st.Ht[m * S + j] = hv_old;
                st.Nt[m * S + j] = nv_old;
            }
            ++st.m;
        }
        // step end of the states whose local solve is over
        for (int i : finished) {
            BatchState& st = B[i];
            sp_handle* h = st.h;
            const int k = st.k, d = st.order[st.step].second, L = h->L;
            spk::normalize(s, h->dx.p, site_ptr(h, k), st.n, nullptr);
            if (reduced(h)) {
                double th, pn, xx;
                rayleigh64(h, k, site_ptr(h, k), th, pn, xx);
                st.out.theta = th;
                st.out.pnorm = pn;
            }
            if (L > 1) {
                if (d > 0) {
                    move_right(h, k);
                    env_left(h, k);
                    h->center = k + 1;
                } else {
                    move_left(h, k);
                    env_right(h, k);
                    h->center = k - 1;
                }
            }
        }
        if (!finished.empty()) {
            HIPCK(hipStreamSynchronize(s));
            HIPCK(hipGetLastError());
        }
        const auto t1 = std::chrono::steady_clock::now();
        for (int i : finished) {
            BatchState& st = B[i];
            if (!st.out.converged) status = SP_ENOCONV;
            record_step(reps[i], o.verbose, i,
                        {int(st.step / st.sweep_len), st.k, st.order[st.step].second, st.out.iters,
                         st.out.converged ? 1 : 0, st.out.matvecs, st.out.theta, st.out.pnorm, st.out.rnorm,
                         std::chrono::duration<double, std::micro>(t1 - st.t0).count()});
            ++st.step;
            phase[i] = st.step < st.order.size() ? 0 : 2;
        }
    }
    return status;
}

}  // namespace

namespace {

// ---------------------------------------------------------------------------
// Sweeps with the device-resident Davidson iteration.  Every state (one or
// many) advances in rounds: in a round each unfinished state solves the
// local problem at its next site.  The first product (V_0) runs eagerly; then
// one iteration of every state - subspace solve, Ritz pass, restart
// rotation, CGS2, H_eff of the correction (one fused launch for all states
// and quadrature points), Gram pass, residual and convergence bookkeeping -
// is captured once in a HIP graph and replayed until no state iterates (the
// host polls a mapped status record every few replays).  A state whose solve
// has ended is idle in the remaining replays of its round: its passes and
// its fused H_eff tasks return at once.  Then the gauge moves and
// environment updates of all states run eagerly, and the next round starts.

// whether these settings run the device-resident iteration for a sweep of
// nstates states
bool device_solver_ok(const sp_handle* h, const sp_sweep_opts& o, int nstates) {
    const int max_sub = std::max(2, o.max_sub);
    const int keep = std::max(1, std::min(o.keep, max_sub - 1));
    const bool want = o.solver == SP_SOLVER_DEVICE || (o.solver == SP_SOLVER_AUTO && nstates >= 2);
    return want && h->path == SP_PATH_TILED && h->cons.empty() && !h->mlp_use && !h->mlp_rec &&
           max_sub + 1 <= spk::kDevSubMax && keep <= spk::kDevKeepMax;
}

spk::DavInst dev_inst(BatchState& st, const sp_sweep_opts& o, int max_sub, int keep, int max_iter, double* status) {
    sp_handle* h = st.h;
    const long long ld = h->ld;
    const DavLayout lay(h->dav_sub, spk::dav_chunks(int(ld)));
    double* sm = h->dsmall.p;
    spk::DavInst I{};
    I.V = h->dV.p;
    I.HV = h->dHV.p;
    I.NV = h->dNV.p;
    I.ld = ld;
    I.aqd = sm + lay.a;
    I.aq = I.aqd;
    I.dh = h->ddh.p;
    I.dn = h->ddn.p;
    I.floor_ = 1e-8;
    I.x = h->dx.p;
    I.t = h->dt.p;
    I.part_x = sm + lay.px;
    I.pc1 = sm + lay.pc1;
    I.pc2 = sm + lay.pc2;
    I.pn = sm + lay.pn;
    I.pg = sm + lay.pg;
    I.tnorm = sm + lay.tn;
    I.ypart = h->ypart.p;
    I.nypart = h->nypart.p;
    I.gstride = st.n;
    I.G = heff_parts(h, st.k);
    I.Gn = h->G;
    I.m = 0;  // the first Gram pass (V_0, products read from the partials)
    I.mr = 0;
    I.n = st.n;
    I.active = 1;
    I.from_t = 0;
    I.ext = 1;
    I.max_iter = max_iter;
    I.max_sub = max_sub;
    I.keep = keep;
    I.S = max_sub + 1;
    I.nch = st.nch;
    I.tol = o.tol;
    I.drop = metric_drop(h);
    I.Ht = h->dHt.p;
    I.Nt = h->dNt.p;
    I.Qk = sm + lay.q;
    I.status = status;
    return I;
}

int sweep_rounds(std::vector<BatchState>& B, const sp_sweep_opts& o, std::vector<sp_sweep_report*>& reps) {
    hipStream_t s = B[0].h->stream;
    const int max_sub = std::max(2, o.max_sub);
    const int keep = std::max(1, std::min(o.keep, max_sub - 1));
    const int max_iter = std::max(1, o.max_iter);
    const int nb = int(B.size());
    for (auto& st : B) ensure_davidson(st.h, max_sub);
    BatchBufs bb;
    // mapped status (8 doubles per state) and pinned staging of the records
    double *stat = nullptr, *stat_dev = nullptr, *stage = nullptr;
    HIPCK(hipHostMalloc(&stat, size_t(8) * nb * sizeof(double), hipHostMallocMapped | hipHostMallocCoherent));
    HIPCK(hipHostGetDevicePointer((void**)&stat_dev, stat, 0));
    HIPCK(hipHostMalloc(&stage, size_t(nb) * sizeof(spk::DavInst), hipHostMallocDefault));
    hipStream_t gs = nullptr;
    HIPCK(hipStreamCreateWithFlags(&gs, hipStreamNonBlocking));
    struct Cleanup {
        double *a, *b;
        hipStream_t g;
        ~Cleanup() {
            if (a) (void)hipHostFree(a);
            if (b) (void)hipHostFree(b);
            if (g) (void)hipStreamDestroy(g);
        }
    } cleanup{stat, stage, gs};
    DArr<spk::DavInst> dinst;
    dinst.alloc(nb);
    DArr<char> ginst;
    int status = SP_OK;
    const int poll = 4;  // replays between two looks at the status
    for (;;) {
        std::vector<int> idx;
        for (int i = 0; i < nb; ++i)
            if (B[i].step < B[i].order.size()) idx.push_back(i);
        if (idx.empty()) break;
        const int na = int(idx.size());
        int max_n = 0;
        // step start: diagonal, V_0 and its products (eager)
        for (int i : idx) {
            BatchState& st = B[i];
            sp_handle* h = st.h;
            st.k = st.order[st.step].first;
            st.n = int(h->sites[st.k - 1].size);
            st.nch = spk::dav_chunks(st.n);
            st.t0 = std::chrono::steady_clock::now();
            max_n = std::max(max_n, st.n);
            diag(h, st.k, h->ddh.p, h->ddn.p);
            spk::normalize(s, site_ptr(h, st.k), h->dV.p, st.n, nullptr);
        }
        {
            std::vector<int> from_v0(B.size(), 1);
            batch_heff_mixed(B, idx, from_v0, bb, s);
        }
        spk::DavInst* D = reinterpret_cast<spk::DavInst*>(stage);
        for (int q = 0; q < na; ++q) {
            for (int c = 0; c < 8; ++c) stat[8 * q + c] = 0.0;
            D[q] = dev_inst(B[idx[q]], o, max_sub, keep, max_iter, stat_dev + 8 * q);
        }
        HIPCK(hipMemcpyAsync(dinst.p, D, size_t(na) * sizeof(spk::DavInst), hipMemcpyHostToDevice, s));
        spk::bdav_gram(s, dinst.p, na, max_n, 0);
        spk::bdav_start(s, dinst.p, na);
        // H_eff x of the corrections: the instance records on the device for
        // the whole round, each instance gated by its record
        HeffBatch hb;
        for (int q = 0; q < na; ++q)
            hb.add(B[idx[q]].h, B[idx[q]].k, B[idx[q]].h->dt.p,
                   reinterpret_cast<const int*>(reinterpret_cast<const char*>(dinst.p + q) + offsetof(spk::DavInst, ext)));
        hb.finish();
        if (ginst.n < hb.bytes()) ginst.alloc(hb.bytes());
        {
            std::vector<char> rec(hb.bytes());
            hb.pack(rec.data());
            HIPCK(hipMemcpy(ginst.p, rec.data(), rec.size(), hipMemcpyHostToDevice));
        }
        HIPCK(hipStreamSynchronize(s));
        // one iteration of every state, captured on the private stream
        hipGraph_t graph = nullptr;
        hipGraphExec_t exec = nullptr;
        hipError_t ce = hipStreamBeginCapture(gs, hipStreamCaptureModeThreadLocal);
        if (ce == hipSuccess) {
            spk::bdav_solve(gs, dinst.p, na, max_sub);
            spk::bdav_ritz(gs, dinst.p, na, max_n);
            spk::bdav_rotate(gs, dinst.p, na, max_n);
            spk::bdav_cgs(gs, dinst.p, na, max_n, 2);
            spk::bdav_cgs(gs, dinst.p, na, max_n, 0);
            spk::bdav_cgs(gs, dinst.p, na, max_n, 1);
            hb.launch(gs, ginst.p);
            spk::bdav_gram(gs, dinst.p, na, max_n, max_sub);
            spk::bdav_update(gs, dinst.p, na);
            ce = hipStreamEndCapture(gs, &graph);
        }
        hip_check(ce, "capture of the Davidson iteration");
        HIPCK(hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0));
        int replays = 0;
        bool running = true;
        while (running && replays < max_iter + 1) {
            for (int r = 0; r < poll && replays < max_iter + 1; ++r, ++replays) HIPCK(hipGraphLaunch(exec, gs));
            HIPCK(hipStreamSynchronize(gs));
            running = false;
            for (int q = 0; q < na; ++q) running = running || stat[8 * q] != 0.0;
        }
        (void)hipGraphExecDestroy(exec);
        (void)hipGraphDestroy(graph);
        HIPCK(hipGetLastError());
        if (running) throw SpError(SP_EHIP, "internal: a device-resident local solve did not end");
        // step end
        for (int q = 0; q < na; ++q) {
            const double* sq = stat + 8 * q;
            const int err = int(sq[7]);
            if (err == SP_ENORM) throw SpError(SP_ENORM, "projected norm vanishes in the search space");
            if (err != 0) throw SpError(SP_ENAN, "non-finite value in a local solve");
            BatchState& st = B[idx[q]];
            st.out = DavOut{};
            st.out.converged = sq[1] != 0.0;
            st.out.iters = int(sq[2]);
            st.out.matvecs = int(sq[3]);
            st.out.theta = sq[4];
            st.out.rnorm = sq[5];
            st.out.pnorm = sq[6];
            sp_handle* h = st.h;
            const int k = st.k, d = st.order[st.step].second, L = h->L;
            spk::normalize(s, h->dx.p, site_ptr(h, k), st.n, nullptr);
            if (reduced(h)) {
                double th, pn, xx;
                rayleigh64(h, k, site_ptr(h, k), th, pn, xx);
                if (!std::isfinite(th)) throw SpError(SP_ENAN, "non-finite Rayleigh quotient");
                st.out.theta = th;
                st.out.pnorm = pn;
            }
            if (L > 1) {
                if (d > 0) {
                    move_right(h, k);
                    env_left(h, k);
                    h->center = k + 1;
                } else {
                    move_left(h, k);
                    env_right(h, k);
                    h->center = k - 1;
                }
            }
        }
        HIPCK(hipStreamSynchronize(s));
        HIPCK(hipGetLastError());
        const auto t1 = std::chrono::steady_clock::now();
        for (int q = 0; q < na; ++q) {
            const int i = idx[q];
            BatchState& st = B[i];
            if (!st.out.converged) status = SP_ENOCONV;
            record_step(reps[i], o.verbose, i,
                        {int(st.step / st.sweep_len), st.k, st.order[st.step].second, st.out.iters,
                         st.out.converged ? 1 : 0, st.out.matvecs, st.out.theta, st.out.pnorm, st.out.rnorm,
                         std::chrono::duration<double, std::micro>(t1 - st.t0).count()});
            ++st.step;
        }
    }
    return status;
}

}  // namespace

// ---------------------------------------------------------------------------
// Allocation-free H_eff x (sp_heff_apply_noalloc): its per-g partial slots
// live in a fixed device array instead of the handle's buffers.  Every GPU
// that runs the library holds its own copy until the process ends.  Host code
// never passes the array's name to a kernel: its device address on each
// device comes from hipGetSymbolAddress, taken once per device at
// sp_init_mps with that device current.

static __device__ __align__(256) double scratch[2 * kNoAllocSlots];

namespace {
std::mutex g_scratch_mu;
std::map<int, double*> g_scratch_ptr;  // device -> device address of its scratch

// address of the scratch array on `device`; resolved on the first call for
// the device (with that device current), cached afterwards
double* noalloc_scratch(int device) {
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    auto it = g_scratch_ptr.find(device);
    if (it != g_scratch_ptr.end()) return it->second;
    int cur = 0;
    HIPCK(hipGetDevice(&cur));
    if (cur != device) HIPCK(hipSetDevice(device));
    void* ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (cur != device) HIPCK(hipSetDevice(cur));
    hip_check(e, "hipGetSymbolAddress(scratch)");
    if (!ptr) throw SpError(SP_EHIP, "hipGetSymbolAddress(scratch) returned a null address");
    g_scratch_ptr[device] = static_cast<double*>(ptr);
    return static_cast<double*>(ptr);
}
}  // namespace

// ---------------------------------------------------------------------------
// C ABI

namespace {
int guarded(const std::function<int()>& f) {
    try {
        return f();
    } catch (const SpError& e) {
        g_last_error = e.what();
        return e.code;
    } catch (const std::bad_alloc&) {
        g_last_error = "host allocation failed";
        return SP_ENOMEM;
    } catch (const std::exception& e) {
        g_last_error = e.what();
        return SP_EINVAL;
    }
}
}  // namespace

extern "C" {

const char* sp_last_error(void) { return g_last_error.c_str(); }

int sp_init_mps(const sp_problem* p, const sp_mpo* W, const sp_block_table* bonds, const double* init_blocks,
                void* hip_stream, sp_handle** out) {
    return guarded([&]() -> int {
        SP_REQUIRE(p && W && bonds && init_blocks && out, "null argument");
        *out = nullptr;
        SP_REQUIRE(p->L >= 1 && p->d == 4, "need L >= 1 and d == 4");
        SP_REQUIRE(p->precision == SP_FP64 || p->precision == SP_FP32 || p->precision == SP_BF16X3,
                   "precision must be SP_FP64, SP_FP32 or SP_BF16X3");
        SP_REQUIRE(p->precision == SP_FP64 || p->path == SP_PATH_TILED, "reduced precision needs the tiled path");
        SP_REQUIRE(p->path == SP_PATH_TILED || p->path == SP_PATH_PLAIN, "unknown kernel path");
        SP_REQUIRE(p->N >= 0 && p->N <= 2 * p->L, "N out of range");
        SP_REQUIRE((p->N + p->twoS) % 2 == 0, "N and 2S must have the same parity");
        SP_REQUIRE((p->N + p->twoM) % 2 == 0, "N and 2M must have the same parity");
        SP_REQUIRE(p->twoS >= 0 && std::abs(p->twoM) <= p->twoS, "need |M| <= S");
        SP_REQUIRE(p->twoS <= sph::max_seniority(p->N, p->twoM, p->L), "S exceeds the largest seniority");
        SP_REQUIRE(p->G >= 1 && p->G <= 1024, "G out of range");
        std::unique_ptr<sp_handle> h(new sp_handle());
        h->stream = reinterpret_cast<hipStream_t>(hip_stream);
        h->path = p->path;
        h->precision = p->precision;
        h->L = p->L;
        h->N = p->N;
        h->twoS = p->twoS;
        h->twoM = p->twoM;
        h->G = p->G;
        h->inexact = p->G < sph::exact_points(p->N, p->L, p->twoS, p->twoM);
        h->qx.resize(h->G);
        h->qw.resize(h->G);
        h->qc.resize(h->G);
        h->qs.resize(h->G);
        h->qcoef.resize(h->G);
        sph::projector_quadrature(h->G, h->twoS, h->twoM, h->qx.data(), h->qw.data(), h->qc.data(), h->qs.data(),
                                  h->qcoef.data());
        build_mpo(h.get(), W);
        build_bonds(h.get(), bonds);
        {
            int tot = 0;
            for (int k = 0; k <= h->L; ++k) tot += bonds->nsec[k];
            h->tab_nsec.assign(bonds->nsec, bonds->nsec + h->L + 1);
            h->tab_n.assign(bonds->sec_n, bonds->sec_n + tot);
            h->tab_2m.assign(bonds->sec_2m, bonds->sec_2m + tot);
            h->tab_dim.assign(bonds->sec_dim, bonds->sec_dim + tot);
        }
        build_env_layouts(h.get());
        h->plan.resize(h->L);
        long long Tmax = 0, Vmax = 0, qrs = 0, qrr = 0, LTmax = 0;
        for_sites(h->L, [&](int k) {
            build_plan(h.get(), k);
            if (h->path == SP_PATH_TILED) {
                if (!build_fused(h.get(), k)) build_fused(h.get(), k, kHeffLdsMax);
                build_chain(h.get(), k);
            }
            if (h->path == SP_PATH_TILED && h->plan[k - 1].h_rows == 1) {
                // wide MPOs: block products, in the reduced precisions FP64
                // or split BF16
                SitePlan& P1 = h->plan[k - 1];
                P1.h_rows = 0;
                P1.h_lds = 0;
            }
        });
        for (int k = 1; k <= h->L; ++k) {
            const SitePlan& P = h->plan[k - 1];
            // the diagonals use the scratch of the plain path's passes; a tiled
            // state has it for them alone
            const long long dgT = (long long)P.dg_nzl * h->bonds[k - 1].D + (long long)P.dg_nzr * h->bonds[k].D;
            Tmax = std::max({Tmax, P.Tsize, P.Zsize, dgT});
            Vmax = std::max({Vmax, P.Vsize, P.Ztsize, (long long)P.dg_mix.size() * h->bonds[k - 1].D});
            LTmax = std::max({LTmax, P.mix_l.size, P.mix_r.size});
            h->mixes = h->mixes || !P.mix_l.empty() || !P.mix_r.empty();
            qrs = std::max({qrs, P.qr_scratch, P.lq_scratch});
            qrr = std::max({qrr, P.qr_rsize, P.lq_rsize});
        }
        h->T_cap = h->G * std::max(1LL, Tmax);
        h->V_cap = h->G * std::max(1LL, Vmax);
        h->LT_cap = h->path == SP_PATH_TILED ? h->G * std::max(1LL, LTmax) : 1;
        h->qr_scratch_cap = std::max(1LL, qrs);
        h->qr_r_cap = std::max(1LL, qrr);
        for (int k = 1; k <= h->L; ++k) {
            h->Xd_cap = std::max(h->Xd_cap, h->plan[k - 1].Xd_size);
            h->Xr_cap = std::max(h->Xr_cap, h->G * (long long)h->plan[k - 1].rmap_h.size());
            h->y_split_max = std::max(h->y_split_max, h->plan[k - 1].y_split);
        }
        h->Xd_cap = std::max(1LL, h->Xd_cap);
        validate_plans(h.get());
        // every host-side check is done; device work starts here
        HIPCK(hipGetDevice(&h->device));
        alloc_envs(h.get());
        {
            Upload u;
            for (int k = 1; k <= h->L; ++k) upload_plan(h.get(), k, u);
            u.finish(h->plan_mem, h->stream);
        }
        h->T.alloc(h->T_cap);
        h->V.alloc(h->V_cap);
        h->LT.alloc(h->LT_cap + read_pad(h.get()));
        h->diag_part.alloc(size_t(spk::kDiagSplitMax) * std::max(1LL, h->max_site));
        h->qr_scratch.alloc(h->qr_scratch_cap);
        h->qr_r.alloc(h->qr_r_cap);
        h->tmp_site.alloc(h->max_site);
        h->mps.alloc(h->mps_size);
        if (h->path == SP_PATH_TILED) {
            h->Xd.alloc(h->Xd_cap + read_pad(h.get()));
            h->Xr.alloc(h->Xr_cap + read_pad(h.get()));
            h->ypart.alloc(size_t(h->G) * h->y_split_max * h->max_site);
            h->nypart.alloc(size_t(h->G) * h->max_site);
        }
        HIPCK(hipMemcpyAsync(h->mps.p, init_blocks, h->mps_size * sizeof(double), hipMemcpyHostToDevice, h->stream));
        // right-canonical form of sites L..2 and the right environments
        for (int k = h->L; k >= 2; --k) {
            move_left(h.get(), k);
            env_right(h.get(), k);
        }
        h->center = 1;
        HIPCK(hipStreamSynchronize(h->stream));
        HIPCK(hipGetLastError());
        if (h->path == SP_PATH_TILED) (void)noalloc_scratch(h->device);
        *out = h.release();
        return (*out)->inexact ? SP_WINEXACT : SP_OK;
    });
}

int sp_destroy(sp_handle* h) {
    return guarded([&]() -> int {
        if (!h) return SP_OK;
        (void)hipStreamSynchronize(h->stream);
        delete h;
        return SP_OK;
    });
}

int sp_env_update(sp_handle* h, int site, int dir) {
    return guarded([&]() -> int {
        SP_REQUIRE(h, "null handle");
        check_site(h, site);
        SP_REQUIRE(dir == 1 || dir == -1, "dir must be +1 or -1");
        forget_mix(h);
        if (dir > 0) env_left(h, site);
        else env_right(h, site);
        HIPCK(hipGetLastError());
        return SP_OK;
    });
}

int sp_heff_apply(sp_handle* h, int site, const double* x, double* y, double* ny) {
    return guarded([&]() -> int {
        SP_REQUIRE(h && x && y && ny, "null argument");
        check_site(h, site);
        SP_REQUIRE(x != y && x != ny && y != ny, "x, y and ny must not alias");
        forget_mix(h);
        heff_apply(h, site, x, y, ny);
        HIPCK(hipGetLastError());
        return SP_OK;
    });
}

int sp_heff_apply_noalloc(sp_handle* h, int site, const double* x, double* y, double* ny) {
    return guarded([&]() -> int {
        SP_REQUIRE(h && x && y && ny, "null argument");
        check_site(h, site);
        SP_REQUIRE(x != y && x != ny && y != ny, "x, y and ny must not alias");
        SP_REQUIRE(h->path == SP_PATH_TILED, "sp_heff_apply_noalloc: tiled path only");
        const long long need = (long long)heff_parts(h, site) * h->sites[site - 1].size;
        if (need > kNoAllocSlots)
            throw SpError(SP_EINVAL, "sp_heff_apply_noalloc: the site needs " + std::to_string(need) +
                                         " partial slots per output, more than the fixed " +
                                         std::to_string(kNoAllocSlots));
        std::unique_lock<std::mutex> lk(g_scratch_mu);
        auto it = g_scratch_ptr.find(h->device);
        SP_REQUIRE(it != g_scratch_ptr.end(), "internal: scratch address of the device not resolved");
        double* base = it->second;
        lk.unlock();
        forget_mix(h);
        heff_apply(h, site, x, y, ny, false, false, base, base + kNoAllocSlots);
        HIPCK(hipGetLastError());
        return SP_OK;
    });
}

int sp_heff_diag(sp_handle* h, int site, double* dh, double* dn) {
    return guarded([&]() -> int {
        SP_REQUIRE(h && dh && dn, "null argument");
        check_site(h, site);
        diag(h, site, dh, dn);
        HIPCK(hipGetLastError());
        return SP_OK;
    });
}

int sp_sweep(sp_handle* h, const sp_sweep_opts* o, sp_sweep_report* r) {
    return guarded([&]() -> int {
        SP_REQUIRE(h && o, "null argument");
        SP_REQUIRE(o->n_sweeps >= 0 && o->max_iter >= 1 && o->max_sub >= 2 && o->keep >= 1 && o->tol >= 0,
                   "bad sweep options");
        SP_REQUIRE(h->center == 1, "sweeps start with the canonical centre at site 1");
        forget_mix(h);
        if (r) r->n_steps = 0;
        SP_REQUIRE(o->solver >= SP_SOLVER_AUTO && o->solver <= SP_SOLVER_DEVICE, "unknown solver");
        if (device_solver_ok(h, *o, 1)) {
            std::vector<BatchState> B(1);
            std::vector<sp_sweep_report*> reps(1, r);
            B[0].h = h;
            const int L = h->L;
            std::vector<std::pair<int, int>> one;
            for (int k = 1; k < L; ++k) one.push_back({k, +1});
            for (int k = L; k >= 2; --k) one.push_back({k, -1});
            if (L == 1) one.push_back({1, +1});
            B[0].sweep_len = int(one.size());
            for (int sw = 0; sw < o->n_sweeps; ++sw) B[0].order.insert(B[0].order.end(), one.begin(), one.end());
            return sweep_rounds(B, *o, reps);
        }
        int status = SP_OK;
        const int L = h->L;
        for (int sw = 0; sw < o->n_sweeps; ++sw) {
            std::vector<std::pair<int, int>> order;
            for (int k = 1; k < L; ++k) order.push_back({k, +1});
            for (int k = L; k >= 2; --k) order.push_back({k, -1});
            if (L == 1) order.push_back({1, +1});
            for (auto [k, d] : order) {
                const auto t0 = std::chrono::steady_clock::now();
                prepare_constraints(h, k);
                DavOut dv = davidson(h, k, *o);
                if (L > 1) {
                    if (d > 0) {
                        move_right(h, k);
                        env_left(h, k);
                        for (auto& a : h->cons) env_left_mixed(a.get(), k, site_ptr(h, k));
                        h->center = k + 1;
                    } else {
                        move_left(h, k);
                        env_right(h, k);
                        for (auto& a : h->cons) env_right_mixed(a.get(), k, site_ptr(h, k));
                        h->center = k - 1;
                    }
                }
                HIPCK(hipStreamSynchronize(h->stream));
                HIPCK(hipGetLastError());
                const auto t1 = std::chrono::steady_clock::now();
                if (!dv.converged) status = SP_ENOCONV;
                record_step(r, o->verbose, 0,
                            {sw, k, d, dv.iters, dv.converged ? 1 : 0, dv.matvecs, dv.theta, dv.pnorm, dv.rnorm,
                             std::chrono::duration<double, std::micro>(t1 - t0).count()});
            }
        }
        return status;
    });
}

int sp_sweep_batch(sp_handle** hs, int n, const sp_sweep_opts* o, sp_sweep_report* r) {
    return guarded([&]() -> int {
        SP_REQUIRE(hs && o && n >= 1, "bad arguments");
        SP_REQUIRE(o->n_sweeps >= 0 && o->max_iter >= 1 && o->max_sub >= 2 && o->keep >= 1 && o->tol >= 0,
                   "bad sweep options");
        std::vector<BatchState> B(n);
        std::vector<sp_sweep_report*> reps(n, nullptr);
        for (int i = 0; i < n; ++i) {
            sp_handle* h = hs[i];
            SP_REQUIRE(h, "null handle");
            SP_REQUIRE(h->path == SP_PATH_TILED, "batched sweeps need the tiled path");
            SP_REQUIRE(h->cons.empty(), "states with orthogonality constraints sweep with sp_sweep");
            SP_REQUIRE(!h->mlp_use && !h->mlp_rec, "states with a learned preconditioner sweep with sp_sweep");
            SP_REQUIRE(h->stream == hs[0]->stream && h->device == hs[0]->device,
                       "batched handles must share one device and one stream");
            SP_REQUIRE(h->precision == hs[0]->precision, "batched handles must share the precision");
            SP_REQUIRE(h->center == 1, "sweeps start with the canonical centre at site 1");
            for (int j = 0; j < i; ++j) SP_REQUIRE(hs[j] != h, "a handle appears twice in the batch");
            forget_mix(h);
            B[i].h = h;
            const int L = h->L;
            std::vector<std::pair<int, int>> one;
            for (int k = 1; k < L; ++k) one.push_back({k, +1});
            for (int k = L; k >= 2; --k) one.push_back({k, -1});
            if (L == 1) one.push_back({1, +1});
            B[i].sweep_len = int(one.size());
            for (int sw = 0; sw < o->n_sweeps; ++sw) B[i].order.insert(B[i].order.end(), one.begin(), one.end());
            if (r) {
                reps[i] = &r[i];
                r[i].n_steps = 0;
            }
        }
        SP_REQUIRE(o->solver >= SP_SOLVER_AUTO && o->solver <= SP_SOLVER_DEVICE, "unknown solver");
        bool dev = true;
        for (int i = 0; i < n; ++i) dev = dev && device_solver_ok(hs[i], *o, n);
        return dev ? sweep_rounds(B, *o, reps) : sweep_batch(B, *o, reps);
    });
}

int sp_autotune(sp_handle* h, int reps, int* budget_out, int* rows_out, double* usec_out) {
    return guarded([&]() -> int {
        SP_REQUIRE(h && reps >= 1, "bad arguments");
        SP_REQUIRE(h->path == SP_PATH_TILED, "the autotuner tunes the H_eff plans of the tiled path");
        forget_mix(h);
        const int candidates[] = {4608, 9216, 13824, kHeffLdsMax};
        hipStream_t s = h->stream;
        hipEvent_t e0, e1;
        HIPCK(hipEventCreate(&e0));
        HIPCK(hipEventCreate(&e1));
        for (int k = 1; k <= h->L; ++k) {
            SitePlan& P = h->plan[k - 1];
            const double* x = site_ptr(h, k);
            int best_b = 0, best_rc = 0;
            float best = 1e30f;
            auto time_plan = [&](int budget) {
                const int mode = heff_mode(h, k, false);
                auto launch = [&]() { heff_partials(h, k, x, mode, h->ypart.p, h->nypart.p); };
                launch();  // warm-up (also mixes the left environment)
                HIPCK(hipEventRecord(e0, s));
                for (int r = 0; r < reps; ++r) launch();
                HIPCK(hipEventRecord(e1, s));
                HIPCK(hipEventSynchronize(e1));
                float ms = 0.f;
                HIPCK(hipEventElapsedTime(&ms, e0, e1));
                HIPCK(hipGetLastError());
                if (ms < best) {
                    best = ms;
                    best_b = budget;
                    best_rc = P.h_rows;
                }
            };
            // a site's products run the same lists whatever the plan; it sets
            // their arithmetic in the reduced precisions, so the first budget
            // that fits stands for all and in FP64 for the block products too
            for (int b : candidates)
                if (build_fused(h, k, b)) {
                    time_plan(b);
                    break;
                }
            if (best_b == 0 || reduced(h)) {
                P.h_rows = P.h_lds = 0;
                time_plan(0);
            }
            if (best_b > 0) build_fused(h, k, best_b);
            if (budget_out) budget_out[k - 1] = best_b;
            if (rows_out) rows_out[k - 1] = best_rc;
            if (usec_out) usec_out[k - 1] = 1e3 * double(best) / reps;
        }
        (void)hipEventDestroy(e0);
        (void)hipEventDestroy(e1);
        return SP_OK;
    });
}

int sp_heff_plan(const sp_handle* h, int site, int* rows, int* lds_doubles) {
    return guarded([&]() -> int {
        SP_REQUIRE(h && rows, "bad arguments");
        check_site(h, site);
        *rows = h->plan[site - 1].h_rows;
        if (lds_doubles) *lds_doubles = h->plan[site - 1].h_lds;
        return SP_OK;
    });
}

int sp_set_heff_plan(sp_handle* h, int site, int lds_budget, int* rows) {
    return guarded([&]() -> int {
        SP_REQUIRE(h, "bad arguments");
        check_site(h, site);
        SP_REQUIRE(h->path == SP_PATH_TILED, "H_eff plans belong to the tiled path");
        SP_REQUIRE(lds_budget == 0 || (lds_budget >= 1 && lds_budget <= kHeffLdsMax),
                   "LDS budget outside 0..18432 doubles");
        SitePlan& P = h->plan[site - 1];
        HIPCK(hipStreamSynchronize(h->stream));  // the old plan may still be in use
        if (lds_budget == 0 || !build_fused(h, site, lds_budget)) P.h_rows = P.h_lds = 0;
        if (rows) *rows = P.h_rows;
        return SP_OK;
    });
}

int sp_expect(sp_handle* h, const sp_mpo* O, double* value, double* normP) {
    return guarded([&]() -> int {
        SP_REQUIRE(h && O && value, "null argument");
        // a second state with the operator's environments: the same site
        // tensors (its set-up moves the canonical centre to site 1 without
        // changing the state), then <O P>/<P> at its centre
        std::vector<double> blocks(h->mps_size);
        HIPCK(hipMemcpyAsync(blocks.data(), h->mps.p, h->mps_size * sizeof(double), hipMemcpyDeviceToHost, h->stream));
        HIPCK(hipStreamSynchronize(h->stream));
        sp_problem p{h->L, 4, h->N, h->twoS, h->twoM, h->G, SP_FP64, h->path};
        sp_block_table bt{h->tab_nsec.data(), h->tab_n.data(), h->tab_2m.data(), h->tab_dim.data()};
        sp_handle* t = nullptr;
        const int rc = sp_init_mps(&p, O, &bt, blocks.data(), h->stream, &t);
        if (rc < 0) throw SpError(rc, std::string("operator state: ") + g_last_error);
        std::unique_ptr<sp_handle, int (*)(sp_handle*)> guard(t, sp_destroy);
        double np = 0.0;
        const int rc2 = sp_energy(t, value, &np);
        if (rc2 < 0) throw SpError(rc2, g_last_error);
        if (normP) *normP = np;
        return SP_OK;
    });
}

int sp_add_orthogonality(sp_handle* h, sp_handle* lower) {
    return guarded([&]() -> int {
        SP_REQUIRE(h && lower && h != lower, "bad arguments");
        SP_REQUIRE(int(h->cons.size()) < kMaxConstraints, "at most 8 orthogonality constraints");
        SP_REQUIRE(h->center == 1, "constraints are added with the canonical centre at site 1");
        SP_REQUIRE(lower->L == h->L && lower->N == h->N && lower->twoS == h->twoS && lower->twoM == h->twoM &&
                       lower->G == h->G,
                   "the lower state must have the same L, N, S, M and quadrature");
        SP_REQUIRE(lower->tab_nsec == h->tab_nsec && lower->tab_n == h->tab_n && lower->tab_2m == h->tab_2m &&
                       lower->tab_dim == h->tab_dim,
                   "the lower state must have the same block table");
        SP_REQUIRE(lower->device == h->device, "the lower state must live on the same device");
        const int L = h->L;
        // the lower state's tensors as they are now
        std::vector<double> blocks(lower->mps_size);
        HIPCK(hipStreamSynchronize(h->stream));
        HIPCK(hipMemcpyAsync(blocks.data(), lower->mps.p, lower->mps_size * sizeof(double), hipMemcpyDeviceToHost,
                             lower->stream));
        HIPCK(hipStreamSynchronize(lower->stream));
        std::vector<int> w(L + 1);
        long long nw = 0;
        sph::mpo_identity(L, w.data(), nullptr, &nw);
        std::vector<double> wd(nw);
        sph::mpo_identity(L, w.data(), wd.data(), &nw);
        sp_problem p{L, 4, h->N, h->twoS, h->twoM, h->G, SP_FP64, SP_PATH_PLAIN};
        sp_mpo W{w.data(), wd.data()};
        sp_block_table bt{h->tab_nsec.data(), h->tab_n.data(), h->tab_2m.data(), h->tab_dim.data()};
        sp_handle* a = nullptr;
        const int rc = sp_init_mps(&p, &W, &bt, blocks.data(), h->stream, &a);
        if (rc < 0) throw SpError(rc, std::string("constraint state: ") + g_last_error);
        std::unique_ptr<sp_handle> ap(a);
        // mixed right environments against this state's right-canonical sites
        for (int k = L; k >= 2; --k) env_right_mixed(a, k, site_ptr(h, k));
        if (h->conB.n == 0) {
            h->cld = (h->max_site + 63) / 64 * 64;
            h->conB.alloc(size_t(kMaxConstraints) * h->cld);
            const int nch = spk::dav_chunks(int(h->max_site));
            h->conPart.alloc(size_t(2) * nch * kMaxConstraints);
            void* hp = nullptr;
            HIPCK(hipHostMalloc(&hp, (size_t(2) * nch + 8) * sizeof(double), hipHostMallocMapped | hipHostMallocCoherent));
            h->con_pin = static_cast<double*>(hp);
            void* dp = nullptr;
            HIPCK(hipHostGetDevicePointer(&dp, hp, 0));
            h->con_pin_dev = static_cast<double*>(dp);
        }
        HIPCK(hipStreamSynchronize(h->stream));
        HIPCK(hipGetLastError());
        h->cons.push_back(std::move(ap));
        return SP_OK;
    });
}

int sp_clear_orthogonality(sp_handle* h) {
    return guarded([&]() -> int {
        SP_REQUIRE(h, "null argument");
        HIPCK(hipStreamSynchronize(h->stream));
        h->cons.clear();
        h->con_active = 0;
        return SP_OK;
    });
}

int sp_orthogonality_overlaps(sp_handle* h, double* out) {
    return guarded([&]() -> int {
        SP_REQUIRE(h && (out || h->cons.empty()), "null argument");
        const int c = h->center;
        const int n = int(h->sites[c - 1].size);
        const size_t nc = h->cons.size();
        if (nc == 0) return SP_OK;
        // per constraint: B.x, then |lower| (its site 1 carries the norm: the
        // constraint state stays right-canonical) and |x| (x = the centre)
        DArr<double> d;
        d.alloc(2 * h->max_site + 2 * nc + 1);
        double* res = d.p + 2 * h->max_site;
        for (size_t j = 0; j < nc; ++j) {
            sp_handle* a = h->cons[j].get();
            SP_REQUIRE(a->Lvalid[c - 1] && a->Rvalid[c], "constraint environments do not reach the centre");
            constraint_vector(a, c, d.p, d.p + h->max_site);
            spk::multidot(h->stream, d.p, 0, 1, site_ptr(h, c), n, res + j);
            spk::normalize(h->stream, site_ptr(a, 1), d.p, int(a->sites[0].size), res + nc + j);
        }
        spk::normalize(h->stream, site_ptr(h, c), d.p, n, res + 2 * nc);
        std::vector<double> hres(2 * nc + 1);
        HIPCK(hipMemcpyAsync(hres.data(), res, hres.size() * sizeof(double), hipMemcpyDeviceToHost, h->stream));
        HIPCK(hipStreamSynchronize(h->stream));
        HIPCK(hipGetLastError());
        for (size_t j = 0; j < nc; ++j) {
            const double den = hres[nc + j] * hres[2 * nc];
            out[j] = den > 0.0 ? hres[j] / den : 0.0;
        }
        return SP_OK;
    });
}

int sp_mlp_create(int hidden, const float* w_init, long long capacity, sp_mlp** out) {
    return guarded([&]() -> int {
        SP_REQUIRE(out && w_init && hidden >= 1 && hidden <= spk::kMlpMaxHidden && capacity >= 0, "bad arguments");
        auto m = std::make_unique<sp_mlp>();
        m->hidden = hidden;
        HIPCK(hipGetDevice(&m->device));
        const long long P = spk::mlp_size(hidden);
        m->w.alloc(P);
        HIPCK(hipMemcpy(m->w.p, w_init, P * sizeof(float), hipMemcpyHostToDevice));
        m->m.alloc(P);
        m->v.alloc(P);
        HIPCK(hipMemset(m->m.p, 0, P * sizeof(double)));
        HIPCK(hipMemset(m->v.p, 0, P * sizeof(double)));
        m->cap = capacity;
        if (capacity > 0) {
            m->F.alloc(size_t(capacity) * spk::kMlpIn);
            m->Y.alloc(capacity);
        }
        m->nparts = 256;
        m->gpart.alloc(size_t(m->nparts) * (P + 1));
        m->scal.alloc(4096);
        *out = m.release();
        return SP_OK;
    });
}

int sp_mlp_set_scope(sp_mlp* m, int scope) {
    return guarded([&]() -> int {
        SP_REQUIRE(m, "null argument");
        SP_REQUIRE(scope == SP_MLP_VECTOR || scope == SP_MLP_NBLOCK, "unknown model scope");
        SP_REQUIRE(m->rows == 0 || scope == m->scope, "the model holds training pairs of the other scope");
        m->scope = scope;
        return SP_OK;
    });
}

int sp_mlp_destroy(sp_mlp* m) {
    return guarded([&]() -> int {
        if (m) {
            (void)hipDeviceSynchronize();
            delete m;
        }
        return SP_OK;
    });
}

int sp_mlp_get(sp_mlp* m, float* w_out, long long* rows) {
    return guarded([&]() -> int {
        SP_REQUIRE(m, "null argument");
        HIPCK(hipDeviceSynchronize());
        if (w_out) HIPCK(hipMemcpy(w_out, m->w.p, spk::mlp_size(m->hidden) * sizeof(float), hipMemcpyDeviceToHost));
        if (rows) *rows = m->rows;
        return SP_OK;
    });
}

int sp_mlp_dataset(sp_mlp* m, long long first, long long count, float* F_out, float* Y_out) {
    return guarded([&]() -> int {
        SP_REQUIRE(m && F_out && Y_out && first >= 0 && count >= 0 && first + count <= m->rows, "bad arguments");
        HIPCK(hipDeviceSynchronize());
        if (count == 0) return SP_OK;
        HIPCK(hipMemcpy(F_out, m->F.p + first * spk::kMlpIn, count * spk::kMlpIn * sizeof(float),
                        hipMemcpyDeviceToHost));
        HIPCK(hipMemcpy(Y_out, m->Y.p + first, count * sizeof(float), hipMemcpyDeviceToHost));
        return SP_OK;
    });
}

int sp_mlp_forward(sp_mlp* m, const float* F, long long n, float* y, void* stream) {
    return guarded([&]() -> int {
        SP_REQUIRE(m && (n == 0 || (F && y)) && n >= 0, "bad arguments");
        hipStream_t s = static_cast<hipStream_t>(stream);
        spk::mlp_forward(s, m->w.p, m->hidden, F, n, y);
        HIPCK(hipGetLastError());
        return SP_OK;
    });
}

int sp_mlp_train_step(sp_mlp* m, const float* F, const float* Y, long long n, double lr, double* loss, void* stream) {
    return guarded([&]() -> int {
        SP_REQUIRE(m && F && Y && n >= 1 && lr > 0.0, "bad arguments");
        hipStream_t s = static_cast<hipStream_t>(stream);
        const int parts = int(std::min<long long>(m->nparts, (n + 63) / 64));
        spk::mlp_grad(s, m->w.p, m->hidden, F, Y, 0, 1, n, m->gpart.p, parts);
        m->step++;
        spk::mlp_adam(s, m->w.p, m->m.p, m->v.p, m->hidden, m->gpart.p, parts, 1.0 / double(n), lr, m->step,
                      m->scal.p);
        double l = 0.0;
        HIPCK(hipMemcpyAsync(&l, m->scal.p, sizeof(double), hipMemcpyDeviceToHost, s));
        HIPCK(hipStreamSynchronize(s));
        if (loss) *loss = l;
        return SP_OK;
    });
}

int sp_mlp_train(sp_mlp* m, int epochs, long long batch, double lr, double* loss_out, void* stream) {
    return guarded([&]() -> int {
        SP_REQUIRE(m && epochs >= 0 && batch >= 1 && lr > 0.0, "bad arguments");
        SP_REQUIRE(m->rows > 0, "no recorded training pairs");
        hipStream_t s = static_cast<hipStream_t>(stream);
        const long long rows = m->rows;
        const long long nb = std::min<long long>((rows + batch - 1) / batch, 4096);
        for (int e = 0; e < epochs; ++e) {
            // batch b: rows b, b + nb, b + 2 nb, ... (interleaves the solves)
            for (long long b = 0; b < nb; ++b) {
                const long long count = (rows - b + nb - 1) / nb;
                const int parts = int(std::min<long long>(m->nparts, (count + 63) / 64));
                spk::mlp_grad(s, m->w.p, m->hidden, m->F.p, m->Y.p, b, nb, count, m->gpart.p, parts);
                m->step++;
                spk::mlp_adam(s, m->w.p, m->m.p, m->v.p, m->hidden, m->gpart.p, parts, 1.0 / double(count), lr,
                              m->step, m->scal.p + b);
            }
            std::vector<double> l(nb);
            HIPCK(hipMemcpyAsync(l.data(), m->scal.p, nb * sizeof(double), hipMemcpyDeviceToHost, s));
            HIPCK(hipStreamSynchronize(s));
            double tot = 0.0;
            for (double x : l) tot += x;
            if (loss_out) loss_out[e] = tot / double(nb);
        }
        HIPCK(hipGetLastError());
        return SP_OK;
    });
}

int sp_set_precond(sp_handle* h, sp_mlp* use, sp_mlp* record) {
    return guarded([&]() -> int {
        SP_REQUIRE(h, "null argument");
        for (sp_mlp* m : {use, record})
            if (m) SP_REQUIRE(m->device == h->device, "the model must live on the state's device");
        if (record) SP_REQUIRE(record->cap > 0, "the recording model has no room for training pairs");
        if (use && record)
            SP_REQUIRE(use->scope == record->scope, "the model in use and the recording one differ in scope");
        HIPCK(hipStreamSynchronize(h->stream));
        h->mlp_use = use;
        h->mlp_rec = record;
        return SP_OK;
    });
}

int sp_energy(sp_handle* h, double* E, double* normP) {
    return guarded([&]() -> int {
        SP_REQUIRE(h && E && normP, "null argument");
        const int k = h->center;
        const int n = int(h->sites[k - 1].size);
        ensure_davidson(h, std::max(h->dav_sub, 2));
        forget_mix(h);
        // always FP64 (also with SP_FP32)
        heff_apply(h, k, site_ptr(h, k), h->dHV.p, h->dNV.p, false, true);
        double* sm = h->dsmall.p;
        spk::multidot(h->stream, h->dHV.p, 0, 1, site_ptr(h, k), n, sm);
        spk::multidot(h->stream, h->dNV.p, 0, 1, site_ptr(h, k), n, sm + 1);
        spk::multidot(h->stream, site_ptr(h, k), 0, 1, site_ptr(h, k), n, sm + 2);
        HIPCK(hipMemcpyAsync(h->pin, sm, 3 * sizeof(double), hipMemcpyDeviceToHost, h->stream));
        HIPCK(hipStreamSynchronize(h->stream));
        const double xy = h->pin[0], xny = h->pin[1], xx = h->pin[2];
        if (!(xx > 0.0) || !(std::fabs(xny) / xx >= 1e-12)) {
            *E = NAN;
            *normP = xx > 0.0 ? xny / xx : 0.0;
            throw SpError(SP_ENORM, "projected norm vanishes");
        }
        *E = xy / xny;
        *normP = xny / xx;
        return SP_OK;
    });
}

int sp_site_size(const sp_handle* h, int site, long long* n) {
    return guarded([&]() -> int {
        SP_REQUIRE(h && n, "null argument");
        check_site(h, site);
        *n = h->sites[site - 1].size;
        return SP_OK;
    });
}

int sp_get_site(sp_handle* h, int site, double* host) {
    return guarded([&]() -> int {
        SP_REQUIRE(h && host, "null argument");
        check_site(h, site);
        HIPCK(hipMemcpyAsync(host, site_ptr(h, site), h->sites[site - 1].size * sizeof(double),
                             hipMemcpyDeviceToHost, h->stream));
        HIPCK(hipStreamSynchronize(h->stream));
        return SP_OK;
    });
}

int sp_set_site(sp_handle* h, int site, const double* host) {
    return guarded([&]() -> int {
        SP_REQUIRE(h && host, "null argument");
        check_site(h, site);
        HIPCK(hipMemcpyAsync(site_ptr(h, site), host, h->sites[site - 1].size * sizeof(double),
                             hipMemcpyHostToDevice, h->stream));
        HIPCK(hipStreamSynchronize(h->stream));
        invalidate_for_site(h, site);
        return SP_OK;
    });
}

int sp_center(const sp_handle* h, int* site) {
    return guarded([&]() -> int {
        SP_REQUIRE(h && site, "null argument");
        *site = h->center;
        return SP_OK;
    });
}

int sp_heff_flops(const sp_handle* h, int site, double* flops) {
    return guarded([&]() -> int {
        SP_REQUIRE(h && flops, "null argument");
        check_site(h, site);
        *flops = h->plan[site - 1].heff_flops;
        return SP_OK;
    });
}

int sp_heff_batch_profile(sp_handle** hs, int n, const int* sites, int reps, double* out) {
    return guarded([&]() -> int {
        SP_REQUIRE(hs && sites && out && n >= 1 && reps >= 1, "bad arguments");
        hipStream_t s = hs[0]->stream;
        HeffBatch hb;
        double groups = 0.0;
        double flops = 0.0, bytes = 0.0;
        for (int i = 0; i < n; ++i) {
            sp_handle* h = hs[i];
            SP_REQUIRE(h, "null handle");
            check_site(h, sites[i]);
            const int k = sites[i];
            SP_REQUIRE(h->path == SP_PATH_TILED && h->plan[k - 1].h_rows > 0, "every site must have a fused plan");
            SP_REQUIRE(h->stream == s && h->device == hs[0]->device && h->precision == hs[0]->precision,
                       "one device, stream and precision");
            SP_REQUIRE(h->Lvalid[k - 1] && h->Rvalid[k], "environments are not built");
            for (int j = 0; j < i; ++j) SP_REQUIRE(hs[j] != h, "a handle appears twice");
            forget_mix(h);
            hb.add(h, k, site_ptr(h, k), nullptr);
            const SitePlan& P = h->plan[k - 1];
            groups += double(P.c_heff.tiles.size()) * h->G;
            flops += P.heff_flops;
            const double G = h->G, xs = double(h->sites[k - 1].size);
            bytes += 8.0 * (G * h->env[k - 1].size + G * h->env[k].size + xs + 2.0 * G * xs);
        }
        hb.finish();
        std::vector<char> rec(hb.bytes());
        hb.pack(rec.data());
        DArr<char> dinst;
        dinst.upload(rec, s);
        HIPCK(hipStreamSynchronize(s));
        auto launch_on = [&](hipStream_t st) { hb.launch(st, dinst.p); };
        auto launch = [&]() { launch_on(s); };
        launch();  // warm-up
        hipEvent_t e0, e1;
        HIPCK(hipEventCreate(&e0));
        HIPCK(hipEventCreate(&e1));
        HIPCK(hipEventRecord(e0, s));
        for (int r = 0; r < reps; ++r) launch();
        HIPCK(hipEventRecord(e1, s));
        HIPCK(hipEventSynchronize(e1));
        float ms = 0.f;
        HIPCK(hipEventElapsedTime(&ms, e0, e1));
        HIPCK(hipGetLastError());
        out[0] = 1e3 * double(ms) / reps;
        out[1] = flops;
        out[2] = bytes;
        out[3] = groups;

        // The same launches captured once in a HIP graph (on a private
        // stream: the handles' stream may be the null stream) and replayed.
        // Every checked replay follows eager work that clears the partials,
        // and its partials must equal the eager launch's bit for bit.
        std::vector<std::vector<double>> ref(n), got(n);
        auto partials = [&](std::vector<std::vector<double>>& dst) {
            for (int i = 0; i < n; ++i) {
                const size_t xs = hs[i]->sites[sites[i] - 1].size, m = heff_parts(hs[i], sites[i]) * xs, mn = hs[i]->G * xs;
                dst[i].resize(m + mn);
                HIPCK(hipMemcpy(dst[i].data(), hs[i]->ypart.p, m * sizeof(double), hipMemcpyDeviceToHost));
                HIPCK(hipMemcpy(dst[i].data() + m, hs[i]->nypart.p, mn * sizeof(double), hipMemcpyDeviceToHost));
            }
        };
        launch();
        HIPCK(hipStreamSynchronize(s));
        partials(ref);
        hipStream_t gs = nullptr;
        hipGraph_t graph = nullptr;
        hipGraphExec_t exec = nullptr;
        HIPCK(hipStreamCreateWithFlags(&gs, hipStreamNonBlocking));
        HIPCK(hipStreamBeginCapture(gs, hipStreamCaptureModeThreadLocal));
        launch_on(gs);
        HIPCK(hipStreamEndCapture(gs, &graph));
        HIPCK(hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0));
        double maxdiff = 0.0;
        for (int c = 0; c < 3; ++c) {
            for (int i = 0; i < n; ++i) {
                const long long xs = hs[i]->sites[sites[i] - 1].size;
                spk::fill(s, hs[i]->ypart.p, heff_parts(hs[i], sites[i]) * xs, 0.0);
                spk::fill(s, hs[i]->nypart.p, hs[i]->G * xs, 0.0);
            }
            HIPCK(hipStreamSynchronize(s));
            HIPCK(hipGraphLaunch(exec, gs));
            HIPCK(hipStreamSynchronize(gs));
            partials(got);
            for (int i = 0; i < n; ++i)
                for (size_t e = 0; e < ref[i].size(); ++e)
                    maxdiff = std::max(maxdiff, std::fabs(got[i][e] - ref[i][e]));
        }
        HIPCK(hipEventRecord(e0, gs));
        for (int r = 0; r < reps; ++r) HIPCK(hipGraphLaunch(exec, gs));
        HIPCK(hipEventRecord(e1, gs));
        HIPCK(hipEventSynchronize(e1));
        float gms = 0.f;
        HIPCK(hipEventElapsedTime(&gms, e0, e1));
        (void)hipGraphExecDestroy(exec);
        (void)hipGraphDestroy(graph);
        (void)hipStreamDestroy(gs);
        (void)hipEventDestroy(e0);
        (void)hipEventDestroy(e1);
        HIPCK(hipGetLastError());
        out[4] = 1e3 * double(gms) / reps;
        out[5] = maxdiff;
        return SP_OK;
    });
}

int sp_heff_profile(sp_handle* h, int site, int reps, const double* x, double* y, double* ny, double* out) {
    return guarded([&]() -> int {
        SP_REQUIRE(h && x && y && ny && out && reps >= 1, "bad arguments");
        check_site(h, site);
        if (!h->Lvalid[site - 1] || !h->Rvalid[site]) throw SpError(SP_ESTATE, "environments are not built");
        forget_mix(h);
        SitePlan& P = h->plan[site - 1];
        hipStream_t s = h->stream;
        const bool plain = h->path == SP_PATH_PLAIN;
        const spk::BufSet b = bufset(h, site, x, y, ny, nullptr);
        const int n = int(h->sites[site - 1].size);
        hipEvent_t ev[4];
        for (auto& e : ev) HIPCK(hipEventCreate(&e));
        double ms[3] = {0, 0, 0};
        double premix_ms = 0.0;
        if (!plain && !P.mix_l.empty()) {
            // the pre-mixed left environment is built once per local problem
            // and reused by every product of the solve: timed on its own,
            // outside the products
            h->lt_site = -1;
            HIPCK(hipEventRecord(ev[0], s));
            premix_left(h, site, heff_mode(h, site, false));
            HIPCK(hipEventRecord(ev[1], s));
            HIPCK(hipEventSynchronize(ev[1]));
            float t = 0.f;
            HIPCK(hipEventElapsedTime(&t, ev[0], ev[1]));
            premix_ms = t;
        }
        for (int r = 0; r < reps; ++r) {
            HIPCK(hipEventRecord(ev[0], s));
            if (plain) {
                P.p1.launch(s, b, P.coef.p);
            } else {
                heff_apply(h, site, x, nullptr, nullptr, true);
            }
            HIPCK(hipEventRecord(ev[1], s));
            if (plain) P.mixl.launch(s, b, P.coef.p);
            HIPCK(hipEventRecord(ev[2], s));
            if (plain) {
                P.yout.launch(s, b, P.coef.p);
            } else {
                spk::gsum2(s, h->ypart.p, h->nypart.p, n, heff_parts(h, site), h->G, n, y, ny);
            }
            HIPCK(hipEventRecord(ev[3], s));
            HIPCK(hipEventSynchronize(ev[3]));
            for (int i = 0; i < 3; ++i) {
                float t = 0.f;
                HIPCK(hipEventElapsedTime(&t, ev[i], ev[i + 1]));
                ms[i] += t;
            }
        }
        for (auto& e : ev) (void)hipEventDestroy(e);
        const double G = h->G, xs = double(h->sites[site - 1].size);
        const double Lb = G * h->env[site - 1].size, Rb = G * h->env[site].size;
        for (int i = 0; i < 3; ++i) out[i] = ms[i] / reps;
        if (plain) {
            out[3] = P.p1.flops;
            out[4] = P.mixl.flops;
            out[5] = P.yout.flops;
            out[6] = 8.0 * (Lb + xs + G * P.Tsize);
            out[7] = 8.0 * (G * P.Tsize + G * P.Vsize);
            out[8] = 8.0 * (G * P.Vsize + G * P.Tsize + Rb + 2.0 * xs);
        } else {
            // the product into per-g partials: environments and x read once,
            // per-g partials written
            out[1] = premix_ms;
            out[3] = P.heff_flops;
            out[4] = G * P.mix_l.flops;
            out[5] = 2.0 * G * xs;
            out[6] = 8.0 * (Lb + Rb + xs + 2.0 * G * xs);
            out[7] = 0.0;
            out[8] = 8.0 * (2.0 * G * xs + 2.0 * xs);
        }
        HIPCK(hipGetLastError());
        return SP_OK;
    });
}

int sp_quadrature(int G, int twoS, int twoM, double* x, double* w, double* coef) {
    return guarded([&]() -> int {
        SP_REQUIRE(G >= 1 && G <= 1024 && x && w && coef, "bad arguments");
        SP_REQUIRE(twoS >= 0 && std::abs(twoM) <= twoS && (twoS - twoM) % 2 == 0, "need |M| <= S, S - M integer");
        std::vector<double> c(G), s(G);
        sph::projector_quadrature(G, twoS, twoM, x, w, c.data(), s.data(), coef);
        return SP_OK;
    });
}

int sp_exact_points(int N, int K, int twoS, int twoM) { return sph::exact_points(N, K, twoS, twoM); }

int sp_mpo_hubbard(int L, double t, double U, int* w, double* data, long long* n) {
    return guarded([&]() -> int {
        SP_REQUIRE(L >= 1 && w && n, "bad arguments");
        return sph::mpo_hubbard(L, t, U, w, data, n);
    });
}
int sp_mpo_s2(int L, int* w, double* data, long long* n) {
    return guarded([&]() -> int {
        SP_REQUIRE(L >= 1 && w && n, "bad arguments");
        return sph::mpo_s2(L, w, data, n);
    });
}
int sp_mpo_identity(int L, int* w, double* data, long long* n) {
    return guarded([&]() -> int {
        SP_REQUIRE(L >= 1 && w && n, "bad arguments");
        return sph::mpo_identity(L, w, data, n);
    });
}

int sp_mpo_site_op(int L, int p, const double* op, int* w, double* data, long long* n) {
    return guarded([&]() -> int {
        SP_REQUIRE(L >= 1 && p >= 1 && p <= L && op && w && n, "bad arguments");
        return sph::mpo_site_op(L, p, op, w, data, n);
    });
}
int sp_mpo_epq(int L, int p, int q, int* w, double* data, long long* n) {
    return guarded([&]() -> int {
        SP_REQUIRE(L >= 1 && p >= 1 && p <= L && q >= 1 && q <= L && w && n, "bad arguments");
        return sph::mpo_epq(L, p, q, w, data, n);
    });
}
int sp_mpo_spin_corr(int L, int X, int Y, int* w, double* data, long long* n) {
    return guarded([&]() -> int {
        SP_REQUIRE(L >= 1 && X >= 1 && X <= L && Y >= 1 && Y <= L && w && n, "bad arguments");
        return sph::mpo_spin_corr(L, X, Y, w, data, n);
    });
}

int sp_mpo_abinitio(int K, const double* h, const double* eri, int* w, double* data, long long* n) {
    return guarded([&]() -> int {
        SP_REQUIRE(K >= 2 && K <= 64 && h && eri && w && n, "bad arguments");
        const int r = sph::mpo_abinitio(K, h, eri, w, data, n);
        SP_REQUIRE(r != -2, "ab-initio MPO: a bond needs more than 4096 channels");
        SP_REQUIRE(r == 0, "ab-initio MPO: internal error");
        return 0;
    });
}

int sp_mpo_abinitio_component(int K, int p, const double* h, const double* eri, int* w, double* data, long long* n) {
    return guarded([&]() -> int {
        SP_REQUIRE(K >= 2 && K <= 64 && h && eri && w && n, "bad arguments");
        SP_REQUIRE(p >= 1 && p <= K, "orbital p out of range");
        const int r = sph::mpo_abinitio(K, h, eri, w, data, n, p - 1);
        SP_REQUIRE(r != -2, "ab-initio MPO: a bond needs more than 4096 channels");
        SP_REQUIRE(r == 0, "ab-initio MPO: internal error");
        return 0;
    });
}

int sp_mpo_hubbard_component(int L, int p, double t, double U, int* w, double* data, long long* n) {
    return guarded([&]() -> int {
        SP_REQUIRE(L >= 2 && L <= 64 && w && n, "bad arguments");
        SP_REQUIRE(p >= 1 && p <= L, "site p out of range");
        // the open chain as integrals: h = -t on nearest neighbours, (pp|pp) = U
        std::vector<double> hh(size_t(L) * L, 0.0), eri(size_t(L) * L * L * L, 0.0);
        for (int q = 0; q + 1 < L; ++q) hh[size_t(q) * L + q + 1] = hh[size_t(q + 1) * L + q] = -t;
        for (int q = 0; q < L; ++q) eri[((size_t(q) * L + q) * L + q) * L + q] = U;
        const int r = sph::mpo_abinitio(L, hh.data(), eri.data(), w, data, n, p - 1);
        SP_REQUIRE(r == 0, "Hubbard component MPO: internal error");
        return 0;
    });
}

int sp_small_gen_lowest(int m, const double* H, const double* N, double drop, double* theta, double* a,
                        int* rank) {
    return guarded([&]() -> int {
        SP_REQUIRE(m >= 1 && H && N && theta && a && rank, "bad arguments");
        const int r = sph::gen_lowest(m, H, N, drop, theta, a, nullptr, rank);
        if (r < 0) throw SpError(SP_ENAN, "subspace eigensolver failed");
        if (r == 0) throw SpError(SP_ENORM, "the metric vanishes");
        return SP_OK;
    });
}

int sp_small_gen_lowest_gpu(int m, double* H, double* N, double drop, int need_all, int keep, double* theta,
                            double* a, double* Qk, int* rank) {
    return guarded([&]() -> int {
        SP_REQUIRE(m >= 1 && m < spk::kDevSubMax && H && N && theta && a && rank, "bad arguments");
        SP_REQUIRE(!need_all || (Qk && keep >= 1 && keep <= spk::kDevKeepMax), "bad restart arguments");
        const int r = spk::dev_small_solve(m, H, N, drop, need_all, keep, theta, a, Qk);
        SP_REQUIRE(r >= 0, "device subspace solve failed");
        *rank = r;
        if (r == 0) throw SpError(SP_ENORM, "the projected metric vanishes");
        return SP_OK;
    });
}

int sp_small_eigh(int n, double* a, double* ev, double* vec) {
    return guarded([&]() -> int {
        SP_REQUIRE(n >= 0 && a && ev && vec, "bad arguments");
        if (sph::sym_eigh(n, a, ev, vec) != 0) throw SpError(SP_ENAN, "eigensolver did not converge");
        return SP_OK;
    });
}

}  // extern "C"
